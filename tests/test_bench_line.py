"""bench.py's line on stdout stays short whatever else is measured."""
import json

import bench


def test_the_line_has_its_keys_and_fits():
    third = 1e6 / 3.0
    result = {k: third for k in bench.HEADLINE}
    result.update(metric="m" * 80, unit="tokens/s", n_gpus=1, steps=1000, warmup=200, higher_is_better=True, scaling="weak", vs_baseline=None, dtype="bf16",
                  data="synthetic", config={f"setting_{i}": 4096 for i in range(14)}, stage_us={f"stage_{i}": third for i in range(4)},
                  ms_per_step_blocks_p10_p50_p90=[third] * 3, roofline={"kernel": "k" * 110, "how": "h" * 120, **{f"figure_{i}": third for i in range(8)}},
                  cpu_baseline={"value": third, "unit": "tokens/s", "cores": 16, "kind": "oracle", "sample": "s" * 100})
    result["sweep"] = [dict(G=g, us=third) for g in range(400)]
    line, rest = bench.split_result(result)
    assert len(line) <= bench.HEADLINE_CHARS and "\n" not in line
    got = json.loads(line)
    assert set(got) == set(bench.HEADLINE) and set(rest) == {"sweep"}
    assert abs(got["value"] / third - 1.0) < 1e-6
