"""What the host code launches, without a GPU: the library on top of a recorder in the place of the HIP runtime (launch_record.py)."""
import re

import pytest

from launch_record import record

LLAMA = dict(d=4096, hq=32, hkv=8, dh=128, groups=64, words=1024)
SMALL = dict(d=768, hq=12, hkv=12, dh=64, groups=16, words=256)
# calls of every kernel that asks for more than 64 KiB of dynamic LDS
LARGE_LDS = [
    dict(entry="layer", n_local=1024, n_nonlocal=3072, causal=True, **LLAMA),
    dict(entry="block", n_local=300, n_nonlocal=300, norm="layernorm", mlp="gelu_erf", dff=3072, **SMALL),
    dict(entry="block", n_local=1024, n_nonlocal=0, norm="rmsnorm", mlp="swiglu", dff=14336, **LLAMA),
    dict(entry="step", hq=64, hkv=8, dh=128, n_local=8001, n_nonlocal=40000, groups=32, words=1024),
    dict(entry="step", hq=32, hkv=8, dh=128, n_local=100, n_nonlocal=300, groups=32, words=1024, dtype="f32"),
    dict(entry="stats", groups=64, dg=64, words=1024, tokens=16384),
    dict(entry="stats", groups=129, dg=8, words=1024, tokens=16384),
]


def test_the_cap_on_dynamic_lds_is_raised_on_every_device(tmp_path):
    """Device 0, then device 1, then 0 again in one process: no launch asks for more than the cap of its kernel on its device."""
    calls = [dict(c, device=d) for d in (0, 1, 70, 0) for c in LARGE_LDS]
    results = record(calls, tmp_path)
    for c, r in zip(calls, results):
        assert r["rc"] == "ok" and r["launches"], c
        assert any(lds > 64 * 1024 for _, _, _, lds, _ in r["launches"]), c
        for name, _, _, lds, cap in r["launches"]:
            assert lds <= cap, f"device {c['device']}: {name} with {lds} bytes of dynamic LDS, cap {cap}"


def test_a_refused_cap_is_an_error_that_does_not_last(tmp_path):
    calls = [dict(c, fail_attributes=f) for c in LARGE_LDS for f in (True, False)]
    for c, r in zip(calls, record(calls, tmp_path)):
        assert (r["rc"] == "ok") == (not c["fail_attributes"]), (c, r["rc"])


def kernels(result):
    assert result["rc"] == "ok", result["rc"]
    return [name for name, *_ in result["launches"]]


def test_the_sort_of_the_statistics(tmp_path):
    """One launch for many groups, or for a large codebook and a number of segments that is no multiple of eight; three launches otherwise."""
    from test_gpu_training import ONE_LAUNCH_SORTS
    cases = [(t, g, k, True) for t, g, k in ONE_LAUNCH_SORTS]
    cases += [(16384, 64, 1024, True), (16384, 64, 256, True), (8000, 64, 256, False), (16384, 1, 256, False), (16384, 32, 1024, False),
              (7000, 1, 1024, True), (8000, 1, 1024, False), (718, 32, 1024, False), (16385, 64, 1024, False), (16384, 64, 1025, False), (0, 64, 1024, False)]
    results = record([dict(entry="stats", tokens=t, groups=g, words=k, dg=8) for t, g, k, _ in cases], tmp_path)
    for (t, g, k, one), r in zip(cases, results):
        names = kernels(r)
        assert ("sort_group_kernel" in names) == one and ("sort_place_kernel" in names) == (not one), (t, g, k, names)


EPILOGUES = {0: "", 1: " residual", 2: " slice", 3: " gelu_tanh", 4: " gelu_erf", 5: " swiglu"}


def forms(result):
    """The products of a call, as wave<row tiles, column tiles, stages> or tile<rows, columns>, with what they carry."""
    out = []
    for name in kernels(result):
        m = re.match(r"gemm_wave_kernel<(\d, \d, \d), (\w+), (\w+), (\d)>", name)
        if m:
            gather, enc = m[2] == "true", m[3] == "true"
            out.append(f"wave<{m[1]}>" + " GATHER" * gather + " ENC" * enc + EPILOGUES[int(m[4])])
        m = re.match(r"gemm_nt_bf16_kernel<(\d+, \d+), \d, \d, (\w+), (\w+), (\d)>", name)
        if m:
            out.append(f"tile<{m[1]}>" + " ENC" * (m[3] == "true") + EPILOGUES[int(m[4])])
    return out


def test_the_forms_the_gpu_tests_name(tmp_path):
    """The products, layers and blocks of the GPU tests run on the forms named beside them."""
    from test_gpu_block import MLP_LAUNCHES
    from test_gpu_layer import GATHERED_TILES, MODEL_OF_WIDTH, PROJECTION_LAUNCHES
    from test_gpu_projection import PRODUCTS
    model = {d: dict(d=d, hq=hq, hkv=hkv, dh=dh, causal=True, bias=True) for d, (hq, hkv, dh) in MODEL_OF_WIDTH.items()}
    for (m, n, k, form), r in zip(PRODUCTS, record([dict(entry="project", m=m, n=n, k=k) for m, n, k, _ in PRODUCTS], tmp_path)):
        assert forms(r) == [form], (m, n, k)
    calls = [dict(model[d], entry="layer", n_local=tl, n_nonlocal=tn, groups=g, words=w) for d, tl, tn, g, w, _ in PROJECTION_LAUNCHES]
    for case, r in zip(PROJECTION_LAUNCHES, record(calls, tmp_path)):
        assert forms(r)[0] == case[-1].replace("> GATHER", ">" if case[-1].startswith("tile") else "> GATHER"), (case, forms(r))
    tiles = [(d, groups, words, rows, form) for d, groups, words in GATHERED_TILES for rows, form in (((700, 700), "tile<128, 256>"), ((1100, 600), "tile<256, 256>"))]
    calls = [dict(entry="layer", d=d, hq=32, hkv=8, dh=128, causal=True, n_local=tl, n_nonlocal=tn, groups=groups, words=words)
             for d, groups, words, (tl, tn), _ in tiles]
    for case, r in zip(tiles, record(calls, tmp_path)):
        assert forms(r)[0].replace(" ENC", "") == case[-1], (case, forms(r))
    calls = [dict(model[d], entry="block", n_local=t, n_nonlocal=0, groups=g, words=w, mlp=mlp, dff=f, norm="layernorm")
             for d, t, g, w, mlp, f, _ in MLP_LAUNCHES]
    for case, r in zip(MLP_LAUNCHES, record(calls, tmp_path)):
        assert set(case[-1]) <= set(forms(r)), (case, forms(r))


@pytest.mark.parametrize("m,n,k,slow", [
    (2000, 4096, 64, "wave"),       # us on the form it has against the wavefront-private one: 10.8 / 16.4
    (6000, 1024, 512, "wave"),      # 16.6 / 24.7
    (2000, 4096, 256, "wave"),      # 13.9 / 18.3
    (718, 4096, 128, "wave"),       # 6.8 / 8.7
    (64, 1024, 4096, "tile"),       # 6.4 / 32.0
    (1000, 4096, 4096, "tile"),     # 36.6 / 46.1
])
def test_short_and_long_contractions(m, n, k, slow, tmp_path):
    """A product whose contraction is short next to its outputs is not cut into many small workgroups, each with a start and a reduction of its own."""
    (form,) = forms(record([dict(entry="project", m=m, n=n, k=k)], tmp_path)[0])
    assert not form.startswith(slow), form


def test_score_products_of_wide_groups(tmp_path):
    """32 groups of 128 channels: six products at a time over K = 128.  (79 us for 718 tokens on 128 x 128 tiles, 117 on 32 x 32.)"""
    for tokens in (718, 2000):
        r = record([dict(entry="encode", d=4096, groups=32, words=1024, tokens=tokens)], tmp_path)[0]
        assert all(f.startswith("tile") for f in forms(r)[:5]), forms(r)


def test_where_the_encode_of_the_local_rows_runs(tmp_path):
    """In the projection launch where its last round has room for it, also if that takes another tile; in the attention launch of 128-wide heads where
    units are idle anyway; and not six items behind one another on sixteen workgroups."""
    def layer(d, **more):
        hq, hkv, dh = {768: (12, 12, 64), 4096: (32, 8, 128)}[d]
        return dict(entry="layer", d=d, hq=hq, hkv=hkv, dh=dh, causal=True, **more)
    calls = [layer(768, n_local=342, n_nonlocal=342, before=114, groups=32, words=256), layer(768, n_local=212, n_nonlocal=636, before=318, groups=32, words=1024),
             layer(4096, n_local=1100, n_nonlocal=1100, before=366, groups=64, words=1024), layer(4096, n_local=208, n_nonlocal=416, before=208, groups=64, words=1024)]
    a, b, c, d = record(calls, tmp_path)
    assert forms(a)[0] == forms(b)[0] == "wave<2, 2, 1> GATHER ENC"
    assert forms(c)[0] == "tile<256, 256> ENC"
    assert "ENC" not in forms(d)[0] and any(re.match(r"attn_bf16_kernel<128, .*, true>", k) for k in kernels(d))
    assert not any("vq_encode" in k for r in (a, b, c, d) for k in kernels(r))


def test_the_decode_step_on_heads_of_64(tmp_path):
    """A score table only for one group per head and a small codebook (19 000 + 19 000 rows, two groups, K = 1024: 22.3 us on the vector ALU, 25.7 with a
    table, 23.7 gathering); a third workgroup per unit where it shortens what a wavefront walks."""
    step = dict(entry="step", hq=12, hkv=12, dh=64)
    calls = [dict(step, n_local=19000, n_nonlocal=19000, groups=24, words=1024), dict(step, n_local=10000, n_nonlocal=30000, groups=12, words=256),
             dict(step, n_local=4832, n_nonlocal=4832, groups=24, words=16)]
    kernel, grid = zip(*[r["launches"][0][:2] for r in record(calls, tmp_path)])
    assert kernel == ("decode_stream_kernel<64, 1, 4, 2, false>", "decode_stream_kernel<64, 1, 8, 1, true>", "decode_stream_kernel<64, 1, 4, 2, false>")
    assert [g[0] for g in grid] == [64, 21, 42]


def test_the_forms_of_the_codebook_update(tmp_path):
    """Four channels per thread for widths of whole 16-byte pieces at aligned addresses, else a channel per thread."""
    cases = [(64, 0, "bf16", True), (12, 0, "f32", True), (1024, 0, "bf16", True), (6, 0, "bf16", False), (1028, 0, "bf16", False), (64, 2, "bf16", False),
             (64, 4, "f32", False)]
    results = record([dict(entry="update", groups=3, words=40, dg=dg, skew=skew, dtype=dtype) for dg, skew, dtype, _ in cases], tmp_path)
    for case, r in zip(cases, results):
        assert any("update4" in k for k in kernels(r)) == case[3], case


def test_gathered_rows_do_not_hide_that_weights_come_from_memory(tmp_path):
    """Layers 4096 wide with one round of 64 x 64 tiles: two stages (54 us, one stage 58)."""
    results = record([dict(entry="layer", d=4096, hq=32, hkv=8, dh=128, n_local=m, n_nonlocal=n, causal=True, before=before, groups=groups, words=256)
                      for m, n, before, groups in ((83, 83, 41, 32), (87, 87, 43, 16), (73, 125, 62, 16), (100, 100, 50, 64))], tmp_path)
    for r in results:
        assert kernels(r)[0].startswith("gemm_wave_kernel<2, 2, 2, true"), kernels(r)


def test_the_forms_of_the_fp32_encode(tmp_path):
    """(tokens, groups, codewords, group length): shared 0, in stages 1, a token per wavefront 2, and without LDS 3; in 16-byte pieces or not."""
    cases = [(64, 4, 256, 48, 0, True), (500, 1, 1024, 768, 0, True), (500, 1, 1024, 1028, 1, True), (500, 1, 1024, 1027, 1, False), (3, 4, 300, 7, 0, False),
             (1024, 2, 16, 384, 2, True), (1028, 2, 16, 384, 0, True), (256, 4, 64, 48, 2, True), (257, 4, 64, 48, 0, True), (64, 1, 64, 512, 0, True),
             (64, 1, 64, 768, 2, True), (64, 1, 64, 1100, 2, True), (4000, 4, 64, 32, 3, True), (64, 4, 65, 32, 0, True), (4000, 4, 128, 12, 3, True), (64, 4, 128, 16, 0, True),
             (64, 4, 128, 3, 3, False)]
    results = record([dict(entry="encode", dtype="f32", tokens=t, groups=g, words=k, d=g * dg) for t, g, k, dg, _, _ in cases], tmp_path)
    for case, r in zip(cases, results):
        assert kernels(r) == [f"vq_encode_f32_kernel<{case[4]}, {str(case[5]).lower()}>"], (case, kernels(r))


def test_tokens_per_wavefront_of_the_bf16_encode(tmp_path):
    """64 where 32 would make more than one round of 512 workgroups, and for more than 256 codewords from 256 items on."""
    cases = [(1000, 64, 256, 1, 512), (1025, 64, 256, 2, 320), (1000, 64, 512, 2, 256), (768, 64, 1024, 1, 384), (769, 64, 1024, 2, 256), (2048, 32, 16, 1, 512),
             (2049, 32, 16, 2, 288)]
    results = record([dict(entry="encode", tokens=t, groups=g, words=k, d=64 * g) for t, g, k, _, _ in cases], tmp_path)
    for (t, g, k, blocks, grid), r in zip(cases, results):
        assert [(n, s[0]) for n, s, *_ in r["launches"]] == [(f"vq_encode_bf16_fast_kernel<{blocks}>", grid)], (t, g, k, r["launches"])


def test_workgroups_per_group_of_the_sort(tmp_path):
    """A group's codes in ranges on up to four workgroups while all of them fit 256 units and the partial sums' place holds the transposed codes; else one."""
    cases = [(16384, 48, 1024, 8, 4), (16384, 64, 1024, 64, 4), (16384, 65, 1024, 8, 2), (16384, 128, 1024, 8, 2), (16384, 129, 1024, 8, 1), (16384, 64, 1024, 6, 1)]
    results = record([dict(entry="stats", tokens=t, groups=g, words=k, dg=dg) for t, g, k, dg, _ in cases], tmp_path)
    for (t, g, k, dg, parts), r in zip(cases, results):
        (name, grid), = [(n, s) for n, s, *_ in r["launches"] if n in ("sort_group_kernel", "sort_whole_group_kernel")]
        assert (name == "sort_group_kernel") == (parts > 1) and grid[:2] == [g, parts], (t, g, k, dg, name, grid)


def test_attention_of_short_sequences(tmp_path):
    """32 query rows per workgroup where those make a single round of 256, unless encodes behind them would lose units; the shapes the GPU tests name."""
    from test_gpu_kv_variant import SHORT
    layer = lambda dh, h, n, m=96: dict(entry="layer", d=64 * h, hq=h, hkv=h, dh=dh, causal=True, n_local=n, n_nonlocal=m, groups=16, words=256)
    calls = [layer(64, 12, 672), layer(64, 12, 673), layer(128, 32, 256, 200), layer(128, 32, 257, 200)]
    for r, name in zip(record(calls, tmp_path), ("attn_short_kernel<64, false, false>", "attn_bf16_kernel<64", "attn_short_kernel<128", "attn_bf16_kernel<128")):
        assert any(k.startswith(name) for k in kernels(r)), (name, kernels(r))
    calls = [dict(entry="kv", d=d, hq=hq, hkv=hkv, dh=128, causal=True, n_local=t // 4, n_nonlocal=t - t // 4, groups=g, words=w) for d, hq, hkv, t, g, w in SHORT]
    calls.append(dict(calls[0], n_local=256, n_nonlocal=768))
    results = record(calls, tmp_path)
    for c, r in zip(calls[:-1], results):
        assert "attn_short_kernel<128, false, true>" in kernels(r), (c, kernels(r))
    assert "attn_bf16_kernel<128, true, false, 2, true>" in kernels(results[-1])


def test_walks_cut_between_workgroups(tmp_path):
    """The shapes the GPU tests name, and none where whole walks are a round of their own or the call brings no scratch for the parts."""
    from test_gpu_layer import CUT_WALKS
    calls = [dict(entry="layer", d=64 * hq, hq=hq, hkv=hkv, dh=128, cls=cls, causal=causal, n_local=t, n_nonlocal=n, groups=16, words=256)
             for t, n, hq, hkv, cls, causal, _, _, _ in CUT_WALKS]
    for (t, n, hq, _, cls, _, _, whole, parts), r in zip(CUT_WALKS, record(calls, tmp_path)):
        blocks = -(-(t + cls) // 128)
        merge = [(k, g[0]) for k, g, *_ in r["launches"] if k.startswith("attn_merge")]
        assert merge == [(f"attn_merge_kernel<{parts}>", 4 * hq * (blocks - whole))], (t, n, merge)
        (grid,) = [g[0] for k, g, *_ in r["launches"] if k.startswith("attn_cut_kernel")]
        assert grid >= hq * (whole + (blocks - whole) * parts)
    calls = [dict(LLAMA, entry=e, n_local=t, n_nonlocal=3072, causal=True) for e in ("layer", "kv") for t in (640, 1024)]
    for r in record(calls, tmp_path):
        assert not any(k.startswith(("attn_cut", "attn_merge")) for k in kernels(r)), kernels(r)


def test_more_whole_walks_than_units(tmp_path):
    """The longest of all heads first where walks differ in length; heads that the XCDs do not share evenly one after the other."""
    calls = [dict(LLAMA, entry="layer", n_local=1531, n_nonlocal=2565, causal=c) for c in (True, False)]
    calls.append(dict(entry="layer", d=640, hq=20, hkv=4, dh=128, groups=16, words=256, n_local=1700, n_nonlocal=64, causal=True))
    for r, name in zip(record(calls, tmp_path), ("attn_cut_kernel", "attn_bf16_kernel", "attn_bf16_kernel")):
        assert any(k.startswith(name) for k in kernels(r)) and not any(k.startswith("attn_merge") for k in kernels(r)), (name, kernels(r))


def test_rotary_positions_are_one_launch(tmp_path):
    """Queries, keys and rebuilt keys together; eight heads of a row to a thread, so that 12 heads are two of them; no blocks for a matrix without rows."""
    block = dict(entry="block", causal=True, norm="rmsnorm", mlp="swiglu", dff=768, rope=10000.0, groups=16, words=256)
    calls = [dict(block, d=768, hq=12, hkv=12, dh=64, n_local=100, n_nonlocal=n, before=b) for n, b in ((300, 200), (300, 0))]
    calls.append(dict(block, d=512, hq=4, hkv=2, dh=128, n_local=33, n_nonlocal=66, before=66, dtype="f32"))
    rows = [(8 * 2 * 100, 8 * 2 * 100, 8 * 2 * 200), (8 * 2 * 100, 8 * 2 * 100), (64 * 33, 64 * 33, 64 * 66)]
    for c, threads, r in zip(calls, rows, record(calls, tmp_path)):
        assert [g[0] for k, g, *_ in r["launches"] if k.startswith("rope_kernel")] == [sum(-(-t // 256) for t in threads)], (c, r["launches"])


def test_reading_ahead_beside_the_attention(tmp_path):
    """Workgroups behind the 32-row attention of a block read the weights that follow, two lines of 128 bytes a thread, or up to four on the units that are
    left; none in a layer by itself."""
    small = dict(SMALL, n_nonlocal=60, causal=True, norm="layernorm", mlp="gelu_tanh", dff=3072)
    lines = (768 * 768 + 2 * 768 * 3072) * 2 // 128
    want = [(64, -(-lines // 1024)), (512, 64), (640, 16), (672, 4)]
    results = record([dict(small, entry="block", n_local=t) for t, _ in want], tmp_path)
    for (t, wgs), r in zip(want, results):
        (grid,) = [g[0] for k, g, *_ in r["launches"] if k.startswith("attn_short")]
        assert grid == -(-t // 32) * 12 + wgs, (t, grid)
    r = record([dict(SMALL, entry="layer", n_local=64, n_nonlocal=60, causal=True)], tmp_path)[0]
    assert [g[0] for k, g, *_ in r["launches"] if k.startswith("attn_short")] == [24]


def test_rebuilt_rows_of_a_block_come_with_its_first_normalisation(tmp_path):
    """Slices of whole 8 bytes but not 16; a launch of their own for others, and none where the projections fetch codewords themselves."""
    block = dict(entry="block", d=768, hq=12, hkv=12, dh=64, n_local=100, causal=True, norm="layernorm", mlp="gelu_tanh", dff=3072, words=256)
    calls = [dict(block, n_nonlocal=300, groups=64), dict(block, n_nonlocal=300, groups=64, before=0), dict(block, n_nonlocal=300, groups=128), dict(block, n_nonlocal=300, groups=32)]
    with_norm, no_rows, own, none = (kernels(r) for r in record(calls, tmp_path))
    assert with_norm[0].startswith("norm_decode_kernel") and not any("vq_decode" in k for k in with_norm)
    assert own[0].startswith("norm_wave_kernel") and any("vq_decode_kernel" in k for k in own)
    assert not any("decode" in k for k in no_rows + none)


def test_normalisation_by_wavefronts_of_narrow_rows(tmp_path):
    """Up to 1024 values a wavefront per row, wider ones a workgroup."""
    block = dict(entry="block", hq=4, hkv=4, dh=64, n_local=33, n_nonlocal=66, causal=True, norm="rmsnorm", mlp="gelu_tanh", dff=256, groups=8, words=16)
    for d, name in ((64, "norm_wave_kernel"), (1024, "norm_wave_kernel"), (1088, "norm_kernel")):
        names = kernels(record([dict(block, d=d)], tmp_path)[0])
        assert sum(k.startswith(name) for k in names) == 2, (d, names)


@pytest.mark.parametrize("dg", [128, 192, 256])
def test_encode_of_wide_groups(dg, tmp_path):
    """32 tokens per workgroup streamed; the matrix-core body where that would make many rounds, or two short ones; score products for few groups."""
    stream, fast, wide = "vq_encode_bf16_stream_kernel", f"vq_encode_bf16_fast{dg}_kernel", "vq_encode_bf16_wide_kernel"
    body = fast if dg != 192 else stream
    few = {128: (4096, 4097), 192: (4096, None), 256: (6144, 6145)}[dg]
    cases = [(17, 16, 1024, stream), (512, 16, 1024, stream), (1024, 16, 1024, stream), (1025, 16, 1024, body), (513, 16, 512, body), (513, 16, 32, stream),
             (1025, 16, 16, body), (512, 16, 256, wide if dg == 256 else stream), (512, 16, 128, stream), (17, 16, 1022, wide),
             (few[0], 2, 1024, "gemm"), (192, 8, 1024, stream if dg == 128 else "gemm"), (193, 8, 1024, stream)]
    if dg != 192:
        cases += [(few[1], 2, 1024, stream), (8193, 2, 1024, fast), (4097, 2, 256, fast), (4097, 2, 254, wide)]
    results = record([dict(entry="encode", tokens=t, groups=g, words=k, d=dg * g) for t, g, k, _ in cases], tmp_path)
    for (t, g, k, name), r in zip(cases, results):
        assert kernels(r)[0].startswith(name), (t, g, k, kernels(r))
    if dg == 192:
        return
    beside = "attn_short_kernel<129"               # in the attention's launch, as long as its blocks and the encode's have a unit each
    last = 160 if dg == 256 else 128
    for rows, name in ((17, beside), (last, beside), (last + 1, stream), (700, stream if dg == 256 else fast), (1200, fast)):
        r = record([dict(entry="layer", d=4096, hq=32, hkv=8, dh=128, causal=True, n_local=rows, n_nonlocal=64, groups=4096 // dg, words=1024)], tmp_path)[0]
        assert [k for k in kernels(r) if k.startswith(("vq_encode", "attn_short_kernel<129", "vq_argmin"))][0].startswith(name), (rows, kernels(r))
        assert sum(k.startswith(("vq_encode", "attn_short_kernel<129", "vq_argmin")) for k in kernels(r)) == 1


@pytest.mark.parametrize("dg", [128, 256])
def test_encode_of_wide_groups_off_a_16_byte_boundary(dg, tmp_path):
    """The body's 16-byte transfers to LDS want x, the codebook and the norms on such a boundary; others keep the kernel for wide groups."""
    call = dict(entry="encode", tokens=4100, groups=16, words=1024, d=16 * dg)
    on, *off = record([call] + [dict(call, skew={a: n}) for a, n in (("x", 8), ("codebook", 2), ("cnorm", 4))], tmp_path)
    assert kernels(on) == [f"vq_encode_bf16_fast{dg}_kernel"]
    for r in off:
        assert len(kernels(r)) == 1 and kernels(r)[0].startswith("vq_encode_bf16_wide_kernel"), kernels(r)


def test_planning_the_attention_costs_the_host_little(tmp_path):
    """128-wide heads have walks to plan, 64-wide ones none: 32 blocks of 4096 rows and a layer whose heads have 800 query blocks, within twice the time of those
    (seen 1.0 - 1.1; a search over all pieces, repeated with every plan of the call, took 25 and 37 times as long)."""
    layer = dict(entry="layer", d=1024, groups=16, words=1024, causal=True, n_local=100000, n_nonlocal=64, repeat=200)
    stack = dict(entry="stack", layers=32, d=4096, groups=64, words=1024, causal=True, n_local=4096, n_nonlocal=2565, norm="rmsnorm", mlp="swiglu", dff=14336,
                 repeat=40)
    calls = [dict(layer, hq=2, hkv=2, dh=64), dict(layer, hq=1, hkv=1, dh=128), dict(stack, hq=64, hkv=16, dh=64), dict(stack, hq=32, hkv=8, dh=128)]
    us = [r["us"] for r in record(calls, tmp_path)]
    assert us[1] < 2 * us[0] and us[3] < 2 * us[2], us


def test_scratch_for_the_parts_of_walks_is_what_a_launch_fills(tmp_path):
    """The layer's workspace is Q, K, V, the peers' K and V and the heads' outputs, and behind them the parts of cut walks (64 KiB and 1 KiB each) of this
    launch or of that with pre-projected codebooks; none where both walk whole."""
    def up(n, m):
        return -(-n // m) * m

    def parts(r):
        return sum(g[0] // 4 * int(k.split("<")[1][:-1]) for k, g, *_ in r["launches"] if k.startswith("attn_merge"))

    shapes = [dict(LLAMA, n_local=1531, n_nonlocal=2565), dict(LLAMA, n_local=512, n_nonlocal=3584), dict(LLAMA, n_local=1024, n_nonlocal=3072),
              dict(LLAMA, n_local=185, n_nonlocal=3076, hq=40, d=2560), dict(LLAMA, n_local=5017, n_nonlocal=131, hq=4, hkv=4, d=256, groups=32),
              dict(LLAMA, n_local=28, n_nonlocal=3182, groups=16), dict(LLAMA, n_local=253, n_nonlocal=6982, hq=16, hkv=2, groups=16)]
    entries = ("layer", "preprojected", "kv")
    results = record([dict(c, entry=e, causal=True) for c in shapes for e in entries], tmp_path)
    some = 0
    for i, c in enumerate(shapes):
        q, v, dq, dkv = c["n_local"], c["n_nonlocal"], c["hq"] * 128, c["hkv"] * 128
        layer = [q * dq, q * dkv, up(q, 64) * dkv, v * dkv, up(v, 64) * dkv, q * dq]
        for per, sizes in ((results[3 * i:3 * i + 2], layer), (results[3 * i + 2:3 * i + 3], layer + [q * dkv])):
            n = max(parts(r) for r in per)
            some += n > 0
            if c["d"] // c["groups"] <= 64 or len(per) == 1:                 # wide groups keep scores in it, too
                assert {r["bytes"] for r in per} == {sum(up(2 * s, 256) for s in sizes) + n * (128 * 128 + 256) * 4}, c
    assert 0 < some < 2 * len(shapes)


def test_short_form_keeps_walks_beside_encodes_with_units_of_their_own(tmp_path):
    """32 query rows per workgroup and the encodes on the units that are left, as long as those are done in about the time of a walk; parts of walks beyond."""
    short = [("kv", 84, 588, 32), ("kv", 40, 1000, 16), ("kv", 200, 1000, 16), ("layer", 128, 1000, 64)]
    cut = [("kv", 40, 4096, 16), ("kv", 84, 4096, 32), ("layer", 128, 4096, 64)]
    results = record([dict(LLAMA, entry=e, n_local=t, n_nonlocal=n, groups=g, causal=True) for e, t, n, g in short + cut], tmp_path)
    for i, (c, r) in enumerate(zip(short + cut, results)):
        assert any(k.startswith("attn_short" if i < len(short) else "attn_cut") for k in kernels(r)), (c, kernels(r))


def test_codebooks_of_a_block_per_wavefront(tmp_path):
    """Groups of 256 values: more than 224 and up to 256 codewords stay with the kernel for wide groups."""
    sizes = [(132, True), (224, True), (228, False), (256, False), (260, True), (320, True)]
    for (k, streamed), r in zip(sizes, record([dict(entry="encode", tokens=64, groups=16, words=k, d=4096) for k, _ in sizes], tmp_path)):
        assert kernels(r)[0].startswith("vq_encode_bf16_stream_kernel" if streamed else "vq_encode_bf16_wide_kernel"), (k, kernels(r))


def test_cut_walks_of_other_entry_points(tmp_path):
    """The shapes of the GPU tests: the layer that quantises K and V after projection, with both encodes aboard, and blocks."""
    from test_gpu_block import CUT as BLOCKS
    from test_gpu_kv_variant import CUT as KV
    common = dict(dh=128, hkv=4, causal=True, words=256, norm="rmsnorm", mlp="gelu_tanh", dff=256, rope=10000.0)
    calls = [dict(common, entry="kv", d=64 * h, hq=h, n_local=n // 16, n_nonlocal=n // 16 * 15, groups=8) for h, n in KV]
    calls += [dict(common, entry="block", d=64 * h, hq=h, n_local=n // d, n_nonlocal=n - n // d, groups=16) for h, n, d in BLOCKS]
    for aboard, c, r in zip((True, True, True, False), calls, record(calls, tmp_path)):
        assert any(k.startswith("attn_merge") for k in kernels(r)), (c, kernels(r))
        assert any(k.startswith("attn_cut_kernel<false, true") for k in kernels(r)) == aboard and not any("vq_encode" in k for k in kernels(r) if aboard), (c, kernels(r))


def test_rebuilt_rows_come_with_the_normalisation_of_wide_rows_too(tmp_path):
    call = dict(entry="block", d=1088, hq=4, hkv=2, dh=64, n_local=33, n_nonlocal=66, causal=True, norm="rmsnorm", mlp="gelu_tanh", dff=128, groups=16, words=256)
    assert kernels(record([call], tmp_path)[0])[0] == "norm_decode_kernel<unsigned char, false>"


def test_encode_bodies_of_wide_groups_by_codebook(tmp_path):
    """From 2^17 elements on, where score products were used, the norm is added to the finished sum (tests/test_gpu_vq.py)."""
    sizes = [(128, 1020, "_small"), (128, 1024, ""), (256, 508, "_small"), (256, 512, "")]
    for (dg, k, form), r in zip(sizes, record([dict(entry="encode", tokens=8200, groups=16, words=k, d=16 * dg) for dg, k, _ in sizes], tmp_path)):
        assert kernels(r) == [f"vq_encode_bf16_fast{dg}_kernel{form}"], (dg, k, kernels(r))


def test_encode_of_one_group_beside_many_rows(tmp_path):
    """A layer's single group has score products whatever its codebook's size; the body that replaces them for many rows adds the norm once, as they do."""
    common = dict(entry="layer", hkv=2, dh=64, groups=1, n_nonlocal=64)
    layers = [dict(common, d=dg, hq=dg // 64, words=k, n_local=t) for dg, k, t in ((128, 512, 4000), (128, 512, 12000), (256, 256, 17000))]
    for c, r, enc in zip(layers, record(layers, tmp_path), ("vq_argmin_scores_kernel", "vq_encode_bf16_fast128_kernel", "vq_encode_bf16_fast256_kernel")):
        assert [k.split("<")[0] for k in kernels(r) if k.startswith("vq_")] == [enc], (c, kernels(r))


def test_large_tiles_of_fp32_products_have_one_form(tmp_path):
    """Tiles of 64 hold too much for the form that copies its one problem's arguments."""
    call = dict(entry="block", dtype="f32", hq=1, hkv=1, dh=64, n_local=700, n_nonlocal=0, norm="layernorm", mlp="gelu_tanh", dff=64, groups=1, words=16)
    small, large = (kernels(r) for r in record([dict(call, d=192), dict(call, d=1536)], tmp_path))
    assert not any(k.startswith("gemm_f32_kernel<4") for k in small) and any(k.endswith(", true>") for k in small if k.startswith("gemm_f32")), small
    assert [k for k in large if k.startswith("gemm_f32_kernel<4")] == 2 * ["gemm_f32_kernel<4, false>"], large
