"""What the host code launches, without a GPU: the library on top of a recorder in the place of the HIP runtime (launch_record.py)."""
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
