"""GPU parity of the bf16 product behind the projections, at the edges of its forms: astra_vq_project_codebook with one group is a plain
C = A . B^T with fp32 output.  Bar: fp32 sums of exact bf16 products in another order, 1e-5 of the largest sum of magnitudes."""
import numpy as np
import pytest

from paper_2505_19342_amd import workloads as wl

pytestmark = pytest.mark.gpu


# rows, columns, contraction, the form that runs them: wave<row tiles of 32, column tiles, stages> or tile<rows, columns> (tests/test_launches.py
# checks that they do)
PRODUCTS = [
    (4, 8, 64, "wave<1, 1, 2>"),            # one contraction slice: three of the four wavefronts of a workgroup have none
    (32, 32, 256, "wave<1, 1, 2>"),         # one tile, one slice per wavefront
    (33, 40, 320, "wave<1, 1, 2>"),         # one row and eight columns beyond a tile, five slices over four wavefronts
    (60, 768, 768, "wave<1, 1, 2>"),        # ring of two stages, three slices per wavefront
    (260, 1032, 192, "wave<1, 1, 2>"),      # several column tiles, the last one of eight columns
    (100, 2056, 576, "wave<2, 1, 2>"),      # nine slices over four wavefronts, four rows beyond a tile
    (228, 2056, 64, "wave<2, 2, 2>"),
    (256, 4096, 1024, "wave<2, 2, 2>"),
    (516, 2056, 64, "wave<2, 2, 1>"),       # two workgroups per unit
    (228, 4104, 2112, "wave<4, 2, 1>"),
    (1028, 2056, 2112, "wave<4, 4, 1>"),    # 33 slices, the reduction in four passes
    (1028, 2056, 64, "tile<128, 128>"),     # a loop that is all prologue and tail
    (516, 4096, 512, "tile<128, 128>"),
    (1024, 4096, 576, "tile<128, 128>"),
    (1028, 4104, 64, "tile<128, 256>"),
    (2052, 4104, 64, "tile<256, 256>"),
    # slices in halves: four to seven per wavefront (prologue, pairs in steady state, one to three in the tail), and one more for some of them
    *[(252, 8312, k, "wave<4, 4, 1>") for k in (1024, 1280, 1536, 1600, 1664, 1728, 1792)],
    # the loop in halves: two tiles of 64 (no more than the prologue fetches), three to seven (its steady part comes from four on, two at a time)
    *[(1028, 4104, k, "tile<128, 256>") for k in (128, 192, 256, 320, 448)],
    *[(2052, 4104, k, "tile<256, 256>") for k in (128, 192, 256, 320, 448)],
]


@pytest.mark.parametrize("m,n,k,form", PRODUCTS)
def test_product_forms(m, n, k, form):
    import torch
    from gpu_util import to_dev, to_host, DEV
    from paper_2505_19342_amd import binding as B
    rng = np.random.default_rng(m + n + k)
    a = wl.round_to_bf16(rng.standard_normal((m, k), dtype=np.float32))
    b = wl.round_to_bf16(rng.standard_normal((n, k), dtype=np.float32))
    out = torch.full((1, m, n), float("nan"), dtype=torch.float32, device=DEV)
    B.astra_vq_project_codebook(B.vq_desc("bf16", k, 1, m), to_dev(a[None], "bf16"), to_dev(b, "bf16"), n, out)
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    scale = (np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64).T).max()
    assert np.abs(to_host(out)[0] - ref).max() <= 1e-5 * scale


@pytest.mark.parametrize("m,n,k", [(1, 8, 1), (17, 24, 7), (33, 40, 16), (64, 192, 192), (50, 72, 1028), (250, 584, 100), (500, 520, 66), (900, 840, 130)])
def test_f32_product(m, n, k):
    """Tiles of 16, 32 and 64, contractions of part of a slice, of no whole 16-byte pieces, and of several rounds of slices.  Bar: 2 sqrt(k) roundings of 2^-24
    of the sum of magnitudes (each of the k products and sums may round; their errors add as a random walk)."""
    import torch
    from gpu_util import to_dev, to_host, DEV
    from paper_2505_19342_amd import binding as B
    rng = np.random.default_rng(m + n + k)
    a, b = rng.standard_normal((m, k), dtype=np.float32), rng.standard_normal((n, k), dtype=np.float32)
    out = torch.full((1, m, n), float("nan"), dtype=torch.float32, device=DEV)
    B.astra_vq_project_codebook(B.vq_desc("f32", k, 1, m), to_dev(a[None], "f32"), to_dev(b, "f32"), n, out)
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    scale = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64).T
    assert np.all(np.abs(to_host(out)[0] - ref) <= 2 * np.sqrt(k) * 2.0 ** -24 * scale)
