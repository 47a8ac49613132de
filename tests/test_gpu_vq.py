"""GPU parity: grouped VQ encode / decode through the C ABI against the CPU oracle on the same
seeded inputs.  Codes are bit-exact except at near-ties (oracle best/second-best gap < 1e-5
relative), which are counted; decode is bit-exact."""
import numpy as np
import pytest

import oracle
from paper_2505_19342_amd import workloads as wl

pytestmark = pytest.mark.gpu

NEAR_TIE = 1e-5


def make(seed, T, G, K, dg, dtype, dist="normal"):
    rng = np.random.default_rng(seed)
    x = wl._embeddings(rng, T, G * dg, dist) if T > 0 else np.zeros((0, G * dg), np.float32)
    cb = rng.standard_normal((G, K, dg), dtype=np.float32)
    if dtype == "bf16":
        x, cb = wl.round_to_bf16(x), wl.round_to_bf16(cb)
    return x, cb


ENCODE_CASES = [
    # (T, G, K, dg, dtype, dist)     spans several 128-token tiles and a ragged tail unless noted
    (64, 4, 256, 48, "f32", "normal"),            # tiny ViT layer
    (300, 4, 256, 48, "f32", "normal"),
    (33, 3, 1000, 20, "f32", "normal"),           # uint16 codes, K not a multiple of the wave
    (5, 2, 300, 132, "f32", "normal"),            # two chunks of 64 values and a piece, five tokens over blocks of four
    (6, 2, 70, 520, "f32", "normal"),
    (3, 4, 300, 7, "f32", "normal"),              # slices of no whole 16-byte pieces
    # fp32 forms: slices that wait in LDS whole and in stages, a token per wavefront out of LDS and without it; codebooks around a wavefront's and a workgroup's lanes
    (9, 2, 300, 1024, "f32", "normal"),           # one full stage
    (9, 1, 257, 1028, "f32", "normal"),           # a stage and a piece; two rounds of codewords
    (5, 1, 256, 1027, "f32", "normal"),           # the same value by value
    (6, 1, 129, 2048, "f32", "normal"),           # two full stages
    (7, 3, 64, 1040, "f32", "normal"),            # a token per wavefront, staged twice
    (7, 2, 16, 2050, "f32", "normal"),            # the same value by value, K of a quarter wavefront
    (600, 4, 32, 40, "f32", "normal"),            # 600 workgroups: shared
    (13, 4, 32, 40, "f32", "normal"),             # 16 workgroups: a token per wavefront
    (9, 3, 128, 12, "f32", "normal"),             # without LDS, two codewords per lane
    (9, 3, 129, 12, "f32", "normal"),             # one codeword too many for that
    (9, 5, 64, 32, "f32", "normal"),              # two chunks of 16 values
    (9, 5, 64, 29, "f32", "normal"),              # value by value
    (9, 5, 65, 36, "f32", "normal"),
    (2, 5, 33, 1, "f32", "normal"),               # a single value
    (256, 16, 256, 48, "bf16", "normal_shift"),   # ViT-Base
    (256, 32, 256, 24, "bf16", "student_t5"),     # GPT-2 small (dg padded to 32)
    (1024, 64, 1024, 64, "bf16", "rms_normal"),   # Llama-3-8B shape, full size
    (300, 16, 256, 48, "bf16", "normal"),         # ragged tail
    (1, 2, 16, 8, "bf16", "normal"),              # single token, K below one MFMA tile
    (130, 64, 16, 12, "bf16", "normal"),          # sweep corner: dg = 12 (unaligned slices), K = 16
    (200, 4, 1024, 192, "bf16", "normal"),        # sweep: dg spans 3 LDS tiles
    (140, 1, 1024, 768, "bf16", "normal"),        # vanilla VQ (G = 1), dg = 768
    (257, 5, 100, 40, "bf16", "normal"),          # K not a multiple of 32, dg not a multiple of 16
    # every contraction-step count of the fast body (dg <= 64), with and without the zero-filled odd piece, ragged K
    (200, 8, 512, 32, "bf16", "normal"),          # two steps, every slot transferred
    (150, 3, 260, 56, "bf16", "normal"),          # four steps, the last piece zero-filled; K = 2 tiles + 4 codewords
    (100, 5, 132, 16, "bf16", "normal"),          # one step; second tile holds 4 codewords
    (70, 2, 1024, 8, "bf16", "normal"),           # one step, upper half of it zero-filled
    # two token blocks per wavefront (256 items of 256 tokens or more): every contraction-step count, one to eight tiles, runs of several items
    (300, 128, 132, 8, "bf16", "normal"),
    (513, 128, 260, 24, "bf16", "student_t5"),
    (257, 200, 100, 40, "bf16", "normal"),
    (1100, 128, 1000, 64, "bf16", "rms_normal"),  # 640 items: runs of two, a group's last item next to the first of the next group
    (4500, 40, 600, 56, "bf16", "normal"),        # 720 items of five tiles, the last one of 88 codewords
    # wide groups (dg a multiple of 64 above 64): the kernel that streams both operands over dg
    (300, 1, 1024, 4096, "bf16", "rms_normal"),   # Llama width with the paper's G = 1; ragged token tail
    (1024, 2, 1024, 2048, "bf16", "rms_normal"),  # G = 2, full row count
    (37, 3, 1001, 128, "bf16", "normal"),         # K odd: scalar norm loads, last pass ragged against the 32-codeword blocks
    (65, 2, 2500, 320, "bf16", "normal"),         # three passes over the codewords, odd number of 64-chunks
    (5, 6, 16, 64 * 3, "bf16", "normal"),         # K below one block of a single wavefront
    # even slices that are no whole 16-byte pieces (tiles fetched as 32-bit words), and odd ones (value by value)
    (512, 64, 1024, 12, "bf16", "normal"),        # sweep corner at its largest codebook: 8 codeword tiles
    (130, 3, 300, 2, "bf16", "normal"),           # shortest even slice; K = 2 tiles + 44 codewords
    (77, 5, 129, 6, "bf16", "normal"),            # second tile holds one codeword
    (140, 2, 520, 62, "bf16", "normal"),          # longest such slice: the last thread pass of a tile is ragged
    (90, 4, 257, 36, "bf16", "student_t5"),       # three contraction steps, the third partly padding
    (60, 7, 200, 20, "bf16", "normal"),           # 140 values per row: rows are not 16-byte multiples
    (50, 3, 150, 7, "bf16", "normal"),            # odd slice length
    (40, 1, 300, 33, "bf16", "normal"),           # odd, three contraction steps
]


@pytest.mark.parametrize("T,G,K,dg,dtype,dist", ENCODE_CASES)
def test_encode_matches_oracle(T, G, K, dg, dtype, dist):
    from gpu_util import compare_codes, gpu_vq_encode
    x, cb = make(100 + T + G, T, G, K, dg, dtype, dist)
    ref, gap = oracle.vq_encode(x, cb, return_gap=True)
    got = gpu_vq_encode(x, cb, dtype)
    n_tie = compare_codes(got, ref, gap, NEAR_TIE)
    print(f"near-tie disagreements: {n_tie} of {ref.size}")
    assert n_tie <= max(2, ref.size // 2000)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_encode_codewords_and_exact_ties(dtype):
    from gpu_util import gpu_vq_decode, gpu_vq_encode
    rng = np.random.default_rng(7)
    G, K, dg = 3, 64, 16
    cb = rng.standard_normal((G, K, dg), dtype=np.float32)
    if dtype == "bf16":
        cb = wl.round_to_bf16(cb)
    cb[:, 40] = cb[:, 7]                       # duplicate codeword: 7 must win over 40
    x = np.concatenate([cb[g] for g in range(G)], axis=1)
    got = gpu_vq_encode(x, cb, dtype)
    expect = np.repeat(np.arange(K)[:, None], G, axis=1)
    expect[40] = 7
    assert np.array_equal(got, expect)
    assert np.array_equal(got, oracle.vq_encode(x, cb))
    assert np.array_equal(gpu_vq_decode(got, cb, dtype), x)          # decode(encode(c)) == c


@pytest.mark.parametrize("T,G", [(40, 3), (300, 130)])          # one token block per wavefront, two
def test_encode_ties_wherever_they_lie(T, G):
    """Equal codewords in one quad, in the two halves of a wavefront, in other blocks and tiles: the lowest index wins; and a codebook of equal codewords."""
    from gpu_util import gpu_vq_encode
    rng = np.random.default_rng(11)
    K, dg = 300, 16
    cb = wl.round_to_bf16(rng.standard_normal((G, K, dg), dtype=np.float32))
    sets = [(5, 6, 7), (1, 12), (9, 13, 41), (100, 101, 131, 299), (250, 251)]
    for s in sets:
        cb[:, list(s)] = cb[:, s[:1]]
    pick = rng.choice([i for s in sets for i in s], size=(T, G))
    x = cb[np.arange(G)[None], pick].reshape(T, G * dg)
    first = {i: s[0] for s in sets for i in s}
    assert np.array_equal(gpu_vq_encode(x, cb, "bf16"), np.vectorize(first.get)(pick))
    cb[:] = cb[:, :1]
    assert not gpu_vq_encode(x, cb, "bf16").any()


@pytest.mark.parametrize("T,G,K,dg", [(300, 1, 1024, 4096), (257, 2, 1000, 384), (100, 7, 1024, 128), (64, 4, 16, 192), (33, 16, 256, 48)])
def test_encode_with_workspace_matches_oracle_and_the_plain_entry_point(T, G, K, dg):
    """astra_vq_encode_ws: wide groups run as score products + an argmin pass (seven groups: two launches of products);
    the last two shapes (a small codebook per group, narrow groups) must fall through to astra_vq_encode's kernels."""
    import torch
    from gpu_util import DEV, codes_to_host, compare_codes, empty_codes, gpu_vq_encode, to_dev
    from paper_2505_19342_amd import binding as B
    x, cb = make(300 + T + G, T, G, K, dg, "bf16", "normal")
    ref, gap = oracle.vq_encode(x, cb, return_gap=True)
    desc = B.vq_desc("bf16", G * dg, G, K)
    cbd, xd = to_dev(cb, "bf16"), to_dev(x, "bf16")
    cnorm = torch.empty((G, K), dtype=torch.float32, device=DEV)
    B.astra_vq_prepare(desc, cbd, cnorm)
    need = B.astra_vq_encode_workspace_bytes(desc, T)
    uses_ws = dg % 64 == 0 and dg > 64 and K * dg >= 1 << 17
    assert need >= (T * G * K * 4 if uses_ws else 256)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    codes = empty_codes(T, G, K)
    B.astra_vq_encode_ws(desc, xd, T, cbd, cnorm, codes, ws)
    torch.cuda.synchronize()
    got = codes_to_host(codes, K)
    n_tie = compare_codes(got, ref, gap, NEAR_TIE)
    assert n_tie <= max(2, ref.size // 2000)
    plain = gpu_vq_encode(x, cb, "bf16")
    assert (got != plain).sum() <= max(2, ref.size // 2000)        # both obey the near-tie rule; they may differ only there
    if uses_ws:
        with pytest.raises(B.AstraError, match="workspace"):
            B.astra_vq_encode_ws(desc, xd, T, cbd, cnorm, codes, torch.empty(256, dtype=torch.uint8, device=DEV))


def test_wide_group_encodes_on_seeded_random_shapes():
    """Twelve seeded shapes with wide groups (token counts, codebook sizes and group widths that are multiples of nothing
    in particular beyond what the kernels need): astra_vq_encode and astra_vq_encode_ws against the oracle."""
    import torch
    from gpu_util import DEV, codes_to_host, compare_codes, empty_codes, gpu_vq_encode, to_dev
    from paper_2505_19342_amd import binding as B
    rng = np.random.default_rng(2024)
    for case in range(12):
        T = int(rng.integers(1, 400))
        G = int(rng.integers(1, 5))
        dg = 64 * int(rng.integers(2, 9))
        K = 8 * int(rng.integers(1, 330))
        x, cb = make(900 + case, T, G, K, dg, "bf16", "normal")
        ref, gap = oracle.vq_encode(x, cb, return_gap=True)
        got = gpu_vq_encode(x, cb, "bf16")
        compare_codes(got, ref, gap, NEAR_TIE)
        desc = B.vq_desc("bf16", G * dg, G, K)
        cbd, xd = to_dev(cb, "bf16"), to_dev(x, "bf16")
        cnorm = torch.empty((G, K), dtype=torch.float32, device=DEV)
        B.astra_vq_prepare(desc, cbd, cnorm)
        ws = torch.empty(B.astra_vq_encode_workspace_bytes(desc, T), dtype=torch.uint8, device=DEV)
        codes = empty_codes(T, G, K)
        B.astra_vq_encode_ws(desc, xd, T, cbd, cnorm, codes, ws)
        torch.cuda.synchronize()
        n_tie = compare_codes(codes_to_host(codes, K), ref, gap, NEAR_TIE)
        print(f"case {case}: T {T} G {G} K {K} dg {dg}: ok ({n_tie} near-ties)")


def test_wide_group_encode_exact_ties_across_wavefronts_and_passes():
    """Duplicate codewords that land in different half-waves, wavefronts and passes of the wide-group kernel: the lowest
    index must win every time."""
    from gpu_util import gpu_vq_encode
    rng = np.random.default_rng(17)
    G, K, dg = 2, 2304, 128
    cb = wl.round_to_bf16(rng.standard_normal((G, K, dg), dtype=np.float32))
    dup = {5: 4, 200: 9, 1030: 3, 2050: 1029, 2303: 131, 36: 32}        # later index -> the earlier codeword it copies
    for later, first in dup.items():
        cb[:, later] = cb[:, first]
    x = np.concatenate([cb[g] for g in range(G)], axis=1)                   # token k is codeword k in both groups
    got = gpu_vq_encode(x, cb, "bf16")
    expect = np.repeat(np.arange(K)[:, None], G, axis=1)
    for later, first in dup.items():
        expect[later] = first
    assert np.array_equal(got, expect)
    assert np.array_equal(got, oracle.vq_encode(x, cb))


def test_f32_encode_of_long_slices_keeps_pace():
    """500 tokens of 768 values against 1024 codewords take about as long as one group as they do as two: 91 us and 49.  (Longer slices were once read
    value by value from memory, 438 us and 51.)"""
    import torch
    from gpu_util import DEV
    from paper_2505_19342_amd import binding as B
    took = []
    for groups in (1, 2):
        x, cb = torch.randn(500, 768, device=DEV), torch.randn(groups, 1024, 768 // groups, device=DEV)
        desc = B.vq_desc("f32", 768, groups, 1024)
        codes, cnorm = torch.empty(500, groups, dtype=torch.int16, device=DEV), torch.empty(groups, 1024, device=DEV)
        times = []
        for _ in range(6):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(10):
                B.astra_vq_encode(desc, x, 500, cb, cnorm, codes)
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end))
        took.append(min(times))
    assert took[0] < 4 * took[1], took


DECODE_CASES = [(192, 4, 256, 48, "f32"), (768, 16, 256, 48, "bf16"), (777, 32, 256, 24, "bf16"),
                (3072, 64, 1024, 64, "bf16"), (50, 64, 16, 12, "bf16"), (9, 3, 5, 7, "bf16"), (11, 2, 300, 5, "f32")]


@pytest.mark.parametrize("T,G,K,dg,dtype", DECODE_CASES)
def test_decode_is_bit_exact(T, G, K, dg, dtype):
    from gpu_util import gpu_vq_decode
    rng = np.random.default_rng(T)
    cb = rng.standard_normal((G, K, dg), dtype=np.float32)
    if dtype == "bf16":
        cb = wl.round_to_bf16(cb)
    codes = rng.integers(0, K, size=(T, G)).astype(np.int32)
    codes[0, :] = K - 1
    codes[-1, :] = 0
    got = gpu_vq_decode(codes, cb, dtype)
    assert np.array_equal(got.view(np.uint32), oracle.vq_decode(codes, cb).view(np.uint32))


def test_empty_inputs_and_argument_errors():
    import torch
    from gpu_util import DEV, gpu_vq_decode, gpu_vq_encode, to_dev
    from paper_2505_19342_amd import binding as B
    cb = np.ones((2, 4, 8), dtype=np.float32)
    assert gpu_vq_encode(np.zeros((0, 16), np.float32), cb, "bf16").shape == (0, 2)
    assert gpu_vq_decode(np.zeros((0, 2), np.int32), cb, "bf16").shape == (0, 16)
    cbd = to_dev(cb, "bf16")
    cn = torch.empty((2, 4), dtype=torch.float32, device=DEV)
    with pytest.raises(B.AstraError):      # G does not divide D
        B.astra_vq_prepare(B.VqDesc(B.ASTRA_BF16, B.ASTRA_CODE_U8, 16, 3, 4), cbd, cn)
    with pytest.raises(B.AstraError):      # uint8 codes cannot hold K = 1024
        B.astra_vq_prepare(B.VqDesc(B.ASTRA_BF16, B.ASTRA_CODE_U8, 16, 2, 1024), cbd, cn)
    with pytest.raises(B.AstraError):      # NULL output
        B.astra_vq_prepare(B.vq_desc("bf16", 16, 2, 4), cbd, None)


@pytest.mark.parametrize("T,G,K", [(257, 32, 1024), (4100, 2, 100), (300, 28, 4), (520, 17, 68), (2100, 64, 64), (600, 32, 256)])
def test_groups_of_128_values(T, G, K):
    """64 tokens per wavefront on tiles of 64 codewords (tests/test_launches.py): ragged tiles and token blocks, a codebook of one quad, a single tile, 8- and
    16-bit codes, workgroups of more than one item whose next tokens are of the next group."""
    from gpu_util import compare_codes, gpu_vq_encode
    x, cb = make(40 + T + G, T, G, K, 128, "bf16", "normal")
    ref, gap = oracle.vq_encode(x, cb, return_gap=True)
    n_tie = compare_codes(gpu_vq_encode(x, cb, "bf16"), ref, gap, NEAR_TIE)
    assert n_tie <= max(2, ref.size // 2000)
    cb[:, K // 2:] = cb[:, :K // 2]                          # every codeword twice: the lower one
    assert gpu_vq_encode(x, cb, "bf16").max() < K // 2


@pytest.mark.parametrize("T,G,K", [(513, 16, 1024), (4100, 2, 100), (300, 28, 4), (520, 17, 68), (1100, 40, 64), (700, 16, 256)])
def test_groups_of_256_values(T, G, K):
    """32 tokens per wavefront, half a unit's codeword fragments held (tests/test_launches.py): the edges of the groups of 128 above."""
    from gpu_util import compare_codes, gpu_vq_encode
    x, cb = make(60 + T + G, T, G, K, 256, "bf16", "normal")
    ref, gap = oracle.vq_encode(x, cb, return_gap=True)
    n_tie = compare_codes(gpu_vq_encode(x, cb, "bf16"), ref, gap, NEAR_TIE)
    assert n_tie <= max(2, ref.size // 2000)
    cb[:, K // 2:] = cb[:, :K // 2]                          # every codeword twice: the lower one
    assert gpu_vq_encode(x, cb, "bf16").max() < K // 2


@pytest.mark.parametrize("dg", [128, 192, 256])
@pytest.mark.parametrize("T,G,K", [(17, 32, 1024), (512, 16, 1024), (33, 7, 4), (700, 20, 32), (100, 9, 100), (64, 3, 260), (300, 13, 2052)])
def test_streamed_wide_groups(T, G, K, dg):
    """32 tokens per workgroup, codewords dealt to eight wavefronts in blocks of 32: fewer blocks than wavefronts, ragged blocks, more than a ring of steps."""
    from gpu_util import compare_codes, gpu_vq_encode
    x, cb = make(70 + T + G + dg, T, G, K, dg, "bf16", "normal")
    ref, gap = oracle.vq_encode(x, cb, return_gap=True)
    n_tie = compare_codes(gpu_vq_encode(x, cb, "bf16"), ref, gap, NEAR_TIE)
    assert n_tie <= max(2, ref.size // 2000)
    cb[:, K // 2:] = cb[:, :K // 2]                          # every codeword twice: the lower one
    assert gpu_vq_encode(x, cb, "bf16").max() < K // 2


def distances_of_few_units(T, G, K, dg):
    """Codewords of one norm n, and products with x that move the nearest by 1.5 or 3 units in the last place of n, a quarter of one per 16 values: added to n
    one by one the quarters would be lost and the lowest code win.  The nearest to the even tokens is K - 1, to the odd ones K - 2."""
    n = dg if dg == 192 else 3 * dg // 4                       # 96 or 192, halfway between two powers of two
    x = np.zeros((T, G, dg), np.float32)
    x[:, :, :n] = 2.0 ** (np.floor(np.log2(n)) - 23) / 128
    x[1::2] *= -1.0
    rng = np.random.default_rng(91)
    half = np.repeat([1.0, -1.0], n // 2).astype(np.float32)
    cb = np.zeros((G, K, dg), np.float32)
    cb[:, :, :n] = rng.permuted(np.broadcast_to(half, (G, K, n)), axis=2)                   # x.c = 0
    cb[:, K - 1, :n], cb[:, K - 2, :n] = 1.0, -1.0
    return x.reshape(T, -1), cb


@pytest.mark.parametrize("T,G,K,dg", [(40, 7, 1024, 128), (40, 7, 1024, 192), (40, 16, 1024, 256), (8200, 2, 1024, 128), (8200, 2, 512, 256)])
def test_distances_of_wide_groups_are_rounded_once(T, G, K, dg):
    """-2 x.c is summed by itself and the norm added once.  Streamed encodes, and both forms of the matrix-core body (vq_encode_fast_wide) for codebooks of 2^17
    elements, whose score products they stand in for."""
    from gpu_util import gpu_vq_encode
    x, cb = distances_of_few_units(T, G, K, dg)
    codes = gpu_vq_encode(x, cb, "bf16")
    assert (codes[0::2] == K - 1).all() and (codes[1::2] == K - 2).all()


@pytest.mark.parametrize("T,K,D", [(4000, 512, 128), (12000, 512, 128), (17000, 256, 256)])
def test_distances_of_one_group_in_a_layer_are_rounded_once(T, K, D):
    """A codebook of any size: by score products, and by the bodies that stand in for them beside many rows (as tests/test_launches.py checks)."""
    from gpu_util import LayerOnGpu
    cfg = wl.LayerConfig("one_group", "bf16", D, D // 64, 2, 64, T, 1, 1, K)
    x, cb = distances_of_few_units(T, 1, K, D)
    rng = np.random.default_rng(92)
    data = {n: wl.round_to_bf16(rng.standard_normal((D, 128 if n in ("wk", "wv") else D), dtype=np.float32)) for n in ("wq", "wk", "wv", "wo")}
    layer = LayerOnGpu(cfg, dict(data, codebook=cb), x, np.zeros((0, 1), np.int64), 0)
    layer.run()
    codes = layer.results()[1]
    assert (codes[0::2] == K - 1).all() and (codes[1::2] == K - 2).all()
