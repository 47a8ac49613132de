"""GPU parity: the whole per-device layer (encode + decode + projections + mixed-precision attention +
output projection) through astra_layer_forward against the CPU oracle, on the seeded workloads.
Bars: codes bit-exact except counted near-ties (oracle gap < 1e-5 relative); layer output max-abs
<= 1e-4 (fp32) / 2e-2 (bf16)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2505_19342_amd import workloads as wl

pytestmark = pytest.mark.gpu

Y_TOL = {"f32": 1e-4, "bf16": 2e-2}
NEAR_TIE = 1e-5


def run_case(cfg, rank, biases=False):
    from gpu_util import LayerOnGpu, compare_codes
    data = wl.generate(cfg)
    view = wl.device_view(cfg, data, rank)
    codes_nl = oracle.vq_encode(view["x_nonlocal"], data["codebook"])       # what the peers would have sent
    b = None
    if biases:
        rng = np.random.default_rng(99)
        dq, dkv = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
        b = [(0.1 * rng.standard_normal(n)).astype(np.float32) for n in (dq, dkv, dkv, cfg.d_model)]
        if cfg.dtype == "bf16":
            b = [wl.round_to_bf16(v) for v in b]
    kw = {} if b is None else dict(bq=b[0], bk=b[1], bv=b[2], bo=b[3])
    y_ref, codes_ref, gap = oracle.layer_forward(
        view["x_local"], codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"], data["wo"],
        n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads, n_cls=cfg.n_cls, causal=cfg.causal,
        n_before=view["n_before"], return_gap=True, **kw)
    layer = LayerOnGpu(cfg, data, view["x_local"], codes_nl, view["n_before"], biases=b)
    layer.run()
    y, codes = layer.results()
    n_tie = compare_codes(codes, codes_ref, gap, NEAR_TIE)
    err = np.abs(y - y_ref).max()
    print(f"{cfg.name} rank {rank}: max abs err {err:.3e} (|y| max {np.abs(y_ref).max():.3f}), near-tie codes {n_tie}/{codes.size}")
    assert err <= Y_TOL[cfg.dtype]
    assert n_tie <= max(2, codes.size // 2000)
    return err


@pytest.mark.parametrize("rank", [0, 1, 3])
def test_tiny_vit_f32(rank):
    run_case(wl.TINY_VIT, rank)


@pytest.mark.parametrize("rank", [0, 3])
def test_vit_base_bf16_with_class_row(rank):
    run_case(wl.VIT_BASE, rank)


@pytest.mark.parametrize("rank", [0, 2, 3])
def test_gpt2_small_bf16_causal(rank):
    run_case(wl.GPT2_SMALL, rank)


def test_biases_f32_and_bf16():
    run_case(wl.TINY_VIT, 1, biases=True)
    run_case(wl.VIT_BASE, 1, biases=True)


def test_f32_launches_of_large_and_small_tiles():
    """The fp32 product runs on the largest of 64 x 64, 32 x 32 and 16 x 16 tiles of which a launch has 192 (the tiny shape: the smallest): a
    longer sequence with ragged rows takes the large ones for the projections and, with two heads of 96, output values
    beyond the first 64 lanes in the attention."""
    cfg = dataclasses.replace(wl.TINY_VIT, name="f32_long", seq_len=1500, n_q_heads=2, n_kv_heads=2, head_dim=96, seed=17)
    run_case(cfg, 1, biases=True)


@pytest.mark.parametrize("groups,words,seq_len", [(32, 300, 256), (64, 256, 300), (96, 16, 1100)])
def test_f32_rows_gathered_value_by_value(groups, words, seq_len):
    """fp32 products whose gathered slices (6, 3 and 2 values) are no whole 16-byte pieces, on tiles of 16 to 64."""
    run_case(dataclasses.replace(wl.TINY_VIT, name="f32_gather", n_groups=groups, codebook_size=words, seq_len=seq_len, seed=18), 1, biases=True)


@pytest.mark.parametrize("i_dev", [0, 1, 2])
@pytest.mark.parametrize("i_k", [0, 1, 2])
@pytest.mark.parametrize("i_g", [0, 1, 2, 3])
def test_sweep_points(i_g, i_k, i_dev):
    """Every point of the sweep on the ViT-Base shape: G in {1, 4, 16, 64} x K in {16, 256, 1024} x {2, 4, 8} devices
    (group widths 768, 192, 48 and 12: the last is not a multiple of the 16-byte operand piece, so the peers' rows are
    rebuilt by the decode kernel instead of inside the projection's operand loader)."""
    cfg = wl.sweep_config(i_g, i_k, i_dev)
    run_case(cfg, cfg.n_dev - 1 if i_g == i_k else 1)


def test_uneven_split_and_ragged_shapes():
    # a device holding 100 of 420 tokens: nothing in the ABI assumes an even split
    from gpu_util import LayerOnGpu, compare_codes
    cfg = dataclasses.replace(wl.GPT2_SMALL, name="uneven", seq_len=420, seed=77)
    data = wl.generate(cfg)
    lo, hi = 130, 230
    x_local = data["x"][lo:hi]
    x_nl = np.concatenate([data["x"][:lo], data["x"][hi:]])
    codes_nl = oracle.vq_encode(x_nl, data["codebook"])
    y_ref, codes_ref, gap = oracle.layer_forward(x_local, codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"],
                                                 data["wo"], n_q_heads=12, n_kv_heads=12, causal=True, n_before=lo,
                                                 return_gap=True)
    layer = LayerOnGpu(cfg, data, x_local, codes_nl, lo)
    layer.run()
    y, codes = layer.results()
    compare_codes(codes, codes_ref, gap, NEAR_TIE)
    assert np.abs(y - y_ref).max() <= Y_TOL["bf16"]


@pytest.mark.parametrize("rank", [3, 0])
def test_llama3_8b_shape_full_size(rank):
    """The benchmark workload at full size, same launch configuration as bench.py times."""
    run_case(wl.LLAMA3_8B, rank)


@pytest.mark.parametrize("seq_len,lo,fused", [(3917, 2917, True), (1000, 0, True), (1900, 900, False), (5100, 3070, False)])
def test_llama_dims_ragged_rows_in_every_projection_tile_shape(seq_len, lo, fused):
    """Llama-3-8B widths with row counts that are multiples of nothing: the last seq_len - lo tokens on this device,
    so the last tile of every projection and the last token block of the encode are ragged.  The cases take the
    launch shapes of the projections: 256x256 tiles with the encode on the units left over (the configuration
    bench.py times), 192 tiles of 128x256 with the encode on the units left over (no visible peers), 256 tiles of
    128x256 that fill the chip (the attention launch then takes the encode), and 288 tiles of 256x256, which are dealt
    into two launches (one of 256x256 tiles that fills its round, one on smaller tiles)."""
    from gpu_util import LayerOnGpu, compare_codes
    from paper_2505_19342_amd import binding as B
    cfg = dataclasses.replace(wl.LLAMA3_8B, name="llama_ragged", seq_len=seq_len, seed=41)
    data = wl.generate(cfg)
    x_local, x_nl = data["x"][lo:], data["x"][:lo]
    codes_nl = oracle.vq_encode(x_nl, data["codebook"])
    y_ref, codes_ref, gap = oracle.layer_forward(x_local, codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"],
                                                 data["wo"], n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads, causal=True,
                                                 n_before=lo, return_gap=True)
    layer = LayerOnGpu(cfg, data, x_local, codes_nl, lo)
    assert B.astra_layer_encode_fused(layer.desc) == fused
    layer.run()
    y, codes = layer.results()
    n_tie = compare_codes(codes, codes_ref, gap, NEAR_TIE)
    err = np.abs(y - y_ref).max()
    print(f"llama dims, {seq_len - lo} local / {lo} non-local rows: max abs err {err:.3e}, near-tie codes {n_tie}/{codes.size}")
    assert err <= Y_TOL["bf16"]
    assert n_tie <= max(2, codes.size // 2000)


# width, local rows, visible peer rows, groups, codewords, and the form of the projection launch (GATHER: the peers' rows from their codes; ENC: with
# the encode), as tests/test_launches.py checks
MODEL_OF_WIDTH = {256: (4, 2, 64), 320: (5, 5, 64), 512: (4, 2, 128), 640: (10, 10, 64), 768: (12, 12, 64), 1024: (8, 8, 128), 2048: (16, 4, 128), 4096: (32, 8, 128)}
PROJECTION_LAUNCHES = [
    (256, 36, 14, 4, 16, "wave<1, 1, 2> GATHER ENC"),
    (512, 27, 6, 4, 256, "wave<1, 1, 2> GATHER"),
    (768, 104, 0, 64, 16, "wave<2, 1, 2>"),
    (768, 108, 0, 32, 256, "wave<2, 1, 2> ENC"),
    (256, 865, 95, 16, 16, "wave<2, 2, 1> GATHER ENC"),
    (768, 153, 70, 8, 16, "wave<2, 2, 1> GATHER"),
    (256, 802, 425, 4, 1024, "wave<2, 2, 2> GATHER ENC"),        # 16-bit codes
    (2048, 116, 140, 32, 256, "wave<2, 2, 2> GATHER"),
    (4096, 131, 0, 8, 1024, "wave<4, 2, 1>"),
    (768, 834, 0, 32, 16, "wave<4, 2, 1> ENC"),
    (768, 733, 0, 16, 1024, "wave<4, 4, 1> ENC"),
    (768, 590, 197, 16, 1024, "wave<4, 4, 1> GATHER ENC"),
    (2048, 1015, 25, 16, 16, "wave<4, 4, 1> GATHER"),
    (256, 3401, 0, 8, 256, "wave<4, 4, 1> ENC"),                 # one slice of 64 per wavefront
    (320, 1673, 500, 8, 256, "wave<4, 4, 1> GATHER ENC"),        # two for the first
    (512, 1675, 200, 8, 256, "wave<4, 4, 1> GATHER ENC"),        # two
    (640, 627, 500, 16, 1024, "wave<4, 4, 1> GATHER ENC"),       # three and two
    (512, 925, 180, 8, 1024, "tile<128, 128> GATHER"),
]


@pytest.mark.parametrize("d,n_local,n_nonlocal,groups,words,form", PROJECTION_LAUNCHES)
def test_projection_launches_with_ragged_rows(d, n_local, n_nonlocal, groups, words, form):
    """Every form of the projection launch on rows that end inside a tile, causal, with biases: stores to rows and to the transposed V, gathered
    rows, the encode alongside."""
    from gpu_util import LayerOnGpu, compare_codes
    hq, hkv, dh = MODEL_OF_WIDTH[d]
    cfg = wl.LayerConfig("forms", "bf16", d, hq, hkv, dh, n_local + n_nonlocal, 1, groups, words, causal=True, seed=61)
    data = wl.generate(cfg)
    rng = np.random.default_rng(62)
    b = [wl.round_to_bf16((0.1 * rng.standard_normal(n)).astype(np.float32)) for n in (hq * dh, hkv * dh, hkv * dh, d)]
    x_nl, x_local = data["x"][:n_nonlocal], data["x"][n_nonlocal:]
    codes_nl = oracle.vq_encode(x_nl, data["codebook"])
    y_ref, codes_ref, gap = oracle.layer_forward(x_local, codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"], data["wo"],
                                                 n_q_heads=hq, n_kv_heads=hkv, causal=True, n_before=n_nonlocal, return_gap=True,
                                                 bq=b[0], bk=b[1], bv=b[2], bo=b[3])
    layer = LayerOnGpu(cfg, data, x_local, codes_nl, n_nonlocal, biases=b)
    layer.run()
    y, codes = layer.results()
    n_tie = compare_codes(codes, codes_ref, gap, NEAR_TIE)
    assert np.abs(y - y_ref).max() <= Y_TOL["bf16"]
    assert n_tie <= max(2, codes.size // 2000)


@pytest.mark.parametrize("d,hq,hkv,dh,groups,words,n_local,n_nonlocal", [
    (768, 12, 12, 64, 16, 256, 100, 20),         # the peers' rows end inside a tile, and the padding after them has a tile of its own
    (768, 12, 12, 64, 16, 256, 256, 777),
    (4096, 32, 8, 128, 64, 1024, 40, 100),       # 16-bit codes
    (4096, 32, 8, 128, 64, 1024, 150, 449),      # tiles of 128 rows
    (4096, 32, 8, 128, 64, 1024, 1000, 2917),    # the large tiles
])
def test_codewords_that_no_code_names_do_not_matter(d, hq, hkv, dh, groups, words, n_local, n_nonlocal):
    """Three codewords of a group are used, the others are NaN in one call and finite in the other: the same output, bit for bit.
    (Rows beyond the peers' last token pad the transposed V; their weight is zero, but zero times a NaN is not.)"""
    import torch
    from gpu_util import LayerOnGpu
    cfg = wl.LayerConfig("unused", "bf16", d, hq, hkv, dh, n_local + n_nonlocal, 2, groups, words, seed=51)
    data = wl.generate(cfg)
    codes_nl = np.random.default_rng(52).integers(0, 3, (n_nonlocal, groups)).astype(np.int32)
    y = []
    for fill in (float("nan"), 0.5):
        layer = LayerOnGpu(cfg, data, data["x"][:n_local], codes_nl, 0)
        layer.codebook[:, 3:] = fill
        layer.run()
        torch.cuda.synchronize()
        y.append(layer.y)
    assert bool(torch.isfinite(y[1]).all()) and torch.equal(y[0], y[1])


def test_fused_encode_equals_the_standalone_encode_and_calls_repeat_bit_exactly():
    """The encode inside the projection launch and astra_vq_encode run the same arithmetic in the same order: equal codes,
    bit for bit.  Two calls of the layer, and the call with stage events, give identical bits too."""
    import torch
    from gpu_util import LayerOnGpu, empty_codes
    from paper_2505_19342_amd import binding as B
    cfg = wl.LLAMA3_8B
    data = wl.generate(cfg)
    view = wl.device_view(cfg, data, 2)
    codes_nl = oracle.vq_encode(view["x_nonlocal"], data["codebook"])
    layer = LayerOnGpu(cfg, data, view["x_local"], codes_nl, view["n_before"])
    assert B.astra_layer_encode_fused(layer.desc)
    layer.run()
    torch.cuda.synchronize()
    y1, c1 = layer.y.clone(), layer.codes_local.clone()
    alone = empty_codes(cfg.n_local, cfg.n_groups, cfg.codebook_size)
    B.astra_vq_encode(layer.desc.vq, layer.x_local, cfg.n_local, layer.codebook, layer.cnorm, alone)
    torch.cuda.synchronize()
    assert torch.equal(alone, c1)
    layer.y.zero_()
    layer.codes_local.zero_()
    layer.run()
    torch.cuda.synchronize()
    assert torch.equal(layer.y, y1) and torch.equal(layer.codes_local, c1)
    layer.y.zero_()
    layer.codes_local.zero_()
    ev = B.HipEvents(7)
    B.astra_layer_forward_profiled(layer.desc, layer.x_local, layer.codes_nonlocal, layer.codebook, layer.cnorm, *layer.w,
                                   *layer.b, layer.y, layer.codes_local, layer.workspace, ev.handles)
    torch.cuda.synchronize()
    assert torch.equal(layer.y, y1) and torch.equal(layer.codes_local, c1)
    assert ev.elapsed_ms(0, 4) > 0


def test_workspace_too_small_is_an_error():
    import torch
    from gpu_util import DEV, LayerOnGpu
    from paper_2505_19342_amd import binding as B
    cfg = wl.TINY_VIT
    data = wl.generate(cfg)
    view = wl.device_view(cfg, data, 0)
    layer = LayerOnGpu(cfg, data, view["x_local"], np.zeros((cfg.n_nonlocal, cfg.n_groups), np.int32), 0)
    layer.workspace = torch.empty(256, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.AstraError):
        layer.run()


# contraction, groups, codewords: one to six tiles of 64, groups that end inside a tile, 8- and 16-bit codes
GATHERED_TILES = [(64, 8, 256), (128, 2, 1024), (192, 8, 256), (256, 4, 1024), (320, 40, 1024), (384, 6, 256)]


@pytest.mark.parametrize("n_local,n_nonlocal,form", [(700, 700, "tile<128, 256>"), (1100, 600, "tile<256, 256>")])
@pytest.mark.parametrize("d,groups,words", GATHERED_TILES)
def test_gathered_rows_over_few_contraction_tiles(d, groups, words, n_local, n_nonlocal, form):
    """The large tiles' loop fetches a tile's codes four half steps before its rows: contractions of as few tiles as the prologue and the first steps
    span.  Logits of standard deviation 5, so that a wrong row of K-hat or V-hat is the whole output of some query.  Bar: bf16 rounding of queries and keys
    moves such a logit by up to 0.05, probabilities by 5 %; 0.1 of the largest output is twice what that gives."""
    import torch
    from gpu_util import DEV, empty_codes
    from paper_2505_19342_amd import binding as B
    hq, hkv, dh = 32, 8, 128
    g = torch.Generator(device=DEV)
    g.manual_seed(d + n_local)
    rnd = lambda *s, std=1.0: (torch.randn(s, generator=g, device=DEV) * std).to(torch.bfloat16)
    x, cb = rnd(n_local, d), rnd(groups, words, d // groups)
    wq, wk = rnd(hq * dh, d, std=(5 / d) ** 0.5), rnd(hkv * dh, d, std=(5 / d) ** 0.5)
    wv, wo = rnd(hkv * dh, d, std=d ** -0.5), rnd(d, hq * dh, std=1 / 64)
    codes = torch.randint(0, words, (n_nonlocal, groups), generator=g, device=DEV)
    desc = B.LayerDesc(B.vq_desc("bf16", d, groups, words), B.attn_desc("bf16", hq, hkv, dh, 0, n_local, n_nonlocal, True, n_nonlocal))
    cnorm = torch.empty((groups, words), dtype=torch.float32, device=DEV)
    B.astra_vq_prepare(desc.vq, cb, cnorm)
    y = torch.empty((n_local, d), dtype=torch.float32, device=DEV)
    B.astra_layer_forward(desc, x, codes.to(torch.uint8 if words <= 256 else torch.int16), cb, cnorm, wq, wk, wv, wo, None, None, None, None, y,
                          empty_codes(n_local, groups, words), torch.empty(B.astra_layer_workspace_bytes(desc), dtype=torch.uint8, device=DEV))
    rows = torch.cat([cb[torch.arange(groups, device=DEV), codes].reshape(n_nonlocal, d).float(), x.float()])
    q = (x.float() @ wq.float().T).view(n_local, hkv, hq // hkv, dh).permute(1, 2, 0, 3)
    k, v = [(rows @ w.float().T).view(-1, hkv, 1, dh).permute(1, 2, 0, 3) for w in (wk, wv)]
    hidden = torch.ones((n_local, n_nonlocal + n_local), dtype=torch.bool, device=DEV).triu(n_nonlocal + 1)
    p = ((q @ k.transpose(-1, -2).contiguous()) * dh ** -0.5).masked_fill(hidden, float("-inf")).softmax(-1)
    ref = (p @ v).permute(2, 0, 1, 3).reshape(n_local, hq * dh) @ wo.float().T
    assert float((y - ref).abs().max()) <= 0.1 * float(ref.abs().max())
    assert float((y - ref).norm() / ref.norm()) <= 2e-2


@pytest.mark.parametrize("n_local,n_nonlocal,hq,hkv,n_cls,causal,lost", [
    (1, 0, 2, 1, 0, True, None),             # one row, one key: seven of the eight wavefronts have no tile
    (32, 0, 4, 4, 1, False, None),           # a second block of one row
    (31, 480, 12, 12, 0, True, None),        # eight tiles and one key's worth of a ninth for the first wavefront
    (33, 513, 12, 4, 0, True, None),         # grouped heads; nine tiles of peers, the last of one row
    (100, 700, 12, 12, 1, False, "some"),
    (100, 700, 12, 12, 0, True, "tiles"),    # the first and third tile lost whole: two wavefronts without a key before the local rows
    (40, 200, 4, 4, 0, True, "all"),
    (150, 1100, 16, 8, 0, True, None),       # three tiles for a wavefront
    (672, 96, 12, 12, 0, True, None),        # 252 blocks of 32 rows: the last round number of heads that is a single round
    (673, 96, 12, 12, 0, True, None),        # 264: the other kernel
])
def test_short_sequences_of_64_wide_heads(n_local, n_nonlocal, hq, hkv, n_cls, causal, lost):
    """Attention on blocks of 32 query rows whose wavefronts walk the tiles for themselves: fewer tiles than wavefronts, ragged ends, masks."""
    _short_sequence(64, n_local, n_nonlocal, hq, hkv, n_cls, causal, lost)


@pytest.mark.parametrize("n_local,n_nonlocal,hq,hkv,n_cls,causal,lost", [
    (1, 0, 2, 1, 0, True, None),
    (31, 225, 4, 2, 1, False, None),         # eight tiles of 32 keys of peers, the last of one; a class row makes whole blocks
    (33, 257, 4, 4, 0, True, None),          # nine, and a second block of one row
    (100, 700, 4, 4, 0, True, "some"),
    (100, 700, 4, 4, 1, False, "tiles"),     # both halves of a word of arrivals, and a half alone
    (40, 200, 4, 1, 0, True, "all"),
    (256, 200, 32, 8, 0, True, None),        # 256 blocks: a single round
    (257, 200, 32, 8, 0, True, None),        # the other kernel
])
def test_short_sequences_of_128_wide_heads(n_local, n_nonlocal, hq, hkv, n_cls, causal, lost):
    """The same on tiles of 32 keys."""
    _short_sequence(128, n_local, n_nonlocal, hq, hkv, n_cls, causal, lost)


# query and key rows, heads, KV heads, class rows, causal, lost codes; blocks of a head walked whole, parts of the others (as tests/test_launches.py checks)
CUT_WALKS = [
    (100, 4096, 4, 4, 0, True, "tiles", 0, 8),      # one block, its last group with four rows; heads that the XCDs do not share evenly
    (20, 4096, 4, 4, 0, True, "all", 0, 8),         # three groups without a row; seven parts without a key
    (255, 1900, 4, 4, 1, False, "some", 0, 8),      # a class row, the encode behind the parts
    (300, 4096, 8, 2, 0, True, None, 0, 8),         # the last part crosses the diagonal; a block of 44 rows
    (520, 2500, 16, 4, 0, True, "some", 0, 3),      # parts of unequal length, a block of 8 rows
    (520, 600, 64, 8, 0, True, None, 4, 3),         # whole walks first, the ragged block in parts
    (520, 600, 64, 8, 0, True, "some", 4, 3),
    (520, 600, 52, 4, 0, True, "tiles", 4, 3),      # heads that the XCDs do not share evenly
    (520, 300, 52, 4, 0, True, None, 4, 4),
    (130, 1500, 52, 4, 0, True, None, 0, 2),        # every other number of parts
    (70, 4096, 64, 8, 0, True, "some", 0, 4),
    (130, 4096, 24, 8, 0, True, None, 0, 5),
    (130, 4096, 20, 4, 0, True, "tiles", 0, 6),
    (70, 4096, 36, 4, 0, True, None, 0, 7),
]


@pytest.mark.parametrize("lost", [None, "some"])
def test_more_whole_walks_than_units(lost):
    """320 blocks of 128 rows on 256 units, the longest of all heads first."""
    _short_sequence(128, 520, 100, 64, 8, 0, True, lost)


@pytest.mark.parametrize("n_local,n_nonlocal,hq,hkv,n_cls,causal,lost,whole,parts", CUT_WALKS)
def test_walks_cut_between_workgroups(n_local, n_nonlocal, hq, hkv, n_cls, causal, lost, whole, parts):
    """Parts of a walk in scratch and their sum; without the scratch the walks are whole, and the call is taken all the same."""
    _short_sequence(128, n_local, n_nonlocal, hq, hkv, n_cls, causal, lost, minimal=True)


@pytest.mark.parametrize("n_local,n_nonlocal,hq,hkv,n_cls,causal,lost,groups,words", [
    (17, 60, 8, 2, 0, True, None, 4, 300), (100, 300, 8, 2, 0, True, "some", 2, 256), (65, 64, 12, 4, 1, False, None, 4, 100),
    (128, 200, 16, 4, 0, True, None, 8, 1024), (33, 0, 8, 8, 0, True, None, 2, 4)])
def test_encodes_of_wide_groups_beside_the_attention(n_local, n_nonlocal, hq, hkv, n_cls, causal, lost, groups, words):
    """Groups of 128, 192 and 256 values, streamed by workgroups behind the 32-row attention's (tests/test_launches.py)."""
    _short_sequence(128, n_local, n_nonlocal, hq, hkv, n_cls, causal, lost, groups=groups, words=words)


def _short_sequence(dh, n_local, n_nonlocal, hq, hkv, n_cls, causal, lost, minimal=False, groups=16, words=256):
    from gpu_util import LayerOnGpu, compare_codes
    d = 64 * hq
    cfg = wl.LayerConfig("short", "bf16", d, hq, hkv, dh, n_local + n_nonlocal, 1, groups, words, n_cls=n_cls, causal=causal, seed=71)
    data = wl.generate(cfg)
    rows = data["x"]
    cls_rows = rows[-n_cls:] if n_cls else rows[:0]
    x_nl = rows[:n_nonlocal]
    x_local = np.concatenate([cls_rows, rows[n_nonlocal:n_nonlocal + n_local]])
    codes_nl = oracle.vq_encode(x_nl, data["codebook"])
    valid = None
    if lost:
        valid = np.ones(n_nonlocal, dtype=bool)
        if lost == "some":
            valid = np.random.default_rng(5).random(n_nonlocal) >= 0.3
        elif lost == "tiles":
            valid[:64] = valid[128:192] = False
            if dh == 128:
                valid[288:320] = valid[384:416] = False
        else:
            valid[:] = False
    n_before = n_nonlocal if causal else 0
    y_ref, codes_ref, gap = oracle.layer_forward(x_local, codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"], data["wo"], n_q_heads=hq,
                                                 n_kv_heads=hkv, n_cls=n_cls, causal=causal, n_before=n_before, return_gap=True, valid_nonlocal=valid)
    layer = LayerOnGpu(cfg, data, x_local, codes_nl, n_before)
    layer.run(valid_nonlocal=valid)
    y, codes = layer.results()
    compare_codes(codes, codes_ref, gap, NEAR_TIE)
    assert np.abs(y - y_ref).max() <= Y_TOL["bf16"]
    if minimal:
        eb, dq, dkv, up = 2, hq * dh, hkv * dh, lambda n, m: -(-n // m) * m
        n_vis, n_q = n_nonlocal, n_cls + n_local
        smallest = sum(up(n * eb, 256) for n in (n_q * dq, n_q * dkv, up(n_q, 64) * dkv, n_vis * dkv, up(n_vis, 64) * dkv, n_q * dq))
        assert layer.workspace.numel() > smallest
        layer.workspace = layer.workspace[:smallest]
        layer.y.zero_()
        layer.run(valid_nonlocal=valid)
        assert np.abs(layer.results()[0] - y_ref).max() <= Y_TOL["bf16"]
