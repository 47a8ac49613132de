"""GPU parity: one whole Transformer block on one device (norm1 -> Astra layer -> residual -> norm2 -> MLP ->
residual; Sec. 3.1) through astra_block_forward against the CPU oracle, on the seeded block workloads.
Bars: block output max-abs <= 1e-4 (fp32); for bf16 the layer's 2e-2 plus 2^-6 rms(out - x): the two bf16-stored
MLP intermediates (norm2 output, hidden activation) each carry a relative rounding error of up to 2^-9 per element,
which reaches every output as a random sum proportional to the output's own scale (about 2^-9 * 1.5 rms, largest of
millions of outputs about 5.3 sigma; tests/test_oracle_block.py reproduces the figure on the CPU).  The normalised tensor h, which is what gets quantised:
fp32 within 1e-5; bf16 bit-equal to the oracle's (fp64 norm, rounded once) except for a counted few elements that
sit on a rounding boundary and come out one bf16 step away (or within 2e-6 where the result cancels to near zero).  Codes of group slices whose h agrees with the
oracle's: bit-exact except near-ties (oracle gap < 1e-5 relative); codes of the few slices whose h differs: any
codeword that the differing h can justify (its distance to the oracle's h exceeds the best by no more than
2 |e| (|h - c'| + |h - c*|), e the difference of the two h slices)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2505_19342_amd import workloads as wl

pytestmark = pytest.mark.gpu

OUT_TOL = {"f32": 1e-4, "bf16": 2e-2}
NEAR_TIE = 1e-5


def peer_codes(bcfg, data, x_nonlocal):
    """What the peers would have sent: the codes of THEIR norm1 outputs, in the layer's element type."""
    cfg = bcfg.layer
    h = oracle.norm(x_nonlocal, bcfg.norm_kind, bcfg.eps, data["g1"], data["be1"]).astype(np.float32)
    if cfg.dtype == "bf16":
        h = wl.round_to_bf16(h)
    return oracle.vq_encode(h, data["codebook"])


def run_case(bcfg, rank, in_place=False, valid=None):
    from gpu_util import BlockOnGpu, check_h_and_codes
    cfg = bcfg.layer
    data = wl.generate_block(bcfg)
    view = wl.device_view(cfg, data, rank)
    codes_nl = peer_codes(bcfg, data, view["x_nonlocal"])
    names = ("bq", "bk", "bv", "bo", "b1", "b2")
    out_ref, codes_ref, gap, h_ref = oracle.block_forward(
        view["x_local"], codes_nl, data["codebook"], data["wq"], data["wk"], data["wv"], data["wo"],
        norm_kind=bcfg.norm_kind, eps=bcfg.eps, g1=data["g1"], g2=data["g2"], be1=data["be1"], be2=data["be2"],
        mlp_kind=bcfg.mlp_kind, w1=data["w1"], w2=data["w2"], n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads,
        n_cls=cfg.n_cls, causal=cfg.causal, n_before=view["n_before"], valid_nonlocal=valid,
        h_is_bf16=cfg.dtype == "bf16", rope_base=bcfg.rope_base, **{n: data.get(n) for n in names})
    blk = BlockOnGpu(bcfg, data, view["x_local"], codes_nl, view["n_before"], in_place=in_place)
    blk.run(valid)
    out, codes, h = blk.results()
    n_tie, n_slices, n_other = check_h_and_codes(cfg.dtype, cfg.n_cls, h, h_ref, codes, codes_ref, gap, data["codebook"])
    err = np.abs(out - out_ref).max()
    print(f"{bcfg.name} rank {rank}: max abs err {err:.3e} (|out| max {np.abs(out_ref).max():.2f}), near-tie codes {n_tie}/{codes.size}, "
          f"slices with a differing h {n_slices} ({n_other} of them chose another codeword)")
    tol = OUT_TOL[cfg.dtype]
    if cfg.dtype == "bf16":
        tol += 2.0 ** -6 * float(np.sqrt(np.mean((out_ref - view["x_local"]) ** 2)))
    assert err <= tol, f"{err:.3e} > {tol:.3e}"
    assert n_tie <= max(2, codes.size // 2000)
    return out


@pytest.mark.parametrize("rank", [0, 3])
def test_tiny_vit_block_f32(rank):
    run_case(wl.TINY_VIT_BLOCK, rank)


@pytest.mark.parametrize("rank", [0, 2])
def test_vit_base_block_bf16_layernorm_gelu_erf_class_row(rank):
    run_case(wl.VIT_BASE_BLOCK, rank)


@pytest.mark.parametrize("rank", [0, 3])
def test_gpt2_small_block_bf16_layernorm_gelu_tanh_causal(rank):
    run_case(wl.GPT2_SMALL_BLOCK, rank)


def small_llama(seq_len=1148, d_ff=1792, seed=51, dtype="bf16"):
    """Llama-3-8B widths (D 4096, 32/8 heads of 128, G 64, K 1024) with fewer rows and a narrower MLP: 287 local rows
    (ragged against every tile size) and d_ff = 7 * 256."""
    layer = dataclasses.replace(wl.LLAMA3_8B, name="llama_small", seq_len=seq_len, seed=seed, dtype=dtype)
    return dataclasses.replace(wl.LLAMA3_8B_BLOCK, name="llama_small_block", layer=layer, d_ff=d_ff)


@pytest.mark.parametrize("rank", [1, 3])
def test_llama_width_block_bf16_rmsnorm_swiglu(rank):
    run_case(small_llama(), rank)


def test_split_contraction_with_ragged_rows():
    """287 rows x 4096 columns is 32 large tiles, d_ff = 16384: the second MLP product is cut into 8 slices of the
    contraction whose partial sums are added in a fixed order by a reduction kernel (with the residual)."""
    run_case(small_llama(d_ff=16384, seed=55), 2)


def test_swiglu_ragged_hidden_width_and_f32_gate():
    """d_ff that is not a multiple of the gate tile (64 | d_ff only), and the fp32 path's separate gate kernel."""
    layer = dataclasses.replace(wl.GPT2_SMALL, name="swiglu_ragged", seq_len=420, seed=52)
    run_case(dataclasses.replace(wl.LLAMA3_8B_BLOCK, name="swiglu_ragged_block", layer=layer, d_ff=1216), 1)
    layer = dataclasses.replace(wl.TINY_VIT, name="swiglu_f32", seed=53)
    run_case(dataclasses.replace(wl.LLAMA3_8B_BLOCK, name="swiglu_f32_block", layer=layer, d_ff=200, norm_kind="rmsnorm"), 2)


def test_large_tiles_with_a_ragged_gate_tile():
    """1024 local rows and d_ff = 65 * 64: the gated GEMM runs on 256 x 256 tiles whose last column tile is half empty."""
    layer = dataclasses.replace(wl.GPT2_SMALL, name="swiglu_big_ragged", seq_len=4096, seed=54)
    run_case(dataclasses.replace(wl.LLAMA3_8B_BLOCK, name="swiglu_big_ragged_block", layer=layer, d_ff=4160), 2)


def test_block_in_place_equals_out_of_place_and_repeats_bit_exactly():
    a = run_case(wl.GPT2_SMALL_BLOCK, 1)
    b = run_case(wl.GPT2_SMALL_BLOCK, 1, in_place=True)
    np.testing.assert_array_equal(a, b)
    c = run_case(wl.GPT2_SMALL_BLOCK, 1)
    np.testing.assert_array_equal(a, c)


def test_block_with_lost_codes():
    bcfg = wl.GPT2_SMALL_BLOCK
    rng = np.random.default_rng(5)
    valid = (rng.random(bcfg.layer.n_nonlocal) > 0.1).astype(np.uint8)
    a = run_case(bcfg, 3, valid=valid)
    b = run_case(bcfg, 3)
    assert np.abs(a - b).max() > 1e-3          # the lost rows matter


def test_llama3_8b_block_full_size():
    run_case(wl.LLAMA3_8B_BLOCK, 3)


@pytest.mark.parametrize("rank", [0, 1, 3])
def test_llama_width_block_with_rotary_positions(rank):
    """Optional rotary positions (outside the paper): Q, K and K-hat turned at their sequence positions before Eq. 1;
    rank 0 has no visible non-local rows, rank 3 the most."""
    a = run_case(dataclasses.replace(small_llama(seed=56), rope_base=500000.0), rank)
    b = run_case(small_llama(seed=56), rank)
    assert np.abs(a - b).max() > 1e-3          # the rotation matters


def test_rotary_positions_fp32_and_head_dim_64():
    """The fp32 path (a pair per thread) on a causal variant of the tiny model, and the bf16 path with 64-wide heads."""
    layer = dataclasses.replace(wl.TINY_VIT, name="tiny_causal_f32", n_cls=0, causal=True, seed=57)
    run_case(dataclasses.replace(wl.TINY_VIT_BLOCK, name="tiny_causal_block_f32", layer=layer, rope_base=10000.0), 2)
    run_case(dataclasses.replace(wl.GPT2_SMALL_BLOCK, name="gpt2_small_rope_block", rope_base=10000.0), 2)


def test_rotary_positions_need_a_causal_layer():
    """A layer that is not causal carries no row positions: the descriptor is refused (no workspace size, no launch)."""
    import torch
    from gpu_util import BlockOnGpu
    from paper_2505_19342_amd import binding as B
    bcfg = wl.TINY_VIT_BLOCK
    data = wl.generate_block(bcfg)
    view = wl.device_view(bcfg.layer, data, 0)
    codes_nl = peer_codes(bcfg, data, view["x_nonlocal"])
    blk = BlockOnGpu(bcfg, data, view["x_local"], codes_nl, view["n_before"])
    bad = B.block_desc(blk.desc.layer, bcfg.norm_kind, bcfg.mlp_kind, bcfg.d_ff, bcfg.eps, 10000.0)
    assert B.astra_block_workspace_bytes(bad) == 0
    blk.x_out.fill_(-7.0)
    with pytest.raises(B.AstraError):
        B.astra_block_forward(bad, blk.weights, blk.x, blk.codes_nonlocal, None, blk.x_out, blk.codes_local, blk.h, blk.workspace)
    torch.cuda.synchronize()
    assert bool((blk.x_out == -7.0).all())


# width, rows, groups, codewords, MLP, hidden width, and forms among the block's products with their epilogues, as tests/test_launches.py checks
MLP_LAUNCHES = [
    (256, 1032, 32, 256, "gelu_tanh", 512, ("wave<2, 1, 2> residual", "wave<2, 2, 2> gelu_tanh", "wave<1, 1, 2> residual")),
    (512, 76, 8, 256, "gelu_erf", 3072, ("wave<2, 1, 2> gelu_erf",)),
    (512, 94, 8, 16, "gelu_tanh", 3072, ("wave<2, 1, 2> gelu_tanh",)),
    (512, 93, 16, 16, "swiglu", 2048, ("wave<2, 1, 2> swiglu",)),
    (1024, 1049, 8, 16, "swiglu", 512, ("wave<2, 2, 1> residual", "wave<2, 2, 1> swiglu")),
    (256, 522, 32, 1024, "gelu_tanh", 2048, ("wave<2, 2, 1> gelu_tanh",)),
    (256, 357, 8, 1024, "gelu_erf", 3072, ("wave<2, 2, 1> gelu_erf",)),
    (512, 1072, 8, 16, "swiglu", 512, ("wave<2, 2, 2> residual",)),
    (256, 70, 4, 256, "swiglu", 3072, ("wave<2, 2, 2> swiglu",)),
    (256, 172, 16, 16, "gelu_erf", 3072, ("wave<2, 2, 2> gelu_erf",)),
    (256, 655, 32, 1024, "gelu_tanh", 3072, ("tile<128, 128> gelu_tanh",)),
    (256, 667, 4, 16, "gelu_erf", 3072, ("tile<128, 128> gelu_erf",)),
    (256, 333, 8, 256, "swiglu", 3072, ("tile<128, 128> swiglu",)),
    (1024, 1048, 8, 16, "gelu_tanh", 3072, ("wave<4, 2, 1> residual",)),
    (2048, 355, 8, 256, "swiglu", 3072, ("wave<4, 4, 1> swiglu",)),
    (2048, 283, 8, 1024, "swiglu", 2048, ("wave<4, 2, 1> swiglu",)),
    (2048, 1047, 8, 1024, "swiglu", 512, ("wave<4, 4, 1> residual", "tile<128, 128> residual")),
]


@pytest.mark.parametrize("d,rows,groups,words,mlp,d_ff,forms", MLP_LAUNCHES)
def test_products_of_the_block_with_ragged_rows(d, rows, groups, words, mlp, d_ff, forms):
    from test_gpu_layer import MODEL_OF_WIDTH
    hq, hkv, dh = MODEL_OF_WIDTH[d]
    layer = wl.LayerConfig("forms", "bf16", d, hq, hkv, dh, rows, 1, groups, words, causal=True, seed=63)
    run_case(wl.BlockConfig("forms_block", layer, "layernorm", mlp, d_ff, 1e-5, True), 0)


@pytest.mark.parametrize("rows", [3, 4100])
@pytest.mark.parametrize("mlp,gate,up,down", [("swiglu", (-88.0, 0.0), 2.0 ** 100, 2.0 ** 20), ("gelu_tanh", (-10.0, -0.03125), None, 2.0 ** 120)])
def test_activations_far_out_on_the_negative_side(mlp, gate, up, down, rows):
    """Where 1 / (1 + e^z) is below the smallest normal number the activation itself is not: silu(-88) = -5.3e-37.  Rows of ones make
    the pre-activation exactly the sum of `gate`; `up` and `down` bring the product back into sight.  The bar is the hidden value's bf16 rounding
    and one step more."""
    import torch
    from gpu_util import DEV
    from paper_2505_19342_amd import binding as B
    D, F = 64, 2048
    layer = B.LayerDesc(B.vq_desc("bf16", D, 1, 16), B.attn_desc("bf16", 1, 1, 64, 0, rows, 0, False, 0))
    desc = B.block_desc(layer, "rmsnorm", mlp, F, 0.0, 0.0)
    zeros = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16, device=DEV)
    t = dict(codebook=zeros(1, 16, D), cnorm=torch.zeros((1, 16), device=DEV), wq=zeros(64, D), wk=zeros(64, D), wv=zeros(64, D), wo=zeros(D, 64),
             w1=zeros(2 * F if up else F, D), w2=zeros(D, F), norm1_gain=torch.ones(D, device=DEV), norm2_gain=torch.ones(D, device=DEV))
    t["w1"][0, 0], t["w1"][0, 1] = gate
    if up:
        t["w1"][F, 0] = up
    t["w2"][5, 0] = down
    x = torch.ones((rows, D), device=DEV)
    out = torch.empty_like(x)
    ws = torch.empty(B.astra_block_workspace_bytes(desc), dtype=torch.uint8, device=DEV)
    codes = torch.empty((rows, 1), dtype=torch.uint8, device=DEV)
    B.astra_block_forward(desc, B.block_weights(**t), x, None, None, out, codes, None, ws)
    torch.cuda.synchronize()
    v = np.float64(sum(gate))
    act = v / (1.0 + np.exp(-v)) if up else v / (1.0 + np.exp(-2.0 * 0.7978845608028654 * (v + 0.044715 * v ** 3)))
    step = act * (up or 1.0) * down
    assert abs(step) > 0.05
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got[:, 5] - 1.0 - step) <= 2.0 ** -8 * abs(step)) and np.all(np.delete(got, 5, axis=1) == 1.0)


def test_block_argument_errors_launch_nothing():
    import torch
    from gpu_util import BlockOnGpu
    from paper_2505_19342_amd import binding as B
    bcfg = wl.TINY_VIT_BLOCK
    data = wl.generate_block(bcfg)
    view = wl.device_view(bcfg.layer, data, 0)
    codes_nl = peer_codes(bcfg, data, view["x_nonlocal"])
    blk = BlockOnGpu(bcfg, data, view["x_local"], codes_nl, view["n_before"])
    blk.x_out.fill_(-7.0)
    small = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(B.AstraError, match="workspace"):
        B.astra_block_forward(blk.desc, blk.weights, blk.x, blk.codes_nonlocal, None, blk.x_out, blk.codes_local, blk.h, small)
    bad = B.block_desc(blk.desc.layer, "layernorm", "gelu_erf", 0, 1e-6)
    with pytest.raises(B.AstraError):
        B.astra_block_forward(bad, blk.weights, blk.x, blk.codes_nonlocal, None, blk.x_out, blk.codes_local, blk.h, blk.workspace)
    assert B.astra_block_workspace_bytes(bad) == 0
    w = B.block_weights(**{k: v for k, v in blk.tensors.items() if k != "w2"})
    with pytest.raises(B.AstraError, match="NULL"):
        B.astra_block_forward(blk.desc, w, blk.x, blk.codes_nonlocal, None, blk.x_out, blk.codes_local, blk.h, blk.workspace)
    torch.cuda.synchronize()
    assert bool((blk.x_out == -7.0).all())


@pytest.mark.parametrize("words,seq_len", [(256, 420), (1024, 420), (16, 8)])
def test_slices_of_no_whole_16_bytes(words, seq_len):
    """64 groups of 12 channels: the peers' rows are rebuilt by the launch of the first normalisation; 8- and 16-bit codes, pieces that fill no whole
    workgroup, and six rows of peers."""
    layer = dataclasses.replace(wl.GPT2_SMALL, name="gpt2_64_groups", n_groups=64, codebook_size=words, seq_len=seq_len, seed=81)
    run_case(dataclasses.replace(wl.GPT2_SMALL_BLOCK, name="gpt2_64_groups_block", layer=layer), 3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("norm_kind", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("d", [64, 832, 1024, 1088])
def test_widths_of_the_normalisation(d, norm_kind, dtype):
    """A wavefront per row up to 1024 values (lanes without any, a ragged last quarter, all of them), a workgroup beyond."""
    layer = wl.LayerConfig("norm_widths", dtype, d, 2, 1, 64, 99, 3, 8, 16, causal=True, seed=82)
    run_case(wl.BlockConfig("norm_widths_block", layer, norm_kind, "gelu_tanh", 128, 1e-5, norm_kind == "layernorm"), 2)


@pytest.mark.parametrize("words", [256, 300])
@pytest.mark.parametrize("norm_kind", ["layernorm", "rmsnorm"])
def test_rebuilt_rows_beside_the_normalisation_of_wide_rows(norm_kind, words):
    """16 groups of 68 channels: a workgroup per row of 1088 values, the peers' rows in the workgroups behind them; 8- and 16-bit codes."""
    layer = wl.LayerConfig("wide_decode", "bf16", 1088, 4, 2, 64, 99, 3, 16, words, causal=True, seed=83)
    run_case(wl.BlockConfig("wide_decode_block", layer, norm_kind, "gelu_tanh", 128, 1e-5, norm_kind == "layernorm"), 2)


# heads, tokens, devices: walks in parts (as tests/test_launches.py checks), with the encode behind them and without
CUT = [(4, 2400, 16), (20, 1600, 4)]


@pytest.mark.parametrize("heads,seq_len,n_dev", CUT)
def test_walks_cut_between_workgroups(heads, seq_len, n_dev):
    """The parts lie behind everything else that the block keeps in its workspace."""
    layer = wl.LayerConfig("block_cut", "bf16", 64 * heads, heads, 4, 128, seq_len, n_dev, 16, 256, causal=True, seed=84)
    run_case(wl.BlockConfig("block_cut", layer, "rmsnorm", "gelu_tanh", 256, 1e-5, False, rope_base=10000.0), n_dev - 1)
