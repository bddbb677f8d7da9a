"""The matrix-core kernel whose waves each take a part of K (kpart.hip), at the
edges of its tiles: 16, 32 and 64 weight rows, 16 and 32 tokens, fewer and
more super-blocks than waves, and the routes its rule draws."""
import numpy as np
import pytest

import gate
from gpu_util import to_gpu
from parity import Ref, kernel_of
from paper_2605_20706_amd import binding, layout, synth
from paper_2605_20706_amd.layout import F16, MXFP4, Q4_0, Q4_1, Q4_K, Q5_0, Q5_1, Q5_K, Q6_K, Q8_0

# (M, K, n_tok): one row; a ragged row tile; 9 super-blocks over 8 waves; a
# token tile and one more token; 32 tokens and one more; the most tokens; then
# 32 and 64 rows a workgroup with 16 and 32 tokens, ragged rows and tokens
SHAPES = [(1, 256, 9), (17, 512, 16), (65, 2304, 13), (100, 4096, 17), (130, 2048, 33), (49, 768, 128),
          (6150, 768, 13), (12300, 768, 13), (3001, 1024, 77), (4111, 768, 99)]
# 2 to 8 tokens (two and four pairs are loaded) with 16, 32 and 64 rows a workgroup
FEW = [(33, 4096, 3), (70, 6400, 6), (12300, 2048, 8), (33, 2048, 4), (33, 4096, 4), (33, 512, 6), (4100, 2048, 3),
       (6150, 4096, 3), (6150, 4096, 7), (16001, 2048, 3), (16001, 2048, 7), (12300, 2048, 4), (12300, 4096, 3),
       (12300, 4096, 8)]


def run_check(oracle_mod, fmt, M, K, n_tok):
    import torch
    kern = kernel_of(fmt, M, K, n_tok)
    print("kpart fmt=%d M=%d K=%d n_tok=%d -> %s" % (fmt, M, K, n_tok, kern), flush=True)
    W = synth.gen_packed(fmt, M * K, np.random.default_rng([71, fmt, M, K]))
    x = synth.gen_x_seeded([72, K, n_tok], K, n_tok)
    y = binding.matvec(fmt, to_gpu(W), to_gpu(x), M, K)
    torch.cuda.synchronize()
    ref = Ref(oracle_mod, fmt, W, x, M, K)
    gate.check(y.cpu().numpy(), ref.y, ref.A, ref.F(kern), f32_bound=1e-4, what=(fmt, M, K, n_tok, kern))


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", sorted(layout.FORMAT_NAMES))
@pytest.mark.parametrize("M,K,n_tok", SHAPES)
def test_tile_edges(oracle_mod, fmt, M, K, n_tok):
    run_check(oracle_mod, fmt, M, K, n_tok)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", sorted(layout.FORMAT_NAMES))
@pytest.mark.parametrize("M,K,n_tok", FEW)
def test_few_tokens(oracle_mod, fmt, M, K, n_tok):
    run_check(oracle_mod, fmt, M, K, n_tok)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [f for f in sorted(layout.FORMAT_NAMES) if f != F16])
@pytest.mark.parametrize("M,K,n_tok", [(4111, 1280, 40), (4111, 1792, 33)])
def test_four_waves_for_five_to_seven_super_blocks(oracle_mod, fmt, M, K, n_tok):
    """More than a round of workgroups: two a compute unit."""
    run_check(oracle_mod, fmt, M, K, n_tok)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [f for f in sorted(layout.FORMAT_NAMES) if f not in (F16, Q8_0)])
@pytest.mark.parametrize("M,K,n_tok", [(100, 2048, 8), (100, 2048, 13), (100, 2048, 40), (6200, 768, 12), (3100, 768, 40)])
def test_offsets_cancel(oracle_mod, fmt, M, K, n_tok):
    """Activations of 16 bits in +-[1, 2): two bf16 parts hold them whole, and a
    block's product less its offset fits in float32, so what is left is the
    rounding of K / 32 block values: at most 8 additions a wave and 8 waves, each
    2^-24 of a partial sum that grows as the root, 2^-24 * 2, and again for the
    formats with a term of their own for the minimum."""
    import torch
    assert binding.kernel_name(fmt, M, K, n_tok).startswith("kpart_kernel<")
    rng = np.random.default_rng([80, fmt])
    W = synth.gen_packed(fmt, M * K, rng)
    x = (rng.integers(2 ** 15, 2 ** 16, (n_tok, K)) * 2.0 ** -15 * rng.choice([-1, 1], (n_tok, K))).astype(np.float32)
    y = binding.matvec(fmt, to_gpu(W), to_gpu(x), M, K)
    torch.cuda.synchronize()
    ref = x.astype(np.float64) @ oracle_mod.dequant(fmt, W, M * K).reshape(M, K).astype(np.float64).T
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 2 * 2 * 2.0 ** -24 * np.linalg.norm(ref)


@pytest.mark.gpu
@pytest.mark.parametrize("K", [768, 1280])
def test_q8_0_half_super_blocks(oracle_mod, K):
    """Q8_0 with 64 rows a workgroup: units of half a super-block, fewer than
    the waves and two for some, on ragged rows and tokens."""
    M, n_tok = 1003, 401
    assert binding.kernel_name(Q8_0, M, K, n_tok).replace(" ", "") == "kpart_kernel<1,2,4,16,2>"
    run_check(oracle_mod, Q8_0, M, K, n_tok)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [F16, Q8_0, Q4_K])
def test_rows_of_several_matrices(oracle_mod, fmt):
    """One launch over three matrices with ragged row counts."""
    import torch
    Ms, K, n_tok = [33, 1, 70], 4096, 11
    assert binding.launch_count_multi(fmt, Ms, K, n_tok) == 1
    kern = binding.kernel_name_multi(fmt, Ms, K, n_tok)
    Ws = [synth.gen_packed(fmt, m * K, np.random.default_rng([73, fmt, i])) for i, m in enumerate(Ms)]
    x = synth.gen_x_seeded([74, K], K, n_tok)
    ys = binding.matvec_multi(fmt, [to_gpu(w) for w in Ws], to_gpu(x), Ms, K)
    torch.cuda.synchronize()
    for w, m, y in zip(Ws, Ms, ys):
        ref = Ref(oracle_mod, fmt, w, x, m, K)
        gate.check(y.cpu().numpy(), ref.y, ref.A, ref.F(kern), f32_bound=1e-4, what=(fmt, m, kern))


@pytest.mark.gpu
@pytest.mark.parametrize("n_tok", [5, 40])
def test_f16_keeps_float32(n_tok):
    """f16 weights: float32 activations in three bf16 parts, so the error stays
    that of float32 sums of at most K terms, taken here as 2^-20 sum |w x|,
    also for subnormal weights and activations 2^+-40 apart in different
    tokens."""
    import torch
    M, K = 50, 2048
    rng = np.random.default_rng(75)
    w = (rng.standard_normal((M, K)) * 0.02).astype(np.float16)
    w[::3] = (rng.standard_normal((len(w[::3]), K)) * 2e-6).astype(np.float16)
    x = rng.standard_normal((n_tok, K)).astype(np.float32)
    x[1] *= np.float32(2.0 ** 40)
    x[2] *= np.float32(2.0 ** -40)
    y = binding.matvec(F16, to_gpu(w.reshape(-1).view(np.uint8)), to_gpu(x), M, K)
    torch.cuda.synchronize()
    w64, x64 = w.astype(np.float64), x.astype(np.float64)
    assert (np.abs(y.cpu().numpy() - x64 @ w64.T) <= 2.0 ** -20 * (np.abs(x64) @ np.abs(w64).T)).all()


# one row tile (two token counts), two and four, with 16 and 32 tokens
F16_TILES = [(50, 2048, 5), (50, 1024, 20), (6200, 256, 33), (12300, 256, 37), (12300, 512, 16), (12300, 2048, 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,n_tok", F16_TILES)
def test_f16_all_bits(M, K, n_tok):
    """A weight row of zeros and a single one, or the smallest subnormal,
    returns its activations bit for bit: all 24 bits, whatever their size and
    that of the others (the smallest weight's outputs stay above 2^-126)."""
    import torch
    assert binding.kernel_name(F16, M, K, n_tok).startswith("kpart_kernel<")
    rng = np.random.default_rng(77)
    w = np.zeros((M, K), np.float16)
    col = rng.integers(0, K, M)
    w[np.arange(M), col] = np.where(np.arange(M) % 2, 1, 2.0 ** -24)
    x = rng.standard_normal((n_tok, K)).astype(np.float32) * np.exp2(rng.integers(-60, 1, (n_tok, K))).astype(np.float32)
    x[1] = rng.standard_normal(K).astype(np.float32) * np.float32(2.0 ** -95)
    x[2] *= np.float32(2.0 ** 120)
    y = binding.matvec(F16, to_gpu(w.reshape(-1).view(np.uint8)), to_gpu(x), M, K)
    torch.cuda.synchronize()
    assert (y.cpu().numpy() == x[:, col] * w.astype(np.float32)[np.arange(M), col]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("big", [1e5, 1e9, 1e12, 1e30, 3e38])
@pytest.mark.parametrize("M,K,n_tok", F16_TILES)
def test_f16_range_within_a_chunk(M, K, n_tok, big):
    """Large activations that meet zero weights take nothing from the others'
    products: float32 sums of at most K terms, 2^-20 sum |w x|. Every other
    token has one in each 64 columns, the last also a subnormal one beside."""
    import torch
    rng = np.random.default_rng(78)
    w = (rng.standard_normal((M, K)) * 0.02).astype(np.float16)
    x = rng.standard_normal((n_tok, K)).astype(np.float32)
    at = np.arange(0, K, 64) + rng.integers(0, 64, K // 64)
    w[:, at] = 0
    x[::2, at] = np.float32(big)
    x[-1] = x[0]
    x[-1, np.delete(np.arange(K), at)[::3]] = np.float32(2.0 ** -140)
    y = binding.matvec(F16, to_gpu(w.reshape(-1).view(np.uint8)), to_gpu(x), M, K)
    torch.cuda.synchronize()
    w64, x64 = w.astype(np.float64), x.astype(np.float64)
    assert (np.abs(y.cpu().numpy() - x64 @ w64.T) <= 2.0 ** -20 * (np.abs(x64) @ np.abs(w64).T)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("n_tok", [5, 20])
def test_f16_infinities_and_nan(n_tok):
    """Infinite and NaN weights and activations give what float32 products and
    sums give, and leave every other output alone."""
    import torch
    M, K = 40, 2304
    rng = np.random.default_rng(76)
    w = (rng.standard_normal((M, K)) * 0.02).astype(np.float16)
    x = rng.standard_normal((n_tok, K)).astype(np.float32)
    w[3, 700], w[17, 0], w[39, 2303] = np.inf, -np.inf, np.nan
    x[1, 5], x[4, 1000] = np.inf, np.nan
    x[2, 700] = 0.0  # times the infinite weight: NaN
    y = binding.matvec(F16, to_gpu(w.reshape(-1).view(np.uint8)), to_gpu(x), M, K)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = (x[:, None, :].astype(np.float64) * w[None].astype(np.float64)).sum(-1)
    assert (np.isnan(y) == np.isnan(ref)).all()
    inf = np.isinf(ref)
    assert (y[inf] == ref[inf]).all()
    fine = np.isfinite(ref)
    assert np.isfinite(y[fine]).all() and np.abs(y[fine] - ref[fine]).max() < 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,n_tok", [(40, 2304, 6), (40, 6400, 3), (12300, 2048, 8)])
def test_q8_0_infinities_and_range(M, K, n_tok):
    """Q8_0 up to 8 tokens: infinite and NaN activations, and finite ones above
    bfloat16's largest, give what float32 products and sums give; tiny ones keep
    their bits. Rows 1 and up hold one code each, so that they are exact."""
    import torch
    assert binding.kernel_name(Q8_0, M, K, n_tok).endswith(", 3>")
    rng = np.random.default_rng(79)
    q = np.zeros((M, K), np.int8)
    col = rng.integers(256, K, M)
    q[np.arange(M), col] = 1
    q[0] = 1
    W = layout.pack_q8_0(q.reshape(-1), np.ones(M * K // 32, np.float16))
    x = rng.standard_normal((n_tok, K)).astype(np.float32)
    x[0, 3], x[1, 4] = np.inf, np.float32(-3.4e38)
    x[2] *= np.float32(2.0 ** -110)
    y = binding.matvec(Q8_0, to_gpu(W), to_gpu(x), M, K)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    assert y[0, 0] == np.inf and y[1, 0] == np.float32(-3.4e38)
    assert np.isnan(y[0, 1:]).all() and (y[1:, 1:] == x[1:, col[1:]]).all()  # inf x 0: NaN


def test_every_form_is_launched():
    """Every instantiation that a format selects over a grid of shapes is one
    that the shapes above launch on the GPU (no GPU here)."""
    for fmt in layout.FORMAT_NAMES:
        covered = {binding.kernel_name(fmt, *s) for s in SHAPES + FEW + [(1003, 768, 401)]}
        for M in (1, 100, 1000, 3000, 4096, 6150, 8192, 9000, 12300, 14336, 16384, 20000, 33000, 65536, 128256):
            for K in (256, 768, 1024, 1280, 2048, 2304, 3072, 4096, 6400, 8192, 14336):
                for n_tok in (2, 3, 4, 5, 6, 8, 9, 13, 16, 17, 33, 64, 77, 100, 128, 200, 401, 700, 1000):
                    kern = binding.kernel_name(fmt, M, K, n_tok)
                    assert kern in covered or not kern.startswith("kpart_kernel<"), (fmt, M, K, n_tok, kern)


def test_routes():
    """Where the rule draws its lines, and the launches of each side (no GPU)."""
    name, count = binding.kernel_name, binding.launch_count
    for fmt in layout.FORMAT_NAMES:
        if fmt != F16:
            assert count(fmt, 4096, 4096, 16) == 1 and name(fmt, 4096, 4096, 16).startswith("kpart_kernel<"), fmt
    assert name(Q8_0, 2048, 2048, 5).startswith("gemv_kernel<1, 5")      # 10240 activations: the vector kernel
    assert name(Q8_0, 2048, 2048, 6) == "kpart_kernel<1, 1, 1, 4, 3>"     # three bf16 parts
    assert name(F16, 2048, 2048, 3).startswith("gemv_kernel<")
    assert name(F16, 2048, 2048, 4) == "kpart_kernel<0, 1, 1, 2, 3>"
    assert name(Q4_0, 65536, 4096, 64) == "gemm32_kernel<2, 8>"         # tall: the tiled kernel
    assert name(Q4_0, 1024, 4096, 64) == "kpart_kernel<2, 2, 1, 16, 2>"
    assert name(Q4_0, 1024, 4096, 129) == "gemm32_kernel<2, 8>"
    assert name(Q4_K, 1000, 1 << 24, 12) == "gemm32_kernel<3, 8>"       # beyond 32-bit lane offsets
    assert count(F16, 2048, 2048, 34) == 2 and count(F16, 4096, 4096, 34) == 1


def test_routes_of_few_tokens():
    """Up to 8 tokens: one round of workgroups, and not a second one with little
    in it; long K over few rows stays with the pair-step kernel (no GPU)."""
    def here(fmt, M, K, n_tok):
        return binding.kernel_name(fmt, M, K, n_tok).startswith("kpart_kernel<")
    for n_tok in (6, 7):
        for fmt in (Q4_0, Q4_K, Q4_1):
            assert not here(fmt, 4096, 14336, n_tok) and not here(fmt, 3000, 12288, n_tok)
            assert here(fmt, 3000, 6144, n_tok) and here(fmt, 8192, 14336, n_tok) and not here(fmt, 10240, 4096, n_tok)
    for n_tok in (2, 5, 8):
        for fmt in (Q5_0, Q5_1, Q5_K, Q6_K, MXFP4):
            assert here(fmt, 4096, 14336, n_tok) and here(fmt, 8192, 4096, n_tok)
            assert not here(fmt, 20000, 3072, n_tok) and not here(fmt, 9600, 11008, n_tok)
        assert here(Q5_K, 16384, 4096, n_tok) and not here(Q5_K, 16384, 3072, n_tok)  # 12 super-blocks over 8 waves
    assert here(Q8_0, 4096, 14336, 2) and not here(Q8_0, 512, 14336, 2) and not here(Q8_0, 6144, 4096, 2)
    assert here(F16, 14336, 4096, 2) and not here(F16, 512, 14336, 2) and here(F16, 512, 2048, 4)
