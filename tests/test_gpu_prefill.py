"""Prefill (more than 16 tokens; every quantized format) on the matrix
cores against the oracle: several row and token tiles with ragged tails, the
tiled kernels' K-split launch (partial products added into a zeroed y) with an
uneven last split and a half coefficient window, and their unsplit launch.

Bar: the gate, and the float32 bound 1e-4 * sum |w*x| + 2^-17 * F (the
activations enter the matrix cores as a bf16 high/low pair, exact to 2^-17;
F the term mass of the biased-code form, tests/gate.py)."""
import numpy as np
import pytest

import gate
from gpu_util import gpu_matvec, to_gpu
from parity import reference
from paper_2605_20706_amd import binding, synth
from paper_2605_20706_amd.layout import F16, MXFP4, Q1_0, Q2_K, Q4_0, Q4_1, Q4_K, Q5_0, Q5_1, Q5_K, Q6_K, Q8_0

pytestmark = pytest.mark.gpu


def run(oracle_mod, fmt, M, K, n_tok, seed):
    W = synth.gen_packed(fmt, M * K, np.random.default_rng([seed, fmt, M, K]))
    x = synth.gen_x_seeded([seed + 1, fmt, K], K, n_tok)
    kern = binding.kernel_name(fmt, M, K, n_tok)
    print("prefill fmt=%d M=%d K=%d n_tok=%d kernel=%s" % (fmt, M, K, n_tok, kern), flush=True)
    y = gpu_matvec(fmt, W, x, M, K, Wg=to_gpu(W))
    y_ref, A, F = reference(oracle_mod, fmt, W, x, M, K, kern)
    gate.check(y, y_ref, A, F, f32_bound=1e-4, what=(fmt, M, K, n_tok))


@pytest.mark.parametrize("fmt", [Q4_0, Q4_K, Q4_1, Q8_0, Q5_0, Q5_1, Q5_K, Q6_K, Q2_K, MXFP4, Q1_0])
@pytest.mark.parametrize("M,K,n_tok", [
    (1100, 4352, 100),  # ragged rows and tokens, 17 super-blocks: K split over the waves
    (300, 1024, 17),    # 17 tokens (one past a token tile), the same kernel
    (8192, 512, 240),   # 16 x 4 tiles of the tiled kernel, unsplit (two super-blocks)
    (41, 2048, 67),     # 41 rows, K split over the waves
])
def test_prefill_tiles(oracle_mod, fmt, M, K, n_tok):
    run(oracle_mod, fmt, M, K, n_tok, 50)


TILED = [(Q8_0, "gemm_kernel<1, 4, 2>")] + [(f, "gemm32_kernel<%d, 8>" % f) for f in (
    Q4_0, Q4_K, Q4_1, Q5_0, Q5_1, Q5_K, Q6_K, Q2_K, MXFP4, Q1_0)]


@pytest.mark.parametrize("fmt,kern", TILED)
@pytest.mark.parametrize("M,K,n_tok,q8_tok,launches", [
    (1100, 4352, 200, 1030, 2),  # ragged rows and tokens; K split with a shorter last part
    (300, 1024, 145, 1025, 1),   # one row tile, one token past a token tile; unsplit (4 super-blocks)
    (41, 2048, 150, 1059, 2),    # most of the row tile masked; two K splits; an output with a fill tail
])
def test_tiled_kernels(oracle_mod, fmt, kern, M, K, n_tok, q8_tok, launches):
    """The tiled kernels, beyond the tokens that the kernel with K split over
    its waves takes (128; Q8_0: 1024)."""
    n_tok = q8_tok if fmt == Q8_0 else n_tok
    assert (binding.kernel_name(fmt, M, K, n_tok), binding.launch_count(fmt, M, K, n_tok)) == (kern, launches)
    run(oracle_mod, fmt, M, K, n_tok, 52)


@pytest.mark.parametrize("fmt", [F16])
@pytest.mark.parametrize("M,K,n_tok", [(300, 2304, 517), (1, 256, 64)])
def test_token_blocks_one_launch(oracle_mod, fmt, M, K, n_tok):
    """f16: 517 tokens in one launch of the kernel with K split over its
    waves, and (K = 256, one row) 64 tokens on it too."""
    assert binding.launch_count(fmt, M, K, n_tok) == 1
    run(oracle_mod, fmt, M, K, n_tok, 70)


@pytest.mark.parametrize("fmt", [Q4_0, Q4_K])
def test_prefill_repeat_equal(oracle_mod, fmt):
    """The unsplit launch, and the kernel with K split over its waves, write y
    with plain stores: two calls give the same bits. The split launch adds
    partials in any order: two calls agree to the float32 rounding of those
    additions."""
    import torch
    for M, K, n_tok, exact in [(8192, 512, 240, True), (1100, 4352, 100, True), (1100, 4352, 200, False)]:
        W = to_gpu(synth.gen_packed(fmt, M * K, np.random.default_rng([60, fmt, M])))
        x = to_gpu(synth.gen_x_seeded([61, fmt], K, n_tok))
        a = binding.matvec(fmt, W, x, M, K)
        b = binding.matvec(fmt, W, x, M, K)
        torch.cuda.synchronize()
        if exact:
            assert torch.equal(a, b), (M, K, n_tok)
        else:
            d = (a - b).abs().max().item()
            assert d <= 1e-5 * a.abs().max().item(), (M, K, n_tok, d)
