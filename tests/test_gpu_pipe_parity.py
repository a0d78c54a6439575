"""GPU parity of the matrix kernel whose loads run in waves of their own (csrc/pipe_kernel.h) through the C ABI: every code
width, its three ways to split K at small sizes (tests/test_gpu_pipe_tiles.py has every tile), ragged columns, column segments,
against the CPU oracle; single weights bit for bit; the same bits alone and in a shared launch.  Few rows of 8, 6 or 3 bits at few
tokens run the streaming kernels."""
import numpy as np
import pytest

import workloads as wl
from workloads import Keep
from parity_util import NORM_TOL, NORM_TOL_BF16, TOL, TOL_BF16, linear_err, normwise_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(uref):
    import torch
    import paper_2512_03383_amd as uq
    assert torch.cuda.is_available(), "gpu tests need an MI355X"
    uq.lib()
    uref.set_threads(min(16, uref.max_threads()))
    return uq, torch


def dev16(torch, a, fmt):
    if fmt == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def gen(rng, N, K, bits, fmt, sym=False):
    w = wl.gen_linear(rng, N, K, fmt=fmt) if bits == 4 else \
        wl.gen_linear8(rng, N, K, fmt=fmt) if bits == 8 else wl.gen_linear_bits(rng, N, K, bits, fmt=fmt)
    if sym:
        w["zeros"] = None
    return w


def oracle_linear(uref, bits, w, x, keep, fmt, rows=None):
    if bits == 4:
        return uref.w4_linear(w["qweight"], w["scales"], w["zeros"], x, keep, fmt=fmt, rows=rows)
    return uref.wq_linear(bits, w["qweight"], w["scales"], w["zeros"], x, keep, fmt=fmt, rows=rows)


# (stored rows, stored columns, rule): rows around multiples of 32 and 64, 8..11 groups (whole and partial slabs of one,
# two and four groups, windows of scales that end inside the row), columns that end inside a block of eight, segments
SHAPES = [
    (129, 1024, Keep()),
    (33, 1152, Keep(n_keep=31, k_keep=1149)),
    (200, 1408, Keep(n_keep=191, k_keep=1033)),
    (320, 1280, Keep(n_keep=5 * 54, row_seg_stride=64, row_seg_keep=54, row_seg_limit=320)),
    (257, 1280, Keep(k_keep=10 * 108, col_seg_stride=128, col_seg_keep=108)),
    (97, 1152, Keep(n_keep=90, k_keep=18 * 54, col_seg_stride=64, col_seg_keep=54)),
]


# tokens around 16, 32, 48, 64, 96, 112 and 128.  So few rows take the smallest tiles: 16 or 32 tokens x 32 rows up to 64 tokens (or
# what else serves them), 64 x 64 above
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M", [2, 16, 17, 33, 48, 64, 65, 96, 113, 129])
@pytest.mark.parametrize("N,K,keep", SHAPES)
def test_linear_parity(env, uref, N, K, keep, M, fmt, bits):
    uq, torch = env
    rng = wl.rng_for(60, N + M + bits)
    w = gen(rng, N, K, bits, fmt, sym=M in (17, 64))
    qw = uq.QuantLinear.from_numpy(w, bits=bits)
    nk, kk = uq.kept_dims(qw, keep)
    x = wl.gen_activations(rng, M, kk, fmt=fmt)
    ref = oracle_linear(uref, bits, w, x, keep, fmt)
    tdt = torch.bfloat16 if fmt == "bf16" else torch.float16
    pad = M % 4          # odd and even leading dimensions; what lies between the rows must not matter
    xb = torch.full((M, kk + pad), float("nan"), dtype=tdt, device="cuda")
    xb[:, :kk] = dev16(torch, x, fmt)
    yb = torch.full((M, nk + pad), -5.0, dtype=tdt, device="cuda")
    uq.uniql_w4_linear(qw, keep, xb[:, :kk], yb[:, :nk])
    torch.cuda.synchronize()
    assert torch.all(yb[:, nk:] == -5.0), "wrote past n_keep"
    y = yb[:, :nk].float().cpu().numpy()
    assert linear_err(y, ref) <= (TOL_BF16 if fmt == "bf16" else TOL)
    if nk >= 64:
        assert normwise_err(y, ref) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL)


# taller matrices: the 64- and 96-row tiles of 33..64 tokens, the 64-row tiles of fewer
@pytest.mark.parametrize("bits,fmt", [(4, "f16"), (4, "bf16"), (8, "f16"), (6, "bf16"), (3, "f16")])
@pytest.mark.parametrize("M", [6, 12, 20, 40, 60])
@pytest.mark.parametrize("N,K,keep", [(9400, 1024, Keep(n_keep=9318)), (25000, 1152, Keep(k_keep=1100)),
                                      (6500, 4224, Keep(n_keep=6401))])
def test_tall_matrices(env, uref, N, K, keep, M, bits, fmt):
    uq, torch = env
    rng = wl.rng_for(61, N + M + bits)
    w = gen(rng, N, K, bits, fmt)
    qw = uq.QuantLinear.from_numpy(w, bits=bits)
    nk, kk = uq.kept_dims(qw, keep)
    x = wl.gen_activations(rng, M, kk, fmt=fmt)
    rows = np.unique(np.concatenate([[0, 15, 16, 31, 95, 96, nk - 2, nk - 1], rng.integers(0, nk, 64)])).astype(np.int32)
    ref = oracle_linear(uref, bits, w, x, keep, fmt, rows=rows)
    y = uq.uniql_w4_linear(qw, keep, dev16(torch, x, fmt))
    y2 = uq.uniql_w4_linear(qw, keep, dev16(torch, x, fmt))
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    assert linear_err(y.float().cpu().numpy()[:, rows], ref) <= (TOL_BF16 if fmt == "bf16" else TOL)


@pytest.mark.parametrize("bits", [4, 8, 6, 3])
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M", [16, 40, 128])
def test_one_hot_activations_return_the_weights(env, uref, M, fmt, bits):
    """A token that is one at a single column returns that column of the matrix, bit for bit: every position of a code in a
    lane's window, every step, both classes of pairs.  640 rows, or 6400 for the way that tall matrices take."""
    uq, torch = env
    rng = wl.rng_for(62, bits)
    N, K = (6400 if M == 40 else 640), 1024
    w = gen(rng, N, K, bits, fmt)
    qw = uq.QuantLinear.from_numpy(w, bits=bits)
    ref = uq.uniql_w4_dequant(qw).view(torch.int16)          # (bit-exact against the oracle in its own tests)
    for k0 in range(0, 256, M):
        cols = torch.arange(k0, k0 + M, device="cuda") % K
        x = torch.zeros((M, K), dtype=torch.bfloat16 if fmt == "bf16" else torch.float16, device="cuda")
        x[torch.arange(M, device="cuda"), cols] = 1.0
        y = uq.uniql_w4_linear(qw, None, x)
        torch.cuda.synchronize()
        # (a zero weight may have either sign: no sum can tell)
        want = ref[:, cols].T
        assert torch.equal(torch.where(want == -32768, 0, want), torch.where(y.view(torch.int16) == -32768, 0, y.view(torch.int16))), (bits, k0)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M", [40, 100])
def test_shared_launch_gives_the_same_bits(env, M, fmt):
    """q, k and v of 40 and 100 tokens (one launch) and a set that has to be split, against one call each."""
    uq, torch = env
    rng = wl.rng_for(63, M)
    for spec in ([(640, 1280), (160, 1280), (161, 1280)], [(700, 1152), (6500, 1152), (64, 1024), (48, 896)]):
        ws = [uq.QuantLinear.from_numpy(gen(rng, N, K, 4, fmt)) for N, K in spec]
        xs = [dev16(torch, wl.gen_activations(rng, M, K, fmt=fmt), fmt) for _, K in spec]
        ys = [torch.empty((M, N), dtype=xs[0].dtype, device="cuda") for N, _ in spec]
        uq.uniql_w4_linear_multi(ws, [None] * len(ws), xs, ys)
        torch.cuda.synchronize()
        for W, x, y in zip(ws, xs, ys):
            assert torch.equal(y, uq.uniql_w4_linear(W, None, x))


# the last block of a prefix: every number of columns in it, in the first block and in later blocks of a group, groups 1, 2, 3 and 4
# of a slab of four; 47 tokens (one and a half tiles of 32), 50 (64), 130 (two tiles, the second with two tokens).  NaN lies
# between the rows of x, and the last row ends with the array.
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("N,M", [(420, 47), (6410, 50), (200, 130)])
def test_ends_of_a_prefix(env, uref, N, M, fmt, bits):
    uq, torch = env
    rng = wl.rng_for(64, N + M + bits)
    K = 1536
    w = gen(rng, N, K, bits, fmt)
    qw = uq.QuantLinear.from_numpy(w, bits=bits)
    rows = np.arange(N) if N < 1000 else np.unique(np.concatenate([[0, 63, 64, N - 1], rng.integers(0, N, 40)]))
    rows = rows.astype(np.int32)
    tdt = torch.bfloat16 if fmt == "bf16" else torch.float16
    for i, kk in enumerate([1025, 1042, 1123, 1252, 1285, 1390, 1415, 1527, 1535, 1032]):
        assert uq.uniql_w4_linear_kernel(N, K, Keep(k_keep=kk), M, bits=bits, bf16=fmt == "bf16")[0] == 2
        x = wl.gen_activations(rng, M, kk, fmt=fmt)
        ref = oracle_linear(uref, bits, w, x, Keep(k_keep=kk), fmt, rows=rows)
        ld = kk + (0, 1, 3, 8)[i % 4]
        flat = torch.full(((M - 1) * ld + kk,), float("nan"), dtype=tdt, device="cuda")
        xb = flat.as_strided((M, kk), (ld, 1))
        xb.copy_(dev16(torch, x, fmt))
        y = uq.uniql_w4_linear(qw, Keep(k_keep=kk), xb)
        torch.cuda.synchronize()
        y = y.float().cpu().numpy()[:, rows]
        assert linear_err(y, ref) <= (TOL_BF16 if fmt == "bf16" else TOL), kk
        assert normwise_err(y, ref) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL), kk
