"""GPU parity of the ring kernel (csrc/ring_kernel.h): every slot of tokens and number of row fragments, ragged rows and columns, segments of
every stride, rows around the shortest that it takes, tokens next to infinities; against the CPU oracle."""
import numpy as np
import pytest

import workloads as wl
from parity_util import TOL, TOL_BF16, linear_err
from test_gpu_pipe_tiles import FORMATS, check, env, np16, oracle, weight   # noqa: F401 (env: the fixture)
from workloads import Keep

pytestmark = pytest.mark.gpu

TOKENS = [2, 4, 5, 8, 9, 16, 17, 31, 32]


def run(env, uref, N, K, M, keep, cols, fmt, zeros, pad, rows, bits=4):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(N + K + M)
    W = weight(env, g, N, K, bits, fmt, zeros=zeros)
    nk, kk = uq.kept_dims(W, keep)
    xb = torch.full((M, kk + pad), float("nan"), dtype=W.scales.dtype, device="cuda")
    xb[:, :kk] = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    yb = torch.full((M + 2, nk + 3), -5.0, dtype=W.scales.dtype, device="cuda")
    uq.uniql_w4_linear(W, keep, xb[:, :kk], yb[1:M + 1, :nk])
    torch.cuda.synchronize()
    assert torch.all(yb[0] == -5.0) and torch.all(yb[-1] == -5.0) and torch.all(yb[:, nk:] == -5.0), "wrote beside the output"
    rows = np.unique(np.asarray(rows).clip(0, nk - 1)).astype(np.int64)
    ref = oracle(uref, W, np.ascontiguousarray(np16(xb[:, :kk], fmt)), cols, fmt, torch.from_numpy(rows).cuda())
    check(yb[1:M + 1, :nk].float().cpu().numpy()[:, rows], ref, fmt)


# rows: one, two and three fragments of 16 a block (256, 512 and more row tiles); columns: the shortest rows (sixteen groups), a last group with an odd
# number of kept columns, one kept column in it
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", TOKENS)
@pytest.mark.parametrize("N,K,kk", [(61, 2048, 2048), (4089, 2048, 1921), (4117, 2304, 2291), (8200, 2176, 2049), (9589, 2176, 2174)])
def test_prefixes(env, uref, N, K, kk, M, fmt):   # noqa: F811
    rng = wl.rng_for(76, N + M)
    rows = np.concatenate([np.arange(0, N, 256), [15, 16, 47, 48, N - 17, N - 4, N - 1], rng.integers(0, N, 40)])
    uq, _ = env
    ld = kk + (-kk) % 8
    choice = uq.uniql_w4_linear_kernel(N, K, Keep(n_keep=N - 2, k_keep=kk), M, bf16=fmt == "bf16", ldx=ld)
    assert choice[0] == 1
    run(env, uref, N, K, M, Keep(n_keep=N - 2, k_keep=kk), Keep(k_keep=kk), fmt, M % 2 == 0, ld - kk, rows)


# taller matrices: five and six fragments of 16 a block, and 12801 and 16260 rows, which would have four and go to other kernels
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [9, 16, 19, 32])
@pytest.mark.parametrize("N,kk", [(12801, 2048), (16260, 2048), (16393, 2051), (19203, 2175), (21001, 2173), (24570, 2050)])
def test_tall_prefixes(env, uref, N, kk, M, fmt):   # noqa: F811
    rng = wl.rng_for(77, N + M)
    rows = np.concatenate([np.arange(0, N, 512), [15, 16, 63, 64, 79, 80, 111, 112, 127, 128, N - 17, N - 4, N - 1], rng.integers(0, N, 40)])
    run(env, uref, N, 2176, M, Keep(n_keep=N - 2, k_keep=kk), Keep(k_keep=kk), fmt, M % 2 == 0, (-kk) % 8, rows)


# up to 8 tokens, three fragments, and from five tokens on six: rows of up to 32 groups up to 639 row tiles, shorter and longer ones above
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M,N,K,kk", [(M, *size) for M in (2, 4, 5, 8) for size in ((10226, 2176, 2171), (10243, 4352, 4225), (12290, 4224, 4224), (11999, 1920, 1913), (12001, 2432, 2427), (22003, 4352, 4350), (24578, 4224, 4098))
                                      if M > 4 or size[0] < 12000 or size[0] == 12290])
def test_tall_prefixes_of_few_tokens(env, uref, N, K, kk, M, fmt):   # noqa: F811
    rng = wl.rng_for(79, N + M)
    rows = np.concatenate([np.arange(0, N, 512), [15, 16, 63, 64, 79, 80, 111, 112, 127, 128, N - 17, N - 4, N - 1], rng.integers(0, N, 40)])
    ld = kk + (-kk) % 8
    assert env[0].uniql_w4_linear_kernel(N, K, Keep(n_keep=N - 2, k_keep=kk), M, bf16=fmt == "bf16", ldx=ld)[3] == 8
    run(env, uref, N, K, M, Keep(n_keep=N - 2, k_keep=kk), Keep(k_keep=kk), fmt, M % 2 == 0, ld - kk, rows)


# gate and up with h = SiLU(g) * u: three or four pairs of fragments a block, one round and more; rows kept apart; one matrix without zero points.
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [9, 15, 16])
@pytest.mark.parametrize("N,K,keep", [(10233, 2048, Keep(k_keep=1921)), (12185, 4096, Keep(k_keep=3968)), (16300, 2176, Keep(n_keep=16299)), (20011, 2304, Keep(k_keep=2302)),
                                      (24573, 2048, Keep()), (14400, 2176, Keep(n_keep=12000, row_seg_stride=96, row_seg_keep=80, row_seg_limit=14400))])
def test_gated_pair(env, uref, N, K, keep, M, fmt):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(N + K + M)
    ws = [weight(env, g, N, K, 4, fmt, zeros=i == 0) for i in range(2)]
    nk, kk = uq.kept_dims(ws[0], keep)
    xb = torch.full((M, kk + (-kk) % 8), float("nan"), dtype=ws[0].scales.dtype, device="cuda")
    x = xb[:, :kk]
    x.copy_(torch.randn((M, kk), generator=g, device="cuda"))
    hb = torch.full((M + 2, nk + 3), -5.0, dtype=x.dtype, device="cuda")
    uq.uniql_w4_gate_up_silu_batch(ws, [keep] * 2, x, hb[1:M + 1, :nk])
    torch.cuda.synchronize()
    assert torch.all(hb[0] == -5.0) and torch.all(hb[-1] == -5.0) and torch.all(hb[:, nk:] == -5.0), "wrote beside the output"
    rows = np.unique(np.concatenate([np.arange(0, nk, 512), [15, 16, 31, 32, 47, 48, 63, 64, nk - 17, nk - 4, nk - 1]]).clip(0, nk - 1)).astype(np.int64)
    stored = rows // keep.row_seg_keep * keep.row_seg_stride + rows % keep.row_seg_keep if keep.row_seg_stride else rows
    go, up = (oracle(uref, w, np.ascontiguousarray(np16(x, fmt)), Keep(k_keep=kk), fmt, torch.from_numpy(stored).cuda()).astype(np.float64) for w in ws)
    ref = go * up / (1.0 + np.exp(-go))
    # (element by element alone: a few products carry a token's norm, and the rounding of one is up to 2^-8 of it in bfloat16)
    assert linear_err(hb[1:M + 1, :nk].float().cpu().numpy()[:, rows], ref) <= (TOL_BF16 if fmt == "bf16" else TOL)


# the two matrices with row rules of their own (the same number of kept rows) and of different heights
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [9, 16])
@pytest.mark.parametrize("K,heights,keeps", [
    (2048, (12000, 14400), (Keep(n_keep=12000, k_keep=2045), Keep(n_keep=12000, k_keep=2045, row_seg_stride=96, row_seg_keep=80, row_seg_limit=14400))),
    (2176, (20480, 16005), (Keep(n_keep=16000, row_seg_stride=128, row_seg_keep=100, row_seg_limit=20480), Keep(n_keep=16000))),
    (2304, (15000, 16000), (Keep(n_keep=11000, row_seg_stride=60, row_seg_keep=44, row_seg_limit=15000), Keep(n_keep=11000, row_seg_stride=64, row_seg_keep=44, row_seg_limit=16000)))])
def test_gated_pair_of_two_row_rules(env, uref, K, heights, keeps, M, fmt):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(K + M)
    ws = [weight(env, g, N, K, 4, fmt, zeros=i == 1) for i, N in enumerate(heights)]
    nk, kk = uq.kept_dims(ws[0], keeps[0])
    assert (nk, kk) == uq.kept_dims(ws[1], keeps[1])
    x = torch.zeros((M, kk + (-kk) % 8), dtype=ws[0].scales.dtype, device="cuda")[:, :kk]
    x.copy_(torch.randn((M, kk), generator=g, device="cuda"))
    h = torch.empty((M, nk), dtype=x.dtype, device="cuda")
    uq.uniql_w4_gate_up_silu_batch(ws, list(keeps), x, h)
    rows = np.unique(np.concatenate([np.arange(0, nk, 256), np.arange(40, 240, 20), [15, 16, 31, 32, nk - 17, nk - 1]])).astype(np.int64)
    go, up = (oracle(uref, w, np.ascontiguousarray(np16(x, fmt)), Keep(k_keep=kk), fmt,
                     torch.from_numpy(rows // k.row_seg_keep * k.row_seg_stride + rows % k.row_seg_keep if k.row_seg_stride else rows).cuda()).astype(np.float64) for w, k in zip(ws, keeps))
    # (element by element alone, as above)
    assert linear_err(h.float().cpu().numpy()[:, rows], go * up / (1.0 + np.exp(-go))) <= (TOL_BF16 if fmt == "bf16" else TOL)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [3, 16, 24])
@pytest.mark.parametrize("stride,keep", [(8, 8), (16, 10), (16, 14), (32, 26), (64, 38), (64, 64), (128, 8), (128, 94), (128, 108), (128, 126)])
def test_segments(env, uref, stride, keep, M, fmt):   # noqa: F811
    N, K = 203, 2176
    k = Keep(k_keep=K // stride * keep, col_seg_stride=stride, col_seg_keep=keep)
    run(env, uref, N, K, M, k, k, fmt, M % 2 == 0, M % 3, np.concatenate([np.arange(0, N, 97), [N - 1]]))


# the same with rows of 33 to 96 groups and 17 tokens and more
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M,N,K,stride,keep", [(17, 207, 4224, 128, 94), (32, 3070, 8192, 64, 50), (24, 4095, 4352, 128, 126), (31, 1001, 12288, 128, 96), (18, 2563, 8320, 32, 24)])
def test_segments_of_long_rows(env, uref, M, N, K, stride, keep, fmt):   # noqa: F811
    k = Keep(k_keep=K // stride * keep, col_seg_stride=stride, col_seg_keep=keep)
    assert env[0].uniql_w4_linear_kernel(N, K, k, M, bf16=fmt == "bf16", ldx=k.k_keep + M % 3)[3] == 8
    run(env, uref, N, K, M, k, k, fmt, M % 2 == 0, M % 3, np.concatenate([np.arange(0, N, 97), [N - 1]]))


# rows of 8 to 15 groups, whose window of zero points ends in the next row, or, the last row's, starts in the one before
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [2, 7, 16, 31])
@pytest.mark.parametrize("N,K,kk", [(2, 1024, 1024), (17, 1152, 1029), (47, 1408, 1407), (600, 1920, 1921 - 128), (4117, 1280, 1274), (5000, 1920, 1920), (9577, 1664, 1650)])
def test_short_rows(env, uref, N, K, kk, M, fmt):   # noqa: F811
    rng = wl.rng_for(80, N + M)
    ld = kk + (-kk) % 8
    assert env[0].uniql_w4_linear_kernel(N, K, Keep(k_keep=kk), M, bf16=fmt == "bf16", ldx=ld)[3] == 8
    run(env, uref, N, K, M, Keep(k_keep=kk), Keep(k_keep=kk), fmt, (N + M) % 4 != 0, ld - kk, np.concatenate([np.arange(0, N, 256), np.arange(max(0, N - 20), N), rng.integers(0, N, 30)]))


# rows of one to three runs of groups a wave, fewer groups than the loads in flight, more, and the windows of eight scales and sixteen zero points
# at the row's end
@pytest.mark.parametrize("M", [2, 8, 16, 32])
@pytest.mark.parametrize("K", [2048, 2176, 3072, 3200, 4096 + 128 * 7, 18944, 40960])
def test_row_lengths(env, uref, K, M):   # noqa: F811
    N = 36
    run(env, uref, N, K, M, Keep(), Keep(), "f16", True, 0, np.arange(N))
    run(env, uref, N, K, M, Keep(k_keep=K - 128), Keep(k_keep=K - 128), "bf16", False, 0, np.arange(N))


# the same bits in a shared launch, whose blocks have more rows (four, six, seven and eight fragments), as alone
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [2, 8, 16, 30])
@pytest.mark.parametrize("sizes", [(5000, 6300, 5003, 4999), (12285, 12270, 999), (8000, 8100), (12285, 12270, 5003), (9001, 16401)])
def test_shared_launch(env, uref, sizes, M, fmt):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(M)
    K = 2176
    ws = [weight(env, g, N, K, 4, fmt, zeros=i != 1) for i, N in enumerate(sizes)]
    x = torch.randn((M, K), generator=g, device="cuda").to(ws[0].scales.dtype)
    ys = [torch.empty((M, w.N), dtype=x.dtype, device="cuda") for w in ws]
    uq.MultiCall(ws, [None] * len(ws), [x] * len(ws), ys).run()
    for w, y in zip(ws, ys):
        assert torch.equal(y, uq.uniql_w4_linear(w, None, x))


# the same for tall matrices of long rows at up to 8 tokens, and for rows of fewer than sixteen groups beside longer ones
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M,shapes", [(2, ((12285, 4352), (999, 4224))), (8, ((22003, 4224), (5003, 4224), (300, 5248))), (16, ((9001, 2176), (16401, 2176))), (30, ((16401, 2176), (5003, 1152))),
                                      (8, ((4096, 1152), (4096, 2176), (77, 1024))), (24, ((6003, 1920), (2048, 4096)))])
def test_shared_launch_of_tall_and_short(env, uref, M, shapes, fmt):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(M)
    ws = [weight(env, g, N, K, 4, fmt, zeros=i != 1) for i, (N, K) in enumerate(shapes)]
    assert all(uq.uniql_w4_linear_kernel(N, K, None, M, bf16=fmt == "bf16")[3] == 8 for N, K in shapes)
    xs = [torch.randn((M, K), generator=g, device="cuda").to(ws[0].scales.dtype) for _, K in shapes]
    ys = [torch.empty((M, w.N), dtype=x.dtype, device="cuda") for w, x in zip(ws, xs)]
    uq.MultiCall(ws, [None] * len(ws), xs, ys).run()
    for w, x, y in zip(ws, xs, ys):
        assert torch.equal(y, uq.uniql_w4_linear(w, None, x))
    rows = np.unique(np.array([0, 15, 16, ws[0].N // 2, ws[0].N - 1]))
    ref = oracle(uref, ws[0], np.ascontiguousarray(np16(xs[0], fmt)), Keep(k_keep=shapes[0][1]), fmt, torch.from_numpy(rows).cuda())
    check(ys[0].float().cpu().numpy()[:, rows], ref, fmt)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [7, 16, 32])
@pytest.mark.parametrize("keep", [Keep(k_keep=2045), Keep(k_keep=2054), Keep(k_keep=17 * 102, col_seg_stride=128, col_seg_keep=102), Keep(k_keep=68 * 26, col_seg_stride=32, col_seg_keep=26)])
def test_tokens_next_to_infinities(env, uref, keep, M, fmt):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(M)
    W = weight(env, g, 5000, 2176, 4, fmt)
    kk = uq.kept_dims(W, keep)[1]
    x = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    clean = uq.uniql_w4_linear(W, keep, x)
    bad = torch.arange(M, device="cuda") % 3 == 1
    x2 = x.clone()
    x2[bad] = torch.where(torch.rand((int(bad.sum()), kk), generator=g, device="cuda") < 0.5, float("inf"), float("nan")).to(x.dtype)
    y = uq.uniql_w4_linear(W, keep, x2)
    assert torch.equal(y[~bad], clean[~bad]) and torch.all(torch.isfinite(clean))


# bfloat16 scales whose unpack takes the wide form, beside ordinary ones
@pytest.mark.parametrize("M", [8, 24])
def test_largest_scales(env, uref, M):   # noqa: F811
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(M)
    W = weight(env, g, 200, 2176, 4, "bf16")
    W.scales[::7, 3] = 2.0 ** 118
    x = torch.zeros((M, 2176), dtype=torch.bfloat16, device="cuda")
    x[:, 3 * 128:4 * 128] = (torch.randn((M, 128), generator=g, device="cuda") * 1e-20).bfloat16()
    y = uq.uniql_w4_linear(W, None, x)
    ref = oracle(uref, W, np16(x, "bf16"), Keep(), "bf16", torch.arange(200, device="cuda"))
    check(y.float().cpu().numpy()[:, ::7], ref[:, ::7], "bf16")
    assert torch.all(torch.isfinite(y.float()))


# codes of 8, 6 and 3 bits: one to six fragments a block, windows of the codes inside words (3 bits, 17 tokens and more), loads that hold more units
# than the tile has, rows as in test_prefixes
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits", [8, 6, 3])
@pytest.mark.parametrize("M", [5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("N,K,kk", [(2061, 2176, 2049), (3061, 2304, 2177), (3061, 4608, 4481), (3050, 5248, 5248), (5003, 2432, 2305), (9018, 2304, 2291), (13005, 2560, 2559), (17003, 2432, 2430), (22003, 2304, 2304)])
def test_wide_prefixes(env, uref, N, K, kk, M, bits, fmt):   # noqa: F811
    uq, _ = env
    ld = kk + (-kk) % 8
    choice = uq.uniql_w4_linear_kernel(N, K, Keep(n_keep=N - 2, k_keep=kk), M, bits=bits, bf16=fmt == "bf16", ldx=ld)
    if choice[3] != 8:
        assert (N == 5003 and bits != 6) or (N == 13005 and bits == 3)
        return
    rng = wl.rng_for(78, N + M)
    rows = np.concatenate([np.arange(0, N, 512), [15, 16, 31, 47, 48, 63, 64, 79, 80, 95, 96, N - 17, N - 4, N - 1], rng.integers(0, N, 40)])
    run(env, uref, N, K, M, Keep(n_keep=N - 2, k_keep=kk), Keep(k_keep=kk), fmt, M % 2 == 0, ld - kk, rows, bits)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits", [8, 6, 3])
@pytest.mark.parametrize("M", [7, 16, 24])
@pytest.mark.parametrize("stride,keep", [(8, 2), (8, 6), (16, 10), (32, 4), (32, 26), (64, 38), (128, 8), (128, 94), (128, 126)])
def test_wide_segments(env, uref, stride, keep, M, bits, fmt):   # noqa: F811
    uq, _ = env
    N, K = 3003, 2432
    k = Keep(k_keep=K // stride * keep, col_seg_stride=stride, col_seg_keep=keep)
    assert uq.uniql_w4_linear_kernel(N, K, k, M, bits=bits, bf16=fmt == "bf16", ldx=K // stride * keep + M % 3)[3] == 8
    run(env, uref, N, K, M, k, k, fmt, M % 2 == 0, M % 3, np.concatenate([np.arange(0, N, 97), [N - 1]]), bits)
