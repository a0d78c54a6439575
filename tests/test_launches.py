"""What the library launches, on the CPU (tests/launches.py)."""
import pytest

import launches as la
import pipe_shapes as ps
import paper_2512_03383_amd as uq


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    directory = tmp_path_factory.mktemp("recorder")
    return lambda calls, **kw: la.record(calls, directory, **kw)


def linear(N, K, M, keep={}, **kw):
    return dict(specs=[(N, K, keep)], M=M, **kw)


# The limit of a kernel's dynamic LDS belongs to the kernel, whichever thread sets it: if calls set what they need themselves, one thread may
# lower it between another's set and launch.  Every call sets the same value, at least what any needs.
def test_limit_of_lds_does_not_depend_on_the_call(record):
    calls = [linear(N, K, M, bits=bits) for bits in (4, 8, 6, 3) for K in (2048, 4096, 5248, 10496, 14336, 18944) for N in (600, 4096, 9000) for M in (4, 8, 16, 32)]
    calls += [dict(specs=[(N, K, {})] * 2, M=M, glu=glu) for N, K in ((12185, 4096), (14336, 2048), (20000, 3584)) for M in (12, 32) for glu in (True, False) if not (glu and M > 16)]
    limits = {}
    for rc, launches in record(calls):
        assert rc == 0
        for x in launches:
            assert x.lds <= max(x.limit, 64 * 1024)
            assert limits.setdefault(x.kernel, x.limit) == x.limit, x.kernel
    assert sum("w_ring_kernel" in k for k in limits) > 20


def reported(kernel):
    """What uniql_w4_linear_kernel says of a launch of this kernel."""
    name, args = kernel.rstrip(">").split("<")
    a = [int(x) if x.isdigit() else x == "true" for x in args.split(",")]
    if name == "w_ring_kernel":
        return (1, a[0], 16 * a[1], 8)
    if name == "w_pipe_kernel":
        return (2, 16 * a[0], 16 * a[1] * a[2], a[3] * a[4])
    return {"w4_smallm_kernel": (1, 0, 0, 0), "w8_gemv_kernel": (0, 0, 0, 0), "wb_gemv_kernel": (0, 0, 0, 0), "w4_prefill_kernel": (3, 256, 256, 1)}.get(name, (4,))


@pytest.mark.parametrize("bits", [4, 8, 6, 3])
@pytest.mark.parametrize("keep", [{}, dict(col_seg_stride=128, col_seg_keep=102), dict(col_seg_stride=32, col_seg_keep=24)])
def test_the_report_names_the_kernel_that_is_launched(record, keep, bits):
    sizes = [(N, K, M) for N in (300, 2048, 4096, 6410, 9472, 13000, 18944, 26000) for K in (1152, 2176, 4096, 5120, 8192) for M in (2, 5, 8, 9, 16, 17, 32, 48, 130, 1000)]
    calls = [linear(N, K, M, keep, bits=bits, bf16=(N + M) % 2 == 1) for N, K, M in sizes]
    seen = set()
    for (N, K, M), call, (rc, launches) in zip(sizes, calls, record(calls)):
        choice = uq.uniql_w4_linear_kernel(N, K, uq.KeepDesc(**keep), M, bits=bits, bf16=call["bf16"])
        want = reported(launches[0].kernel)
        assert rc == 0 and len(launches) == 1 and choice[:len(want)] == want, (N, K, M, launches[0].kernel, choice)
        seen.add(launches[0].kernel.split("<")[0])
    assert {"w_ring_kernel", "w_pipe_kernel"} <= seen


# decode batches of tall and short matrices: one launch where one kernel takes them all
@pytest.mark.parametrize("M", [2, 5, 8])
def test_decode_batches_of_mixed_heights(record, M):
    sets = [[(12288, 8192, {}), (1024, 8192, {}), (1024, 8192, {})], [(10240, 5120, {}), (1024, 5120, {})], [(12200, 1920, {}), (1024, 1920, {})],
            [(9700, 4096, {}), (4096, 4096, {})], [(4096, 1536, {}), (4096, 4096, {})], [(2048, 1024, {}), (1024, 2048, {}), (300, 1920, {})], [(8192, 4096, {}), (1024, 4096, {}), (1024, 4096, {})]]
    assert [len(launches) for _, launches in record([dict(specs=s, M=M) for s in sets])] == [1] * len(sets)
    tall = [[(12288, K, {}), (1024, K, {}), (1024, K, {})] for K in (2048, 2560, 4096)]
    assert [[len(launches) for _, launches in record([dict(specs=s, M=M, bf16=b) for s in tall])] for b in (False, True)] == ([[1, 1, 2], [1, 1, 1]] if M > 4 else [[2, 2, 2], [1, 1, 2]])


# rows of fewer than sixteen groups and longer ones in one launch
@pytest.mark.parametrize("M", [12, 24])
def test_decode_batches_of_mixed_lengths(record, M):
    sets = [[(4096, 1536, {}), (4096, 4096, {})], [(2048, 1024, {}), (1024, 2048, {})], [(6384, 1920, {}), (6384, 14336, {}), (200, 1024, {})]]
    assert [len(launches) for _, launches in record([dict(specs=s, M=M) for s in sets])] == [1] * len(sets)


# the last round of a grid as halves: two blocks for each of its tiles
@pytest.mark.parametrize("bf16", [False, True])
def test_last_round_goes_out_as_halves(record, bf16):
    calls = [linear(N, K, M, ps.halves_rule(K, N, segments), bits=bits, bf16=bf16) for bits, K, N, M, segments, _ in ps.HALVES]
    for (bits, K, N, M, segments, tokens), (rc, launches) in zip(ps.HALVES, record(calls)):
        tile = reported(launches[0].kernel)[1:3]
        halves, tiles = ps.half_tiles(N - 3, M, tile)
        assert rc == 0 and tile[0] == tokens and halves > 0 and launches[0].blocks == tiles + halves, (bits, K, N, M, launches)


# lines that are rounds of the compute units follow the device's number of them
@pytest.mark.parametrize("cus", [256, 128])
def test_rounds_are_the_devices(record, cus):
    def ring(bits, M, *row_tiles):
        return ["w_ring_kernel" in launches[0].kernel for _, launches in record([linear(16 * n, 4096, M, bits=bits) for n in row_tiles], compute_units=cus)]
    for bits in (8, 3):   # one round of the pipelined kernel's 32-row tiles
        assert ring(bits, 16, cus, cus + 1, 2 * cus, 2 * cus + 1) == [True, False, False, True]
    assert ring(3, 16, 3 * cus, 3 * cus + 1, 4 * cus, 4 * cus + 1) == [True, False, False, True]   # four fragments a block
