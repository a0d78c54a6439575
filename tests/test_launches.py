"""What the library launches, on the CPU (tests/launches.py)."""
import pytest

import launches as la


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    directory = tmp_path_factory.mktemp("recorder")
    return lambda calls: la.record(calls, directory)


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
