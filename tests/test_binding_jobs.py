"""The binding's two ways of writing a hop_mix job down give the same bytes; what only ctypes takes or refuses goes there."""
import ctypes as C

import numpy as np
import pytest

from paper_1902_01064_amd import hop


@pytest.mark.parametrize("n", [0, 1, 5, 31, 32])
def test_packed_jobs_equal_the_structures(n):
    rnd = np.random.default_rng(n)
    ptr = lambda: int(rnd.integers(16, 1 << 47))
    jobs = [dict(out=ptr(), g=g, eta=0.01 * n, src=[ptr() for _ in range(n)], w=list(rnd.random(n)), **more)
            for g, more in ((None, {}), (ptr(), dict(vel=ptr(), mu=0.9)), (0, dict(vel=None)))]
    assert hop._pack_jobs(jobs) == bytes(hop._fill_jobs(jobs))
    jobs[0]["w"] = np.asarray(jobs[0]["w"], dtype=np.float32)
    assert hop._pack_jobs(jobs) == bytes(hop._fill_jobs(jobs))


@pytest.mark.parametrize("job", [dict(src=[np.int64(64)], w=[1.0]), dict(out=None), dict(w=[1.0, 2.0]), dict(w=[1e300]),
                                 dict(w=iter([1.0])), dict(g=1.5), dict(src=[64] * 33, w=[0.0] * 33), dict(eta="0.5")])
def test_other_jobs_are_not_packed(job):
    with pytest.raises(Exception):
        hop._pack_jobs([dict(dict(out=64, src=[64], w=[1.0]), **job)])


def test_the_library_call_takes_structures_and_packed_jobs_only():
    """One structure, an array of them, a pointer to them or nothing, as for every structure that a call takes; no bare addresses."""
    call, job = hop.load().hop_mix, hop.hop_mix_job()
    for jobs in (job, (hop.hop_mix_job * 2)(), C.pointer(job), C.byref(job), bytes(job)):
        assert call(jobs, 0, 1, None) == 0
    assert call(None, 0, 1, None) == call(None, 1, 1, None) == -1
    for jobs in (4096, "jobs", hop.hop_opts()):
        with pytest.raises(C.ArgumentError):
            call(jobs, 0, 1, None)
