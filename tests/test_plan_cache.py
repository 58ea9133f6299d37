"""The plans conv_fwd_fused keeps between calls: reused for a repeated problem, bounded, closed on
eviction and when their thread ends (host only: plans are host objects)."""
import ctypes
import threading

import pytest

from paper_1910_00078_amd import cvx


def _args(c, stream=0):
    return (cvx.CVX_BF16, (1, c, 6, 6), (4, c, 3, 3), (1, 1), (1, 1), (1, 1), 1, None, stream, None)


def test_a_repeated_problem_reuses_its_plan_and_the_cache_stays_bounded():
    cache = cvx._PlanCache()
    first = cache.get(_args(8), _args(8))
    assert cache.get(_args(8), _args(8)) is first
    assert cache.get(_args(8, stream=16), _args(8, stream=16)) is not first       # another stream, another handle
    for c in range(9, 9 + cache.LIMIT):
        cache.get(_args(c), _args(c))
    assert len(cache.plans) == cache.LIMIT
    assert first.h is None                                                        # evicted and closed
    assert cache.get(_args(8), _args(8)).y_shape == (1, 4, 6, 6)


def test_a_threads_plans_are_its_own_and_are_closed_with_it():
    seen = []

    def work():
        seen.append(cvx._per_thread.plans.get(_args(8), _args(8)))
        assert seen[0].h is not None

    t = threading.Thread(target=work)
    t.start()
    t.join()
    mine = cvx._per_thread.plans.get(_args(8), _args(8))
    assert mine is not seen[0]
    assert seen[0].h is None


@pytest.mark.gpu
def test_what_no_plan_is_made_for_finds_none():
    """Arguments that equal a kept problem's without being of its types are refused before and after it is kept."""
    import torch
    x, w = (torch.zeros(shape, dtype=torch.bfloat16, device="cuda") for shape in ((1, 8, 6, 6), (4, 8, 3, 3)))
    for _ in range(2):
        for wrong in (dict(groups=1.0), dict(policy=0.0), dict(policy=None)):
            with pytest.raises(ctypes.ArgumentError):
                cvx.conv_fwd_fused(x, w, pad=1, **wrong)
        assert cvx.conv_fwd_fused(x, w, pad=1).shape == (1, 4, 6, 6)
        assert cvx.conv_fwd_fused(x, w, pad=1, groups=True, policy=False).shape == (1, 4, 6, 6)
