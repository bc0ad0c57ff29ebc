"""When device memory of a plan may serve the next one: after all work on the
device, on every stream, and back to the system when asked for."""

import pytest

import latgen

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _lattice(n=8):
    return latgen.bcc(n, ("uniform", 0.05, 0.12), 0.05, seed=n)


def _long_work(torch, stream):
    """Some ten milliseconds of other work on another stream; its end as an event."""
    a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(stream):
        for _ in range(40):
            a @ a
        done.record()
    return done


@pytest.mark.parametrize("how", ["destroy", "larger records", "larger second records"])
def test_memory_is_given_up_only_after_work_on_other_streams(how):
    """The other stream could be replaying a graph of the plan's calls."""
    import torch

    from paper_2405_15197_amd import Mesher

    m, other = Mesher(_lattice()), torch.cuda.Stream()
    try:
        r = m.run(6)
        if how == "larger second records":
            m.retriangulate(6, r=m.alloc({k: 8 * v + 64 for k, v in r.totals.items()}))
        _long_work(torch, other).synchronize()  # (the first product prepares itself)
        done = _long_work(torch, other)
        assert not done.query()
        if how == "destroy":
            m.close()
        elif how == "larger records":
            m.count(300)
        else:
            from paper_2405_15197_amd import latmesh

            latmesh.lm_retriangulate(m.plan, 60, m.outputs(r))
        assert done.query()
    finally:
        torch.cuda.synchronize()
        m.close()


def test_kept_memory_is_released_on_request():
    import torch

    from paper_2405_15197_amd import Mesher, latmesh

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    live = Mesher(_lattice(6))
    want = live.count(12)
    latmesh.lm_release_memory()
    before = free()
    plans = [Mesher(_lattice(24)) for _ in range(3)]
    for m in plans:
        m.count(16)
    used = before - free()
    for m in plans:
        m.close()
    del plans
    latmesh.lm_release_memory()
    assert used > 128 * MIB
    assert before - free() <= 8 * MIB  # the runtime's own
    latmesh.lm_release_memory()  # nothing left: no effect
    assert live.count(12) == want
    live.close()
