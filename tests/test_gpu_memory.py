"""Device memory of handles: the registered allocator, the blocks that freed
handles leave for the next one."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


class Refusing:
    """torch's caching allocator, but nothing past a limit."""

    def __init__(self, limit):
        from paper_1902_01458_amd import _lib
        self.asked, self.live = [], set()

        def alloc(nbytes, stream, ctx):
            self.asked.append(int(nbytes))
            if nbytes > limit:
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), stream=stream or 0)
            self.live.add(p)
            return p

        def free(ptr, ctx):
            self.live.remove(ptr)
            torch.cuda.caching_allocator_delete(ptr)

        self.lib = _lib.lib()
        self.callbacks = (_lib.ALLOC_FN(alloc), _lib.FREE_FN(free))
        self.none = (_lib.ALLOC_FN(), _lib.FREE_FN())

    def __enter__(self):
        assert self.lib.rr_set_allocator(*self.callbacks, None) == 0
        return self

    def __exit__(self, *_):
        assert self.lib.rr_set_allocator(*self.none, None) == 0


def test_the_allocator_decides_what_fits():
    """A batch whose factors exceed the device is the registered allocator's to
    refuse (it may hold memory elsewhere): it is asked for all of them, and
    what it gave before comes back."""
    w = W.small("nm", 64, 32, nu=1e-2)
    prob = rr().BurgersProblem.from_workload(w)
    shifts = 400_000
    with Refusing(1 << 30) as a:
        with pytest.raises(rr().RRError) as e:
            rr().factor(prob, [1.0] * shifts, "fp64", k_max=2)
        assert e.value.status == 6  # RR_ERR_NOMEM
        assert max(a.asked) >= 16 * 16 * w.n * shifts > torch.cuda.mem_get_info()[1]
        assert not a.live
        f = rr().factor(prob, [1.0], "fp64", k_max=2)
        f.check()
        f.free()
        assert not a.live


def test_what_no_device_holds_is_out_of_memory():
    w = W.small("nm", 64, 32, nu=1e-2)
    prob = rr().BurgersProblem.from_workload(w)
    for prec in ("fp64", "mixed"):
        with pytest.raises(rr().RRError) as e:
            rr().factor(prob, [1.0] * 1_000_000, prec, k_max=2)
        assert e.value.status == 6
    f = rr().factor(prob, [1.0], "fp64", k_max=2)
    f.check()
    f.free()


def test_blocks_of_freed_handles_are_given_back_on_request():
    w = W.small("rm", 128, 64, nu=1e-2)
    prob = rr().BurgersProblem.from_workload(w)
    rr().release_memory()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    f = rr().factor(prob, [0.5, 1.0, 2.0, 3.0], "fp64", k_max=16)
    f.check()
    held = f.nbytes()
    f.free()
    assert before - torch.cuda.mem_get_info()[0] > held // 2 > 50 << 20  # kept for the next handle
    live = rr().factor(prob, [0.5], "fp64", k_max=16)
    B = torch.randn((1, 16, w.n), dtype=torch.complex128, device="cuda")
    X = live.solve(B)
    rr().release_memory()  # a live handle's blocks stay
    assert torch.equal(live.solve(B), X)
    live.check()
    live.free()
    rr().release_memory()
    del B, X
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] <= 16 << 20
