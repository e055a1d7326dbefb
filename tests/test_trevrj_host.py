"""What TrevrJ and Tree ask for in memory, without a GPU: stand-ins for the
tree or the library record the calls."""
import ctypes

import pytest
import torch

from paper_2310_15235_amd import api


class _Tree:
    reserved = 0

    def __init__(self, x, y, z, m, rho, kappa, lum, **opts):
        self.shape = tuple(lum.shape)

    def reserve_adjoint(self, active=None):
        _Tree.reserved += 1

    def compute_J(self, active=None, bg=None):
        return torch.zeros(self.shape, dtype=torch.float64)

    def compute_J_backward(self, gJ, active=None, bg=None):
        return gJ, gJ, gJ.sum(0)


# room for an adjoint only where one can follow
@pytest.mark.parametrize("grad,mode,want", [(True, None, 1), (False, None, 0),
                                            (True, torch.no_grad, 0),
                                            (True, torch.inference_mode, 0)])
def test_room_only_where_gradients_are_recorded(monkeypatch, grad, mode, want):
    monkeypatch.setattr(api, "Tree", _Tree)
    _Tree.reserved = 0
    v = [torch.ones(5) for _ in range(5)] + [torch.ones(2, 5) for _ in range(2)]
    if grad:
        for a in v[4:]:
            a.requires_grad_(True)
    if mode is None:
        J = api.TrevrJ.apply(*v, None, None, {})
    else:
        with mode():
            J = api.TrevrJ.apply(*v, None, None, {})
    assert _Tree.reserved == want
    assert J.requires_grad == (want == 1)
    if want:
        g = torch.autograd.grad(J.sum(), v[4:])
        assert [tuple(a.shape) for a in g] == [(5,), (2, 5), (2, 5)]


# a forward whose room for the adjoint does not fit the memory runs without it
@pytest.mark.parametrize("reserve", [False, True])
def test_forward_without_room_where_memory_is_short(monkeypatch, reserve):
    class Lib:
        room = False
        need = 0

        def trevr_scratch_needed(self, handle, out):
            ctypes.cast(out, ctypes.POINTER(ctypes.c_size_t))[0] = self.need
            return api.OK

        def trevr_tree_tune(self, handle, key, value):
            if key == api.TUNE_ADJOINT:
                self.room = bool(value)
                self.need = 5000 if value else self.need
            return api.OK

        def trevr_last_error(self):
            return b"short"

        def forward(self, ptr, size):
            self.need = 9000 if self.room else 3000
            return api.E_CAPACITY if size < self.need else api.OK

    class Torch:
        def __getattr__(self, name):
            return getattr(torch, name)

        def empty(self, n, **kw):
            if n > 8000:
                raise torch.OutOfMemoryError("short")
            return torch.empty(n, **kw)

    L = Lib()
    monkeypatch.setattr(api, "lib", lambda: L)
    monkeypatch.setattr(api, "_torch", Torch)
    monkeypatch.setattr(api, "workspace_bytes", lambda p, n: (100, 1000))
    T = api.Tree.__new__(api.Tree)
    T.n, T.B, T.nside, T.params, T.handle, T._owned = 100, 1, 1, None, None, False
    T.device = "cpu"
    T._scratch = torch.empty(1000, dtype=torch.uint8)
    if reserve:
        T.reserve_adjoint()
        assert T.scratch.numel() == 5000
    T._call_with_scratch(L.forward, "forward")
    assert not L.room and 3000 <= T.scratch.numel() <= 8000
