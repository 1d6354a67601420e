"""How much memory a gradient call takes that allocates its own workspace: the
required size, and room for further segments' step states within its limits."""
import pytest
import torch

import paper_1107_4107_amd as aw

N, T, CK = 1000, 400, 100       # 4 segments
CASES = [(6, aw.grad_workspace_bytes), (12, aw.ftle_grad_workspace_bytes)]


def _sizes(rows, need):
    e = aw.Ensemble(eps=1e-2, n_steps=T, ic_kind="explicit", n_orbits=N, tangent=rows == 12)
    nb = need(e, CK)
    seg = nb - (2 * N * (T // 8) if rows == 12 else 0) - 8 * rows * N * 5
    assert seg == 8 * rows * N * 26     # 26 kept steps of a segment at most
    return e, nb, seg


@pytest.fixture
def asked(monkeypatch):
    """The sizes asked of the allocator, which refuses those in `refuse`."""
    got, refuse, empty = [], set(), torch.empty

    def fake(shape, **kw):
        got.append(shape[0])
        if shape[0] in refuse:
            raise torch.OutOfMemoryError("out of memory")
        return empty(shape, **kw)
    monkeypatch.setattr(torch, "empty", fake)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    return got, refuse


@pytest.mark.parametrize("rows,need", CASES)
def test_keep_bytes_bounds_the_memory(rows, need, asked):
    e, nb, seg = _sizes(rows, need)
    got, _ = asked
    for keep, segs in ((0, 0), (seg - 1, 0), (seg, 1), (2 * seg + 7, 2), (100 * seg, 3)):
        w = aw._adjoint_workspace(e, CK, nb, rows, False, "cpu", keep)
        assert w.numel() == nb + segs * seg, keep
    assert aw._adjoint_workspace(e, CK, nb, rows, True, "cpu", 100 * seg).numel() == nb


@pytest.mark.parametrize("rows,need", CASES)
def test_default_room_follows_the_free_memory(rows, need, asked, monkeypatch):
    e, nb, seg = _sizes(rows, need)
    got, refuse = asked
    monkeypatch.setattr(aw, "KEEP_UNASKED_BYTES", 0)
    for free, segs in ((1 << 40, 3), (4 * (nb + 2 * seg) + 40, 2), (4 * nb, 0), (0, 0)):
        monkeypatch.setattr(aw, "_free_bytes", lambda dev: free)
        assert aw._adjoint_workspace(e, CK, nb, rows, False, "cpu").numel() == nb + segs * seg, free
    monkeypatch.setattr(aw, "_free_bytes", lambda dev: 1 << 40)
    monkeypatch.setattr(aw, "KEEP_BYTES", nb + seg)
    assert aw._adjoint_workspace(e, CK, nb, rows, False, "cpu").numel() == nb + seg


@pytest.mark.parametrize("rows,need", CASES)
def test_a_refused_workspace_falls_back_to_the_required_size(rows, need, asked):
    e, nb, seg = _sizes(rows, need)
    got, refuse = asked
    refuse.add(nb + 3 * seg)
    assert aw._adjoint_workspace(e, CK, nb, rows, False, "cpu").numel() == nb
    assert got == [nb + 3 * seg, nb]
    refuse.add(nb)
    with pytest.raises(torch.OutOfMemoryError):
        aw._adjoint_workspace(e, CK, nb, rows, False, "cpu")


def test_the_public_calls_take_keep_bytes():
    import inspect
    for fn in (aw.indicator_grad, aw.ftle_grad, aw.IndicatorJ.forward, aw.IndicatorL.forward):
        p = inspect.signature(fn).parameters["keep_bytes"]
        assert p.default is None and list(inspect.signature(fn).parameters)[-1] == "keep_bytes"
