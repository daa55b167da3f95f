"""The binding's native half: what it refuses before it looks at memory (no GPU needed unless marked)."""
import ctypes
import weakref

import pytest
import torch

from paper_1512_06216_amd import binding as psd


def _plan():
    return psd.plan_layer(psd.LAYER_FC, 8, 8, 2, 2)


class _AlmostPlan(ctypes.Structure):                # the fields of a plan that are looked at first, and nothing behind them
    _fields_ = [("M", ctypes.c_int64), ("N", ctypes.c_int64), ("B", ctypes.c_int64), ("P", ctypes.c_int64)]


@pytest.mark.parametrize("wrong", [b"", bytes(ctypes.sizeof(psd.Plan)), bytearray(256), _AlmostPlan(8, 8, 2, 2), psd.SspState(),
                                   (psd.Plan * 2)(), {"P": 2}, None],
                         ids=["no_bytes", "bytes", "bytearray", "half_a_plan", "state", "array", "dict", "none"])
def test_only_a_plan_is_read_as_a_plan(wrong):
    t, two = torch.zeros(64), [torch.zeros(16)] * 2
    for call in (lambda: psd.pack_factors(wrong, two, two, psd.F32, t, 8, t, 8),
                 lambda: psd.sync_fc_sfb(wrong, psd.F32, t, 8, t, 8, t, t, 0.1, 0.9),
                 lambda: psd.sync_fc_sfb_static(wrong, psd.F32, t, 8, t, 8, t, t, 0.1, 0.9),
                 lambda: psd._native().sync_fc_sfb_blocks(wrong, psd.F32, two, 8, two, 8, t, t, 0.1, 0.9, 0.0, None),
                 lambda: psd.sync_fc_bias(wrong, psd.F32, t, 8, t, t, 0.1, 0.9)):
        with pytest.raises(TypeError):
            call()


def test_a_subclass_of_plan_is_a_plan():
    class Mine(psd.Plan):
        pass
    mine = Mine()
    ctypes.memmove(ctypes.byref(mine), ctypes.byref(_plan()), ctypes.sizeof(psd.Plan))
    with pytest.raises(ValueError, match="U must be a contiguous CUDA tensor"):
        psd.sync_fc_bias(mine, psd.F32, torch.zeros(64), 8, torch.zeros(8), torch.zeros(8), 0.1, 0.9)


@pytest.mark.parametrize("wrong", [bytes(ctypes.sizeof(psd.SspState)), bytearray(ctypes.sizeof(psd.SspState)), b"", psd.Plan(), None],
                         ids=["bytes", "bytearray", "no_bytes", "plan", "none"])
def test_only_a_state_is_read_and_written_as_a_state(wrong):
    ring = (ctypes.c_void_p * 1)(1)
    with pytest.raises(TypeError, match="an SspState expected"):
        psd._native().ssp_clock_fc(wrong, _plan(), psd.F32, None, None, ring, 8, ring, 8, None, None, 0.1, 0.9, 0.0, None, 0)


def test_rings_and_tables_are_as_long_as_the_call_reads_them():
    ext, plan = psd._native(), _plan()
    state, ring, short = psd.SspState(s=2), (ctypes.c_void_p * 3)(), (ctypes.c_void_p * 2)()
    for u, v in ((short, ring), (ring, short), ((ctypes.c_int64 * 3)(), ring), (ring, bytes(24))):
        with pytest.raises(TypeError, match="pointers expected"):
            ext.ssp_clock_fc(state, plan, psd.F32, None, None, u, 8, v, 8, None, None, 0.1, 0.9, 0.0, None, 0)
    for wrong in ((psd.DenseSegment * 1)(), (psd.LayerTask * 2)(), bytes(1000), psd.DenseSegment(), None):
        with pytest.raises(TypeError, match="DenseSegments expected"):
            ext.sync_dense_ps_multi(2, wrong, 0.1, 0.9, 0.0, 0)
    for wrong in ((psd.LayerTask * 1)(), (psd.DenseSegment * 9)(), bytes(1000), psd.LayerTask(), None):
        with pytest.raises(TypeError, match="LayerTasks expected"):
            ext.sync_iteration(2, wrong, 0.1, 0.9, 0.0, 0)
    # ... and what fits goes through to the library's own checks
    assert ext.sync_dense_ps_multi(2, (psd.DenseSegment * 2)(), 0.1, 0.9, 0.0, 0) == psd.E_INVALID
    assert ext.sync_iteration(0, (psd.LayerTask * 1)(), 0.1, 0.9, 0.0, 0) == psd.E_INVALID


def test_an_iterator_of_tensors_is_no_sequence():
    t, two, plan = torch.zeros(64), [torch.zeros(16)] * 2, _plan()
    layer = psd.SspFc.__new__(psd.SspFc)
    layer.plan, layer.dtype, layer.state, layer.ldu, layer.ldv = plan, psd.F32, psd.SspState(), 8, 8
    layer.U_ring = layer.V_ring = (ctypes.c_void_p * 1)(1)
    for call in (lambda: psd.pack_factors(plan, iter(two), two, psd.F32, t, 8, t, 8),
                 lambda: psd.sync_fc_sfb_blocks(plan, psd.F32, two, 8, (x for x in two), 8, t, t, 0.1, 0.9),
                 lambda: psd.sync_dense_ps(iter(two), t, t, 0.1, 0.9, 1),
                 lambda: layer.clock(iter(two), two, t, t, 0.1, 0.9)):
        with pytest.raises(TypeError, match="has no len"):
            call()


class _MadeWhenRead:
    """A sequence that makes its tensors as it is read, and knows which of them are still there."""

    def __init__(self, make, P, says=None):
        self.make, self.P, self.says, self.refs = make, P, P if says is None else says, []

    def __len__(self):
        return self.says

    def __getitem__(self, i):
        if i >= self.P:
            raise IndexError(i)
        t = self.make()
        self.refs.append(weakref.ref(t))
        return t


class _LastArgument:
    """Stands for a stream, which the calls look at last, after the tensors' pointers are taken."""

    def __init__(self, *sequences):
        self.sequences, self.alive = sequences, None

    @property
    def cuda_stream(self):
        self.alive = [r() is not None for s in self.sequences for r in s.refs]
        return torch.cuda.current_stream().cuda_stream


@pytest.mark.gpu
def test_tensors_of_a_sequence_live_until_the_library_is_called():
    dev, plan = "cuda:0", psd.plan_layer(psd.LAYER_FC, 64, 32, 16, 3)
    ones = lambda *shape: _MadeWhenRead(lambda: torch.ones(*shape, device=dev), 3)
    W, Mom = torch.zeros(32, 64, device=dev), torch.zeros(32, 64, device=dev)
    U, ldu, V, ldv = psd.alloc_factors(plan, psd.F32, dev)
    layer = psd.SspFc(plan, psd.F32, 0, dev)
    d, v, G = lambda: ones(16, 32), lambda: ones(16, 64), lambda: ones(32 * 64)
    for call, sequences in ((lambda s, x, y: psd.pack_factors(plan, x, y, psd.F32, U, ldu, V, ldv, stream=s), (d(), v())),
                            (lambda s, x, y: psd.sync_fc_sfb_blocks(plan, psd.F32, x, 0, y, 0, W, Mom, 0.1, 0.9, stream=s), (d(), v())),
                            (lambda s, x, y: layer.clock(x, y, W, Mom, 0.1, 0.9, stream=s), (d(), v())),
                            (lambda s, x: psd.sync_dense_ps(x, W, Mom, 0.1, 0.9, 1, stream=s), (G(),))):
        last = _LastArgument(*sequences)
        call(last, *sequences)
        assert last.alive == [True] * (3 * len(sequences))
    torch.cuda.synchronize()
    assert bool((U[:, :32] == 1).all()) and bool((V[:, :64] == 1).all())


@pytest.mark.gpu
def test_a_sequence_shorter_than_it_says_is_refused():
    dev, plan = "cuda:0", psd.plan_layer(psd.LAYER_FC, 64, 32, 16, 3)
    short, full = _MadeWhenRead(lambda: torch.ones(16, 64, device=dev), 2, says=3), [torch.ones(16, 64, device=dev)] * 3
    W, Mom = torch.zeros(32, 64, device=dev), torch.zeros(32, 64, device=dev)
    for x, y in ((short, full), (full, short)):
        with pytest.raises(ValueError, match="need P per-worker blocks"):
            psd.sync_fc_sfb_blocks(plan, psd.F32, x, 0, y, 0, W, Mom, 0.1, 0.9)
