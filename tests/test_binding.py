"""The binding's native half: what it refuses before it looks at memory (no GPU needed unless marked)."""
import ctypes

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
