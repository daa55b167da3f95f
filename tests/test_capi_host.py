"""Host-only checks of the C-ABI library: it loads, exports what include/psd.h declares,
its integer logic equals the oracle bit for bit, and bad arguments come back as status
codes before anything is launched (no GPU needed)."""
import ctypes
import itertools
import os
import re

import pytest

from oracle import psd_oracle as orc
from paper_1512_06216_amd import binding as psd
from tests.conftest import ROOT


def test_library_exports_every_declared_symbol():
    text = open(os.path.join(ROOT, "include", "psd.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(psd_[a-z0-9_]+)\s*\(", text))
    assert declared == set(psd.SIGNATURES), declared ^ set(psd.SIGNATURES)
    L = psd.lib()
    for name in declared:
        assert getattr(L, name) is not None
    assert L.psd_version() == 2


def test_struct_layouts_match_the_header():
    assert ctypes.sizeof(psd.Plan) == 4 * 8 + 4 * 4 + 3 * 8
    assert ctypes.sizeof(psd.DenseSegment) == 8 + 4 + 4 + 3 * 8
    assert ctypes.sizeof(psd.LayerTask) == ctypes.sizeof(psd.Plan) + 8 + 2 * 8 + 4 * 8 + 8 + 2 * 8 + 2 * 8 + 8 + 3 * 8


GRID = list(itertools.product([1, 3, 128, 256, 1000, 4096, 9216], [1, 2, 128, 1000, 4096, 21841],
                              [1, 32, 64, 128, 256, 4000], [1, 2, 3, 4, 8, 16, 33, 64]))


def test_plan_equals_oracle_on_a_grid():
    for kind in (psd.LAYER_FC, psd.LAYER_CONV):
        for M, N, B, P in GRID:
            got = psd.plan_layer(kind, M, N, B, P).as_dict()
            want = orc.plan_layer(kind, M, N, B, P)
            assert got == want, (kind, M, N, B, P)


def test_plan_paper_example_and_config2_discrepancy():
    p = psd.plan_layer(psd.LAYER_FC, 4096, 4096, 256, 4)
    assert (p.cost_sfb, p.cost_ps_dense, p.cost_sf_ps) == (18874368, 134217728, 75497472)
    # 4096 -> 1000 at B=256, P=8: Algorithm 3 as printed sends factors to the server,
    # the SFB-vs-full-matrix comparison of the prose picks SFB
    p = psd.plan_layer(psd.LAYER_FC, 4096, 1000, 256, 8)
    assert p.route_alg3 == psd.ROUTE_SF_PS and p.route_vs_dense == psd.ROUTE_SFB


def test_plan_errors():
    L = psd.lib()
    out = psd.Plan()
    assert L.psd_plan_layer(psd.LAYER_FC, 4, 4, 4, 4, None) == psd.E_NULL
    for args in [(2, 4, 4, 4, 4), (1, 0, 4, 4, 4), (1, 4, -1, 4, 4), (1, 4, 4, 0, 4), (1, 4, 4, 4, 0), (1, 4, 4, 4, 65)]:
        assert L.psd_plan_layer(*args, ctypes.byref(out)) == psd.E_INVALID
    assert L.psd_plan_layer(1, 2 ** 31, 2 ** 31, 1, 4, ctypes.byref(out)) == psd.E_OVERFLOW
    assert L.psd_plan_layer(1, 2 ** 62, 2 ** 62, 1, 2, ctypes.byref(out)) == psd.E_OVERFLOW
    with pytest.raises(OverflowError):
        orc.plan_layer(1, 2 ** 31, 2 ** 31, 1, 4)
    # largest cost just fits
    p = psd.plan_layer(1, 2 ** 30, 2 ** 30, 1, 4).as_dict()
    assert p == orc.plan_layer(1, 2 ** 30, 2 ** 30, 1, 4)
    assert b"overflow" in L.psd_status_string(psd.E_OVERFLOW)


def test_shard_range_equals_oracle():
    for n in list(range(1, 30)) + [97, 34848, 307200, 884736, 21841 * 4096, 2 ** 40 - 1]:
        for S in [1, 2, 3, 7, 8, 16, 29]:
            if S > n:
                continue
            for s in {0, S // 2, S - 1}:
                assert psd.shard_range(n, S, s) == orc.shard_range(n, S, s)
    L = psd.lib()
    b, e = ctypes.c_int64(), ctypes.c_int64()
    for n, S, s in [(4, 5, 0), (4, 0, 0), (4, 2, 2), (4, 2, -1), (0, 1, 0)]:
        assert L.psd_shard_range(n, S, s, ctypes.byref(b), ctypes.byref(e)) == psd.E_INVALID
    assert L.psd_shard_range(4, 2, 0, None, ctypes.byref(e)) == psd.E_NULL


def test_factor_ld():
    # rows of 128-byte multiples: 32 fp32 or 64 bf16 elements
    assert psd.factor_ld(1000, psd.F32) == 1024 and psd.factor_ld(1025, psd.F32) == 1056
    assert psd.factor_ld(21841, psd.BF16) == 21888 and psd.factor_ld(4096, psd.BF16) == 4096
    assert psd.factor_ld(1, psd.BF16) == 64 and psd.factor_ld(9216, psd.F32) == 9216
    assert psd.lib().psd_factor_ld(0, psd.F32) == 0 and psd.lib().psd_factor_ld(8, 7) == 0


def _fake(addr):
    return ctypes.c_void_p(addr)


def test_device_entry_points_reject_bad_arguments_before_launching():
    L = psd.lib()
    plan = psd.plan_layer(psd.LAYER_FC, 8, 8, 2, 2)
    f32p = ctypes.POINTER(ctypes.c_float)
    good = (f32p * 2)(ctypes.cast(0x1000, f32p), ctypes.cast(0x2000, f32p))
    odd = (f32p * 2)(ctypes.cast(0x1004, f32p), ctypes.cast(0x2000, f32p))
    null = (f32p * 2)(ctypes.cast(0x1000, f32p), None)
    U, V, W, Mom = _fake(0x10000), _fake(0x20000), _fake(0x30000), _fake(0x40000)
    pp = ctypes.byref(plan)
    # pack
    assert L.psd_pack_factors(None, good, good, psd.F32, U, 8, V, 8, None) == psd.E_NULL
    assert L.psd_pack_factors(pp, good, good, psd.F32, None, 8, V, 8, None) == psd.E_NULL
    assert L.psd_pack_factors(pp, null, good, psd.F32, U, 8, V, 8, None) == psd.E_NULL
    assert L.psd_pack_factors(pp, odd, good, psd.F32, U, 8, V, 8, None) == psd.E_INVALID
    assert L.psd_pack_factors(pp, good, good, 5, U, 8, V, 8, None) == psd.E_INVALID
    assert L.psd_pack_factors(pp, good, good, psd.F32, U, 4, V, 8, None) == psd.E_INVALID      # ld < N
    assert L.psd_pack_factors(pp, good, good, psd.F32, U, 9, V, 8, None) == psd.E_INVALID      # ld*4 % 16
    assert L.psd_pack_factors(pp, good, good, psd.BF16, U, 12, V, 8, None) == psd.E_INVALID    # ld*2 % 16
    assert L.psd_pack_factors(pp, good, good, psd.F32, _fake(0x10004), 8, V, 8, None) == psd.E_INVALID
    # sfb
    assert L.psd_sync_fc_sfb(pp, psd.F32, U, 8, V, 8, None, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_NULL
    assert L.psd_sync_fc_sfb(pp, 9, U, 8, V, 8, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID
    assert L.psd_sync_fc_sfb(pp, psd.F32, U, 8, V, 8, W, W, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID
    assert L.psd_sync_fc_sfb(pp, psd.F32, U, 8, V, 8, _fake(0x30008), Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID
    assert L.psd_sync_fc_sfb(pp, psd.BF16, U, 8, V, 7, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID
    bad = psd.Plan()
    ctypes.memmove(ctypes.byref(bad), ctypes.byref(plan), ctypes.sizeof(plan))
    bad.P = 0
    assert L.psd_sync_fc_sfb(ctypes.byref(bad), psd.F32, U, 8, V, 8, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID
    # bias
    assert L.psd_sync_fc_bias(pp, psd.F32, U, 8, None, Mom, 0.1, 0.9, 0.0, None) == psd.E_NULL
    assert L.psd_sync_fc_bias(pp, psd.F32, U, 8, W, W, 0.1, 0.9, 0.0, None) == psd.E_INVALID
    assert L.psd_sync_fc_bias(pp, psd.F32, U, 6, W, Mom, 0.1, 0.9, 0.0, None) == psd.E_INVALID       # ld < N
    assert L.psd_sync_fc_bias(pp, 3, U, 8, W, Mom, 0.1, 0.9, 0.0, None) == psd.E_INVALID
    assert L.psd_sync_fc_bias(pp, psd.BF16, U, 8, W, Mom, 0.1, 0.9, -0.5, None) == psd.E_INVALID
    # dense
    assert L.psd_sync_dense_ps(16, 2, None, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_NULL
    assert L.psd_sync_dense_ps(16, 2, null, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_NULL
    assert L.psd_sync_dense_ps(16, 0, good, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps(16, 65, good, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps(16, 2, good, W, Mom, 0.1, 0.9, 0.0, 17, None) == psd.E_INVALID     # S > n
    assert L.psd_sync_dense_ps(16, 2, good, W, Mom, 0.1, 0.9, 0.0, 0, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps(-1, 2, good, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps(16, 2, odd, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps(0, 2, good, W, Mom, 0.1, 0.9, 0.0, 1, None) == psd.OK              # empty layer: no-op
    assert L.psd_sync_dense_ps(16, 2, good, W, Mom, 0.1, 0.9, -1e-4, 1, None) == psd.E_INVALID     # negative weight decay
    assert L.psd_sync_dense_ps(16, 2, good, W, Mom, 0.1, 0.9, float('nan'), 1, None) == psd.E_INVALID
    assert L.psd_sync_fc_sfb(pp, psd.F32, U, 8, V, 8, W, Mom, 0.1, 0.9, -1.0, None, 0, None) == psd.E_INVALID
    # multi
    seg = (psd.DenseSegment * 1)()
    seg[0].n, seg[0].P, seg[0].S = 16, 2, 1
    seg[0].G = ctypes.cast(good, ctypes.POINTER(f32p))
    seg[0].W, seg[0].Mom = ctypes.cast(0x30000, f32p), ctypes.cast(0x40000, f32p)
    assert L.psd_sync_dense_ps_multi(0, seg, 0.1, 0.9, 0.0, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps_multi(17, seg, 0.1, 0.9, 0.0, None) == psd.E_INVALID
    assert L.psd_sync_dense_ps_multi(1, None, 0.1, 0.9, 0.0, None) == psd.E_NULL
    seg[0].P = 17
    assert L.psd_sync_dense_ps_multi(1, seg, 0.1, 0.9, 0.0, None) == psd.E_INVALID
    seg[0].P, seg[0].n = 2, 0
    assert L.psd_sync_dense_ps_multi(1, seg, 0.1, 0.9, 0.0, None) == psd.OK                       # nothing to do
    # iteration
    assert L.psd_sync_iteration(1, None, 0.1, 0.9, 0.0, 0) == psd.E_NULL
    task = (psd.LayerTask * 1)()
    task[0].plan = psd.plan_layer(psd.LAYER_CONV, 8, 8, 2, 2)
    assert L.psd_sync_iteration(0, task, 0.1, 0.9, 0.0, 0) == psd.E_INVALID
    assert L.psd_sync_iteration(1, task, 0.1, 0.9, 0.0, 7) == psd.E_INVALID
    assert L.psd_sync_iteration(1, task, 0.1, 0.9, 0.0, 0) == psd.E_UNSUPPORTED                   # PS route without G
    for s in (0, -1, -2, -3, -4, -5, -99):
        assert L.psd_status_string(s)


def test_sizes_beyond_what_the_kernels_index_are_refused_before_launching():
    L = psd.lib()
    U, V, W, Mom = _fake(0x10000), _fake(0x20000), _fake(0x30000), _fake(0x40000)
    # the reconstruct kernels use 32-bit byte offsets into each stacked factor matrix
    plan = psd.plan_layer(psd.LAYER_FC, 8, 2 ** 21, 256, 8)          # U: 2048 x 2^21 bf16 = 8.6 GB
    assert L.psd_sync_fc_sfb(ctypes.byref(plan), psd.BF16, U, 2 ** 21, V, 8, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_UNSUPPORTED
    assert L.psd_sync_fc_sfb(ctypes.byref(plan), psd.F32, U, 2 ** 21, V, 8, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_UNSUPPORTED
    # M, N, K beyond 2^31 are invalid for the device entry points (the plan itself is fine)
    plan = psd.plan_layer(psd.LAYER_FC, 2 ** 31, 8, 1, 1)
    assert L.psd_sync_fc_sfb(ctypes.byref(plan), psd.F32, U, 8, V, 2 ** 31, W, Mom, 0.1, 0.9, 0.0, None, 0, None) == psd.E_INVALID


def test_binding_fails_loudly_without_the_library(monkeypatch):
    monkeypatch.setattr(psd, "_lib", None)
    monkeypatch.setattr(psd, "LIB_PATH", "/nonexistent/libpsd.so")
    with pytest.raises(RuntimeError, match="not built"):
        psd.plan_layer(psd.LAYER_FC, 4, 4, 4, 4)


def test_tune_hook_accepts_listed_values_only():
    L = psd.lib()
    for knob, good, bad in ((psd.TUNE_SFB_BF16_TILE, (0, 1, 2, -1), (3, -2, 100)), (psd.TUNE_SFB_F32_TILE, (1, 2, -1), (0, 3)),
                            (psd.TUNE_SFB_BF16_SKEW_US, (0, 20, 200, -1), (201, -2))):
        for v in good:
            assert L.psd_tune_set(knob, v) == psd.OK
        for v in bad:
            assert L.psd_tune_set(knob, v) == psd.E_INVALID
    assert L.psd_tune_set(3, 0) == psd.E_INVALID and L.psd_tune_set(-1, 0) == psd.E_INVALID


def test_factor_matrices_past_the_32_bit_offset_reach_are_refused_on_the_host():
    """The reconstruction kernels address each stacked factor matrix with 32-bit byte offsets.  A layer
    whose U or V would be larger is refused with PSD_E_UNSUPPORTED during validation, before anything is
    launched (the pointers below are never dereferenced)."""
    L = psd.lib()
    fake = ctypes.c_void_p(0x10000000)               # aligned, non-null, never touched
    # VGG-16's first FC layer is fine even at fp32 (25088 x 2048 x 4 B = 205 MB) ...
    # ... a 2^20-wide layer at K = 2048 is not (4 GiB of bf16, 8 GiB of fp32)
    big = psd.plan_layer(psd.LAYER_FC, 1 << 20, 256, 256, 8)
    for dtype in (psd.BF16, psd.F32):
        ldu, ldv = psd.factor_ld(big.N, dtype), psd.factor_ld(big.M, dtype)
        st = L.psd_sync_fc_sfb(ctypes.byref(big), dtype, fake, ldu, fake, ldv, fake, ctypes.c_void_p(0x20000000),
                               0.01, 0.9, 0.0, None, 0, None)
        assert st == psd.E_UNSUPPORTED, (dtype, st)


def test_workspace_query_and_argument_checks():
    """psd_sfb_workspace_bytes is host logic: a layer that leaves most compute units without a tile asks
    for 2-4 partial dW matrices, a layer with a tile per compute unit or more for none; a workspace that
    is too small, misaligned or NULL with a non-zero size is refused before anything is launched."""
    L = psd.lib()
    fake = lambda a: ctypes.c_void_p(a)
    small = psd.plan_layer(psd.LAYER_FC, 1024, 1000, 256, 8)      # 64 tiles of 128 x 128
    fc8 = psd.plan_layer(psd.LAYER_FC, 4096, 1000, 256, 8)        # 256 tiles: one per compute unit already
    fc6 = psd.plan_layer(psd.LAYER_FC, 9216, 4096, 256, 8)
    tiny = psd.plan_layer(psd.LAYER_FC, 256, 128, 32, 4)          # K = 128: too short to split
    for dtype in (psd.BF16, psd.F32):
        need = psd.sfb_workspace_bytes(small, dtype)
        per = (1000 * 1024 + 3) // 4 * 4 * 4
        assert need % per == 0 and 2 <= need // per <= 4 and need % 16 == 0, (dtype, need)
        for plan in (fc8, fc6, tiny):
            assert psd.sfb_workspace_bytes(plan, dtype) == 0
        ldu, ldv = psd.factor_ld(small.N, dtype), psd.factor_ld(small.M, dtype)
        args = (ctypes.byref(small), dtype, fake(0x10000000), ldu, fake(0x20000000), ldv, fake(0x30000000),
                fake(0x40000000), 0.01, 0.9, 0.0)
        assert L.psd_sync_fc_sfb(*args, fake(0x50000000), need - 16, None) == psd.E_WORKSPACE
        assert L.psd_sync_fc_sfb(*args, None, need, None) == psd.E_NULL
        assert L.psd_sync_fc_sfb(*args, fake(0x50000008), need, None) == psd.E_INVALID
    assert L.psd_sfb_workspace_bytes(None, psd.BF16) == 0 and L.psd_sfb_workspace_bytes(ctypes.byref(small), 7) == 0
    assert b"workspace" in L.psd_status_string(psd.E_WORKSPACE)


def test_ssp_clock_bookkeeping_against_a_literal_ring():
    """psd_ssp_slots against a literal simulation: a deque of the last s+1 clocks' slots; the update of
    clock c is due at clock c + s (so that the reader at clock c + s + 1 sees it, Section 3.2)."""
    L = psd.lib()
    for s in range(0, 6):
        st = psd.SspState()
        assert L.psd_ssp_init(ctypes.byref(st), s) == psd.OK and (st.s, st.clock) == (s, 0)
        slot_of_clock = {}
        for t in range(0, 20):
            a, b = ctypes.c_int32(), ctypes.c_int32()
            assert L.psd_ssp_slots(ctypes.byref(st), ctypes.byref(a), ctypes.byref(b)) == psd.OK
            assert 0 <= a.value <= s
            # the push slot must not hold an update that is still pending (clocks t-s .. t-1, except the one due now
            # when s = 0 where push == due)
            pending = {slot_of_clock[c] for c in range(max(0, t - s + 1), t)}
            assert a.value not in pending
            slot_of_clock[t] = a.value
            if t < s:
                assert b.value == -1
            else:
                assert b.value == slot_of_clock[t - s]
                assert orc.ssp_updates_visible(t + 1, s) == t - s + 1          # after this clock: clocks 0 .. t-s applied
            st.clock += 1
    st = psd.SspState()
    assert L.psd_ssp_init(None, 0) == psd.E_NULL
    assert L.psd_ssp_init(ctypes.byref(st), -1) == psd.E_INVALID
    assert L.psd_ssp_init(ctypes.byref(st), psd.MAX_STALENESS + 1) == psd.E_INVALID
    assert L.psd_ssp_slots(ctypes.byref(st), None, None) == psd.E_NULL


def test_blocks_in_place_support_rule_and_argument_checks():
    """Which layers the reconstruction can read straight from the per-worker blocks, and what the entry
    point says about bad arguments -- all decided on the host before anything is launched."""
    L = psd.lib()
    sup = lambda plan, dt, ldu, ldv: bool(L.psd_sfb_blocks_supported(ctypes.byref(plan), dt, ldu, ldv))
    for (M, N, B, P, dt, ldu, ldv), ok in (
            ((4096, 1000, 256, 8, psd.F32, 1000, 4096), True), ((9216, 4096, 16, 64, psd.F32, 4096, 9216), True),
            ((9216, 4096, 16, 8, psd.BF16, 4096, 9216), False),       # bf16 k-stages are 32 rows
            ((9216, 4096, 32, 8, psd.BF16, 4096, 9216), True),
            ((4096, 21841, 256, 8, psd.BF16, 21888, 4096), True),     # padded rows of an odd-width layer
            ((4096, 21841, 256, 8, psd.BF16, 21841, 4096), False),    # rows not a multiple of 16 bytes
            ((256, 128, 11, 4, psd.F32, 128, 256), False),            # a stage would straddle two blocks
            ((256, 130, 16, 4, psd.F32, 130, 256), False), ((256, 130, 16, 4, psd.F32, 132, 256), True),
            ((256, 128, 16, 4, psd.F32, 124, 256), False)):           # rows shorter than the layer is wide
        plan = psd.plan_layer(psd.LAYER_FC, M, N, B, P)
        assert sup(plan, dt, ldu, ldv) == ok, (M, N, B, P, dt, ldu, ldv)
    plan = psd.plan_layer(psd.LAYER_FC, 256, 130, 16, 2)
    assert L.psd_sfb_blocks_supported(None, psd.F32, 132, 256) == 0 and not sup(plan, 7, 132, 256)
    fake = 0x10000000
    ptrs = (ctypes.POINTER(ctypes.c_float) * 2)(*[ctypes.cast(fake + 0x100000 * i, ctypes.POINTER(ctypes.c_float)) for i in range(2)])
    pp = ctypes.cast(ptrs, ctypes.POINTER(ctypes.POINTER(ctypes.c_float)))
    W, Mom = ctypes.c_void_p(fake + 0x800000), ctypes.c_void_p(fake + 0x900000)

    def call(plan_ref, up, vp, w, mom, wd=0.0, dt=psd.F32, ldu=130, ldv=256):    # ldu = 130: unsupported, never launched
        return L.psd_sync_fc_sfb_blocks(plan_ref, dt, up, ldu, vp, ldv, w, mom, 0.1, 0.9, wd, None)
    assert call(ctypes.byref(plan), pp, pp, W, Mom) == psd.E_UNSUPPORTED
    assert call(None, pp, pp, W, Mom) == psd.E_NULL
    assert call(ctypes.byref(plan), None, pp, W, Mom) == psd.E_NULL
    assert call(ctypes.byref(plan), pp, pp, None, Mom) == psd.E_NULL
    assert call(ctypes.byref(plan), pp, pp, W, W) == psd.E_INVALID
    assert call(ctypes.byref(plan), pp, pp, ctypes.c_void_p(fake + 4), Mom) == psd.E_INVALID
    assert call(ctypes.byref(plan), pp, pp, W, Mom, wd=-1.0) == psd.E_INVALID
    assert call(ctypes.byref(plan), pp, pp, W, Mom, dt=5) == psd.E_INVALID
    ptrs[1] = ctypes.cast(fake + 8, ctypes.POINTER(ctypes.c_float))
    assert call(ctypes.byref(plan), pp, pp, W, Mom) == psd.E_INVALID
    ptrs[1] = ctypes.cast(None, ctypes.POINTER(ctypes.c_float))
    assert call(ctypes.byref(plan), pp, pp, W, Mom) == psd.E_NULL


def test_a_batch_whose_product_with_the_workers_wraps_is_refused():
    """psd_plan_layer returns no such plan, but the structure is the caller's to fill: 64 workers of 2^58 samples are 2^64."""
    L = psd.lib()
    plan = psd.Plan(M=64, N=32, B=2 ** 58, P=64, kind=psd.LAYER_FC)
    fake = lambda i: ctypes.c_void_p(0x10000000 + 0x100000 * i)
    ptrs = (ctypes.POINTER(ctypes.c_float) * 64)(*[ctypes.cast(0x20000000, ctypes.POINTER(ctypes.c_float))] * 64)
    pp = ctypes.cast(ptrs, ctypes.POINTER(ctypes.POINTER(ctypes.c_float)))
    for dtype in (psd.F32, psd.BF16):
        assert L.psd_sfb_blocks_supported(ctypes.byref(plan), dtype, 32, 64) == 0
        assert L.psd_sfb_workspace_bytes(ctypes.byref(plan), dtype) == 0
        args = (fake(2), fake(3), 0.1, 0.9, 0.0)
        assert L.psd_sync_fc_sfb_blocks(ctypes.byref(plan), dtype, pp, 32, pp, 64, *args, None) == psd.E_INVALID
        assert L.psd_sync_fc_sfb(ctypes.byref(plan), dtype, fake(0), 32, fake(1), 64, *args, None, 0, None) == psd.E_INVALID
        assert L.psd_sync_fc_bias(ctypes.byref(plan), dtype, fake(0), 32, *args, None) == psd.E_INVALID
    assert L.psd_pack_factors(ctypes.byref(plan), pp, pp, psd.F32, fake(0), 32, fake(1), 64, None) == psd.E_INVALID


def _big_step(ev_ready=None):
    """Two parameter-server layers below three 3500 -> 3500 layers with bf16 factors; every address is made up."""
    f32p = ctypes.POINTER(ctypes.c_float)
    ptrs = (f32p * 2)(ctypes.cast(0x10000000, f32p), ctypes.cast(0x20000000, f32p))
    pp = ctypes.cast(ptrs, ctypes.POINTER(f32p))
    tasks = (psd.LayerTask * 5)()
    for i, t in enumerate(tasks):
        t.W, t.Mom = ctypes.cast(0x30000000 + i * 0x10000000, f32p), ctypes.cast(0x38000000 + i * 0x10000000, f32p)
        t.stream, t.ev_ready, t.S, t.factor_dtype = 0x1000 * (i + 1), ev_ready, 1, psd.BF16
        if i < 2:
            t.plan, t.G = psd.plan_layer(psd.LAYER_CONV, 1000, 1, 16, 2), pp
        else:
            t.plan, t.delta_p, t.act_p = psd.plan_layer(psd.LAYER_FC, 3500, 3500, 16, 2), pp, pp
            t.U, t.ldu, t.V, t.ldv = 0x90000000, 3520, 0xa0000000, 3520
    return tasks, ptrs


@pytest.mark.parametrize("layer,field,value,status", [(4, "ldu", 3501, psd.E_INVALID), (4, "U", None, psd.E_NULL), (4, "ldv", 3508, psd.E_INVALID),
                                                      (4, "factor_dtype", 5, psd.E_INVALID), (4, "act_p", None, psd.E_NULL)])
def test_iteration_without_events_comes_to_a_refused_layer_before_the_layers_below_it(layer, field, value, status):
    """Without readiness events the issue order is top-down: the top layer is refused before anything is launched
    (a launch would be PSD_E_HIP here, where there is no GPU)."""
    tasks, keep = _big_step()
    setattr(tasks[layer], field, value)
    assert psd.lib().psd_sync_iteration(5, tasks, 0.1, 0.9, 0.0, psd.RULE_ALG3) == status


def test_workspace_query_follows_a_pinned_tile():
    """1024 -> 1000: 64 tiles of 128 x 128 take four partial sums, 128 tiles of 64 x 128 two, 32 of 128 x 256 four."""
    plan = psd.plan_layer(psd.LAYER_FC, 1024, 1000, 256, 8)
    for knob, dtype, want in ((psd.TUNE_SFB_F32_TILE, psd.F32, {-1: 4, 1: 2, 2: 4}), (psd.TUNE_SFB_BF16_TILE, psd.BF16, {-1: 4, 0: 4, 1: 4, 2: 4})):
        try:
            for tile, partials in want.items():
                psd.tune_set(knob, tile)
                assert psd.sfb_workspace_bytes(plan, dtype) == partials * 1024 * 1000 * 4, (dtype, tile)
        finally:
            psd.tune_set(knob, -1)
