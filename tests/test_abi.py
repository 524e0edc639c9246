"""The C-ABI library loads, exports every symbol include/*.h declares, and
its host-side routines (no GPU) agree with the oracle and reject bad input."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle import tca_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    names = set()
    for header in ("tca.h", "tca_diag.h"):       # the method's boundary, and the diagnostics beside it
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(tca_[a-z_0-9]+)\s*\(", text))
    return sorted(names)


def test_the_boundary_header_holds_no_diagnostics():
    text = open(os.path.join(ROOT, "include", "tca.h")).read()
    assert "tca_probe" not in text and "tca_diag" not in text


def test_library_exports_every_declared_symbol():
    import paper_2512_09238_amd.binding as tb
    names = _declared_symbols()
    assert "tca_select" in names and "tca_prefill" in names and "tca_decode" in names
    assert "tca_calibrate_budgets" in names
    for n in names:
        assert hasattr(tb.lib, n), n
        assert n in tb.EXPORTS, f"{n} has no ctypes signature"
    assert set(tb.EXPORTS) == set(names)


def test_host_candidates_match_oracle():
    import paper_2512_09238_amd.binding as tb
    for b, M, sigma in [(128, 14, 1.0), (32, 5, 0.7), (4, 3, 1.0), (256, 1, 2.0)]:
        got = tb.tca_make_candidates(b, M, sigma)
        np.testing.assert_allclose(got, orc.candidates(b, M, sigma), rtol=1e-13, atol=1e-300)
    for f in (0.001, 0.05, 0.1, 0.25, 0.5, 0.7, 0.77, 0.99, 1.0, 1.5):
        for b in (32, 128):
            np.testing.assert_allclose(tb.tca_config_from_budget(b, 1.0, f), orc.config_from_budget(b, 1.0, f),
                                       rtol=1e-12, atol=1e-15)


def test_host_counts_rows_and_decode_budget_match_oracle():
    import paper_2512_09238_amd.binding as tb
    rng = np.random.default_rng(0)
    b = 128
    prm = tb.make_params(4, 2, 128, b, 512, tb.TCA_BF16)
    for m in (0, 1, 7, 256, 1024, 4096):
        P = np.stack([orc.config_from_budget(b, 1.0, f) for f in rng.uniform(0.02, 0.9, 4)])
        for p in P:
            assert list(tb.tca_psi_counts(b, m, p)) == list(orc.psi_counts(m, p))
            assert tb.tca_decode_budget(b, p) == orc.decode_budget(b, p)
        total, rows = tb.tca_select_rows(prm, m, P)
        assert list(rows) == [orc.selected_rows(b, m, p) for p in P] and total == rows.sum()
    assert list(tb.tca_psi_counts(2, 8, [0.25, 0.75])) == [2, 6]
    # a shared selection has one entry per KV head, and needs room for the logits of every query head
    shared = tb.make_params(4, 2, 128, b, 512, tb.TCA_BF16, share=tb.TCA_SHARE_GROUP)
    assert tb.tca_selection_heads(prm) == 4 and tb.tca_selection_heads(shared) == 2
    total, rows = tb.tca_select_rows(shared, 256, P[:2])
    assert list(rows) == [orc.selected_rows(b, 256, p) for p in P[:2]]
    assert tb.tca_select_workspace_bytes(shared, 4096) >= 4 * 4096 * 8


def test_argument_errors_are_codes_not_crashes():
    import paper_2512_09238_amd.binding as tb
    with pytest.raises(tb.TcaError) as e:
        tb.tca_num_counts(48)
    assert e.value.code == tb.TCA_ERR_UNSUPPORTED
    with pytest.raises(tb.TcaError) as e:
        tb.tca_psi_counts(4, 8, [0.5, 0.1, 0.1])
    assert e.value.code == tb.TCA_ERR_INVALID
    bad = tb.make_params(6, 4, 128, 128, 4096, tb.TCA_BF16)
    with pytest.raises(tb.TcaError):
        tb.tca_select_rows(bad, 4, np.ones((6, 8)) / 8)
    assert tb.tca_select_workspace_bytes(bad, 1024) == 0
    for prm in (tb.make_params(4, 2, 96, 128, 4096, tb.TCA_BF16), tb.make_params(4, 2, 128, 128, 100, tb.TCA_BF16),
                tb.make_params(4, 2, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0, 2),
                tb.make_params(4, 2, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0, 0, 2),
                tb.make_params(4, 2, 128, 128, 4096, 7), tb.make_params(256, 256, 128, 128, 4096, 0)):
        with pytest.raises(tb.TcaError):
            tb.tca_select_rows(prm, 4, np.ones((prm.n_q_heads, 8)) / 8)
    # NULL device pointers are rejected before any launch
    ok = tb.make_params(4, 2, 128, 128, 4096, tb.TCA_BF16)
    p = np.ones((4, 8)) / 8
    offs = np.arange(5, dtype=np.int64) * 10
    rc = tb.lib.tca_select(ctypes.byref(ok), None, None, None, 128, 0, 128, p.ctypes.data_as(tb._dbl_p),
                           offs.ctypes.data_as(tb._i64_p), None, None, None, None, None, 0, None)
    assert rc == tb.TCA_ERR_INVALID and b"NULL" in tb.lib.tca_last_error()
    assert tb.lib.tca_strerror(-3) == b"workspace too small or misaligned"
    assert tb.tca_select_workspace_bytes(ok, 131072) > 4 * 131072


@pytest.mark.parametrize("L,d", [(1, 64), (333, 128), (8192, 128)])
def test_calibration_workspace_without_the_digits(L, d):
    """What a bf16 call asks for over the same call in fp32: 4 bytes per element, 16 per 16 rows, rows rounded up to 128."""
    import paper_2512_09238_amd.binding as tb
    bf16, f32 = (tb.tca_calibrate_workspace_bytes(tb.make_params(8, 2, d, 32, 64, t), L, 5) for t in (tb.TCA_BF16, tb.TCA_F32))
    rows = (8 + 2) * (-(-L // 128) * 128)
    assert 0 <= bf16 - f32 - (rows * d * 4 + rows // 16 * 16) < 4 * 256


def test_prefill_query_tiles_by_the_length_of_the_walk():
    """Host logic of the bf16 prefill launch: 256 queries a workgroup in calls of many query tiles, and of fewer (1024 in all
    at least) where each walks a long context; otherwise 128, and rows fetched through their positions do not ask for it."""
    import paper_2512_09238_amd.binding as tb
    wide = tb.make_params(64, 8, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0)
    shared = tb.make_params(64, 8, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0, share=tb.TCA_SHARE_GROUP)
    layer = tb.make_params(32, 8, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0)
    for prm, pos0, n, free, want in ((wide, 0, 4096, False, 128), (wide, 0, 4096, True, 256), (wide, 8192, 4096, False, 128),
                                     (wide, 16384, 4096, False, 256), (wide, 65536, 5000, False, 256), (shared, 65536, 4096, False, 256),
                                     (shared, 0, 5446, False, 128), (wide, 0, 6144, False, 256), (wide, 65536, 2048, False, 128),
                                     (layer, 65536, 4096, False, 128), (layer, 0, 8192, False, 256)):
        Hs = tb.tca_selection_heads(prm)
        offs = np.arange(Hs + 1, dtype=np.int64) * int(0.35 * (pos0 + n))
        start, _ = tb.tca_diag_prefill_xcd_plan(prm, offs, pos0, n, gather_free=free)
        assert start[8] == prm.n_q_heads * -(-n // want), (pos0, n, free)


def test_prefill_cut_into_chunks_where_long_heads_share_a_cu():
    """Host logic of the bf16 prefill launch, calls of 257 to 512 workgroups whose heads keep 20 to 50 % of the rows: cut into
    chunks of keys where the long heads' workgroups meet on a CU, whole where they meet short ones."""
    import paper_2512_09238_amd.binding as tb
    for (Hq, Hkv, d, w), pos0, n, cut in (((4, 1, 64, 128), 32768, 12763, True), ((8, 2, 64, 1024), 65536, 6363, True),
                                          ((28, 4, 64, 1024), 65536, 1755, True), ((12, 4, 128, 4096), 65536, 4187, True),
                                          ((16, 4, 128, 4096), 65536, 3163, False), ((32, 8, 128, 4096), 65536, 1499, False),
                                          ((64, 8, 128, 4096), 65536, 859, False), ((12, 4, 128, 4096), 0, 4187, False)):
        prm = tb.make_params(Hq, Hkv, d, 32, w, tb.TCA_BF16, 0.5, 0.0)
        kept = np.linspace(0.2, 0.5, Hq)[np.random.default_rng(5).permutation(Hq)] * (pos0 + n)
        offs = np.concatenate([[0], np.cumsum(kept.astype(np.int64))])
        ws = tb.tca_prefill_workspace_bytes(prm, n, int(offs[-1]))
        assert (tb.tca_diag_prefill_walk(prm, offs, pos0, n, ws)[2] > 0) == cut, (Hq, pos0, n)


def test_exports_refuse_host_arrays_of_another_type():
    """The exports take their host arrays as pointers of the declared type: one of another type is refused by the binding
    instead of being read as what it is not."""
    import paper_2512_09238_amd.binding as tb
    prm = tb.make_params(4, 2, 128, 128, 512, tb.TCA_BF16)
    p, rows = np.full((4, 8), 1 / 8), np.zeros(4, np.int64)
    as_f32, as_i32 = p.astype(np.float32), rows.astype(np.int32)
    good_p, good_rows = p.ctypes.data_as(tb._dbl_p), rows.ctypes.data_as(tb._i64_p)
    for pp, rr in ((as_f32.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), good_rows), (good_p, as_i32.ctypes.data_as(tb._i32_p)),
                   (p.ctypes.data, good_rows), (good_p, ctypes.byref(ctypes.c_int32(0)))):
        with pytest.raises(ctypes.ArgumentError):
            tb.lib.tca_select_rows(ctypes.byref(prm), 4, pp, rr)
    assert tb.lib.tca_select_rows(ctypes.byref(prm), 4, good_p, good_rows) == rows.sum() > 0
    assert np.array_equal(tb.tca_select_rows(prm, 4, as_f32)[1], rows)          # the wrappers convert


def test_current_stream_without_the_direct_query(monkeypatch):
    import types

    import torch

    import paper_2512_09238_amd.binding as tb
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 100 + dev, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert tb._stream(None) == 103 and tb._stream(5) == 5
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert tb._stream(None) == 77 and tb._stream(5) == 5


def test_probe_rejects_bad_arguments_without_a_gpu():
    import paper_2512_09238_amd.binding as tb
    assert tb.tca_probe_workspace_bytes() >= 1024 * 24
    tf, ghz = ctypes.c_double(0), ctypes.c_double(0)
    rc = tb.lib.tca_probe_mfma(1, 100, ctypes.byref(tf), ctypes.byref(ghz), None, 0, None)
    assert rc == tb.TCA_ERR_INVALID
    rc = tb.lib.tca_probe_mfma(1, 100, None, None, ctypes.c_void_p(256), 1 << 20, None)
    assert rc == tb.TCA_ERR_INVALID
    rc = tb.lib.tca_probe_mfma(1, 0, ctypes.byref(tf), ctypes.byref(ghz), ctypes.c_void_p(256), 1 << 20, None)
    assert rc == tb.TCA_ERR_INVALID
    rc = tb.lib.tca_probe_mfma(1, 100, ctypes.byref(tf), ctypes.byref(ghz), ctypes.c_void_p(256), 16, None)
    assert rc == tb.TCA_ERR_WORKSPACE


def test_prefill_work_split_over_the_xcds():
    """Host logic of the bf16 prefill launch: the ranges the eight XCDs take cover the (head, query tile)
    sequence once, in order; equal regions with few long items per CU keep whole heads per XCD (an item
    more than the CUs divide would cost a whole round); unequal regions move the cuts towards the light
    heads; and the grid is eight times the longest range."""
    import paper_2512_09238_amd.binding as tb
    Hq, Hkv, d, b, w = 32, 8, 128, 128, 4096
    prm = tb.make_params(Hq, Hkv, d, b, w, tb.TCA_BF16, 0.5, 0.0)
    L = 131072
    n_qt = L // 256                                           # long calls: 256 queries per workgroup

    def check(start, n_wg, items):
        assert start[0] == 0 and start[8] == items and (np.diff(start) >= 0).all()
        assert n_wg == 8 * int(np.diff(start).max())

    # equal regions, the whole sequence: equal work is equal counts
    offs = np.arange(Hq + 1, dtype=np.int64) * 70000
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, offs, 0, L)
    check(start, n_wg, Hq * n_qt)
    assert np.abs(np.diff(start) - 4 * n_qt).max() <= 1 and n_wg <= 8 * (4 * n_qt + 1)
    # the last 8192-token chunk of it: 1024 long items on 256 CUs, four rounds only if every XCD takes 128
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, offs, L - 8192, 8192)
    check(start, n_wg, Hq * 32)
    assert np.array_equal(start, np.arange(9) * 128) and n_wg == 1024
    # regions from 5 % to 50 % of the sequence, heavy heads first: the first XCDs take fewer items
    rows = np.linspace(0.5, 0.05, Hq) * L
    offs = np.concatenate([[0], np.cumsum(rows.astype(np.int64))])
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, offs, 0, L)
    check(start, n_wg, Hq * n_qt)
    counts = np.diff(start)
    assert counts[0] < 4 * n_qt < counts[7] and (np.diff(counts) >= 0).all()
    # the work of the ranges, recomputed here from the sizes: within a few per cent of each other
    def work(g):
        h, qt = g // n_qt, n_qt - 1 - g % n_qt
        last = qt * 256 + 255
        return 64 + 4 + (rows[h] * max(0, last - w + 1) / L) / 64
    per_xcd = [sum(work(g) for g in range(start[x], start[x + 1])) for x in range(8)]
    assert max(per_xcd) / min(per_xcd) < 1.05
    # a window-only part has no regions to weigh: equal counts again
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, offs, 0, L, part=tb.TCA_PART_WINDOW)
    check(start, n_wg, Hq * n_qt)
    assert np.abs(np.diff(start) - 4 * n_qt).max() <= 2
    # short calls use 128 queries per workgroup; head counts that are no multiple of 8 have no plan
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, np.arange(Hq + 1, dtype=np.int64) * 1000, 0, 4096)
    check(start, n_wg, Hq * 32)
    prm12 = tb.make_params(12, 4, d, b, w, tb.TCA_BF16, 0.5, 0.0)
    with pytest.raises(ValueError):
        tb.tca_diag_prefill_xcd_plan(prm12, np.arange(13, dtype=np.int64) * 1000, 0, 4096)


@pytest.mark.parametrize("hq,hkv,share,pos0,n", [
    (8, 8, False, 0, 17000), (16, 4, False, 30000, 9001), (64, 8, False, 0, 5446), (64, 8, True, 0, 5446), (32, 8, False, 65536, 3000),
    (32, 8, False, 114688, 8192), (64, 8, True, 65536, 6000), (64, 8, False, 0, 13000), (40, 8, False, 5000, 7777), (24, 8, False, 0, 12345)])
def test_prefill_plan_is_that_of_a_plain_replay(hq, hkv, share, pos0, n):
    """Order and ranges of calls of more than a round and fewer than sixteen against the same rule played through here, every
    candidate, with a heap: what the plan leaves out cannot change its choice."""
    import heapq

    import paper_2512_09238_amd.binding as tb
    w, GS, nh = 4096, hq // hkv if share else 1, hq // 8
    prm = tb.make_params(hq, hkv, 128, 128, w, tb.TCA_BF16, share=tb.TCA_SHARE_GROUP if share else tb.TCA_SHARE_HEAD)
    eight = -(-n // 256) * hq >= 1024                         # rows fetched through idx: the number of items alone decides
    BM, slots = (256, 32) if eight else (128, 64)
    n_qt, end = -(-n // BM), pos0 + n
    assert 8 * slots < hq * n_qt < 8 * slots * 16
    for seed in range(3):
        cap = np.random.default_rng(seed).integers(0, int(0.5 * end), hq // GS)
        offs = np.concatenate([[0], np.cumsum(cap)]).astype(np.int64)
        first = pos0 + BM * np.arange(n_qt)[::-1]
        last = np.minimum(first + BM - 1, end - 1)
        dense = last // 64 - np.maximum(first - w + 1, 0) // 64 + 1
        cost = [4 + dense + np.where(last >= w, (int(cap[h // GS]) * np.maximum(last - w + 1, 0) // end + 63) // 64, 0) for h in range(hq)]
        flat = np.concatenate(cost)

        def ends(xcds):
            worst = 0
            for items in xcds:
                places = [0] * slots
                for c in items:
                    worst = max(worst, places[0] + int(c))
                    heapq.heapreplace(places, places[0] + int(c))
            return worst

        def ranges(st):
            cut = [max(a, b // n_qt * n_qt) for a, b in zip(st[:-1], st[1:])]
            return ends([np.concatenate([flat[m:b], flat[a:m]]) for a, m, b in zip(st[:-1], cut, st[1:])])

        by_head = [x * nh * n_qt for x in range(9)]
        acc = np.cumsum(flat)
        by_work = [0] + [int(np.argmax(acc * 8 >= acc[-1] * x)) + 1 for x in range(1, 8)] + [len(flat)]
        order, heads, _ = tb.tca_diag_prefill_walk(prm, offs, pos0, n, 0, gather_free=True)
        start, _ = tb.tca_diag_prefill_xcd_plan(prm, offs, pos0, n, gather_free=True)
        deal = np.asarray(heads).reshape(8, nh) if order else None
        if deal is None:                                      # dealt out by the last query tile's cost, the costliest first
            deal, have, total = [[] for _ in range(8)], range(8), [0] * 8
            for h in sorted(range(hq), key=lambda h: -cost[h][0]):
                x = min((x for x in have if len(deal[x]) < nh), key=lambda x: (total[x], x))
                deal[x].append(h)
                total[x] += int(cost[h][0])
            deal = np.arange(hq).reshape(8, nh) if share else np.asarray(deal)
        one = ends([np.stack([cost[h] for h in d], 1).ravel() for d in deal])
        two = ends([np.concatenate([cost[h] for h in d]) for d in deal])
        t = min(ranges(by_head), ranges(by_work))
        expected = 0
        if two * 40 < t * 39:
            t, expected = two, 2
        if one * 20 < t * 19:
            expected = 1
        assert order == expected
        if not expected:
            assert list(start) == (by_head if ranges(by_head) <= ranges(by_work) else by_work)


def test_prefill_of_ten_rounds_keeps_a_head_at_a_time():
    """Ten rounds of workgroups, heads of 4 % to 25 %: ranges of equal work, a head at a time.  Taking the heads of an XCD
    side by side, in whole heads, promises an end 4 % earlier and was 10 % later (all stream through one L2)."""
    import paper_2512_09238_amd.binding as tb
    Hq, L = 32, 20000
    prm = tb.make_params(Hq, 8, 128, 128, 4096, tb.TCA_BF16, 0.5, 0.0)
    rows = np.random.default_rng(4).uniform(0.04, 0.25, Hq) * L
    offs = np.concatenate([[0], np.cumsum(rows.astype(np.int64))])
    start, n_wg = tb.tca_diag_prefill_xcd_plan(prm, offs, 0, L)
    n_qt = -(-L // 256)
    assert start[0] == 0 and start[8] == Hq * n_qt and n_wg == 8 * int(np.diff(start).max())
    assert not np.array_equal(start, np.arange(9) * 4 * n_qt)
    assert tb.tca_diag_prefill_walk(prm, offs, 0, L, 1 << 30)[::2] == (0, 0)


def test_prefill_order_and_chunks_of_a_call():
    """The other orders, where they promise enough: by query tile for one window's length, by head for a late chunk whose
    heads keep different numbers of rows; every head is on one XCD.  A call of few query tiles is cut into chunks if its
    workspace has room for them, a part never."""
    import paper_2512_09238_amd.binding as tb
    Hq, w = 32, 4096
    prm = tb.make_params(Hq, 8, 128, 128, w, tb.TCA_BF16, 0.5, 0.0)
    rows = np.random.default_rng(5).permutation(np.linspace(0.03, 0.3, Hq)) * 65536
    offs = np.concatenate([[0], np.cumsum(rows.astype(np.int64))])
    order, heads, chunks = tb.tca_diag_prefill_walk(prm, np.arange(Hq + 1, dtype=np.int64) * 100, 0, w, 1 << 30)
    assert (order, chunks) == (1, 0) and sorted(heads) == list(range(Hq))
    order, heads, chunks = tb.tca_diag_prefill_walk(prm, offs, 65536, 8192, 1 << 30)
    assert (order, chunks) == (2, 0) and sorted(heads) == list(range(Hq))
    sums = [rows[heads[4 * x:4 * x + 4]].sum() for x in range(8)]
    assert max(sums) / min(sums) < 1.1 and all((np.diff(rows[heads[4 * x:4 * x + 4]]) <= 0).all() for x in range(8))
    full = tb.tca_prefill_workspace_bytes(prm, 300, int(offs[-1]))
    assert 96 < tb.tca_diag_prefill_walk(prm, offs, 65536, 300, full)[2] <= 1024
    assert tb.tca_diag_prefill_walk(prm, offs, 65536, 300, 0)[2] == 0
    for part in (tb.TCA_PART_WINDOW, tb.TCA_PART_GLOBAL):
        assert tb.tca_diag_prefill_walk(prm, offs, 65536, 300, full, part=part)[2] == 0
    assert tb.tca_diag_prefill_walk(tb.make_params(12, 4, 128, 128, w, tb.TCA_BF16, 0.5, 0.0), offs[:13], 65536, 300, full)[0::2] >= (-1, 1)
    with pytest.raises(ValueError):
        tb.tca_diag_prefill_walk(tb.make_params(Hq, 8, 128, 128, w, tb.TCA_F32, 0.5, 0.0), offs, 0, w, 0)



def test_binding_loads_torch_before_the_library():
    """One HIP runtime per process: the binding imports torch (which ships its own copy) before it
    loads libtca.so, whatever the caller imported first."""
    import subprocess
    import sys
    code = ("import sys; import paper_2512_09238_amd.binding as tb; "
            "assert 'torch' in sys.modules; print(tb.tca_num_counts(128))")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "8", r.stderr[-500:]


def test_calibration_file_round_trip(tmp_path):
    """The calibrated configurations as a file: doubles come back bit for bit, a file made for
    another layer shape is refused."""
    import paper_2512_09238_amd.binding as tb
    import paper_2512_09238_amd.calibration as calib
    prm = tb.make_params(4, 2, 128, 128, 4096, tb.TCA_BF16)
    cands = tb.tca_make_candidates(128, 14, 1.0)
    pick = np.array([[3, 7, 7, 13], [0, 5, 6, 8]])
    cal = {"p_star": cands[pick], "cand_idx": pick.astype(np.int32), "fallback": np.array([[0, 0, 0, 1], [0, 0, 0, 0]], np.int32)}
    path = os.path.join(tmp_path, "c.json")
    calib.save_calibration(path, prm, cal, 14, 1.0, 0.9, 8192)
    back = calib.load_calibration(path, prm)
    assert np.array_equal(back["p_star"], cal["p_star"]) and back["p_star"].dtype == np.float64
    assert np.array_equal(back["cand_idx"], cal["cand_idx"]) and np.array_equal(back["fallback"], cal["fallback"])
    assert (back["n_layers"], back["n_selection_heads"], back["candidates"], back["calibration_tokens"]) == (2, 4, 14, 8192)
    one = {"p_star": cands[pick[0]], "cand_idx": pick[0].astype(np.int32), "fallback": np.zeros(4, np.int32)}
    calib.save_calibration(path, prm, one, 14, 1.0, 0.9, 8192)          # a single tca_calibrate_budgets result is one layer
    assert calib.load_calibration(path)["p_star"].shape == (1, 4, 8)
    with pytest.raises(ValueError):
        calib.load_calibration(path, tb.make_params(8, 2, 128, 128, 4096, tb.TCA_BF16))
    with open(path, "w") as f:
        f.write('{"format": "something else"}')
    with pytest.raises(ValueError):
        calib.load_calibration(path)


def test_bench_refuses_more_than_one_gpu():
    """Every box has one GPU: bench.py --gpus N with N above 1 ends with a message, before touching a device."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stderr + r.stdout) or "1 GPU" in (r.stderr + r.stdout) or "--gpus" in (r.stderr + r.stdout)


def test_binding_fails_loudly_without_the_library(tmp_path):
    """The product path has no fallback: with no libtca.so to load, importing the binding raises."""
    import shutil
    import subprocess
    import sys
    pkg = tmp_path / "paper_2512_09238_amd"
    shutil.copytree(os.path.join(ROOT, "paper_2512_09238_amd"), pkg,
                    ignore=shutil.ignore_patterns("*.so", "_build", "__pycache__", "csrc"))
    code = "import paper_2512_09238_amd.binding"
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, timeout=300,
                       env={**os.environ, "PYTHONPATH": str(tmp_path)})
    assert r.returncode != 0 and "libtca" in r.stderr
