"""Rows that are not finite: they reach what sees them and nothing else, and never an index."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import tca_oracle as orc
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tb():
    import paper_2512_09238_amd.binding as tb
    return tb


@pytest.fixture(scope="module")
def bufs():
    import paper_2512_09238_amd.buffers as bufs
    return bufs


SELECT_CASES = [
    # tokens, b, shared, what is not finite: every shape of the block ranking, full and with padding
    (64 * 16, 16, False, "nan key"),
    (50 * 16 + 3, 16, True, "nan query"),
    (256 * 2, 2, False, "inf key"),
    (200 * 4, 4, False, "nan query"),
    (300 * 4 + 1, 4, True, "nan key"),
    (1024 * 2, 2, False, "nan key"),
    (1500 * 2, 2, False, "nan key"),
    (4096 * 2, 2, False, "nan query"),
]


@pytest.mark.parametrize("free", [False, True], ids=["compacted", "positions"])
@pytest.mark.parametrize("case", SELECT_CASES, ids=lambda c: f"L{c[0]}-b{c[1]}-share{c[2]}-{c[3].replace(' ', '-')}")
def test_select_keeps_valid_rows_whatever_the_scores(tb, bufs, case, free):
    """A head whose scores are not finite has no ranking, but still keeps the budgets Psi holds, one per block, of rows
    in ascending order; the heads of the other KV head keep what they keep without it."""
    L, b, share, what = case
    print("case", case, free, flush=True)
    Hq, Hkv, d = 4, 2, 64
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, "f32", 61)
    prm = H.params_for(tb, Hq, Hkv, d, b, 4 * b, "f32", share=share)
    Hs = Hkv if share else Hq
    P = np.stack([tb.tca_config_from_budget(b, 1.0, f) for f in np.linspace(0.3, 0.7, Hs)])
    clean, *_ = H.gpu_select(tb, bufs, prm, x, P)
    if what == "nan query":
        x["Q"][0, L - 1, 3] = np.nan
    else:
        x["K"][0, L // 3, 5] = np.nan if what == "nan key" else np.inf
    _, rows = tb.tca_select_rows(prm, L // b, P)
    gb = bufs.GlobalBuffers(prm, rows)
    Qd, Kd, Vd = (bufs.to_device(x[k]) for k in ("Q", "K", "V"))
    tb.tca_select(prm, Qd[:, L - 1].contiguous(), Kd, Vd, L, 0, L, P, gb.offs, gb.n_rows, gb.idx,
                  None if free else gb.Kg, None if free else gb.Vg, bufs.workspace(tb.tca_select_workspace_bytes(prm, L)))
    torch.cuda.synchronize()
    m = L // b
    for h in range(Hs):
        got = H.head_indices(gb, h)
        assert len(got) == rows[h]
        assert got.min() >= 0 and got.max() < m * b and np.all(np.diff(got) > 0)
        assert np.array_equal(np.sort(np.bincount(got // b, minlength=m)), orc.psi_list(b, m, P[h])), f"head {h}"
        o = int(gb.offs[h])
        if not free:
            at = torch.from_numpy(got).cuda()
            assert torch.equal(gb.Kg[o:o + len(got)].view(torch.int32), Kd[h // (Hs // Hkv), at].view(torch.int32))
        if h >= Hs // Hkv:                                           # the KV head without the bad row
            assert np.array_equal(got, H.head_indices(clean, h))


def prefill_call(tb, bufs, Hq, Hkv, d, L, w, dtype, S, Qd, Kd, Vd, free=False, ws_bytes=None, b=16, q0=0):
    """tca_prefill of the queries q0 .. L-1 with the kept positions S (one list per query head): O [Hq, L - q0, d], lse, in float64."""
    prm = H.params_for(tb, Hq, Hkv, d, b, w, dtype)
    gb = bufs.GlobalBuffers(prm, np.array([len(s) for s in S]) + 3)
    for h, s in enumerate(S):
        o, at = int(gb.offs[h]), torch.from_numpy(np.asarray(s, np.int64)).cuda()
        gb.idx[o:o + len(s)] = at.to(torch.int32)
        gb.Kg[o:o + len(s)], gb.Vg[o:o + len(s)] = Kd[h * Hkv // Hq, at], Vd[h * Hkv // Hq, at]
        gb.n_rows[h] = len(s)
    Qt = Qd[:, q0:].contiguous()
    O = torch.full_like(Qt, 7.0)
    lse = torch.full(Qt.shape[:2], 7.0, dtype=torch.float32, device="cuda")
    if ws_bytes is None:
        ws_bytes = tb.tca_prefill_workspace_bytes(prm, L - q0, int(gb.offs[-1]))
    ws = bufs.workspace(ws_bytes)
    tb.tca_prefill(prm, Qt, q0, L - q0, Kd, Vd, L, gb.idx, None if free else gb.Kg, None if free else gb.Vg, gb.offs,
                   gb.n_rows, O, lse, ws)
    torch.cuda.synchronize()
    return O.double().cpu().numpy(), lse.double().cpu().numpy()


def who_sees(Hq, Hkv, L, w, S, kvh, j):
    """[Hq, L] true where query i of head h attends to row j of KV head kvh: in its window, or kept and behind it."""
    i = np.arange(L)
    out = np.zeros((Hq, L), bool)
    for h in range(Hq):
        if h * Hkv // Hq == kvh:
            out[h] = ((i - w < j) & (j <= i)) | ((j <= i - w) & bool(np.isin(j, S[h])))
    return out


F32_CASES = [
    # Hq, Hkv, d, L, w, gather-free, row: 64 queries per workgroup (432 and more), and 16
    (16, 2, 64, 1700, 96, False, 803),
    (32, 4, 128, 900, 64, True, 450),
    (4, 2, 64, 333, 48, False, 100),
    (2, 1, 128, 290, 32, True, 77),
]


def f32_inputs(bufs, case):
    Hq, Hkv, d, L, w, free, j = case
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, "f32", 62)
    rng = np.random.default_rng(63)
    S = [np.unique(np.append(np.setdiff1d(rng.choice(L, L // 3, replace=False), j), [j] if h % 2 == 0 else [])).astype(np.int64)
         for h in range(Hq)]                                         # every other head keeps row j
    return (S,) + tuple(bufs.to_device(x[k]) for k in ("Q", "K", "V"))


@pytest.mark.parametrize("what", ["key", "query"])
@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: f"Hq{c[0]}-d{c[2]}-L{c[3]}-free{c[5]}")
def test_fp32_prefill_shows_a_nan_where_it_is_seen(tb, bufs, case, what):
    """A NaN in a key row makes the outputs of the queries that see it NaN, one in a query row that query's; all others
    keep every bit."""
    Hq, Hkv, d, L, w, free, j = case
    print("case", case, what, flush=True)
    S, Qd, Kd, Vd = f32_inputs(bufs, case)
    clean, clean_lse = prefill_call(tb, bufs, Hq, Hkv, d, L, w, "f32", S, Qd, Kd, Vd, free)
    if what == "key":
        Kd[1 % Hkv, j, 5] = float("nan")
        bad = who_sees(Hq, Hkv, L, w, S, 1 % Hkv, j)
    else:
        Qd[1, j, 5] = float("nan")
        bad = np.zeros((Hq, L), bool)
        bad[1, j] = True
    O, lse = prefill_call(tb, bufs, Hq, Hkv, d, L, w, "f32", S, Qd, Kd, Vd, free)
    assert np.isnan(O[bad]).all()
    assert np.array_equal(O[~bad], clean[~bad]) and np.array_equal(lse[~bad], clean_lse[~bad])


@pytest.mark.parametrize("value", ["inf", "nan"])
@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: f"Hq{c[0]}-d{c[2]}-L{c[3]}-free{c[5]}")
def test_fp32_prefill_keeps_a_value_row_from_those_who_do_not_see_it(tb, bufs, case, value):
    """An infinity or a NaN in a V row: that element of the queries that see the row is not finite, every other element
    and every other query is what it is without (up to the order of a tile's sum: 1e-5 as in the oracle comparison)."""
    Hq, Hkv, d, L, w, free, j = case
    print("case", case, value, flush=True)
    S, Qd, Kd, Vd = f32_inputs(bufs, case)
    clean, clean_lse = prefill_call(tb, bufs, Hq, Hkv, d, L, w, "f32", S, Qd, Kd, Vd, free)
    kvh, e = 1 % Hkv, 37
    Vd[kvh, j, e] = float(value)
    bad = np.zeros((Hq, L, d), bool)
    bad[:, :, e] = who_sees(Hq, Hkv, L, w, S, kvh, j)
    O, lse = prefill_call(tb, bufs, Hq, Hkv, d, L, w, "f32", S, Qd, Kd, Vd, free)
    assert not np.isfinite(O[bad]).any()
    assert np.isfinite(O[~bad]).all() and np.abs(O[~bad] - clean[~bad]).max() <= 1e-5
    assert np.array_equal(lse, clean_lse)


SPLIT_CASES = [
    # Hq, Hkv, d, queries, gather-free, row that is not finite (kept by every other head) or query
    (8, 2, 128, 130, False, 900),
    (16, 2, 64, 300, True, 2500),
    (3, 1, 128, 1, False, 2990),                                     # in the window
    (4, 4, 64, 200, False, "query"),
]


@pytest.mark.parametrize("case", SPLIT_CASES, ids=lambda c: f"Hq{c[0]}-d{c[2]}-n{c[3]}-free{c[4]}-{c[5]}")
def test_prefill_in_chunks_shows_a_nan_where_it_is_seen(tb, bufs, case):
    """A bf16 call cut into chunks of keys and one with the smallest workspace, which is not, are NaN in the same places:
    where a query sees the key row that is NaN, or is NaN itself."""
    Hq, Hkv, d, n, free, j = case
    print("case", case, flush=True)
    L, w = 3000, 256
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, "bf16", 64)
    rng = np.random.default_rng(65)
    at = j if j != "query" else -1
    S = [np.unique(np.append(np.setdiff1d(rng.choice(L - 300, 1500, replace=False), at), [at] if h % 2 == 0 and at >= 0 else [])).astype(np.int64)
         for h in range(Hq)]
    Qd, Kd, Vd = (bufs.to_device(x[k]) for k in ("Q", "K", "V"))
    bad = np.zeros((Hq, L), bool)
    if at >= 0:
        Kd[Hkv - 1, at, 5] = float("nan")
        bad = who_sees(Hq, Hkv, L, w, S, Hkv - 1, at)
    else:
        Qd[Hq - 1, L - 7, 5] = float("nan")
        bad[Hq - 1, L - 7] = True
    total = sum(len(s) + 3 for s in S)
    need = 256 + 512 * d + (total // 64 + Hq + 1 + Hkv * ((n + w) // 64 + 2)) * 128 * d      # clock counters, V^T tiles, rounding
    offs = np.concatenate([[0], np.cumsum([len(s) + 3 for s in S])])
    prm = H.params_for(tb, Hq, Hkv, d, 16, w, "bf16")
    cut = [tb.tca_diag_prefill_walk(prm, offs, L - n, n, size, gather_free=free)[2]
           for size in (tb.tca_prefill_workspace_bytes(prm, n, total), need)]
    assert cut[0] > 0 and cut[1] == 0
    for ws_bytes in (None, need):
        O, _ = prefill_call(tb, bufs, Hq, Hkv, d, L, w, "bf16", S, Qd, Kd, Vd, free, ws_bytes, q0=L - n)
        assert bad[:, L - n:].any()
        assert np.array_equal(np.isnan(O).all(axis=2), bad[:, L - n:]) and np.array_equal(np.isnan(O).any(axis=2), bad[:, L - n:])


@pytest.mark.parametrize("L", [129, 160, 333])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_calibration_shows_a_nan_key(tb, bufs, dtype, d, L):
    """The last key row is seen by the last query alone, but every column mean counts that query: the heads of its KV head
    have no coverage to compare and fall back, the others' results keep every bit."""
    print("case", dtype, d, L, flush=True)
    Hq, Hkv, b, M = 4, 2, 16, 4
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, dtype, 66)
    prm = H.params_for(tb, Hq, Hkv, d, b, b, dtype)
    Qd, Kd = bufs.to_device(x["Q"]), bufs.to_device(x["K"])
    ws = bufs.workspace(tb.tca_calibrate_workspace_bytes(prm, L, M))
    clean = tb.tca_calibrate_budgets(prm, Qd, Kd, L, M, 1.0, 0.5, ws)
    Kd[0, L - 1, 5] = float("nan")
    got = tb.tca_calibrate_budgets(prm, Qd, Kd, L, M, 1.0, 0.5, ws)
    assert np.isnan(got["a"][:2]).all() and got["fallback"][:2].all()
    for name in ("a", "cand_idx", "p_star", "fallback"):
        assert np.array_equal(got[name][2:], clean[name][2:]), name
    assert np.array_equal(got["n"], clean["n"])


DECODE_CASES = [
    # Hq, Hkv, d, shared, rows: every body a step's rows go through, by their type, their length and the queries they meet
    (8, 2, 128, False, "bf16"),
    (8, 2, 128, True, "bf16"),
    (8, 2, 128, False, "fp8"),
    (8, 1, 128, False, "fp8"),
    (6, 2, 128, True, "fp8"),
    (4, 4, 128, False, "fp8"),
    (6, 2, 64, False, "bf16"),
    (4, 2, 64, True, "fp8"),
    (4, 1, 64, False, "f32"),
]
DECODE_L, DECODE_W, DECODE_ROWS = 2003, 160, 300


def decode_setup(tb, bufs, case):
    """A cache of two sequences of DECODE_L tokens, DECODE_ROWS rows a region (the last 20 still inside the window), and one
    step's queries, equal for all heads so that a key row can be set against all of them at once."""
    Hq, Hkv, d, share, rows = case
    fp8 = rows == "fp8"
    prm = H.params_for(tb, Hq, Hkv, d, 16, DECODE_W, "f32" if rows == "f32" else "bf16", share=share)
    Hs = tb.tca_selection_heads(prm)
    g = torch.Generator(device="cuda").manual_seed(67)
    c = bufs.DecodeCache(prm, 2, np.full(Hs, DECODE_ROWS + 5), kv_format=tb.TCA_KV_FP8 if fp8 else tb.TCA_KV_NATIVE)
    for t in (c.Kg, c.Vg, c.ringK, c.ringV):
        if fp8:                                                      # codes of finite numbers
            t.copy_(torch.randint(0, 0x78, t.shape, generator=g, device="cuda") | torch.randint(0, 2, t.shape, generator=g, device="cuda") << 7)
        else:
            t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    for t in (c.Kg_scale, c.Vg_scale, c.ringK_scale, c.ringV_scale):
        if fp8:
            t.copy_(torch.rand(t.shape, generator=g, device="cuda") * 0.01 + 0.001)
    c.length.fill_(DECODE_L)
    c.n_rows.fill_(DECODE_ROWS)
    rng = np.random.default_rng(68)
    for s in range(2):
        for n in range(Hs):
            o = int(c.offs[n])
            old = np.sort(rng.choice(DECODE_L - DECODE_W, DECODE_ROWS - 20, replace=False))
            new = np.sort(rng.choice(np.arange(DECODE_L - DECODE_W + 1, DECODE_L), 20, replace=False))
            c.idx[s, o:o + DECODE_ROWS] = torch.from_numpy(np.append(old, new).astype(np.int32)).cuda()
    dt = torch.float32 if rows == "f32" else torch.bfloat16
    q = torch.randn(2, 1, d, generator=g, device="cuda").expand(2, Hq, d).to(dt).contiguous()
    q = torch.where(q == 0, torch.ones_like(q), q)
    kn, vn = (torch.randn(2, Hkv, d, generator=g, device="cuda").to(dt) for _ in range(2))
    P = np.stack([tb.tca_config_from_budget(16, 1.0, 0.4)] * Hs)

    def step():
        c.length.fill_(DECODE_L)                                     # (no block ends at this position: the regions stay)
        O = torch.full_like(q, 7.0)
        tb.tca_decode(prm, c.view, c.offs, q, kn, vn, P, O, bufs.workspace(tb.tca_decode_workspace_bytes(prm, 2, c.max_head_rows)))
        torch.cuda.synchronize()
        return O
    return c, q, step


def decode_row(c, case, where, row):
    """Row `row` of KV head 0's ring or of the first region, of sequence 1: K, its scale (FP8), and which heads see it."""
    Hq, Hkv, d, share, rows = case
    bad = torch.zeros(2, Hq, dtype=torch.bool)
    G = Hq // Hkv
    if where == "ring":
        bad[1, :G] = True
        return c.ringK[1, 0, row], None if c.ringK_scale is None else c.ringK_scale[1, 0], bad
    bad[1, :G if share else 1] = row < DECODE_ROWS - 20
    return c.Kg[1, row], None if c.Kg_scale is None else c.Kg_scale[1], bad


# rows at the start, inside and at the end of a chunk; the last one of a region is still inside the window, where nobody sees it
DECODE_AT = [("ring", 0), ("ring", 77), ("ring", 159), ("region", 0), ("region", 130), ("region", 279), ("region", 290)]


@pytest.mark.parametrize("at", DECODE_AT, ids=lambda a: f"{a[0]}{a[1]}")
@pytest.mark.parametrize("case", DECODE_CASES, ids=lambda c: f"Hq{c[0]}-Hkv{c[1]}-d{c[2]}-share{c[3]}-{c[4]}")
def test_decode_shows_a_nan_key_where_it_is_seen(tb, bufs, case, at):
    """A NaN in a key row of the ring or of a region (FP8: a NaN code, or a NaN scale) makes the outputs of the heads that see
    the row NaN; every other head keeps every bit."""
    print("case", case, at, flush=True)
    c, _, step = decode_setup(tb, bufs, case)
    clean = step()
    assert torch.isfinite(clean).all()
    k, scale, bad = decode_row(c, case, *at)
    kept = k.clone()
    for what in ("element", "scale"):
        if what == "element":
            k[5] = 0x7F if scale is not None else float("nan")
        elif scale is None:
            break
        else:
            k.copy_(kept)
            scale[at[1]] = float("nan")
        O = step().cpu()
        assert O[bad].isnan().all(), what
        assert torch.equal(O[~bad], clean.cpu()[~bad]), what


@pytest.mark.parametrize("at", [("ring", 0), ("ring", 77), ("region", 0), ("region", 130)], ids=lambda a: f"{a[0]}{a[1]}")
@pytest.mark.parametrize("case", [c for c in DECODE_CASES if c[4] != "fp8"], ids=lambda c: f"Hq{c[0]}-Hkv{c[1]}-d{c[2]}-share{c[3]}-{c[4]}")
def test_decode_gives_a_logit_of_minus_infinity_no_weight(tb, bufs, case, at):
    """Wherever in a chunk the row lies: every output is, bit for bit, that of a logit so small that its term is zero."""
    print("case", case, at, flush=True)
    c, q, step = decode_setup(tb, bufs, case)
    k, _, bad = decode_row(c, case, *at)
    outs = []
    for far in (1e3, float("inf")):
        k.copy_(-torch.sign(q[1, 0]) * far)
        outs.append(step())
    assert bad.any() and torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])
