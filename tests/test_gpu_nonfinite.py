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
