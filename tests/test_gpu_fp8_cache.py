"""GPU parity of the FP8 decode cache (TCA_KV_FP8; an extension around the path): codes and scales
byte for byte against the oracle's quantiser, decode steps against the oracle reading the same
dequantised rows."""
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


def _prefill_into_fp8_cache(tb, bufs, prm, x, P_gpu, L, steps, seq=0, batch=1):
    """tca_select into staging buffers of the native type, then the hand-over into an FP8 cache."""
    b = prm.block
    Hs = tb.tca_selection_heads(prm)
    _, rows = tb.tca_select_rows(prm, L // b, P_gpu)
    extra = np.array([tb.tca_decode_budget(b, p) for p in P_gpu]) * ((L + steps) // b - L // b + 1)
    cache = bufs.DecodeCache(prm, batch, rows + extra, kv_format=tb.TCA_KV_FP8)
    gb = bufs.GlobalBuffers(prm, rows + extra)          # same capacity layout as the cache
    Qd, Kd, Vd = bufs.to_device(x["Q"]), bufs.to_device(x["K"]), bufs.to_device(x["V"])
    ws = bufs.workspace(tb.tca_select_workspace_bytes(prm, L))
    tb.tca_select(prm, Qd[:, L - 1].contiguous(), Kd, Vd, L, 0, L, P_gpu, gb.offs, gb.n_rows, gb.idx, gb.Kg, gb.Vg, ws)
    tb.tca_cache_load_global(prm, cache.view, seq, gb.idx, gb.Kg, gb.Vg, gb.offs, gb.n_rows)
    tb.tca_cache_load_window(prm, cache.view, seq, Kd, Vd, L, L)
    torch.cuda.synchronize()
    return cache, gb


FP8_CASES = [
    # Hq, Hkv, d, L, b, w, steps, share, seed
    (8, 2, 128, 1500 + 100, 128, 256, 140, False, 61),
    (4, 4, 64, 90, 8, 32, 30, False, 62),             # d = 64 (4 codes per lane), several completions, L < 3w
    (6, 2, 128, 700, 32, 128, 40, False, 63),         # G = 3
    (8, 2, 128, 900, 64, 128, 70, True, 64),          # one selection per KV head: every row scored against 4 queries
]


FP8_WIDE_CASES = [
    (8, 1, 128, 700, 32, 128, 40, False, 67),         # groups of more than four: four region rows a lane group ahead, ragged ends
    (5, 1, 128, 395, 16, 64, 20, False, 68),
    (8, 1, 128, 600, 32, 96, 40, True, 69),
    (4, 2, 128, 500, 16, 96, 30, False, 70),          # two queries a row: rows of 128 elements on vector units
    (4, 2, 128, 700, 32, 128, 40, True, 71),
    (6, 2, 128, 600, 32, 96, 40, True, 72),           # three: on the matrix cores
]


@pytest.mark.parametrize("case", FP8_CASES + FP8_WIDE_CASES, ids=lambda c: f"Hq{c[0]}-Hkv{c[1]}-d{c[2]}-L{c[3]}-b{c[4]}-w{c[5]}-n{c[6]}{'-shared' if c[7] else ''}")
def test_fp8_cache_bytes_and_decode_match_oracle(tb, bufs, case):
    Hq, Hkv, d, L, b, w, steps, share, seed = case
    print("case", case, flush=True)
    G = Hq // Hkv
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, "bf16", seed)
    prm = H.params_for(tb, Hq, Hkv, d, b, w, "bf16", share=share)
    Hs = tb.tca_selection_heads(prm)
    fr = wl.budget_fractions(seed + 1, Hs)
    P_gpu = np.stack([tb.tca_config_from_budget(b, 1.0, f) for f in fr])
    P_orc = np.stack([orc.config_from_budget(b, 1.0, f) for f in fr])
    cache, gb = _prefill_into_fp8_cache(tb, bufs, prm, x, P_gpu, L, steps)
    assert int(cache.length[0].item()) == L

    Qf, Kf, Vf = wl.to_f64(x["Q"]), wl.to_f64(x["K"]), wl.to_f64(x["V"])
    sels = (orc.select_all_groups if share else orc.select_all_heads)(Qf[:, L - 1], Kf, b, P_orc, 0.5)
    # the global region: positions, codes and scales byte for byte
    for n in range(Hs):
        kvh = n if share else n // G
        o, cnt = int(cache.offs[n]), int(cache.n_rows[0, n].item())
        S = sels[n].S
        assert cnt == len(S) and np.array_equal(cache.idx[0, o:o + cnt].cpu().numpy(), S), f"head {n}"
        for name, src in (("Kg", Kf), ("Vg", Vf)):
            codes, scale = orc.quantize_rows_fp8(src[kvh][S])
            assert np.array_equal(getattr(cache, name)[0, o:o + cnt].cpu().numpy(), codes), (name, n)
            assert np.array_equal(getattr(cache, name + "_scale")[0, o:o + cnt].cpu().numpy(), scale), (name, n)
    # the ring: rows [L-w, L) at slot = position mod w
    first = max(0, L - w)
    slots = np.arange(first, L) % w
    for name, src in (("ringK", Kf), ("ringV", Vf)):
        codes, scale = orc.quantize_rows_fp8(src[:, first:L])
        assert np.array_equal(getattr(cache, name)[0][:, slots].cpu().numpy(), codes), name
        assert np.array_equal(getattr(cache, name + "_scale")[0][:, slots].cpu().numpy(), scale), name

    ocache = orc.cache_after_prefill(Kf, Vf, sels, kv_quant="fp8")
    dec = wl.decode_inputs(Hq, Hkv, d, steps, "bf16", seed + 2, batch=1, gains=x["gains"])
    qd, kd, vd = (bufs.to_device(dec[k]) for k in ("q", "k_new", "v_new"))
    wsd = bufs.workspace(tb.tca_decode_workspace_bytes(prm, 1, cache.max_head_rows))
    O = torch.full((steps, 1, Hq, d), float("nan"), dtype=qd.dtype, device="cuda")
    for s in range(steps):                      # queued back to back, no host sync in between
        tb.tca_decode(prm, cache.view, cache.offs, qd[s], kd[s], vd[s], P_gpu, O[s], wsd)
    torch.cuda.synchronize()
    Og = bufs.to_host_f64(O)
    assert np.isfinite(Og).all()
    worst = 0.0
    for s in range(steps):
        ref = orc.decode_step(ocache, wl.to_f64(dec["q"][s, 0]), wl.to_f64(dec["k_new"][s, 0]),
                              wl.to_f64(dec["v_new"][s, 0]), b, w, P_orc, share=share, kv_quant="fp8")
        worst = max(worst, np.abs(Og[s, 0] - ref).max())
    print("max abs err over steps", worst, flush=True)
    assert worst <= H.TOL["bf16"]
    assert int(cache.length[0].item()) == L + steps
    # after decoding: prefill set + per-block top-t, positions exact, rows as the oracle's cache reads them
    for n in range(Hs):
        kvh = n if share else n // G
        o, cnt = int(cache.offs[n]), int(cache.n_rows[0, n].item())
        assert np.array_equal(cache.idx[0, o:o + cnt].cpu().numpy(), ocache.S[n]), f"head {n} after decoding"
        got = orc.dequantize_rows_fp8(cache.Kg[0, o:o + cnt].cpu().numpy(), cache.Kg_scale[0, o:o + cnt].cpu().numpy())
        assert np.array_equal(got, ocache.K[kvh][ocache.S[n]]), f"head {n} rows after decoding"


@pytest.mark.parametrize("d", [64, 128])
def test_handover_codes_are_those_of_the_divisions(tb, bufs, d):
    """Codes and scales of rows over the range of bf16, bit for bit: every pair of mantissas of an element and its row's
    largest one, zeros of both signs, rows too small or too large for the quotient without a division, one with an infinity."""
    rng = np.random.default_rng(97)
    w, Hkv = 512, 2
    mant = np.arange(128, dtype=np.uint32)
    bits = np.zeros((Hkv, w, d), np.uint32)
    exps = np.concatenate([rng.integers(100, 150, w - 64), rng.integers(1, 70, 32), rng.integers(190, 255, 32)])
    for r in range(w):
        e = int(exps[r])
        # element 0 is the row's largest; the others lie 1 .. 20 octaves below it and run through the mantissas
        bits[:, r, 0] = e << 7 | mant[r % 128]
        below = np.maximum(e - rng.integers(1, 21, (Hkv, d - 1)), 0)
        bits[:, r, 1:] = below << 7 | mant[(np.arange(d - 1) + r // 128 * 32 + np.arange(Hkv)[:, None] * 64) % 128]
    bits |= rng.integers(0, 2, bits.shape).astype(np.uint32) << 15
    bits[:, :, 3] &= 0x8000                                          # zeros, of either sign
    K = (bits << 16).view(np.float32)
    K[0, 7, 5] = np.inf
    Kd = torch.from_numpy(K).cuda().to(torch.bfloat16)
    prm = H.params_for(tb, Hkv, Hkv, d, 16, w, "bf16")
    cache = bufs.DecodeCache(prm, 1, np.full(Hkv, 16), kv_format=tb.TCA_KV_FP8)
    tb.tca_cache_load_window(prm, cache.view, 0, Kd, Kd.flip(0).contiguous(), w, w)
    torch.cuda.synchronize()
    for kvh in range(Hkv):
        amax = np.abs(K[kvh]).max(1)
        with np.errstate(over="ignore", invalid="ignore"):
            scale = np.where(amax > 0, amax / np.float32(448), np.float32(1)).astype(np.float32)
            finite = np.isfinite(K[kvh] / scale[:, None])
            quot = np.clip(K[kvh] / scale[:, None], np.float32(-448), np.float32(448))
        want = torch.from_numpy(quot).to(torch.float8_e4m3fn).view(torch.uint8).numpy()
        for ring, sc in ((cache.ringK[0, kvh], cache.ringK_scale[0, kvh]), (cache.ringV[0, 1 - kvh], cache.ringV_scale[0, 1 - kvh])):
            assert np.array_equal(sc.cpu().numpy().reshape(-1), scale)
            assert np.array_equal(ring.cpu().numpy().reshape(w, d)[finite], want[finite])


def test_load_global_with_the_native_format_is_a_copy_and_checks_its_arguments(tb, bufs):
    Hq, Hkv, d, L, b, w = 4, 2, 64, 600, 16, 64
    x = wl.prefill_inputs("lowrank", Hq, Hkv, d, L, "bf16", 66)
    prm = H.params_for(tb, Hq, Hkv, d, b, w, "bf16")
    P = np.stack([tb.tca_config_from_budget(b, 1.0, f) for f in (0.1, 0.2, 0.3, 0.4)])
    gb, Qd, Kd, Vd = H.gpu_select(tb, bufs, prm, x, P)
    cache = bufs.DecodeCache(prm, 2, np.diff(gb.offs))
    tb.tca_cache_load_global(prm, cache.view, 1, gb.idx, gb.Kg, gb.Vg, gb.offs, gb.n_rows)
    torch.cuda.synchronize()
    assert torch.equal(cache.n_rows[1], gb.n_rows) and int(cache.n_rows[0].sum().item()) == 0
    for h in range(Hq):
        o, n = int(gb.offs[h]), int(gb.n_rows[h].item())
        assert torch.equal(cache.idx[1, o:o + n], gb.idx[o:o + n])
        assert torch.equal(cache.Kg[1, o:o + n], gb.Kg[o:o + n]) and torch.equal(cache.Vg[1, o:o + n], gb.Vg[o:o + n])
    with pytest.raises(tb.TcaError):
        tb.tca_cache_load_global(prm, cache.view, 2, gb.idx, gb.Kg, gb.Vg, gb.offs, gb.n_rows)      # seq outside the batch
    prm32 = H.params_for(tb, Hq, Hkv, d, b, w, "f32")
    c8 = bufs.DecodeCache(prm, 1, np.diff(gb.offs), kv_format=tb.TCA_KV_FP8)
    with pytest.raises(tb.TcaError) as e:                                                         # FP8 rows need bf16 inputs
        tb.tca_cache_load_global(prm32, c8.view, 0, gb.idx, gb.Kg, gb.Vg, gb.offs, gb.n_rows)
    assert e.value.code == tb.TCA_ERR_UNSUPPORTED


REGION_CASES = [
    # Hq = Hkv, capacities of the heads' regions, rows filled of each
    (4, (0, 33, 0, 64), (0, 33, 0, 40)),             # empty regions between; a workgroup's rows in two heads, and in one
    (2, (32, 32), (32, 1)),                          # regions that end where a workgroup does
    (70, tuple(7 * h % 45 for h in range(70)), tuple(7 * h % 45 // 2 for h in range(70))),       # more heads than lanes
]


@pytest.mark.parametrize("case", REGION_CASES, ids=lambda c: f"H{c[0]}")
@pytest.mark.parametrize("kv", ["native", "fp8"])
def test_load_global_copies_the_filled_rows_of_every_region(tb, bufs, case, kv):
    """Rows below each region's count arrive (FP8: as codes and scales of the same rows), what lies behind is left alone."""
    Hn, cap, rows = case
    print("case", Hn, kv, flush=True)
    d, fp8 = 64, kv == "fp8"
    prm = H.params_for(tb, Hn, Hn, d, 16, 32, "bf16")
    gb = bufs.GlobalBuffers(prm, np.array(cap))
    total = int(gb.offs[-1])
    g = torch.Generator(device="cuda").manual_seed(98)
    for t in (gb.Kg, gb.Vg):
        t.copy_(torch.randn(total, d, generator=g, device="cuda"))
    gb.idx.copy_(torch.arange(total, device="cuda"))
    gb.n_rows.copy_(torch.tensor(rows, dtype=torch.int32))
    cache = bufs.DecodeCache(prm, 2, np.array(cap), kv_format=tb.TCA_KV_FP8 if fp8 else tb.TCA_KV_NATIVE)
    cache.idx.fill_(-7)
    tb.tca_cache_load_global(prm, cache.view, 1, gb.idx, gb.Kg, gb.Vg, gb.offs, gb.n_rows)
    torch.cuda.synchronize()
    full = np.concatenate([np.arange(c) < r for c, r in zip(cap, rows)])
    assert np.array_equal(cache.idx[1].cpu().numpy(), np.where(full, np.arange(total), -7))
    assert (cache.idx[0] == -7).all() and np.array_equal(cache.n_rows[1].cpu().numpy(), rows)
    at = torch.from_numpy(full).cuda()
    for src, dst, scale in ((gb.Kg, cache.Kg, getattr(cache, "Kg_scale", None)), (gb.Vg, cache.Vg, getattr(cache, "Vg_scale", None))):
        if fp8:
            codes, sc = orc.quantize_rows_fp8(src[at].double().cpu().numpy())
            assert np.array_equal(dst[1][at].cpu().numpy(), codes) and np.array_equal(scale[1][at].cpu().numpy().ravel(), np.ravel(sc))
        else:
            assert torch.equal(dst[1][at], src[at])


@pytest.mark.parametrize("rows", [0, 1, 31, 33, 130])
@pytest.mark.parametrize("share", [False, True])
@pytest.mark.parametrize("B", [3, 320])
def test_fp8_decode_reads_regions_from_any_eight_bytes(tb, bufs, rows, share, B):
    """Region rows are read 16 bytes a lane where a row meets one query and chunks are long (320 sequences), 8 bytes elsewhere: buffers
    that start 8 bytes off a 16-byte boundary give the same bits.  Region counts at the edges of a wave's rows, and no region at all."""
    Hq, Hkv, d, b, w = 8, 2, 128, 16, 64
    prm = H.params_for(tb, Hq, Hkv, d, b, w, "bf16", share=share)
    Hs = Hkv if share else Hq
    P = np.stack([tb.tca_config_from_budget(b, 1.0, 0.3)] * Hs)
    g = torch.Generator(device="cuda").manual_seed(99)
    q, k, v = (torch.randn(B, n, d, generator=g, device="cuda").bfloat16() for n in (Hq, Hkv, Hkv))
    cap = np.full(Hs, rows)
    fill = [torch.randint(0, 0x78, (B, max(Hs * rows, 1), d), generator=g, device="cuda", dtype=torch.uint8) for _ in range(2)]
    ring = [torch.randint(0, 0x78, (B, Hkv, w, d), generator=g, device="cuda", dtype=torch.uint8) for _ in range(2)]
    outs = []
    for off in (0, 8):
        c = bufs.DecodeCache(prm, B, cap, kv_format=tb.TCA_KV_FP8)
        moved = []
        for t in (c.Kg, c.Vg):
            big = torch.empty(t.numel() + 16, dtype=torch.uint8, device="cuda")
            moved.append(big[off:off + t.numel()].view(t.shape))
        moved[0].copy_(fill[0]); moved[1].copy_(fill[1]); c.ringK.copy_(ring[0]); c.ringV.copy_(ring[1])
        for t in (c.Kg_scale, c.Vg_scale, c.ringK_scale, c.ringV_scale):
            t.fill_(0.01)
        c.length.fill_(50)
        c.length[:3].copy_(torch.tensor([2000, 40, 1999]))
        c.n_rows.fill_(rows)
        if rows:
            c.idx.copy_((torch.arange(rows, device="cuda") * 3).repeat(Hs)[None].expand(B, -1))
        view = tb.make_cache(B, c.cap_rows, c.idx, moved[0], moved[1], c.n_rows, c.ringK, c.ringV, c.length, tb.TCA_KV_FP8, c.Kg_scale,
                             c.Vg_scale, c.ringK_scale, c.ringV_scale)
        O = torch.full_like(q, float("nan"))
        tb.tca_decode(prm, view, c.offs, q, k, v, P, O, bufs.workspace(tb.tca_decode_workspace_bytes(prm, B, c.max_head_rows)))
        torch.cuda.synchronize()
        outs.append(O)
        for s, T in enumerate((2000, 40, 1999)):
            for h in range(Hq):
                hs, kvh = h * Hs // Hq, h * Hkv // Hq
                n = int((np.arange(rows) * 3 <= T - w).sum())
                o, live = hs * rows, min(T + 1, w)
                keys = torch.cat([m[s, o:o + n] if i == 0 else m[s, kvh, :live] for i, m in ((0, moved[0]), (1, c.ringK))]).view(torch.float8_e4m3fn).double()
                vals = torch.cat([m[s, o:o + n] if i == 0 else m[s, kvh, :live] for i, m in ((0, moved[1]), (1, c.ringV))]).view(torch.float8_e4m3fn).double()
                ks = torch.cat([c.Kg_scale[s, o:o + n], c.ringK_scale[s, kvh, :live]]).double()
                vs = torch.cat([c.Vg_scale[s, o:o + n], c.ringV_scale[s, kvh, :live]]).double()
                p = torch.softmax((keys @ q[s, h].double()) * ks / d ** 0.5, 0)
                assert (O[s, h].double() - (p * vs) @ vals).abs().max().item() <= H.TOL["bf16"], (s, h)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("lengths", [(0,), (700,), (0, 5000, 255, 256, 700, 40), tuple(range(0, 1400, 20)), (1024, 2000, 1500),
                                     (1100,) * 64 + (3, 600, 1024, 0), (1100,) * 64 + (2000, 1024)],
                         ids=["empty", "part", "mixed", "70", "full", "full-but-the-last", "66-full"])
def test_rings_of_any_fill_are_read_once(tb, bufs, lengths):
    """The units of all rings, in the order for full ones and the other: sequences that have just begun, part of a window, all of
    it, more of them than lanes, of which the first decide; every ring row below the fill counts once."""
    Hq, Hkv, d, b, w, B = 4, 2, 128, 16, 1024, len(lengths)
    prm = H.params_for(tb, Hq, Hkv, d, b, w, "bf16")
    P = np.stack([tb.tca_config_from_budget(b, 1.0, 0.3)] * Hq)
    g = torch.Generator(device="cuda").manual_seed(100)
    q, k, v = (torch.randn(B, n, d, generator=g, device="cuda").bfloat16() for n in (Hq, Hkv, Hkv))
    c = bufs.DecodeCache(prm, B, np.zeros(Hq, np.int64))
    c.ringK.copy_(torch.randn(c.ringK.shape, generator=g, device="cuda"))
    c.ringV.copy_(torch.randn(c.ringV.shape, generator=g, device="cuda"))
    c.length.copy_(torch.tensor(lengths))
    O = torch.full_like(q, float("nan"))
    ws = bufs.workspace(tb.tca_decode_workspace_bytes(prm, B, 0))
    ws.fill_(0xFF)
    tb.tca_decode(prm, c.view, c.offs, q, k, v, P, O, ws)
    torch.cuda.synchronize()
    assert c.length.tolist() == [T + 1 for T in lengths]
    for s, T in enumerate(lengths):
        live = min(T + 1, w)
        for h in range(Hq):
            keys, vals = c.ringK[s, h // 2, :live].double(), c.ringV[s, h // 2, :live].double()
            at = T % w                                               # (the step wrote it)
            assert torch.equal(c.ringK[s, h // 2, at], k[s, h // 2]) and torch.equal(c.ringV[s, h // 2, at], v[s, h // 2])
            ref = torch.softmax((keys @ q[s, h].double()) / d ** 0.5, 0) @ vals
            assert (O[s, h].double() - ref).abs().max().item() <= H.TOL["bf16"], (s, h)


def test_more_workgroups_than_one_dimension_of_a_grid_holds(tb, bufs):
    """65535 sequences of 128 heads, 257 units of a step each: 256 threads times 16.8 million are more than 2^32.  The first
    sequence, the last and some between against float64; every output is written."""
    Hq, d, b, w, B, rows = 128, 64, 2, 2, 65535, 1025
    assert B * (2 * Hq + 1) * 256 >= 2 ** 32
    prm = H.params_for(tb, Hq, Hq, d, b, w, "bf16")
    P = np.stack([tb.tca_config_from_budget(b, 1.0, 0.5)] * Hq)
    cap = np.where(np.arange(Hq) == 0, rows, 1)                      # two units, one for every other head
    c = bufs.DecodeCache(prm, B, cap, kv_format=tb.TCA_KV_FP8)
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.zeros(B, Hq, d, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    some = [0, 1, 33333, B - 1]
    for s in some:
        for t in (q, k, v):
            t[s] = torch.randn(Hq, d, generator=g, device="cuda").bfloat16()
        for t in (c.Kg, c.Vg, c.ringK, c.ringV):
            t[s] = torch.randint(0, 0x78, t[s].shape, generator=g, device="cuda", dtype=torch.uint8)
    for t in (c.Kg_scale, c.Vg_scale, c.ringK_scale, c.ringV_scale):
        t.fill_(0.01)
    c.length.fill_(6)                                                # no block completes
    c.n_rows.copy_(torch.from_numpy(cap.astype(np.int32)))
    O = torch.full_like(q, float("nan"))
    tb.tca_decode(prm, c.view, c.offs, q, k, v, P, O, bufs.workspace(tb.tca_decode_workspace_bytes(prm, B, c.max_head_rows)))
    torch.cuda.synchronize()
    assert torch.isfinite(O).all() and (c.length == 7).all()
    for s in some:
        for h in range(Hq):
            at = slice(int(c.offs[h]), int(c.offs[h + 1]))
            code = lambda t: t.view(torch.float8_e4m3fn).double()
            keys, vals = torch.cat([code(c.Kg[s, at]), code(c.ringK[s, h])]) * 0.01, torch.cat([code(c.Vg[s, at]), code(c.ringV[s, h])]) * 0.01
            new = len(keys) - 2                                      # position 6 lies in the ring's row 0
            keys[new], vals[new] = (code(t[s, h, 0]) * x[s, h, 0].double() for t, x in ((c.ringK, c.ringK_scale), (c.ringV, c.ringV_scale)))
            ref = torch.softmax((keys @ q[s, h].double()) / d ** 0.5, 0) @ vals
            assert (O[s, h].double() - ref).abs().max().item() <= H.TOL["bf16"], (s, h)
