"""GPU parity of the Quest decode path (page metadata, page selection, attention over the
selected pages, fused select+attend, dense) against the float64 oracle, through the C ABI.
Later stages are fed the oracle's rounded cache so that both sides start from the same
stored bits."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, tdtype, to_dev, to_np
from helpers import attn_close, topk_set_ok
from paper_2605_28640_amd import synth

pytestmark = pytest.mark.gpu


def _cache_from_oracle(w, T, Tcap):
    """Oracle scan of the workload's prefill, rounded to the storage dtype."""
    w = w.scaled(T=T)
    k, v, g = synth.prefill(w)
    ko, vo, _, _ = oracle.rat_scan(k, v, g)
    kc = np.zeros((w.B, w.Hkv, Tcap, w.D), dtype=np.float32)
    vc = np.zeros_like(kc)
    if w.dtype == "bf16":
        kc[:, :, :T], vc[:, :, :T] = oracle.round_to_bf16(ko), oracle.round_to_bf16(vo)
    else:
        kc[:, :, :T], vc[:, :, :T] = ko.astype(np.float32), vo.astype(np.float32)
    return w, kc, vc


def _forced(Np, n_first, n_local):
    f = np.zeros(Np, dtype=bool)
    f[:n_first] = True
    if n_local:
        f[Np - n_local:] = True
    return f


CASES = [
    # workload, T_valid, Tcap, P, K, n_first, n_local
    (synth.C1, 2048, 2048 + 16, 16, 16, 1, 1),
    (synth.C1, 2041, 2048 + 16, 16, 16, 1, 1),                       # ragged last page
    (synth.C2.scaled(Hq=8, Hkv=2), 4096 + 5, 4096 + 64, 16, 32, 1, 1),  # GQA, bf16, D=128
    (synth.C3.scaled(B=2, Hq=2, Hkv=2), 8192, 8192, 64, 8, 1, 2),     # 64-token pages
    (synth.C1.scaled(dtype="bf16"), 1000, 1024, 32, 5, 0, 0),          # D=64 bf16, nothing forced
    # the paper's own Quest settings (App. A.1; Tables 3-4): T = 4096, 64-token pages with
    # top-16 / 8 / 4, 16-token pages with top-4
    (synth.C3.scaled(B=1, Hq=4, Hkv=4), 4096, 4096 + 64, 64, 16, 1, 1),
    (synth.C3.scaled(B=1, Hq=4, Hkv=4), 4096, 4096 + 64, 64, 8, 1, 1),
    (synth.C3.scaled(B=1, Hq=4, Hkv=4), 4096, 4096 + 64, 64, 4, 1, 1),
    (synth.C3.scaled(B=1, Hq=4, Hkv=4), 4096, 4096 + 64, 16, 4, 1, 1),
    # large pages
    (synth.C3.scaled(B=1, Hq=4, Hkv=2), 8192 + 77, 8192 + 512, 512, 5, 1, 1),
    (synth.C3.scaled(B=2, Hq=2, Hkv=2), 6000, 6144, 256, 6, 0, 1),
]


def _random_cases(seed, n):
    """Seeded random small shapes: head counts and grouping, both head dims and dtypes, every
    page size, ragged lengths, budgets from one page to all of them, 0-2 forced pages per end."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        Hkv = int(rng.integers(1, 4))
        G = int(rng.choice([1, 2, 4]))
        D = int(rng.choice([64, 128]))
        dtype = str(rng.choice(["bf16", "f32"]))
        P = int(rng.choice([16, 32, 64, 128, 256]))
        T = int(rng.integers(P + 1, 2500))
        Np = -(-T // P)
        Tcap = Np * P + P * int(rng.integers(0, 3))
        n_first, n_local = int(rng.integers(0, 3)), int(rng.integers(0, 3))
        forced = min(n_first + n_local, Np)
        K = int(rng.integers(max(1, forced), Np + 1))
        w = synth.C1.scaled(B=int(rng.integers(1, 4)), Hq=Hkv * G, Hkv=Hkv, D=D, dtype=dtype,
                            n_needles=0 if T < 64 else 4)
        out.append((w, T, Tcap, P, K, n_first, n_local))
    return out


CASES += _random_cases(20260528, 12)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_meta_select_attend(rs, knobs, case):
    w, T, Tcap, P, K, n_first, n_local = CASES[case]
    say("quest case", case, w.name, T, Tcap, P, K, n_first, n_local)
    w, kc, vc = _cache_from_oracle(w, T, Tcap)
    _, _, _, q = synth.decode_step(w, 0)
    Np = -(-T // P)
    scale = 1.0 / np.sqrt(w.D)
    dt = tdtype(w.dtype)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, P, dt)
    tkc, tvc, tq = to_dev(kc, w.dtype), to_dev(vc, w.dtype), to_dev(q, w.dtype)
    meta = torch.zeros(w.B, w.Hkv, Tcap // P, 2, w.D, dtype=dt, device="cuda")
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, Np))

    # page metadata: bulk, bit-exact values
    rs.quest_page_meta(s, tkc, meta, 0, T)
    ometa = oracle.quest_page_meta(kc, P, T)
    np.testing.assert_array_equal(to_np(meta), ometa)

    # selection
    idx = torch.full((w.B, w.Hq, K), -7, dtype=torch.int32, device="cuda")
    scores = torch.zeros(w.B, w.Hq, Np, device="cuda")
    rs.quest_select_decode(s, tq, meta, T, K, n_first, n_local, idx, scores, ws)
    osc = oracle.quest_scores(q, ometa, Np)
    np.testing.assert_allclose(to_np(scores), osc, rtol=2e-6, atol=1e-5)
    oidx = oracle.quest_select(osc, K, n_first, n_local)
    gidx = to_np(idx)
    forced = _forced(Np, n_first, n_local)
    same = 0
    for b in range(w.B):
        for h in range(w.Hq):
            ok, why = topk_set_ok(osc[b, h], forced, K, gidx[b, h])
            assert ok, (b, h, why)
            same += np.array_equal(gidx[b, h], oidx[b, h])
    say("  identical index lists:", same, "of", w.B * w.Hq)

    # attention over the oracle's list
    out = torch.zeros(w.B, w.Hq, w.D, dtype=dt, device="cuda")
    lse = torch.zeros(w.B, w.Hq, device="cuda")
    rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, to_dev(oidx), K, None, 0, 0, out, lse, None, ws)
    oout, olse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, oidx)
    ok, worst = attn_close(to_np(out), oout, 2e-2 if w.dtype == "bf16" else 1e-4)
    assert ok, worst
    np.testing.assert_allclose(to_np(lse), olse, rtol=1e-4, atol=1e-4)

    # select-then-attend in one call, emitting its selection: as one persistent launch, as two
    # launches, and with the whole step of a (batch, head) inside one workgroup (the library
    # picks by shape; the knobs force each)
    oout2, _ = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, gidx)
    for two_launch, one_wg in (("0", "0"), ("1", "0"), ("1", "1")):
        knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", two_launch)
        knobs.setenv("RATSPARSE_FUSED_ONE_WG", one_wg)
        out2 = torch.zeros_like(out)
        idx2 = torch.full_like(idx, -7)
        rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, K, meta, n_first, n_local, out2, None, idx2, ws)
        np.testing.assert_array_equal(to_np(idx2), gidx)
        assert attn_close(to_np(out2), oout2, 2e-2 if w.dtype == "bf16" else 1e-4)[0]
        out3 = torch.zeros_like(out)
        lse3 = torch.zeros_like(lse)
        rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, K, meta, n_first, n_local, out3, lse3, None, ws)
        assert torch.equal(out3, out2)  # same result when the selection is not emitted
        _, olse2 = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, gidx)
        np.testing.assert_allclose(to_np(lse3), olse2, rtol=1e-4, atol=1e-4)
    knobs.delenv("RATSPARSE_FUSED_TWO_LAUNCH")
    knobs.delenv("RATSPARSE_FUSED_ONE_WG")
    out4 = torch.zeros_like(out)
    rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, K, meta, n_first, n_local, out4, None, None, ws)  # own choice
    assert attn_close(to_np(out4), oout2, 2e-2 if w.dtype == "bf16" else 1e-4)[0]

    # dense path, and full budget = dense
    outd = torch.zeros_like(out)
    rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, 0, None, 0, 0, outd, lse, None, ws)
    od, odl = oracle.sparse_attn_decode(q, kc, vc, P, T, scale)
    assert attn_close(to_np(outd), od, 2e-2 if w.dtype == "bf16" else 1e-4)[0]
    np.testing.assert_allclose(to_np(lse), odl, rtol=1e-4, atol=1e-4)
    outf = torch.zeros_like(out)
    rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, Np, meta, n_first, n_local, outf, None, None, ws)
    assert attn_close(to_np(outf), od, 2e-2 if w.dtype == "bf16" else 1e-4)[0]
    torch.cuda.synchronize()
    ws.async_status()


@pytest.mark.parametrize("P,K,T", [(16, 1100, 19200 + 7), (64, 300, 64 * 330)])
def test_persistent_launch_with_one_long_item_per_unit(rs, knobs, P, K, T):
    """The persistent launch with its work split as coarsely as it goes: one score item and one attend item
    per (batch, head), so a wave walks 60-70 attention steps inside one item (its list entries come in more
    than once) and every score loop runs many rounds.  Same lists and outputs as the two-launch form, and
    the attention against the oracle."""
    w = synth.C2.scaled(B=1, Hq=2, Hkv=2)
    Tcap = -(-T // P) * P + P
    say("long items", P, K, T)
    w, kc, vc = _cache_from_oracle(w, T, Tcap)
    _, _, _, q = synth.decode_step(w, 0)
    Np = -(-T // P)
    scale = 1.0 / np.sqrt(w.D)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, P, torch.bfloat16)
    tkc, tvc, tq = to_dev(kc, "bf16"), to_dev(vc, "bf16"), to_dev(q, "bf16")
    meta = torch.zeros(w.B, w.Hkv, Tcap // P, 2, w.D, dtype=torch.bfloat16, device="cuda")
    rs.quest_page_meta(s, tkc, meta, 0, T)
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, K))
    res = {}
    for form, env in (("two launches", {"RATSPARSE_FUSED_TWO_LAUNCH": "1", "RATSPARSE_FUSED_ONE_WG": "0"}),
                      ("one launch, coarse", {"RATSPARSE_FUSED_TWO_LAUNCH": "0", "RATSPARSE_FUSED_ONE_WG": "0",
                                              "RATSPARSE_FUSED_SATT": "1", "RATSPARSE_FUSED_SSCORE": "1",
                                              "RATSPARSE_FUSED_FINE": "1"})):
        for k_, v_ in env.items():
            knobs.setenv(k_, v_)
        out = torch.zeros(w.B, w.Hq, w.D, dtype=torch.bfloat16, device="cuda")
        lse = torch.zeros(w.B, w.Hq, device="cuda")
        idx = torch.full((w.B, w.Hq, K), -7, dtype=torch.int32, device="cuda")
        rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, None, K, meta, 1, 1, out, lse, idx, ws)
        torch.cuda.synchronize()
        ws.async_status()
        res[form] = (to_np(idx), to_np(out), to_np(lse))
        for k_ in env:
            knobs.delenv(k_)
    np.testing.assert_array_equal(res["one launch, coarse"][0], res["two launches"][0])
    gidx = res["two launches"][0]
    osc = oracle.quest_scores(q, oracle.quest_page_meta(kc, P, T), Np)
    for h in range(w.Hq):
        ok, why = topk_set_ok(osc[0, h], _forced(Np, 1, 1), K, gidx[0, h])
        assert ok, (h, why)
    oout, olse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, gidx)
    for form in res:
        assert attn_close(res[form][1], oout, 2e-2)[0], form
        np.testing.assert_allclose(res[form][2], olse, rtol=1e-4, atol=1e-4)


def test_incremental_meta_equals_bulk(rs):
    w, kc, vc = _cache_from_oracle(synth.C1.scaled(dtype="bf16"), 200, 256)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, 256, 16, torch.bfloat16)
    tkc = to_dev(kc, "bf16")
    inc = torch.zeros(w.B, w.Hkv, 16, 2, w.D, dtype=torch.bfloat16, device="cuda")
    rs.quest_page_meta(s, tkc, inc, 0, 150)
    for t in range(150, 200):
        rs.quest_page_meta(s, tkc, inc, t, t + 1)
    bulk = torch.zeros_like(inc)
    rs.quest_page_meta(s, tkc, bulk, 0, 200)
    assert torch.equal(inc, bulk)
    np.testing.assert_array_equal(to_np(bulk), oracle.quest_page_meta(kc, 16, 200))


def test_scan_with_meta_equals_separate_page_meta(rs):
    """rat_scan's optional page-metadata update (prefill path and one-token appends across page
    boundaries) leaves exactly what quest_page_meta computes from the stored cache."""
    for dtype, D, P in (("bf16", 128, 16), ("f32", 64, 32)):
        B, H, T0, steps = 1, 2, 300, 70
        Tcap = 384
        r = np.random.default_rng(11)
        mk = lambda n: r.standard_normal((B, H, n, D)).astype(np.float32)
        k, v = mk(T0 + steps), mk(T0 + steps)
        if dtype == "bf16":
            k, v = synth.to_bf16_grid(k), synth.to_bf16_grid(v)
        g = (1 / (1 + np.exp(-(4.2 + 0.5 * r.standard_normal((B, H, T0 + steps, D)))))).astype(np.float32)
        dt = tdtype(dtype)
        s = rs.make_shape(B, H, H, D, Tcap, P, dt)
        kc = torch.zeros(B, H, Tcap, D, dtype=dt, device="cuda")
        vc = torch.zeros_like(kc)
        sk = torch.zeros(B, H, D, device="cuda")
        sv = torch.zeros_like(sk)
        meta = torch.zeros(B, H, Tcap // P, 2, D, dtype=dt, device="cuda")
        ws = rs.Workspace(rs.rat_scan_workspace_bytes(s, T0))
        rs.rat_scan(s, to_dev(k[:, :, :T0], dtype), to_dev(v[:, :, :T0], dtype), to_dev(g[:, :, :T0]), sk, sv, kc, vc,
                    0, T0, ws, meta)
        for t in range(T0, T0 + steps):
            rs.rat_scan(s, to_dev(k[:, :, t:t + 1], dtype), to_dev(v[:, :, t:t + 1], dtype), to_dev(g[:, :, t:t + 1]),
                        sk, sv, kc, vc, t, 1, None, meta)
        want = torch.zeros_like(meta)
        rs.quest_page_meta(s, kc, want, 0, T0 + steps)
        assert torch.equal(meta, want)
        np.testing.assert_array_equal(to_np(meta), oracle.quest_page_meta(to_np(kc), P, T0 + steps))
        ws.async_status()


@pytest.mark.parametrize("slab", ["0", "1"])  # full rows, or 32-channel slabs (chunks four / two times as long)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("P", [16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("in_scan", ["1", "0"])
def test_scan_runs_leave_the_page_bounds(rs, knobs, in_scan, P, D, dtype, slab):
    """Long runs with the page metadata: where the scan kernel can (pages of 16 tokens up
    to the chunk length, a start on a chunk boundary) the bounds leave with the states, else the
    touched pages are recomputed afterwards; runs of both kinds back to back, with ragged ends,
    must leave what one bulk pass over the final cache computes.  The knob switches the first
    kind off, so both paths see every run."""
    knobs.setenv("RATSPARSE_SCAN_META", in_scan)
    knobs.setenv("RATSPARSE_SCAN_SLAB", slab)
    B, H = 2, 20  # 40 (batch, head) pairs: full-row chunks (128 tokens at 128 channels, 256 at 64)
    # (t0, T_new): aligned; aligned and a single chunk; unaligned; unaligned; unaligned and long
    runs = [(0, 256), (256, 100), (356, 156), (512, 521), (1033, 200), (1233, 3000)]  # 512: aligned for every form
    T = 4233
    Tcap = 4608  # a multiple of every page size
    r = np.random.default_rng(17)
    k = synth.to_bf16_grid(r.standard_normal((B, H, T, D)).astype(np.float32))
    v = synth.to_bf16_grid(r.standard_normal((B, H, T, D)).astype(np.float32))
    g = (1 / (1 + np.exp(-(4.2 + 0.5 * r.standard_normal((B, H, T, D)))))).astype(np.float32)
    dt = tdtype(dtype)
    s = rs.make_shape(B, H, H, D, Tcap, P, dt)
    kc = torch.zeros(B, H, Tcap, D, dtype=dt, device="cuda")
    vc = torch.zeros_like(kc)
    sk = torch.zeros(B, H, D, device="cuda")
    sv = torch.zeros_like(sk)
    meta = torch.zeros(B, H, Tcap // P, 2, D, dtype=dt, device="cuda")
    ws = rs.Workspace(rs.rat_scan_workspace_bytes(s, 3000))
    for t0, n in runs:
        rs.rat_scan(s, to_dev(k[:, :, t0:t0 + n], dtype), to_dev(v[:, :, t0:t0 + n], dtype), to_dev(g[:, :, t0:t0 + n]),
                    sk, sv, kc, vc, t0, n, ws, meta)
    want = torch.zeros_like(meta)
    rs.quest_page_meta(s, kc, want, 0, T)
    assert torch.equal(meta, want)
    np.testing.assert_array_equal(to_np(meta), oracle.quest_page_meta(to_np(kc), P, T))
    ws.async_status()


def test_exact_ties_take_the_lowest_index(rs):
    B, H, D, P, Np = 1, 2, 128, 16, 300
    r = np.random.default_rng(3)
    base = synth.to_bf16_grid(r.standard_normal((B, H, 7, P, D)).astype(np.float32))
    pick = r.integers(0, 7, Np)
    kc = base[:, :, pick].reshape(B, H, Np * P, D)  # only 7 distinct pages: scores tie exactly
    q = synth.to_bf16_grid(r.standard_normal((B, H, D)).astype(np.float32))
    s = rs.make_shape(B, H, H, D, Np * P, P, torch.bfloat16)
    meta = torch.zeros(B, H, Np, 2, D, dtype=torch.bfloat16, device="cuda")
    rs.quest_page_meta(s, to_dev(kc, "bf16"), meta, 0, Np * P)
    ws = rs.Workspace(rs.quest_select_decode_workspace_bytes(s, Np * P))
    osc = oracle.quest_scores(q, oracle.quest_page_meta(kc, P, Np * P), Np)
    for K in (1, 10, 64, 299, 300):
        idx = torch.zeros(B, H, K, dtype=torch.int32, device="cuda")
        rs.quest_select_decode(s, to_dev(q, "bf16"), meta, Np * P, K, 0, 0, idx, None, ws)
        np.testing.assert_array_equal(to_np(idx), oracle.quest_select(osc, K, 0, 0))


def test_listed_pages_with_skips_and_any_order(rs):
    w, kc, vc = _cache_from_oracle(synth.C1.scaled(dtype="bf16"), 512, 512)
    _, _, _, q = synth.decode_step(w, 1)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, 512, 16, torch.bfloat16)
    idx = np.array([[[31, 2, -1, 7, 19, 0], [5, -1, -1, 30, 1, 8]]], dtype=np.int32)
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, 505, 6))
    out = torch.zeros(w.B, w.Hq, w.D, dtype=torch.bfloat16, device="cuda")
    rs.sparse_attn_decode(s, to_dev(q, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), 505, 0.125,
                          to_dev(idx), 6, None, 0, 0, out, None, None, ws)
    want, _ = oracle.sparse_attn_decode(q, kc, vc, 16, 505, 0.125, idx)
    assert attn_close(to_np(out), want)[0]


def test_argument_errors_are_reported(rs):
    s = rs.make_shape(1, 2, 2, 128, 256, 16, torch.bfloat16)
    t = torch.zeros(1 << 16, dtype=torch.bfloat16, device="cuda")
    i = torch.zeros(64, dtype=torch.int32, device="cuda")
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, 256, 16))
    with pytest.raises(rs.RatsparseError, match="invalid argument"):
        rs.quest_select_decode(s, t, t, 256, 17, 1, 1, i, None, ws)  # K > Np
    with pytest.raises(rs.RatsparseError, match="invalid argument"):
        rs.quest_select_decode(s, t, t, 256, 2, 2, 2, i, None, ws)  # more forced pages than K
    with pytest.raises(rs.RatsparseError, match="invalid argument"):
        rs.sparse_attn_decode(s, t, t, t, 257, 1.0, None, 0, None, 0, 0, t, None, None, ws)  # T > Tcap
    small = rs.Workspace(0)
    big = rs.make_shape(4, 32, 32, 128, 65536, 16, torch.bfloat16)
    with pytest.raises(rs.RatsparseError, match="workspace too small"):
        rs.sparse_attn_decode(big, t, t, t, 65536, 1.0, None, 0, None, 0, 0, t, None, None, small)


def test_random_selector_five_seeds(rs):
    """The random selector of the paper's H2 analysis (Sec. 2.3): uniform K-subsets of the pages
    drawn on the host, five seeds, evaluated through the listed-pages mode (Eq. 4 unchanged).
    Unsorted lists and a list that misses the newest page are legal inputs."""
    w, kc, vc = _cache_from_oracle(synth.C2.scaled(Hq=8, Hkv=2), 4096 + 5, 4096 + 64)
    T, Tcap, P, K = 4096 + 5, 4096 + 64, 16, 32
    Np = -(-T // P)
    _, _, _, q = synth.decode_step(w, 0)
    scale = 1.0 / np.sqrt(w.D)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, P, torch.bfloat16)
    tkc, tvc, tq = to_dev(kc, "bf16"), to_dev(vc, "bf16"), to_dev(q, "bf16")
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, K))
    for seed in range(5):
        r = np.random.default_rng(1000 + seed)
        ridx = np.stack([np.stack([r.choice(Np, size=K, replace=False) for _ in range(w.Hq)]) for _ in range(w.B)])
        ridx = ridx.astype(np.int32)
        out = torch.zeros(w.B, w.Hq, w.D, dtype=torch.bfloat16, device="cuda")
        lse = torch.zeros(w.B, w.Hq, device="cuda")
        rs.sparse_attn_decode(s, tq, tkc, tvc, T, scale, to_dev(ridx), K, None, 0, 0, out, lse, None, ws)
        want, wlse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, ridx)
        ok, worst = attn_close(to_np(out), want)
        assert ok, (seed, worst)
        np.testing.assert_allclose(to_np(lse), wlse, rtol=1e-4, atol=1e-4)
    torch.cuda.synchronize()
    ws.async_status()


GROUP_CASES = [
    # workload, T_valid, Tcap, P, K, n_first, n_local
    (synth.C2.scaled(Hq=8, Hkv=2), 4096 + 5, 4096 + 64, 16, 32, 1, 1),   # G = 4, bf16
    (synth.C1.scaled(Hq=4, Hkv=2), 2041, 2048 + 16, 16, 16, 1, 1),       # G = 2, fp32, D = 64
    (synth.C2.scaled(B=2, Hq=8, Hkv=1), 3000, 3072, 64, 6, 0, 2),        # G = 8, 64-token pages
    (synth.C2.scaled(Hq=6, Hkv=2), 1000, 1024, 16, 8, 1, 1),             # G = 3: not offered
]


@pytest.mark.parametrize("case", range(len(GROUP_CASES)))
def test_group_shared_selection(rs, case):
    """The option for grouped-query attention: one page list per KV head from the summed
    scores of its query heads, attended by all of them."""
    w, T, Tcap, P, K, n_first, n_local = GROUP_CASES[case]
    say("group case", case, w.name, w.Hq, w.Hkv, T, P, K)
    w, kc, vc = _cache_from_oracle(w, T, Tcap)
    _, _, _, q = synth.decode_step(w, 0)
    Np = -(-T // P)
    G = w.Hq // w.Hkv
    scale = 1.0 / np.sqrt(w.D)
    dt = tdtype(w.dtype)
    tol = 2e-2 if w.dtype == "bf16" else 1e-4
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, P, dt)
    tkc, tvc, tq = to_dev(kc, w.dtype), to_dev(vc, w.dtype), to_dev(q, w.dtype)
    meta = torch.zeros(w.B, w.Hkv, Tcap // P, 2, w.D, dtype=dt, device="cuda")
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, Np))
    rs.quest_page_meta(s, tkc, meta, 0, T)
    ometa = oracle.quest_page_meta(kc, P, T)
    idx = torch.full((w.B, w.Hkv, K), -7, dtype=torch.int32, device="cuda")
    scores = torch.zeros(w.B, w.Hkv, Np, device="cuda")
    if G not in (2, 4, 8):
        with pytest.raises(rs.RatsparseError, match="status 2"):
            rs.quest_select_decode_group(s, tq, meta, T, K, n_first, n_local, idx, scores, ws)
        return
    rs.quest_select_decode_group(s, tq, meta, T, K, n_first, n_local, idx, scores, ws)
    osc = oracle.quest_scores_group(q, ometa, Np)
    np.testing.assert_allclose(to_np(scores), osc, rtol=4e-6, atol=2e-5)
    gidx = to_np(idx)
    forced = _forced(Np, n_first, n_local)
    for b in range(w.B):
        for kvh in range(w.Hkv):
            ok, why = topk_set_ok(osc[b, kvh], forced, K, gidx[b, kvh])
            assert ok, (b, kvh, why)
    # every query head of the group attends the group's list
    per_head = np.repeat(gidx, G, axis=1)
    want, wlse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, per_head)
    out = torch.zeros(w.B, w.Hq, w.D, dtype=dt, device="cuda")
    lse = torch.zeros(w.B, w.Hq, device="cuda")
    rs.sparse_attn_decode_group(s, tq, tkc, tvc, T, scale, idx, K, None, 0, 0, out, lse, None, ws)
    ok, worst = attn_close(to_np(out), want, tol)
    assert ok, worst
    np.testing.assert_allclose(to_np(lse), wlse, rtol=1e-4, atol=1e-4)
    # select, then attend, in one call; same list, same result
    out2 = torch.zeros_like(out)
    idx2 = torch.full_like(idx, -7)
    rs.sparse_attn_decode_group(s, tq, tkc, tvc, T, scale, None, K, meta, n_first, n_local, out2, None, idx2, ws)
    np.testing.assert_array_equal(to_np(idx2), gidx)
    assert torch.equal(out2, out)
    with pytest.raises(rs.RatsparseError, match="status 1"):  # no dense mode
        rs.sparse_attn_decode_group(s, tq, tkc, tvc, T, scale, None, 0, None, 0, 0, out2, None, None, ws)
    torch.cuda.synchronize()
    ws.async_status()


@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 4), ("bf16", 128, 8), ("bf16", 64, 2), ("f32", 128, 2), ("f32", 64, 8), ("f32", 128, 8)])
def test_dense_decode_of_shared_rows(rs, knobs, dtype, D, G):
    """Dense decode under grouped-query attention with the query heads of a KV head taken together (forced, for any
    length it may be asked for) and head by head: both against the oracle.  Lengths around a tile, a wave's step, a
    workgroup's and several splits; rows past T hold NaN; then a page list per KV head with skipped entries."""
    B, Hkv, P, r = 2, 2, 16, np.random.default_rng(G * D)
    Tcap, tol = 4128, 2e-2 if dtype == "bf16" else 1e-4  # (the tolerances of the tests above)
    kc, vc = (r.standard_normal((B, Hkv, Tcap, D)).astype(np.float32) for _ in range(2))
    q = r.standard_normal((B, Hkv * G, D)).astype(np.float32)
    if dtype == "bf16":
        kc, vc, q = (synth.to_bf16_grid(x) for x in (kc, vc, q))
    s = rs.make_shape(B, Hkv * G, Hkv, D, Tcap, P, tdtype(dtype))
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, Tcap, Tcap // P))
    scale, tq = 2.0 / np.sqrt(D), to_dev(q, dtype)
    for T in (1, 15, 17, 127, 129, 500, 1030, 4100):
        dk, dv = kc.copy(), vc.copy()
        dk[:, :, T:], dv[:, :, T:] = np.nan, np.nan
        tk, tv = to_dev(dk, dtype), to_dev(dv, dtype)
        all_pages = np.tile(np.arange(-(-T // P), dtype=np.int32), (B, Hkv * G, 1))
        want, wlse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, all_pages)
        lists = np.sort(np.stack([r.choice(-(-T // P), max(1, -(-T // P) // 2), replace=False) for _ in range(B * Hkv)]), 1)
        lists = lists.reshape(B, Hkv, -1).astype(np.int32)
        lwant, llse = oracle.sparse_attn_decode(q, kc, vc, P, T, scale, np.repeat(lists, G, axis=1))
        given = np.concatenate([lists, np.full((B, Hkv, 1), -1, np.int32)], 2) if lists.shape[2] < -(-T // P) else lists
        for shared in ("1", "0"):
            knobs.setenv("RATSPARSE_ATTEND_SHARED", shared)
            for idx, w, wl in ((None, want, wlse), (given, lwant, llse)):
                out = torch.full((B, Hkv * G, D), 7.0, dtype=tdtype(dtype), device="cuda")
                lse = torch.full((B, Hkv * G), 7.0, device="cuda")
                if idx is None:
                    rs.sparse_attn_decode(s, tq, tk, tv, T, scale, None, 0, None, 0, 0, out, lse, None, ws)
                else:
                    rs.sparse_attn_decode_group(s, tq, tk, tv, T, scale, torch.from_numpy(idx).cuda(), idx.shape[2], None, 0, 0,
                                                out, lse, None, ws)
                ok, worst = attn_close(to_np(out), w, tol)
                assert ok, (T, shared, idx is None, worst)
                np.testing.assert_allclose(to_np(lse), wl, rtol=1e-4, atol=1e-4)
        ws.async_status()


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("scores", ["spread", "ties", "nan"])
def test_few_pages_in_one_workgroup(rs, knobs, dtype, D, scores):
    """The one-workgroup step counts ranks up to 256 pages and takes radix passes beyond, and fetches the pages that are kept
    anyway before it knows the rest: the lists are those of the two-launch form, the outputs (other orders of the same
    rows) agree to float32 rounding through the weights, 2^-20 of their size or one rounding of the storage type."""
    P, B, Hq, Hkv = 16, 2, 4, 2
    for Np, K, n_first, n_local in ((1, 1, 1, 1), (2, 2, 1, 1), (3, 2, 1, 1), (5, 4, 0, 2), (9, 5, 2, 0), (63, 8, 1, 1), (64, 64, 3, 1),
                                    (65, 9, 1, 2), (127, 16, 1, 1), (129, 30, 0, 0), (255, 40, 1, 4), (256, 64, 2, 2), (257, 64, 1, 1)):
        say("few pages", dtype, D, scores, Np, K, n_first, n_local)
        T = Np * P - 5
        gen = torch.Generator(device="cuda")
        gen.manual_seed(Np)
        s = rs.make_shape(B, Hq, Hkv, D, Np * P, P, tdtype(dtype))
        kc, vc = (torch.randn(B, Hkv, Np * P, D, generator=gen, device="cuda").to(tdtype(dtype)) for _ in range(2))
        q = torch.randn(B, Hq, D, generator=gen, device="cuda").to(tdtype(dtype))
        meta = torch.zeros(B, Hkv, Np, 2, D, dtype=tdtype(dtype), device="cuda")
        rs.quest_page_meta(s, kc, meta, 0, T)
        if scores == "ties":
            meta[:] = meta[:, :, :1]
            meta[:, :, 1::3] *= 2
        if scores == "nan":
            meta[:, :, Np // 2:, 1, 0] = -torch.tensor(float("nan"), device="cuda")
        ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, K))
        got = []
        for one_wg in ("0", "1"):
            knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", "1")
            knobs.setenv("RATSPARSE_FUSED_ONE_WG", one_wg)
            out = torch.zeros(B, Hq, D, dtype=tdtype(dtype), device="cuda")
            lse = torch.zeros(B, Hq, device="cuda")
            idx = torch.full((B, Hq, K), -5, dtype=torch.int32, device="cuda")
            rs.sparse_attn_decode(s, q, kc, vc, T, 1.0 / np.sqrt(D), None, K, meta, n_first, n_local, out, lse, idx, ws)
            torch.cuda.synchronize()
            ws.async_status()
            got.append((to_np(out), to_np(lse), to_np(idx)))
        np.testing.assert_array_equal(got[1][2], got[0][2])
        np.testing.assert_allclose(got[1][1], got[0][1], rtol=1e-6, atol=2e-6)
        np.testing.assert_allclose(got[1][0], got[0][0], rtol=2.0 ** -7 if dtype == "bf16" else 1e-5, atol=2e-6)


@pytest.mark.parametrize("P,T,K,Hq,Hkv,D,dtype", [(16, 1024, 5, 2, 2, 128, "bf16"), (16, 1040 - 3, 64, 4, 2, 64, "bf16"), (64, 9001, 100, 2, 1, 128, "f32"),
                                                   (16, 70000, 700, 2, 2, 64, "bf16"), (16, 16 * 12100, 300, 1, 1, 64, "bf16")])
def test_selection_by_every_split_or_by_a_launch_of_its_own(rs, knobs, P, T, K, Hq, Hkv, D, dtype):
    """As two launches the attention's splits select for themselves (a split's part of the list may begin and end inside a
    page); with more keys than fit the LDS, and with a workspace that has no room for them, the first launch selects: the
    same lists, log-sum-exps and outputs bit for bit, with and without the list asked for."""
    say("selection by split", P, T, K, Hq, Hkv, D, dtype)
    knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", "1")
    knobs.setenv("RATSPARSE_FUSED_ONE_WG", "0")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T)
    Np, B = -(-T // P), 1
    s = rs.make_shape(B, Hq, Hkv, D, Np * P, P, tdtype(dtype))
    kc, vc = (torch.randn(B, Hkv, Np * P, D, generator=gen, device="cuda").to(tdtype(dtype)) for _ in range(2))
    q = torch.randn(B, Hq, D, generator=gen, device="cuda").to(tdtype(dtype))
    meta = torch.zeros(B, Hkv, Np, 2, D, dtype=tdtype(dtype), device="cuda")
    rs.quest_page_meta(s, kc, meta, 0, T)
    need = rs.sparse_attn_decode_workspace_bytes(s, T, K)
    keys = -(-(B * Hq * (-(-Np // 4) * 4) * 4) // 256) * 256
    got = []
    for size, with_list in ((need, True), (need - keys - 256, True), (need, False)):
        ws = rs.Workspace(size)
        out = torch.zeros(B, Hq, D, dtype=tdtype(dtype), device="cuda")
        lse = torch.zeros(B, Hq, device="cuda")
        idx = torch.full((B, Hq, K), -5, dtype=torch.int32, device="cuda")
        for _ in range(2):  # (the second time on a workspace that holds the first one's words)
            rs.sparse_attn_decode(s, q, kc, vc, T, 1.0 / np.sqrt(D), None, K, meta, 1, 1, out, lse, idx if with_list else None, ws)
        torch.cuda.synchronize()
        ws.async_status()
        got.append((out, lse, idx))
    assert torch.equal(got[0][2], got[1][2]) and int(got[0][2].min()) == 0 and int(got[0][2].max()) == Np - 1
    for o in got[1:]:
        assert torch.equal(o[0], got[0][0]) and torch.equal(o[1], got[0][1])


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("P", [32, 64, 512])
@pytest.mark.parametrize("form", ["one_wg", "select_by_split", "select_by_launch", "persistent", "step", "listed", "group", "group_listed"])
def test_rows_that_are_not_attended_count_for_nothing(rs, knobs, form, P, dtype, D):
    """Only rows below T_valid of kept pages may reach the result.  Rows from T_valid on hold NaN (tiles of the last page
    begin past it wherever P >= 32), page 0 is not kept and the values of its first 16 rows are infinite or NaN, and given
    lists also name pages past the end: the first one, and one whose first row is 2^32."""
    G = 2 if form.startswith("group") else 1
    B, Hkv, dt, tol = 1, 2, tdtype(dtype), 2e-2 if dtype == "bf16" else 1e-4  # (the tolerances of the tests above)
    Hq, scale = Hkv * G, 1.0 / np.sqrt(D)
    knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", "0" if form == "persistent" else "1")
    knobs.setenv("RATSPARSE_FUSED_ONE_WG", "1" if form == "one_wg" else "0")
    knobs.setenv("RATSPARSE_ATTEND_SHARED", "1")
    for T in (1, 5, 15, 17, P + 1, 2 * P + 3, 63 * P + 17, 70 * P + 16):
        Np = -(-T // P)
        K = min(3, Np - 1) if Np > 1 else 1  # (page 0 is left out where there is another)
        say("rows not attended", form, P, dtype, T, K)
        Tcap = (Np + 1) * P
        gen = torch.Generator(device="cuda").manual_seed(T)
        kc, vc = (torch.randn(B, Hkv, Tcap, D, generator=gen, device="cuda") for _ in range(2))
        q = (torch.randn(B, Hq, D, generator=gen, device="cuda").abs() + 0.1).to(dt)
        meta = torch.zeros(B, Hkv, Tcap // P, 2, D, dtype=dt, device="cuda")
        if Np > 1:
            kc[:, :, :P] = -4.0
            vc[:, :, :16:3], vc[:, :, 1:16:3] = torch.inf, torch.nan
        kc[:, :, T:], vc[:, :, T:] = torch.nan, torch.nan
        kc, vc = kc.to(dt), vc.to(dt)
        s = rs.make_shape(B, Hq, Hkv, D, Tcap, P, dt)
        rs.quest_page_meta(s, kc, meta, 0, T)
        heads = Hkv if G > 1 else Hq
        idx = torch.full((B, heads, K), -5, dtype=torch.int32, device="cuda")
        out, lse = torch.full((B, Hq, D), 7.0, dtype=dt, device="cuda"), torch.full((B, Hq), 7.0, device="cuda")
        need = rs.sparse_attn_decode_workspace_bytes(s, T, max(K, 3))
        if form == "select_by_launch":
            need = rs.sparse_attn_decode_workspace_bytes(s, T, K) - -(-(B * Hq * (-(-Np // 4) * 4) * 4) // 256) * 256 - 256
        ws = rs.Workspace(need)
        if form == "step":
            ws = rs.Workspace(rs.rat_decode_step_workspace_bytes(s, T, K))
            rs.rat_decode_state_set(ws, T - 1)
            state = [torch.randn(B, Hkv, D, generator=gen, device="cuda") for _ in range(2)]
            k, v = (torch.randn(B, Hkv, 1, D, generator=gen, device="cuda").to(dt) for _ in range(2))
            g = torch.rand(B, Hkv, 1, D, generator=gen, device="cuda")
            rs.rat_decode_step(s, k, v, g, *state, kc, vc, meta, q, scale, K, 0, 1, T, out, lse, idx, ws)
        elif form.endswith("listed"):
            if Np > 2:
                K = 3
                idx = torch.tensor([Np - 1, Np, 2 ** 32 // P], dtype=torch.int32, device="cuda").repeat(B, heads, 1)
            else:
                idx[:] = Np - 1
            call = rs.sparse_attn_decode_group if G > 1 else rs.sparse_attn_decode
            call(s, q, kc, vc, T, scale, idx, K, None, 0, 0, out, lse, None, ws)
        else:
            call = rs.sparse_attn_decode_group if G > 1 else rs.sparse_attn_decode
            call(s, q, kc, vc, T, scale, None, K, meta, 0, 1, out, lse, idx, ws)
        torch.cuda.synchronize()
        ws.async_status()
        for b in range(B):
            for h in range(Hq):
                pages = [p for p in idx[b, h // G].tolist() if p < Np]
                assert pages[-1] == Np - 1 and (Np == 1 or 0 not in pages), pages
                rows = torch.cat([torch.arange(p * P, min((p + 1) * P, T)) for p in pages]).cuda()
                x = kc[b, h // G, rows].double() @ q[b, h].double() * scale
                want = torch.softmax(x, 0) @ vc[b, h // G, rows].double()
                ok, worst = attn_close(to_np(out[b, h]), to_np(want), tol)
                assert ok, (T, h, worst)
                np.testing.assert_allclose(float(lse[b, h]), float(torch.logsumexp(x, 0)), rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("B,H,T,K,dtype", [(3, 4, 7473, 0, "f32"), (1, 12, 3000, 0, "bf16"), (7, 8, 1100, 30, "bf16"), (5, 11, 30000, 0, "bf16"), (31, 8, 300, 0, "bf16"),
                                           (1, 18, 33000, 1100, "bf16"), (7, 10, 257, 0, "bf16"), (2, 128, 260, 0, "bf16"), (1, 257, 260, 0, "bf16")])
def test_splits_of_unit_counts_that_do_not_divide_the_chip(rs, knobs, B, H, T, K, dtype):
    """A few units more or fewer than divide 256 or 512 workgroups: dense decode, and two launches with a selection, against
    64-bit attention over the rows kept.  (bfloat16 outputs are rounded once, 2^-8 of a value; float32 sums of 7473
    weights: a few times 2^-24 x 16.)"""
    say("uneven units", B, H, T, K, dtype)
    knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", "1")
    knobs.setenv("RATSPARSE_FUSED_ONE_WG", "0")
    P, D, dt = 16, 128, tdtype(dtype)
    Np = -(-T // P)
    gen = torch.Generator(device="cuda").manual_seed(T)
    kc, vc = (torch.randn(B, H, Np * P, D, generator=gen, device="cuda").to(dt) for _ in range(2))
    q = torch.randn(B, H, D, generator=gen, device="cuda").to(dt)
    s = rs.make_shape(B, H, H, D, Np * P, P, dt)
    meta = torch.zeros(B, H, Np, 2, D, dtype=dt, device="cuda")
    if K:
        rs.quest_page_meta(s, kc, meta, 0, T)
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, K))
    out, lse = torch.zeros(B, H, D, dtype=dt, device="cuda"), torch.zeros(B, H, device="cuda")
    idx = torch.full((B, H, max(K, 1)), -5, dtype=torch.int32, device="cuda")
    rs.sparse_attn_decode(s, q, kc, vc, T, D ** -0.5, None, K, meta if K else None, 1 if K else 0, 1 if K else 0, out, lse, idx if K else None, ws)
    torch.cuda.synchronize()
    ws.async_status()
    tol = 2.0 ** -8 if dtype == "bf16" else 4e-6
    for b in range(B):
        for h in range(H):
            rows = torch.arange(T, device="cuda")
            if K:
                rows = (idx[b, h].long()[:, None] * P + torch.arange(P, device="cuda")).flatten()
                rows = rows[rows < T]
            x = kc[b, h, rows].double() @ q[b, h].double() * D ** -0.5
            want = torch.softmax(x, 0) @ vc[b, h, rows].double()
            assert float((out[b, h].double() - want).abs().max()) <= tol * float(want.abs().max()), (b, h)
            assert abs(float(lse[b, h]) - float(torch.logsumexp(x, 0))) <= 1e-5


def _score_rows(Np, rng):
    """Page scores of several kinds, one row each: spread out, tied, crowded beside outliers, not finite, of extreme range."""
    n = rng.standard_normal(Np)
    rows = [n, 5 + 0.1 * n, rng.integers(0, 10, Np), np.full(Np, 2.5), np.round(n * 8) / 8, np.exp(6 * n), n * 1e-38, n * 5e37]
    for big in (1e30, np.inf):
        x = n.copy()
        x[rng.integers(0, Np, 3)] = big
        rows.append(x)
    rows.append(np.where(rng.random(Np) < 0.3, -np.inf, n))
    rows.append(np.where(n > 0, 0.0, -0.0))
    return np.stack(rows).astype(np.float32)


@pytest.mark.parametrize("Np,K", [(257, 3), (512, 64), (513, 513), (1024, 1023), (1025, 130), (2049, 256), (4096, 2048), (4097, 2),
                                  (5120, 640), (5121, 640)])
def test_selection_over_kinds_of_scores(rs, knobs, Np, K):
    """Selection from scores that are given exactly (a one-hot query picks one channel of the page bounds): the list is that of a
    stable sort, whichever way the selection goes about it (one histogram, ranked bin, radix passes), alone and inside the decode."""
    say("kinds of scores", Np, K)
    D, P = 64, 16
    sc = _score_rows(Np, np.random.default_rng(Np))
    H = sc.shape[0]
    want = np.empty((H, K), np.int64)
    for h in range(H):
        x = sc[h] + 0.0  # -0 to 0
        x[0] = x[-1] = np.inf
        if np.isinf(sc[h]).any():  # forced pages come before infinite ones
            order = np.lexsort((np.arange(Np), -x, ~_forced(Np, 1, 1)))
        else:
            order = np.argsort(-x, kind="stable")
        want[h] = np.sort(order[:K])
    meta = torch.zeros(1, H, Np, 2, D, device="cuda")
    meta[0, :, :, 0, 0] = meta[0, :, :, 1, 0] = torch.from_numpy(sc).cuda()
    q = torch.zeros(1, H, D, device="cuda")
    q[:, :, 0] = 1
    s = rs.make_shape(1, H, H, D, Np * P, P, torch.float32)
    T = Np * P
    idx = torch.full((1, H, K), -5, dtype=torch.int32, device="cuda")
    ws = rs.Workspace(max(rs.quest_select_decode_workspace_bytes(s, T), rs.sparse_attn_decode_workspace_bytes(s, T, K)))
    rs.quest_select_decode(s, q, meta, T, K, 1, 1, idx, None, ws)
    assert np.array_equal(to_np(idx)[0], want)
    kc = torch.zeros(1, H, T, D, device="cuda")
    out, lse = torch.zeros(1, H, D, device="cuda"), torch.zeros(1, H, device="cuda")
    for two, one in (("1", "0"), ("0", "0"), ("0", "1")):
        if one == "1" and (Np > 4096 or K > 1024):
            continue
        knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", two)
        knobs.setenv("RATSPARSE_FUSED_ONE_WG", one)
        idx.fill_(-5)
        rs.sparse_attn_decode(s, q, kc, kc, T, 1.0, None, K, meta, 1, 1, out, lse, idx, ws)
        torch.cuda.synchronize()
        ws.async_status()
        assert np.array_equal(to_np(idx)[0], want), (two, one)


@pytest.mark.parametrize("B,Hq,Hkv,D,T,K,dtype", [
    (1, 64, 64, 128, 512 * 16 + 1, 32, "bf16"), (2, 33, 33, 128, 1031 * 16 - 5, 16, "bf16"), (1, 130, 1, 64, 777 * 16, 40, "bf16"),
    (1, 70, 70, 64, 3001 * 16, 60, "f32"), (3, 32, 32, 128, 40000, 160, "bf16"), (4, 32, 8, 128, 32768, 256, "bf16"),
    (2, 32, 8, 128, 65000, 1015, "bf16"), (4, 32, 32, 128, 32768, 256, "f32"),
    # rows of 128 bytes, shared and the CUs filled or not; more than 450 MB with few and with many page bounds
    (8, 32, 8, 64, 30000, 469, "bf16"), (5, 32, 8, 64, 34918, 545, "bf16"), (7, 16, 16, 128, 50000, 390, "bf16"),
    (16, 32, 32, 64, 38400, 150, "bf16")])
def test_own_choice_of_form_over_fills_of_the_chip(rs, knobs, B, Hq, Hkv, D, T, K, dtype):
    """The library's own choice between one persistent launch and two plain ones (on each side of its lines: few heads, CUs filled
    evenly or not, shared rows), and each form by name: the same lists, and outputs that differ by rounding only.  The pages are scored in steps of
    128 or 256: one step or several, whole or with a remainder."""
    say("own choice of form", B, Hq, Hkv, D, T, K, dtype)
    P, gen = 16, torch.Generator(device="cuda")
    gen.manual_seed(T)
    Np = -(-T // P)
    s = rs.make_shape(B, Hq, Hkv, D, Np * P, P, tdtype(dtype))
    kc, vc = (torch.randn(B, Hkv, Np * P, D, generator=gen, device="cuda").to(tdtype(dtype)) for _ in range(2))
    q = torch.randn(B, Hq, D, generator=gen, device="cuda").to(tdtype(dtype))
    meta = torch.zeros(B, Hkv, Np, 2, D, dtype=tdtype(dtype), device="cuda")
    rs.quest_page_meta(s, kc, meta, 0, T)
    ws = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(s, T, K))
    got = []
    for form in (None, "0", "1"):
        if form is not None:
            knobs.setenv("RATSPARSE_FUSED_TWO_LAUNCH", form)
            knobs.setenv("RATSPARSE_FUSED_ONE_WG", "0")
        out = torch.zeros(B, Hq, D, dtype=tdtype(dtype), device="cuda")
        lse = torch.zeros(B, Hq, device="cuda")
        idx = torch.full((B, Hq, K), -5, dtype=torch.int32, device="cuda")
        rs.sparse_attn_decode(s, q, kc, vc, T, 1.0 / np.sqrt(D), None, K, meta, 1, 1, out, lse, idx, ws)
        torch.cuda.synchronize()
        ws.async_status()
        got.append((to_np(out), to_np(lse), to_np(idx)))
    for other in got[1:]:
        np.testing.assert_array_equal(other[2], got[0][2])
        np.testing.assert_allclose(other[1], got[0][1], rtol=1e-6, atol=2e-6)
        np.testing.assert_allclose(other[0], got[0][0], rtol=2.0 ** -7 if dtype == "bf16" else 1e-5, atol=2e-6)
