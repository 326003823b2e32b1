"""GPU parity of MoBA routing (block means, gate scores, top-K blocks) and of the block-sparse
/ dense causal prefill attention against the float64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, to_dev, to_np
from helpers import attn_close, topk_set_ok
from paper_2605_28640_amd import synth

pytestmark = pytest.mark.gpu


def _setup(w, T, Tcap):
    w = w.scaled(T=T)
    k, v, g = synth.prefill(w)
    ko, vo, _, _ = oracle.rat_scan(k, v, g)
    kc = np.zeros((w.B, w.Hkv, Tcap, w.D), dtype=np.float32)
    vc = np.zeros_like(kc)
    kc[:, :, :T], vc[:, :, :T] = oracle.round_to_bf16(ko), oracle.round_to_bf16(vo)
    q = synth.prefill_queries(w)
    return w, q, kc, vc


CASES = [
    # workload, T, Tcap, block, K, n_first
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 2048, 2048, 512, 3, 0),
    (synth.C4.scaled(B=1, Hq=4, Hkv=2), 1000, 1024, 64, 4, 1),      # GQA, ragged tail block, first block kept
    (synth.C4.scaled(B=2, Hq=2, Hkv=2, D=64), 777, 800, 128, 2, 0),  # D=64, T not a multiple of anything
    (synth.C4.scaled(B=1, Hq=2, Hkv=1), 512, 512, 16, 8, 0),         # small blocks inside one row tile
    (synth.C4.scaled(B=2, Hq=4, Hkv=2), 1024, 1024, 128, 3, 0),      # 8 (batch, head) units: the XCD-aware tile order
    # the paper's own MoBA settings (App. A.1; Tables 3-4): T = 4096, 64-token blocks with
    # top-16 / 8 / 4, 128-token blocks with top-8 / 4
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 4096, 4096, 64, 16, 0),
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 4096, 4096, 64, 8, 1),
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 4096, 4096, 64, 4, 0),
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 4096, 4096, 128, 8, 0),
    (synth.C4.scaled(B=1, Hq=2, Hkv=2), 4096, 4096, 128, 4, 1),
]


def _random_cases(seed, n):
    """Seeded random small shapes: head counts and grouping, both head dims, block sizes from 16
    to 256, ragged lengths, 1-8 picked blocks, 0-1 always-kept leading blocks."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        Hkv = int(rng.integers(1, 3))
        G = int(rng.choice([1, 2]))
        D = int(rng.choice([64, 128]))
        block = int(rng.choice([16, 32, 64, 128, 256]))
        T = int(rng.integers(block + 1, 1400))
        Tcap = -(-T // 16) * 16 + 16 * int(rng.integers(0, 3))
        n_first = int(rng.integers(0, 2))
        K = int(rng.integers(1 + n_first, 9))
        w = synth.C4.scaled(B=int(rng.integers(1, 3)), Hq=Hkv * G, Hkv=Hkv, D=D)
        out.append((w, T, Tcap, block, K, n_first))
    return out


CASES += _random_cases(20260528, 8)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_moba_select_and_sparse_prefill(rs, knobs, case):
    w, T, Tcap, block, K, n_first = CASES[case]
    say("moba case", case, T, Tcap, block, K, n_first)
    w, q, kc, vc = _setup(w, T, Tcap)
    Nb = -(-T // block)
    scale = 1.0 / np.sqrt(w.D)
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, 16, torch.bfloat16)
    tq, tkc, tvc = to_dev(q, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16")
    means = torch.zeros(w.B, w.Hkv, Nb, w.D, device="cuda")
    idx = torch.full((w.B, w.Hq, T, K), -9, dtype=torch.int32, device="cuda")
    ws = rs.Workspace(max(rs.moba_select_prefill_workspace_bytes(s, T, block),
                          rs.sparse_attn_prefill_workspace_bytes(s, T, block, max(K, Nb))))
    rs.moba_select_prefill(s, tq, tkc, T, block, K, n_first, means, idx, ws)
    omeans = oracle.moba_block_means(kc, T, block)
    np.testing.assert_allclose(to_np(means), omeans, rtol=1e-5, atol=1e-6)
    oidx, osc = oracle.moba_select(q, omeans, T, block, K, n_first, want_scores=True)
    gidx = to_np(idx)
    same = 0
    for b in range(w.B):
        for h in range(w.Hq):
            for t in range(T):
                own = t // block
                take = min(K, own + 1)
                sc = np.where(np.isnan(osc[b, h, t, :own + 1]), 0.0, osc[b, h, t, :own + 1])
                forced = np.zeros(own + 1, bool)
                forced[own] = True
                forced[:n_first] = True
                row = gidx[b, h, t]
                assert np.all(row[take:] == -1), (b, h, t, row)
                ok, why = topk_set_ok(sc, forced, take, row[:take])
                assert ok, (b, h, t, why, row)
                same += np.array_equal(row, oidx[b, h, t])
    say("  rows with identical block lists:", same, "of", w.B * w.Hq * T)
    # the gate's other form (block-mean operands shared through LDS by six-wave workgroups, or
    # fetched by each one-wave workgroup; the library picks by size): the same routing bit for bit
    for form in ("0", "1"):
        knobs.setenv("RATSPARSE_GATE_SHARED", form)
        idx2 = torch.full_like(idx, -9)
        rs.moba_select_prefill(s, tq, tkc, T, block, K, n_first, means, idx2, ws)
        assert torch.equal(idx2, idx), form
    knobs.delenv("RATSPARSE_GATE_SHARED")

    # block-sparse attention over the GPU's own routing
    out = torch.zeros(w.B, w.Hq, T, w.D, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros(w.B, w.Hq, T, device="cuda")
    oout, olse = oracle.sparse_attn_prefill(q, kc, vc, T, block, scale, gidx)
    # both forms of the routed kernel (the library picks by shape; the knob forces either):
    # regrouped by block, and - for up to 64 blocks of a multiple of 64 tokens - causal tiles
    # with a bit set of listed blocks per row
    for form in ("0", "1"):
        knobs.setenv("RATSPARSE_PREFILL_MASKED", form)
        out.zero_(), lse.zero_()
        rs.sparse_attn_prefill(s, tq, tkc, tvc, T, block, scale, idx, K, out, lse, ws)
        ok, worst = attn_close(to_np(out), oout)
        assert ok, (form, worst)
        np.testing.assert_allclose(to_np(lse), olse, rtol=2e-3, atol=2e-3)
        say("  sparse prefill, form", form, "worst relative row error", worst)
    knobs.delenv("RATSPARSE_PREFILL_MASKED")
    rs.sparse_attn_prefill(s, tq, tkc, tvc, T, block, scale, idx, K, out, lse, ws)  # the library's own choice
    assert attn_close(to_np(out), oout)[0]

    # dense causal path, and enough blocks = dense
    outd = torch.zeros_like(out)
    rs.sparse_attn_prefill(s, tq, tkc, tvc, T, block, scale, None, 0, outd, lse, ws)
    od, odl = oracle.sparse_attn_prefill(q, kc, vc, T, block, scale)
    ok, worst = attn_close(to_np(outd), od)
    assert ok, worst
    np.testing.assert_allclose(to_np(lse), odl, rtol=2e-3, atol=2e-3)
    if Nb <= 32:
        idx_all = torch.full((w.B, w.Hq, T, Nb), -9, dtype=torch.int32, device="cuda")
        rs.moba_select_prefill(s, tq, tkc, T, block, Nb, n_first, means, idx_all, ws)
        outf = torch.zeros_like(out)
        rs.sparse_attn_prefill(s, tq, tkc, tvc, T, block, scale, idx_all, Nb, outf, None, ws)
        assert attn_close(to_np(outf), od)[0]
    torch.cuda.synchronize()
    ws.async_status()


# (K, n_first, block): register picks (at most 64 blocks; lists of 4, 8, 16), score columns in LDS
# with top lists (more than 64 blocks), and LDS sweeps (K above 16)
@pytest.mark.parametrize("K,n_first,block", [(3, 0, 64), (4, 1, 64), (8, 0, 64), (16, 2, 64), (3, 0, 16), (8, 1, 16),
                                             (13, 0, 16), (20, 0, 64), (24, 1, 16)])
def test_moba_exact_ties_pick_lowest_blocks(rs, K, n_first, block):
    """A cache that repeats with the block length has identical block means, so every gate
    score of a query ties exactly: the routing must keep the query's own block, the first
    n_first blocks, and fill up with the lowest block indices (the oracle's tie rule)."""
    say("moba ties", K, n_first)
    w = synth.C4.scaled(B=1, Hq=2, Hkv=2, T=1024)
    T = 1024 if block == 64 else 1600  # 16 blocks, or 100 blocks of 16 tokens
    w = w.scaled(T=T)
    Nb = T // block
    rng = np.random.default_rng(7)
    one = oracle.round_to_bf16(rng.standard_normal((w.B, w.Hkv, block, w.D)).astype(np.float32))
    kc = np.tile(one, (1, 1, Nb, 1))
    q = oracle.round_to_bf16(rng.standard_normal((w.B, w.Hq, T, w.D)).astype(np.float32))
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, T, 16, torch.bfloat16)
    means = torch.zeros(w.B, w.Hkv, Nb, w.D, device="cuda")
    idx = torch.full((w.B, w.Hq, T, K), -9, dtype=torch.int32, device="cuda")
    ws = rs.Workspace(rs.moba_select_prefill_workspace_bytes(s, T, block))
    rs.moba_select_prefill(s, to_dev(q, "bf16"), to_dev(kc, "bf16"), T, block, K, n_first, means, idx, ws)
    omeans = oracle.moba_block_means(kc, T, block)
    oidx = oracle.moba_select(q, omeans, T, block, K, n_first)
    gidx = to_np(idx)
    for t in (0, 63, 64, 200, 511, 1023, T - 1):
        own = t // block
        # always kept: own block and the first n_first; the rest ties: lowest indices first
        want = sorted(set(list(range(min(K - 1, own))) + [own]))
        want = want + [-1] * (K - len(want))
        assert list(oidx[0, 0, t]) == want, (t, oidx[0, 0, t], want)  # the oracle follows the stated rule
    np.testing.assert_array_equal(gidx, oidx)
    ws.async_status()


@pytest.mark.parametrize("form", ["0", "1"])
def test_lists_are_taken_as_given(rs, knobs, form):
    """The attention follows the lists it is handed, whatever wrote them: rows whose own block is
    not listed do not attend it, rows with an empty list give zeros and a log-sum-exp of -inf,
    entries may come in any order.  Both forms of the routed kernel."""
    knobs.setenv("RATSPARSE_PREFILL_MASKED", form)
    w = synth.C4.scaled(B=1, Hq=4, Hkv=2, T=1536)
    T, block, K = 1536, 128, 4
    w, q, kc, vc = _setup(w, T, T)
    Nb = T // block
    rng = np.random.default_rng(99)
    idx = np.full((w.B, w.Hq, T, K), -1, dtype=np.int32)
    for b in range(w.B):
        for h in range(w.Hq):
            for t in range(T):
                own = t // block
                n = int(rng.integers(0, min(K, own + 1) + 1))  # sometimes nothing at all
                pick = rng.choice(own + 1, size=n, replace=False)  # may or may not hold the own block
                idx[b, h, t, :n] = pick  # unsorted
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, T, 16, torch.bfloat16)
    ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, K))
    out = torch.zeros(w.B, w.Hq, T, w.D, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros(w.B, w.Hq, T, device="cuda")
    scale = 1.0 / np.sqrt(w.D)
    rs.sparse_attn_prefill(s, to_dev(q, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), T, block, scale,
                           torch.from_numpy(idx).cuda(), K, out, lse, ws)
    oout, olse = oracle.sparse_attn_prefill(q, kc, vc, T, block, scale, idx)
    empty = np.all(idx < 0, axis=-1)
    assert empty.any() and (~empty).any()
    got, glse = to_np(out), to_np(lse)
    assert np.all(got[empty] == 0) and np.all(np.isneginf(glse[empty]))
    ok, worst = attn_close(got[~empty], oout[~empty])
    assert ok, worst
    np.testing.assert_allclose(glse[~empty], olse[~empty], rtol=2e-3, atol=2e-3)
    ws.async_status()


@pytest.mark.parametrize("sub", ["1", "2"])  # steps of 32 keys, of 64
@pytest.mark.parametrize("D,Hq,Hkv", [(64, 3, 1), (128, 8, 2)])  # units in launch order; eight units, one per XCD
def test_prefill_tile_edges(rs, knobs, D, Hq, Hkv, sub):
    """Lengths around the edges of the tiles of a step, of the ring of three of them and of the 128-row
    tiles, in every form of the kernel; cache rows past T hold NaN and must not be looked at."""
    knobs.setenv("RATSPARSE_PREFILL_SUB", sub)
    block, K, rng = 64, 3, np.random.default_rng(31)
    for T in (1, 31, 32, 33, 64, 96, 97, 128, 129, 190, 225, 257, 330, 500):
        say("prefill tile edges", D, T)
        w, q, kc, vc = _setup(synth.C4.scaled(B=1, Hq=Hq, Hkv=Hkv, D=D, n_needles=1), T, T + 16)
        dk, dv = kc.copy(), vc.copy()
        dk[:, :, T:], dv[:, :, T:] = np.nan, np.nan
        idx = np.full((1, Hq, T, K), -1, dtype=np.int32)
        for h in range(Hq):
            for t in range(T):
                n = min(K, t // block + 1)
                idx[0, h, t, :n] = np.sort(rng.choice(t // block + 1, size=n, replace=False))
        s = rs.make_shape(1, Hq, Hkv, D, T + 16, 16, torch.bfloat16)
        ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, K))
        scale = 1.0 / np.sqrt(D)
        for form in ("dense", "0", "1"):
            knobs.setenv("RATSPARSE_PREFILL_MASKED", "0" if form == "dense" else form)
            lists = None if form == "dense" else idx
            out = torch.full((1, Hq, T, D), 7.0, dtype=torch.bfloat16, device="cuda")
            lse = torch.full((1, Hq, T), 7.0, device="cuda")
            rs.sparse_attn_prefill(s, to_dev(q, "bf16"), to_dev(dk, "bf16"), to_dev(dv, "bf16"), T, block, scale,
                                   None if lists is None else torch.from_numpy(lists).cuda(), K, out, lse, ws)
            oout, olse = oracle.sparse_attn_prefill(q, kc, vc, T, block, scale, lists)
            ok, worst = attn_close(to_np(out), oout)  # one bf16 step of the output is 4e-3 of it; 2e-2 allows five
            assert ok, (T, form, worst)
            np.testing.assert_allclose(to_np(lse), olse, rtol=2e-3, atol=2e-3)
        ws.async_status()


@pytest.mark.parametrize("sub", ["1", "2"])  # steps of 32 keys, of 64
@pytest.mark.parametrize("D", [64, 128])
def test_blocks_that_no_row_of_a_wave_listed_are_not_looked_at(rs, knobs, D, sub):
    """By bit sets a wave of 32 rows skips the blocks that none of its rows listed: such a block may hold NaN and infinities
    (a weight of zero times them would be NaN) and every row still gets the oracle's result over a clean cache."""
    knobs.setenv("RATSPARSE_PREFILL_SUB", sub)
    knobs.setenv("RATSPARSE_PREFILL_MASKED", "1")
    T, block, Hq, Hkv, r = 1000, 64, 4, 2, np.random.default_rng(D)
    w, q, kc, vc = _setup(synth.C4.scaled(B=1, Hq=Hq, Hkv=Hkv, D=D, n_needles=1), T, T + 24)
    bad = (2, 3, 7)  # blocks that no row lists, those that live in them included
    idx = np.full((1, Hq, T, 3), -1, dtype=np.int32)
    for h in range(Hq):
        for t in range(T):
            may = [j for j in range(t // block + 1) if j not in bad]
            pick = np.sort(r.choice(may, size=min(3, len(may)), replace=False))
            idx[0, h, t, :len(pick)] = pick
    dk, dv = kc.copy(), vc.copy()
    for j, x in zip(bad, (np.nan, np.inf, -np.inf)):
        dk[:, :, j * block:(j + 1) * block], dv[:, :, j * block:(j + 1) * block] = x, x
    s = rs.make_shape(1, Hq, Hkv, D, T + 24, 16, torch.bfloat16)
    ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, 3))
    out = torch.full((1, Hq, T, D), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, Hq, T), 7.0, device="cuda")
    rs.sparse_attn_prefill(s, to_dev(q, "bf16"), to_dev(dk, "bf16"), to_dev(dv, "bf16"), T, block, 1.0 / np.sqrt(D),
                           torch.from_numpy(idx).cuda(), 3, out, lse, ws)
    oout, olse = oracle.sparse_attn_prefill(q, kc, vc, T, block, 1.0 / np.sqrt(D), idx)
    ok, worst = attn_close(to_np(out), oout)
    assert ok, worst
    np.testing.assert_allclose(to_np(lse), olse, rtol=2e-3, atol=2e-3)
    ws.async_status()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("order", ["growing", "falling", "mixed"])
@pytest.mark.parametrize("sub", ["1", "2"])
def test_prefill_scores_that_outgrow_the_reference(rs, knobs, D, order, sub):
    """Row maxima that keep growing by far more than the lazily moved softmax reference allows for, that come first, or
    that jump about, with weights down to nothing in between: every form of the kernel against the oracle."""
    knobs.setenv("RATSPARSE_PREFILL_SUB", sub)
    T, block, K, Hq, Hkv, r = 900, 64, 3, 2, 1, np.random.default_rng(D)
    q = r.standard_normal((1, Hq, T, D)).astype(np.float32)
    d = r.standard_normal(D).astype(np.float32)
    q += 2.0 * d
    size = {"growing": np.linspace(0.0, 6.0, T), "falling": np.linspace(6.0, 0.0, T), "mixed": r.uniform(-6.0, 6.0, T)}[order]
    k = (r.standard_normal((1, Hkv, T, D)) + size[:, None] * d).astype(np.float32)
    v = r.standard_normal((1, Hkv, T, D)).astype(np.float32)
    q, k, v = (oracle.round_to_bf16(x) for x in (q, k, v))
    idx = np.full((1, Hq, T, K), -1, dtype=np.int32)
    for h in range(Hq):
        for t in range(T):
            n = min(K, t // block + 1)
            idx[0, h, t, :n] = np.sort(r.choice(t // block + 1, size=n, replace=False))
    s = rs.make_shape(1, Hq, Hkv, D, T, 16, torch.bfloat16)
    ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, K))
    scale = 1.0 / np.sqrt(D)
    for form in ("dense", "0", "1"):
        knobs.setenv("RATSPARSE_PREFILL_MASKED", "0" if form == "dense" else form)
        lists = None if form == "dense" else idx
        out = torch.full((1, Hq, T, D), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((1, Hq, T), 7.0, device="cuda")
        rs.sparse_attn_prefill(s, to_dev(q, "bf16"), to_dev(k, "bf16"), to_dev(v, "bf16"), T, block, scale,
                               None if lists is None else torch.from_numpy(lists).cuda(), K, out, lse, ws)
        oout, olse = oracle.sparse_attn_prefill(q, k, v, T, block, scale, lists)
        ok, worst = attn_close(to_np(out), oout)  # one bf16 step of the output is 4e-3 of it; 2e-2 allows five
        assert ok, (order, form, worst)
        np.testing.assert_allclose(to_np(lse), olse, rtol=2e-3, atol=2e-3)
    ws.async_status()


@pytest.mark.parametrize("heads,T,D", [
    (56, 4001, 64), (50, 4001, 64),  # seven units per XCD in groups of six; in launch order in groups of 48
    (64, 4001, 128),                 # eight of 128 channels in two groups of four
    (40, 8300, 64), (48, 8300, 64)])  # long heads: five in groups of three, six in groups of four
def test_tile_order_over_many_heads(rs, knobs, heads, T, D):
    """Causal tiles go out over groups of heads with a remainder first: every tile once, whatever the
    grouping, so each head gets the bits it gets in a call with few heads (steps of one length in all calls)."""
    knobs.setenv("RATSPARSE_PREFILL_SUB", "1")
    block, K = 64, 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(heads)
    q, k, v = (torch.randn(1, heads, T, D, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    t = torch.arange(T, device="cuda")[:, None] // block
    idx = torch.sort(torch.where(torch.arange(K, device="cuda") <= t, t - torch.arange(K, device="cuda"), -1), dim=1).values
    idx = idx.to(torch.int32).expand(1, heads, T, K).contiguous()

    def run(lo, hi, lists):
        s = rs.make_shape(1, hi - lo, hi - lo, D, T, 16, torch.bfloat16)
        ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, K))
        out = torch.full((1, hi - lo, T, D), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((1, hi - lo, T), 7.0, device="cuda")
        rs.sparse_attn_prefill(s, *(x[:, lo:hi].contiguous() for x in (q, k, v)), T, block, 0.125,
                               None if lists is None else lists[:, lo:hi].contiguous(), K, out, lse, ws)
        return out, lse

    for lists in (None, idx):
        say("tile order", heads, T, D, lists is not None)
        out, lse = run(0, heads, lists)
        for lo in range(0, heads, 5):
            few, few_lse = run(lo, min(lo + 5, heads), lists)
            assert torch.equal(out[:, lo:lo + 5], few) and torch.equal(lse[:, lo:lo + 5], few_lse), lo


@pytest.mark.parametrize("T,units", [(1100, 28), (1100, 29), (1100, 56), (1100, 57), (1100, 85), (1100, 86), (390, 64), (390, 65), (390, 128)])
def test_launches_around_the_lines_between_the_step_widths(rs, knobs, T, units):
    """Which step width a causal launch takes, and how many workgroups share a CU, depends on its tiles in all and per head:
    on either side of each line (one tile a CU, two turns, two workgroups a CU, three) the launch gives the bits of one of
    the two widths forced, and both forced widths agree with each other as far as bfloat16 weights let them."""
    D, block, K = 128, 64, 4
    gen = torch.Generator(device="cuda").manual_seed(T + units)
    q, k, v = (torch.randn(1, units, T, D, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    t = torch.arange(T, device="cuda")[:, None] // block
    idx = torch.sort(torch.where(torch.arange(K, device="cuda") <= t, t - torch.arange(K, device="cuda"), -1), dim=1).values
    idx = idx.to(torch.int32).expand(1, units, T, K).contiguous()
    s = rs.make_shape(1, units, units, D, T, 16, torch.bfloat16)
    ws = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, block, K))
    knobs.setenv("RATSPARSE_PREFILL_MASKED", "1")
    for lists in (None, idx):
        got = {}
        for sub in (None, "1", "2"):
            knobs.delenv("RATSPARSE_PREFILL_SUB") if sub is None else knobs.setenv("RATSPARSE_PREFILL_SUB", sub)
            out = torch.full((1, units, T, D), 7.0, dtype=torch.bfloat16, device="cuda")
            lse = torch.full((1, units, T), 7.0, device="cuda")
            rs.sparse_attn_prefill(s, q, k, v, T, block, D ** -0.5, lists, K, out, lse, ws)
            got[sub] = (out, lse)
        assert any(torch.equal(got[None][0], got[x][0]) and torch.equal(got[None][1], got[x][1]) for x in ("1", "2"))
        ok, worst = attn_close(to_np(got["1"][0]), to_np(got["2"][0]))  # two roundings of the weights: within the 2e-2 of the others
        assert ok, worst
        torch.testing.assert_close(got["1"][1], got["2"][1], rtol=1e-5, atol=1e-5)  # 32-bit sums
    ws.async_status()


@pytest.mark.parametrize("B,Hq,Hkv,D,T,block,K", [
    (1, 3, 1, 128, 1023, 16, 4), (1, 3, 3, 64, 1001, 16, 16), (2, 5, 5, 128, 385, 32, 8), (1, 7, 1, 128, 31, 16, 2),
    (1, 37, 37, 64, 800, 48, 3), (1, 300, 300, 64, 97, 16, 6),
    # more tiles than waves: two to five a wave, the next one's rows sent for under the picks, a last tile of 1, 17 or 12 rows
    (1, 64, 16, 128, 4001, 64, 8), (1, 128, 128, 64, 3217, 64, 16), (1, 257, 257, 64, 1100, 32, 4),
    # (not shared by waves: a list of more than 16 blocks is picked from LDS)
    (1, 2, 1, 128, 12289, 512, 20)])
def test_gate_tiles_of_32_rows(rs, knobs, B, Hq, Hkv, D, T, block, K):
    """Twelve waves of 32 query rows share a unit's block means: tiles that cross several own blocks, a last tile and a last round of
    waves that are part empty, unit counts that do not divide the workgroups, more units than workgroups.  The same lists as with the
    one-wave form, and by the float64 scores no block left out is better than one taken."""
    say("gate tiles", B, Hq, Hkv, D, T, block, K)
    gen = torch.Generator(device="cuda").manual_seed(T)
    s = rs.make_shape(B, Hq, Hkv, D, -(-T // 16) * 16, 16, torch.bfloat16)
    q = torch.randn(B, Hq, T, D, generator=gen, device="cuda").to(torch.bfloat16)
    kc = torch.randn(B, Hkv, s.Tcap, D, generator=gen, device="cuda").to(torch.bfloat16)
    Nb = -(-T // block)
    means = torch.zeros(B, Hkv, Nb, D, device="cuda")
    ws = rs.Workspace(rs.moba_select_prefill_workspace_bytes(s, T, block))
    got = []
    for form in ("0", "1"):
        knobs.setenv("RATSPARSE_GATE_SHARED", form)
        idx = torch.full((B, Hq, T, K), -9, dtype=torch.int32, device="cuda")
        rs.moba_select_prefill(s, q, kc, T, block, K, 0, means, idx, ws)
        torch.cuda.synchronize()
        got.append(to_np(idx))
    np.testing.assert_array_equal(got[1], got[0])
    m = np.repeat(to_np(means).astype(np.float64), Hq // Hkv, axis=1)
    sc = np.matmul(to_np(q.float()).astype(np.float64), m.transpose(0, 1, 3, 2))  # [B, Hq, T, Nb]
    own = np.arange(T) // block
    take = np.minimum(K, own + 1)
    listed = got[1]
    assert np.array_equal((listed >= 0).sum(-1), np.broadcast_to(take, listed.shape[:-1]))
    picked = np.zeros(sc.shape, bool)
    b, h, t, j = np.nonzero(listed >= 0)
    picked[b, h, t, listed[b, h, t, j]] = True
    assert np.array_equal(picked.sum(-1), np.broadcast_to(take, listed.shape[:-1])) and picked[:, :, np.arange(T), own].all()
    ahead = np.arange(Nb) > own[:, None]
    assert not (picked & ahead).any()
    worst_in = np.where(picked & (np.arange(Nb) != own[:, None]), sc, np.inf).min(-1)
    best_out = np.where(picked | ahead, -np.inf, sc).max(-1)
    # (a score is a float32 sum of D products of a bfloat16 and a mean split into bfloat16 terms of 24 bits together)
    bound = (D + 3) * 2.0 ** -23 * np.matmul(np.abs(to_np(q.float()).astype(np.float64)), np.abs(m).transpose(0, 1, 3, 2)).max(-1)
    assert (worst_in >= best_out - 2 * bound).all()
