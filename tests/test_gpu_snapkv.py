"""GPU parity of SnapKV compression (window votes, pooling, top-K positions, gather) and of
dense decode over the compressed cache, against the float64 oracle, through the C ABI."""
import hashlib

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
    return w, synth.window_queries(w), kc, vc


CASES = [
    # workload, T, Tcap, K_keep, pool
    (synth.C5.scaled(B=1, Hq=8, Hkv=2), 4096, 4096, 512, 7),        # G*W = 128 rows: one row tile
    (synth.C5.scaled(B=2, Hq=2, Hkv=2, W=20), 3000, 3008, 300, 7),  # ragged rows, ragged key chunks
    (synth.C5.scaled(B=1, Hq=16, Hkv=2, D=64), 2500, 2560, 100, 1),  # 256 rows: two row tiles; no pooling
    (synth.C5.scaled(B=1, Hq=4, Hkv=4, W=8), 1200, 1216, 1192, 3),   # keep everything
    # the paper's own SnapKV settings (App. A.1; Tables 3-4): T = 4096, a 64-token observation
    # window, 1024 / 512 / 256 positions kept
    (synth.C5.scaled(B=1, Hq=4, Hkv=4, W=64), 4096, 4096, 1024, 7),
    (synth.C5.scaled(B=1, Hq=4, Hkv=4, W=64), 4096, 4096, 512, 7),
    (synth.C5.scaled(B=1, Hq=4, Hkv=2, W=64), 4096, 4096, 256, 7),    # two heads per KV head: 128 window rows
]


def _random_cases(seed, n):
    """Seeded random small shapes: grouping 1-4, both head dims, windows of 4-64 rows, ragged
    lengths, kept counts from a handful to everything, odd pooling kernels 1-9."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        Hkv = int(rng.integers(1, 3))
        G = int(rng.choice([1, 2, 4]))
        D = int(rng.choice([64, 128]))
        W = int(rng.integers(4, 65))
        T = int(rng.integers(W + 40, 2200))
        Tcap = -(-T // 16) * 16 + 16 * int(rng.integers(0, 3))
        K_keep = int(rng.integers(1, T - W + 1)) if rng.random() < 0.8 else T - W
        pool = int(rng.choice([1, 3, 5, 7, 9]))
        w = synth.C5.scaled(B=int(rng.integers(1, 3)), Hq=Hkv * G, Hkv=Hkv, D=D, W=W)
        out.append((w, T, Tcap, K_keep, pool))
    return out


CASES += _random_cases(20260528, 8)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_snapkv_compress_then_decode(rs, knobs, case):
    w, T, Tcap, K_keep, pool = CASES[case]
    say("snapkv case", case, T, Tcap, K_keep, pool, "W", w.W)
    w, qw, kc, vc = _setup(w, T, Tcap)
    W, L = w.W, T - w.W
    scale = 1.0 / np.sqrt(w.D)
    Tco = ((K_keep + W + 32 + 15) // 16) * 16
    s = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tcap, 16, torch.bfloat16)
    ws = rs.Workspace(rs.snapkv_compress_workspace_bytes(s, T, W))
    kco = torch.zeros(w.B, w.Hkv, Tco, w.D, dtype=torch.bfloat16, device="cuda")
    vco = torch.zeros_like(kco)
    idx = torch.full((w.B, w.Hkv, K_keep), -5, dtype=torch.int32, device="cuda")
    votes = torch.zeros(w.B, w.Hkv, L, device="cuda")
    rs.snapkv_compress(s, to_dev(qw, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), T, W, K_keep, pool, scale,
                       kco, vco, Tco, idx, votes, ws)
    ovotes = oracle.snapkv_votes(qw, kc, T, scale)
    opooled = oracle.maxpool1d(ovotes, pool)
    np.testing.assert_allclose(to_np(votes), opooled, rtol=2e-4, atol=1e-9)
    gidx = to_np(idx)
    oidx, okc, ovc = oracle.snapkv_select_gather(opooled, kc, vc, T, W, K_keep)
    same = 0
    for b in range(w.B):
        for h in range(w.Hkv):
            ok, why = topk_set_ok(opooled[b, h], np.zeros(L, bool), K_keep, gidx[b, h])
            assert ok, (b, h, why)
            same += np.array_equal(gidx[b, h], oidx[b, h])
            rows = np.concatenate([gidx[b, h], np.arange(L, T)])
            np.testing.assert_array_equal(to_np(kco)[b, h, :K_keep + W], kc[b, h, rows])  # gathered bit for bit
            np.testing.assert_array_equal(to_np(vco)[b, h, :K_keep + W], vc[b, h, rows])
    say("  identical kept sets:", same, "of", w.B * w.Hkv)
    assert torch.all(kco[:, :, K_keep + W:] == 0)
    # the other form of the selection (pooling + top-K in one workgroup per head for short
    # prefixes, or spread over workgroups; the library picks by length): the same bits
    knobs.setenv("RATSPARSE_SNAP_ONE_WG", "0")
    kco2, vco2, idx2, votes2 = torch.zeros_like(kco), torch.zeros_like(vco), torch.full_like(idx, -5), torch.zeros_like(votes)
    rs.snapkv_compress(s, to_dev(qw, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), T, W, K_keep, pool, scale,
                       kco2, vco2, Tco, idx2, votes2, ws)
    knobs.delenv("RATSPARSE_SNAP_ONE_WG")
    assert torch.equal(idx2, idx) and torch.equal(votes2, votes)
    assert torch.equal(kco2, kco) and torch.equal(vco2, vco)

    # the same with the window rows' log-sum-exp handed in (one sweep over the keys instead of two):
    # from the oracle's causal attention of those rows, and from the GPU's own dense prefill
    q_full = np.zeros((w.B, w.Hq, T, w.D), dtype=np.float32)
    q_full[:, :, L:] = qw
    _, olse = oracle.sparse_attn_prefill(q_full, kc, vc, T, 16, scale, None, t_begin=L, t_end=T)
    glse = torch.zeros(w.B, w.Hq, T, device="cuda")
    gout = torch.zeros(w.B, w.Hq, T, w.D, dtype=torch.bfloat16, device="cuda")
    wsp = rs.Workspace(rs.sparse_attn_prefill_workspace_bytes(s, T, 16, 0))
    rs.sparse_attn_prefill(s, to_dev(q_full, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), T, 16, scale, None, 0,
                           gout, glse, wsp)
    for name, lse_win, band in (("oracle", to_dev(olse.astype(np.float32)), 1e-4),
                                ("prefill", glse[:, :, L:].contiguous(), 2e-3)):
        kco3, vco3 = torch.zeros_like(kco), torch.zeros_like(vco)
        idx3, votes3 = torch.full_like(idx, -5), torch.zeros_like(votes)
        rs.snapkv_compress_lse(s, to_dev(qw, "bf16"), to_dev(kc, "bf16"), to_dev(vc, "bf16"), T, W, K_keep, pool, scale,
                               lse_win, kco3, vco3, Tco, idx3, votes3, ws)
        np.testing.assert_allclose(to_np(votes3), opooled, rtol=2e-4 if name == "oracle" else 5e-3, atol=1e-9)
        g3 = to_np(idx3)
        for b in range(w.B):
            for h in range(w.Hkv):
                ok, why = topk_set_ok(opooled[b, h], np.zeros(L, bool), K_keep, g3[b, h], band=band)
                assert ok, (name, b, h, why)
                rows = np.concatenate([g3[b, h], np.arange(L, T)])
                np.testing.assert_array_equal(to_np(kco3)[b, h, :K_keep + W], kc[b, h, rows])
    wsp.async_status()

    # a decode step over the compressed cache: append through rat_scan, then dense attention
    sc = rs.make_shape(w.B, w.Hq, w.Hkv, w.D, Tco, 16, torch.bfloat16)
    kd, vd, gd, qd = synth.decode_step(w, 0)
    sk = torch.zeros(w.B, w.Hkv, w.D, device="cuda")
    sv = torch.zeros_like(sk)
    rs.rat_scan(sc, to_dev(kd, "bf16"), to_dev(vd, "bf16"), to_dev(gd), sk, sv, kco, vco, K_keep + W, 1, None)
    ws2 = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(sc, K_keep + W + 1, 0))
    out = torch.zeros(w.B, w.Hq, w.D, dtype=torch.bfloat16, device="cuda")
    rs.sparse_attn_decode(sc, to_dev(qd, "bf16"), kco, vco, K_keep + W + 1, scale, None, 0, None, 0, 0, out, None,
                          None, ws2)
    hk, hv = to_np(kco), to_np(vco)
    want, _ = oracle.sparse_attn_decode(qd, hk, hv, 16, K_keep + W + 1, scale)
    assert attn_close(to_np(out), want)[0]
    if K_keep == L:  # nothing dropped: same as dense attention over the full cache
        full_k = np.concatenate([kc[:, :, :T], hk[:, :, T:T + 1]], axis=2)
        full_v = np.concatenate([vc[:, :, :T], hv[:, :, T:T + 1]], axis=2)
        want2, _ = oracle.sparse_attn_decode(qd, full_k, full_v, 16, T + 1, scale)
        assert attn_close(to_np(out), want2)[0]
    torch.cuda.synchronize()
    ws.async_status()


def _compress(rs, q, kc, vc, T, W, keep, pool, scale, lse=None):
    """One call on device tensors: (kept positions, pooled votes, kept K rows)."""
    B, Hkv, Tcap, D = kc.shape
    s = rs.make_shape(B, q.shape[1], Hkv, D, Tcap, 16, torch.bfloat16)
    ws = rs.Workspace(rs.snapkv_compress_workspace_bytes(s, T, W))
    k_out, v_out = (torch.zeros(B, Hkv, keep + W, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    idx = torch.full((B, Hkv, keep), -5, dtype=torch.int32, device="cuda")
    votes = torch.full((B, Hkv, T - W), -1.0, device="cuda")
    if lse is None:
        rs.snapkv_compress(s, q, kc, vc, T, W, keep, pool, scale, k_out, v_out, keep + W, idx, votes, ws)
    else:
        rs.snapkv_compress_lse(s, q, kc, vc, T, W, keep, pool, scale, lse, k_out, v_out, keep + W, idx, votes, ws)
    torch.cuda.synchronize()
    ws.async_status()
    return idx, votes, k_out


@pytest.mark.parametrize("L", [1, 100, 259, 4095, 4096, 4097, 8191, 8192, 8193, 12289, 15359, 15360, 15361, 20481])
def test_selection_over_slices(rs, knobs, L):
    """The spread-out selection takes 4096 positions a workgroup.  Lengths around one slice, several and the longest that
    one workgroup takes; pools without a halo, with one and the widest; keys that repeat, so that equal votes lie on
    both sides of every border.  The kept positions are exactly the first K of a stable descending sort of the
    pooled votes, the pooled votes are the raw ones pooled, and both forms of the selection give the same bits."""
    W, D, Hkv = 16, 64, 2
    T = L + W
    gen = torch.Generator(device="cuda").manual_seed(L)
    period = 37  # of the keys: every vote comes L / 37 times
    kc = torch.randn(1, Hkv, period, D, generator=gen, device="cuda").to(torch.bfloat16)
    kc = kc.repeat(1, 1, -(-T // period), 1)[:, :, :T].contiguous()
    vc = torch.randn(1, Hkv, T, D, generator=gen, device="cuda").to(torch.bfloat16)
    if L > 1000:  # a few positions of their own, at the borders too
        at = torch.tensor([p for p in (0, 1, 4094, 4095, 4096, 4097, 8191, 8192, 12288, L - 1, L // 2) if p < L], device="cuda")
        kc[:, :, at] = torch.randn(1, Hkv, len(at), D, generator=gen, device="cuda").to(torch.bfloat16) * 1.5
    q = torch.randn(1, 2 * Hkv, W, D, generator=gen, device="cuda").to(torch.bfloat16)
    raw = None
    for pool in (1, 7, 63):
        for keep in sorted({1, L // 3 + 1, max(1, L - 1), L}):
            knobs.setenv("RATSPARSE_SNAP_ONE_WG", "0")
            idx, votes, k_out = _compress(rs, q, kc, vc, T, W, keep, pool, 0.3)
            raw = votes if pool == 1 and raw is None else raw
            want = torch.nn.functional.max_pool1d(raw, pool, 1, pool // 2) if pool > 1 else raw
            assert torch.equal(votes, want), (pool, keep)
            first = torch.sort(votes, dim=2, descending=True, stable=True).indices[:, :, :keep].sort(2).values
            assert torch.equal(idx.long(), first), (pool, keep)
            rows = torch.cat([first, torch.arange(L, T, device="cuda").expand(1, Hkv, W)], 2)
            assert torch.equal(k_out, kc.gather(2, rows[..., None].expand(-1, -1, -1, D)))
            if L <= 15360:
                knobs.setenv("RATSPARSE_SNAP_ONE_WG", "1")
                idx1, votes1, k1 = _compress(rs, q, kc, vc, T, W, keep, pool, 0.3)
                assert torch.equal(idx1, idx) and torch.equal(votes1, votes) and torch.equal(k1, k_out), (pool, keep)


def test_long_sweeps_at_64_channels(rs):
    """A hundred megabytes of keys of 64 channels: eight heads at once against each head by itself.
    With the log-sum-exp given the votes are the same bits; without, they differ by the order in which the key
    chunks' sums are added (32 bits, 50 partial sums: 1e-5 leaves a factor of three over 50 x 2^-24)."""
    T, W, D, H, keep = 102433, 32, 64, 8, 1000
    gen = torch.Generator(device="cuda").manual_seed(3)
    kc, vc = (torch.randn(1, H, T, D, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(1, 2 * H, W, D, generator=gen, device="cuda").to(torch.bfloat16)
    lse = torch.randn(1, 2 * H, W, generator=gen, device="cuda") + 11.0
    idx, votes, k_out = _compress(rs, q, kc, vc, T, W, keep, 7, 0.125)
    idx_l, votes_l, k_l = _compress(rs, q, kc, vc, T, W, keep, 7, 0.125, lse)
    for h in range(H):
        one = [x[:, h:h + 1].contiguous() for x in (kc, vc)]
        qh, lh = q[:, 2 * h:2 * h + 2].contiguous(), lse[:, 2 * h:2 * h + 2].contiguous()
        i1, v1, k1 = _compress(rs, qh, *one, T, W, keep, 7, 0.125, lh)
        assert torch.equal(i1[0, 0], idx_l[0, h]) and torch.equal(v1[0, 0], votes_l[0, h]) and torch.equal(k1[0, 0], k_l[0, h])
        _, v2, _ = _compress(rs, qh, *one, T, W, keep, 7, 0.125)
        torch.testing.assert_close(v2[0, 0], votes[0, h], rtol=1e-5, atol=0.0)
        first = torch.sort(votes[0, h], descending=True, stable=True).indices[:keep].sort().values
        assert torch.equal(idx[0, h].long(), first)
        rows = torch.cat([first, torch.arange(T - W, T, device="cuda")])
        assert torch.equal(k_out[0, h], kc[0, h, rows])


@pytest.mark.parametrize("Hq,Hkv,D,W", [(2, 2, 128, 20), (2, 2, 64, 64), (4, 2, 128, 33), (4, 1, 64, 40), (8, 2, 128, 64)])
@pytest.mark.parametrize("grow", [0.0, 0.05])
def test_sweeps_at_the_edges_of_tiles(rs, Hq, Hkv, D, W, grow):
    """One, two and four groups of 32 window rows and more than one tile of them; lengths that leave waves without a tile,
    a tile with one key, and several chunks of keys; scores that keep growing along the keys (the softmax reference moves)
    and ones that don't; the last length also with enough heads for streaming loads.  Against 64-bit softmax sums: the
    votes are sums of W * G weights, each within a few units of float32 rounding of exp2 and of a log-sum-exp of
    magnitude below 2^10, 2^10 * 2^-23 = 1.2e-4 at worst; where the scores don't grow it stays below 16, and its two roundings,
    the exponent's and a few of the sums come to 16 * 2^-24 * 4 = 4e-6."""
    scale = 1.0 / np.sqrt(D)
    for T, B in ((W + 1, 1), (W + 31, 2), (W + 97, 1), (W + 128, 1), (2048 + W + 1, 1), (2 * 2048 + 5, 2), (4001, -(-(81 << 20) // (Hkv * 4001 * D * 2)))):
        say("snapkv edges", Hq, Hkv, D, W, grow, T, B)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(T)
        k = torch.randn(B, Hkv, T, D, generator=gen, device="cuda")
        q = torch.randn(B, Hq, W, D, generator=gen, device="cuda")
        k[..., 0] += grow * torch.arange(T, device="cuda")
        q[..., 0] = 1.0
        k, q = k.bfloat16(), q.bfloat16()
        v = torch.randn(B, Hkv, T, D, generator=gen, device="cuda").bfloat16()
        L = T - W
        keep = max(1, L // 3)
        s = rs.make_shape(B, Hq, Hkv, D, T, 16, torch.bfloat16)
        ws = rs.Workspace(rs.snapkv_compress_workspace_bytes(s, T, W))
        ko, vo = (torch.zeros(B, Hkv, keep + W, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        idx = torch.full((B, Hkv, keep), -5, dtype=torch.int32, device="cuda")
        votes = torch.zeros(B, Hkv, L, device="cuda")
        rs.snapkv_compress(s, q, k, v, T, W, keep, 1, scale, ko, vo, keep + W, idx, votes, ws)
        later = torch.arange(T, device="cuda")[None] > L + torch.arange(W, device="cuda")[:, None]
        for b, h in {(0, 0), (B - 1, Hkv - 1), (B // 2, 0)}:
            want = torch.zeros(L, dtype=torch.float64, device="cuda")
            for g in range(Hq // Hkv):
                x = q[b, h * (Hq // Hkv) + g].double() @ k[b, h].double().T * scale
                want += torch.softmax(x.masked_fill_(later, -torch.inf), 1).sum(0)[:L]
            np.testing.assert_allclose(to_np(votes[b, h]), to_np(want), rtol=2e-4 if grow else 4e-6, atol=1e-9)
        best = torch.sort(votes, dim=2, descending=True, stable=True).indices[:, :, :keep].sort(2).values
        assert torch.equal(best.int(), idx)
        rows = torch.cat([best, torch.arange(L, T, device="cuda").expand(B, Hkv, W)], 2)[..., None].expand(-1, -1, -1, D)
        assert torch.equal(ko, k.gather(2, rows)) and torch.equal(vo, v.gather(2, rows))


def _of_integers(shape, seed):
    """bf16 values of about unit variance from integer arithmetic alone: the same bits wherever they are made."""
    n = int(np.prod(shape))
    x = torch.arange(n, dtype=torch.int64, device="cuda") + (seed << 40)
    total = torch.zeros_like(x)
    for _ in range(2):
        x = (x ^ (x >> 29)) * 0x2545F4914F6CDD1D + 0x1234567
        x = (x ^ (x >> 32)) * 0x5851F42D4C957F2D
        for shift in (0, 16, 32, 48):
            total += (x >> shift) & 0xFFFF
    return ((total.float() - 4 * 65535.0) / 65536.0 * 1.2247449).to(torch.bfloat16).view(shape)


VOTE_DIGESTS = {
    (2, 2, 2, 128, 1000, 20): "67db2d1de6e47aa6",
    (1, 4, 1, 128, 2048, 32): "e0580499a646cead",
    (1, 4, 1, 128, 2049, 32): "04ff56d1c8dd338a",
    (2, 16, 2, 64, 1800, 20): "2e991ac47f2ca60b",
    (1, 4, 2, 128, 3001, 40): "2b9369875b0263ed",
    (1, 4, 1, 64, 65, 64): "2f535acbdc114ba3",
    (1, 8, 2, 128, 9001, 64): "94001a61917985a4",
    (3, 6, 3, 64, 20001, 64): "628e2acac47f6885",
    (8, 32, 32, 128, 4096, 64): "7c6a547590751ff4",
    (1, 8, 8, 64, 102433, 32): "c675b59fdfd0aee0",
    (1, 8, 1, 128, 131072, 32): "f0a351f9c41bee8b",
}


@pytest.mark.parametrize("B,Hq,Hkv,D,T,W", list(VOTE_DIGESTS))
def test_votes_keep_their_bits(rs, B, Hq, Hkv, D, T, W):
    """Which of thousands of positions are kept hangs on the last place of the votes: two on either side of the cut
    often tie to seven digits, and one swapped tie moves a hundred entries of the ascending list.  So the votes' bits do
    not change with the way the sweeps are laid out: these are the digests of the votes that 128-key steps by whole workgroups
    gave, for one and several row tiles, waves without rows, a single key, up to 8, up to 64 and more chunks, with and without
    streaming loads."""
    say("snapkv bits", B, Hq, Hkv, D, T, W)
    k, q = _of_integers((B, Hkv, T, D), 109), _of_integers((B, Hq, W, D), 110)
    _, votes, _ = _compress(rs, q, k, k, T, W, 1, 1, D ** -0.5)
    assert hashlib.sha1(votes.cpu().numpy().tobytes()).hexdigest()[:16] == VOTE_DIGESTS[B, Hq, Hkv, D, T, W]


def test_kept_positions_are_those_of_64_bit_votes(rs):
    """256 heads of 4096 tokens to 512 with pooling: plateaus of seven equal votes, and a cut that falls among thousands of
    votes a part in a million apart.  For these inputs the votes in float32 (3.3e-7 off in the mean, a log-sum-exp of about 9
    rounded to float32 being most of it) select what the 64-bit ones select, in every head."""
    B, H, T, W, D, keep, pool = 8, 32, 4096, 64, 128, 512, 7
    k, q = _of_integers((B, H, T, D), 109), _of_integers((B, H, W, D), 110)
    idx, votes, _ = _compress(rs, q, k, k, T, W, keep, pool, D ** -0.5)
    L = T - W
    later = torch.arange(T, device="cuda")[None] > L + torch.arange(W, device="cuda")[:, None]
    for b in range(B):
        x = torch.matmul(q[b].double(), k[b].double().transpose(1, 2).contiguous()) * D ** -0.5
        want = torch.softmax(x.masked_fill_(later, -torch.inf), 2).sum(1)[:, :L]
        want = torch.nn.functional.max_pool1d(want[None], pool, 1, pool // 2)[0]
        # (64 weights a vote, each exp2 and its argument within a few times 2^-24 x 16)
        assert ((votes[b].double() - want).abs() <= 4e-6 * want).all()
        first = torch.sort(want, dim=1, descending=True, stable=True).indices[:, :keep].sort(1).values
        assert torch.equal(idx[b].long(), first), b


@pytest.mark.parametrize("L,K,pool", [(700, 100, 1), (1025, 1, 3), (4032, 512, 7), (9001, 9000, 1), (10241, 700, 5), (15360, 1920, 1)])
def test_kept_positions_over_kinds_of_votes(rs, L, K, pool):
    """The kept positions are those of a stable sort of the votes the library itself reports: votes spread evenly, all alike,
    a few that hold nearly all of the range over a crowd of near-equal ones, two levels, and over forty octaves."""
    say("kinds of votes", L, K, pool)
    D, W = 64, 32
    T = L + W
    rng = np.random.default_rng(L)
    n = rng.standard_normal(L)
    rows = [0.3 * n, np.zeros(L), np.where(rng.random(L) < 3 / L, 12.0, 0.004 * n), np.where(n > 1, 1.0, 0.0), 9 * n]
    H = len(rows)
    kc = torch.zeros(1, H, T, D, device="cuda")
    kc[0, :, :L, 0] = torch.from_numpy(np.stack(rows)).float().cuda()
    kc = kc.to(torch.bfloat16)
    q = torch.zeros(1, H, W, D, device="cuda")
    q[..., 0] = 1 + 0.01 * torch.arange(W, device="cuda")
    s = rs.make_shape(1, H, H, D, T, 16, torch.bfloat16)
    ws = rs.Workspace(rs.snapkv_compress_workspace_bytes(s, T, W))
    ko, vo = (torch.zeros(1, H, K + W, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    idx = torch.full((1, H, K), -5, dtype=torch.int32, device="cuda")
    votes = torch.zeros(1, H, L, device="cuda")
    rs.snapkv_compress(s, q.to(torch.bfloat16), kc, kc, T, W, K, pool, 1.0, ko, vo, K + W, idx, votes, ws)
    torch.cuda.synchronize()
    for h in range(H):
        want = np.sort(np.argsort(-to_np(votes)[0, h], kind="stable")[:K])
        assert np.array_equal(to_np(idx)[0, h], want), h
        assert torch.equal(ko[0, h, :K], kc[0, h, torch.from_numpy(want).cuda()])


@pytest.mark.parametrize("H,L,K,pool", [(257, 700, 90, 7), (260, 3071, 400, 5), (257, 3072, 3072, 63), (257, 3073, 1, 3), (300, 4064, 500, 7),
                                        (257, 10240, 700, 1), (257, 10241, 1000, 7), (256, 3000, 400, 7)])
def test_more_heads_than_compute_units(rs, knobs, H, L, K, pool):
    """Up to 256 heads and above, on both sides of the lengths where the pooling and the selection change their form: the votes and
    the positions of the launches that spread a head over the chip, and the positions of a stable sort."""
    say("more heads", H, L, K, pool)
    D, W = 64, 32
    T = L + W
    gen = torch.Generator(device="cuda").manual_seed(L + H)
    kc = torch.zeros(1, H, T, D, device="cuda", dtype=torch.bfloat16)
    x = torch.randn(H, L, generator=gen, device="cuda")
    x[1::5] = 0  # all alike
    x[2::5] = torch.where(x[2::5] > 2.5, 12.0, 0.004 * x[2::5])  # a few hold nearly all of the range
    x[3::5] = (x[3::5] > 1).float()
    x[4::5] *= 9
    kc[0, :, :L, 0] = x
    q = torch.zeros(1, H, W, D, device="cuda")
    q[..., 0] = 1 + 0.01 * torch.arange(W, device="cuda")
    s = rs.make_shape(1, H, H, D, T, 16, torch.bfloat16)
    ws = rs.Workspace(rs.snapkv_compress_workspace_bytes(s, T, W))
    got = []
    for form in ("1", "0"):
        knobs.setenv("RATSPARSE_SNAP_ONE_WG", form)
        ko, vo = (torch.zeros(1, H, K + W, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        idx = torch.full((1, H, K), -5, dtype=torch.int32, device="cuda")
        votes = torch.zeros(1, H, L, device="cuda")
        rs.snapkv_compress(s, q.to(torch.bfloat16), kc, kc, T, W, K, pool, 1.0, ko, vo, K + W, idx, votes, ws)
        torch.cuda.synchronize()
        got.append((idx, votes))
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][0], got[1][0])
    want = torch.sort(got[0][1][0], dim=1, descending=True, stable=True).indices[:, :K].sort(1).values
    assert torch.equal(got[0][0][0].long(), want)
