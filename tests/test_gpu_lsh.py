"""GPU parity of stage 1 through the random-hyperplane LSH index (Section 3, Eq. (1)) through the C ABI,
against the CPU oracle's signatures and LSH lookup on the same seeded inputs.

A signature bit is a float decision (the sign of a projection): the GPU sums in float32, the oracle in
double, so a bit whose projection lies within EPS of zero may legitimately differ.  Signatures are compared
bit for bit outside that band; a query's result is compared exactly unless such a near-zero bit could move
an entry across the Hamming radius and that entry could be the top-1 (then it is exempt and counted)."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle
import synth
from tests.compare import MARGIN, SCORE_TOL, compare
from tests.gpu_util import gpu_cache, gpu_lookup, oracle_store, sample_rows, to_dev

pytestmark = pytest.mark.gpu

EPS = 1e-3  # bound on |float32 - double| of a projection (d <= 1024, |r| entries ~ N(0, 1))


@pytest.fixture(scope="module")
def lc():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_01718_amd as m
    return m


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _popcount_rows(x):
    return np.unpackbits(x.view(np.uint8), axis=-1).sum(axis=-1)


def _hamming(sq, sk):
    return np.stack([_popcount_rows(np.bitwise_xor(sk, s[None, :])) for s in sq])


def _lsh_run(lc, sp, w, bits, radius, max_cand=512, rows=None, insert_chunk=None, enable_first=False):
    hp = synth.hyperplanes(bits, sp.d, seed=sp.seed + bits)
    N = w.keys.shape[0]
    if enable_first:
        c = lc.LaCache(max(1, N), sp.d, sp.k_cap, sp.in_dtype, 4096, 0)
        c.enable_lsh(bits, to_dev(hp), max_cand)
        step = insert_chunk or max(1, N)
        for r0 in range(0, N, step):
            c.insert(to_dev(w.keys[r0:r0 + step]), to_dev(w.emb[r0:r0 + step]), to_dev(w.tokens[r0:r0 + step]))
    else:
        c = gpu_cache(lc, sp, w.keys, w.emb, w.tokens, insert_chunk=insert_chunk)
        c.enable_lsh(bits, to_dev(hp), max_cand)
    B = w.queries.shape[0]
    out = c.lookup_lsh(to_dev(w.queries), to_dev(w.la_emb), to_dev(np.ascontiguousarray(w.la_tok[:, :sp.k])),
                       sp.tau_q, sp.tau_r, sp.k, radius)
    g = [t.cpu().numpy() for t in out]
    gsig = c.export_signatures(0, N).cpu().numpy().view(np.uint32) if N else np.zeros((0, bits // 32), np.uint32)
    c.close()
    kq, eq, tok = oracle_store(sp, w.keys, w.emb, w.tokens)
    qq = oracle.quantise(w.queries, sp.in_dtype)
    aq = oracle.quantise(w.la_emb, sp.in_dtype)
    u = np.ascontiguousarray(w.la_tok[:, :sp.k])
    sk, pk = oracle.simhash(kq, hp, bits) if N else (np.zeros((0, bits // 32), np.uint32), np.zeros((0, bits)))
    sq, pq = oracle.simhash(qq, hp, bits)
    o = oracle.lookup_lsh(kq, eq, tok, sk, qq, sq, aq, u, radius, sp.tau_q, sp.tau_r, sp.k)
    return dict(idx=g[0], score=g[1], resp_score=g[2], decision=g[3], n_cand=g[4]), o, gsig, sk, pk, sq, pq, kq, qq


def _check_signatures(gsig, sk, pk):
    """Bits equal wherever the oracle's projection is farther than EPS from zero."""
    if gsig.size == 0:
        return 0
    diff = np.unpackbits((gsig ^ sk).view(np.uint8), axis=-1, bitorder="little").astype(bool)
    near = np.abs(pk) < EPS
    assert not np.any(diff & ~near), f"{int(np.sum(diff & ~near))} signature bits differ away from zero"
    return int(diff.sum())


def _check_lookup(g, o, sk, pk, sq, pq, kq, qq, radius, sp):
    """Exact agreement per query unless a near-zero bit could change the candidate set in a way that matters."""
    B = qq.shape[0]
    if kq.shape[0] == 0:
        assert np.all(g["idx"] == -1) and np.all(g["decision"] == oracle.MISS) and np.all(g["n_cand"] == 0)
        return 0
    H = _hamming(sq, sk)
    nz_k = (np.abs(pk) < EPS).sum(axis=1)
    nz_q = (np.abs(pq) < EPS).sum(axis=1)
    S = (synth.bf16_bits_to_f64(qq) @ synth.bf16_bits_to_f64(kq).T)
    exempt = 0
    for b in range(B):
        border = np.abs(H[b] - radius) <= nz_q[b] + nz_k
        border &= ~((H[b] <= radius) & (H[b] + nz_q[b] + nz_k <= radius))
        best = S[b, o["idx"][b]] if o["idx"][b] >= 0 else -np.inf
        if np.any(border & (S[b] >= best - MARGIN)):
            exempt += 1
            continue
        assert g["n_cand"][b] == o["n_cand"][b] or np.any(border), (b, g["n_cand"][b], o["n_cand"][b])
        assert g["idx"][b] == o["idx"][b], (b, g["idx"][b], o["idx"][b])
        if o["idx"][b] < 0:
            assert np.isnan(g["score"][b]) and g["decision"][b] == oracle.MISS
            continue
        assert abs(float(g["score"][b]) - float(o["score"][b])) <= SCORE_TOL
        near_thr = abs(float(g["score"][b]) - sp.tau_q) < MARGIN or (
            not np.isnan(o["resp_score"][b]) and abs(float(o["resp_score"][b]) - sp.tau_r) < MARGIN)
        if not near_thr:
            assert g["decision"][b] == o["decision"][b], (b, g["decision"][b], o["decision"][b])
            assert np.isnan(g["resp_score"][b]) == np.isnan(o["resp_score"][b])
    return exempt


# d = 1280 and 2176: the query preparation's widest register-resident form and its two-pass form
@pytest.mark.parametrize("name,N,bits,radius,d", [("tiny", 3000, 64, 12, None), ("mid", 20000, 256, 64, None),
                                                  ("mid_paper", 10000, 128, 30, None),
                                                  ("serve_small", 30000, 256, 64, None), ("mid", 4000, 128, 30, 1280),
                                                  ("mid", 3000, 128, 30, 2176)])
def test_lsh_parity(lc, name, N, bits, radius, d):
    extra = {} if d is None else {"d": d}
    sp = synth.spec(name, N=N, B=300, **extra) if name != "serve_small" else synth.spec(name, N=N, B=500)
    w = synth.generate(sp)
    say(f"[case] lsh {name} N={N} d={sp.d} bits={bits} radius={radius}")
    g, o, gsig, sk, pk, sq, pq, kq, qq = _lsh_run(lc, sp, w, bits, radius, insert_chunk=7777)
    flips = _check_signatures(gsig, sk, pk)
    ex = _check_lookup(g, o, sk, pk, sq, pq, kq, qq, radius, sp)
    say(f"[ok] lsh {name}: bit flips near zero {flips}, exempt queries {ex}, mean candidates "
        f"{o['n_cand'].mean():.1f}, hits {int(np.sum(g['decision'] >= 2))}")
    assert ex <= 2


def test_lsh_full_radius_is_the_exact_lookup(lc):
    """radius = bits: every entry is a candidate, so the result is the exact top-1 (judged by the oracle's
    exact lookup with the usual rules)."""
    sp = synth.spec("mid", N=6000, B=200)
    w = synth.generate(sp)
    g, o, *_ = _lsh_run(lc, sp, w, 64, 64, max_cand=sp.N)
    assert np.all(g["n_cand"] == sp.N)
    kq, eq, tok = oracle_store(sp, w.keys, w.emb, w.tokens)
    qq = oracle.quantise(w.queries, sp.in_dtype)
    aq = oracle.quantise(w.la_emb, sp.in_dtype)
    u = np.ascontiguousarray(w.la_tok[:, :sp.k])
    e = oracle.lookup(kq, eq, tok, qq, aq, u, sp.tau_q, sp.tau_r, sp.k)
    compare(g, e, kq, eq, tok, qq, aq, u, sp.tau_q, sp.tau_r, sp.k)


def test_lsh_radius_zero_self_queries_and_inserts_after_enable(lc):
    """Radius 0 is equality of hash keys: a query equal to a stored key always finds it (or the lowest
    identical copy).  Signatures of entries inserted after the index was enabled are maintained."""
    sp = synth.spec("mid", N=5000, B=64)
    w = synth.generate(sp)
    w.queries[:] = w.keys[np.arange(0, 5000, 5000 // 64)[:64]]
    g, o, gsig, sk, pk, sq, pq, kq, qq = _lsh_run(lc, sp, w, 128, 0, enable_first=True, insert_chunk=999)
    _check_signatures(gsig, sk, pk)
    want = np.arange(0, 5000, 5000 // 64)[:64]
    for b in range(64):
        assert g["idx"][b] == oracle.first_identical(kq, int(want[b])), b
        assert g["score"][b] >= 1 - 2 ** -7
    _check_lookup(g, o, sk, pk, sq, pq, kq, qq, 0, sp)


def test_lsh_edges(lc):
    import torch
    sp = synth.spec("tiny", N=10, B=7)
    w = synth.generate(sp)
    hp = to_dev(synth.hyperplanes(64, sp.d, seed=5))
    c = lc.LaCache(100, sp.d, sp.k_cap, sp.in_dtype, 64, 0)
    q, a, t = to_dev(w.queries), to_dev(w.la_emb), to_dev(np.ascontiguousarray(w.la_tok[:, :sp.k]))
    with pytest.raises(lc.LaCacheError):                       # index not enabled
        lc.lacache_lookup_lsh(c, q, a, t, 0.9, 0.85, sp.k, 10)
    c.enable_lsh(64, hp, 8)
    g = [x.cpu().numpy() for x in c.lookup_lsh(q, a, t, 0.9, 0.85, sp.k, 10)]   # empty cache
    assert np.all(g[0] == -1) and np.all(g[3] == 0) and np.all(g[4] == 0) and np.all(np.isnan(g[1]))
    for bad in (-1, 65):
        with pytest.raises(lc.LaCacheError):
            lc.lacache_lookup_lsh(c, q, a, t, 0.9, 0.85, sp.k, bad)
    for bits, mc in ((48, 8), (288, 8), (64, 0)):
        with pytest.raises(lc.LaCacheError):
            lc.lacache_enable_lsh(c, bits, to_dev(synth.hyperplanes(max(bits, 32), sp.d, seed=1)), mc)
    c.close()
    # candidate overflow is reported through n_cand
    sp = synth.spec("tiny", N=2000, B=20)
    w = synth.generate(sp)
    c = gpu_cache(lc, sp, w.keys, w.emb, w.tokens)
    c.enable_lsh(64, hp, 4)
    g = [x.cpu().numpy() for x in c.lookup_lsh(to_dev(w.queries), to_dev(w.la_emb),
                                                to_dev(np.ascontiguousarray(w.la_tok[:, :sp.k])), 0.9, 0.85,
                                                sp.k, 64)]
    assert np.all(g[4] == 2000) and np.all(g[0] >= 0)
    c.close()
    # ensemble caches have no LSH lookup
    c = lc.LaCache(10, sp.d, sp.k_cap, sp.in_dtype, 16, 0, d_resp=(sp.d, 32))
    c.enable_lsh(64, hp, 4)
    with pytest.raises(lc.LaCacheError):
        lc.lacache_lookup_lsh(c, q, a, t, 0.9, 0.85, sp.k, 10)
    c.close()


@pytest.mark.parametrize("bits", list(range(32, 257, 32)))
def test_signatures_at_tile_edges(lc, bits):
    """Every signature width, on inserts whose rows start and end inside and at the edges of the signature
    kernels' tiles (16-row groups, 256-row tiles, a single wave's rows), at both sides of the row count where the bulk
    kernel takes over, at aligned and unaligned first rows; and on the whole store, when the index is replaced by one
    of the opposite hyperplanes (in the same buffers, whose old signatures differ from it in every bit but those of
    zero projections) and by the first again.  Away from EPS the bits equal the float64 signs; a query equal to a
    stored row gets that row's signature (radius 0 finds it)."""
    import torch
    most = max(14000, 2500000 // bits)                # rows that a wave per group and byte takes
    for d, parts in ((100, (37, most + 512, 1, 4097)), (700, (most, 16, 5000)), (200, (most + 1, 255, 6000)),
                     (60, (3 * 512 + most,))):
        N = sum(parts)
        g = torch.Generator().manual_seed(bits * 1000 + d)
        keys = torch.randn((N, d), generator=g).to(torch.bfloat16).cuda()
        keys[N // 2] = 0
        tok = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
        hp = torch.randn((bits, d), generator=g).to(torch.bfloat16).cuda()
        c = lc.LaCache(N, d, 1, lc.BF16, 64, 0)
        c.enable_lsh(bits, hp, 8)
        r0 = 0
        for n in parts:
            c.insert(keys[r0:r0 + n], keys[r0:r0 + n], tok[r0:r0 + n])
            r0 += n
        ones = c.export_signatures(0, N)
        c.enable_lsh(bits, -hp, 8)
        opposite = c.export_signatures(0, N)
        c.enable_lsh(bits, hp, 8)
        assert torch.equal(ones, c.export_signatures(0, N))
        proj = c.export(0, N)[0].view(torch.bfloat16).double() @ hp.double().T
        for sig, p in ((ones, proj), (opposite, -proj)):
            got = ((sig[..., None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).flatten(1).bool()
            bad = (got != (p >= 0)) & (p.abs() >= EPS)
            assert not bad.any(), (d, bad.nonzero()[:10])
            assert got[N // 2].all()                  # a zero vector projects to zero, which counts as >= 0
        rows = torch.randint(N, (64,), generator=g).cuda()
        out = c.lookup_lsh(keys[rows], keys[rows], tok[rows], 0.9, 0.85, 1, 0)
        live = (rows != N // 2).cpu()
        assert torch.equal(out[0].cpu()[live].long(), rows.cpu()[live])
        c.close()


@pytest.mark.parametrize("bits", list(range(32, 257, 32)))
def test_candidate_scan_at_block_edges(lc, bits):
    """The candidates of every signature width, at store sizes around the scan's 16- and 64-entry blocks and its
    turns, and query counts around its 16-query blocks, its largest chunk and the count below which it runs on
    the vector ALU: counts equal to the Hamming distances of the exported signatures (whole numbers), and the
    winner the best of exactly those candidates."""
    import torch
    d, g = 64, torch.Generator().manual_seed(bits)
    hp = torch.randn((bits, d), generator=g).to(torch.bfloat16).cuda()
    for N, B in ((1, 4), (15, 1), (63, 3), (64, 16), (65, 17), (1025, 100), (5000, 480), (4099, 481), (300001, 30)):
        keys = torch.randn((N, d), generator=g).to(torch.bfloat16).cuda()
        q = torch.randn((B, d), generator=g).to(torch.bfloat16).cuda()
        q[0], q[B // 2], q[B - 1] = keys[0], keys[N // 2], keys[N - 1]
        tok = torch.zeros((max(N, B), 1), dtype=torch.int32, device="cuda")
        c, cq = (lc.LaCache(n, d, 1, lc.BF16, 512, 0) for n in (N, B))
        for x, rows in ((c, keys), (cq, q)):
            x.insert(rows, rows, tok[:rows.shape[0]])
            x.enable_lsh(bits, hp, 4096)
        sig = c.export_signatures(0, N).view(torch.uint8)
        sq = cq.export_signatures(0, B).view(torch.uint8)
        unpack = lambda x: ((x[..., None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1).flatten(1)  # noqa: E731
        kb, qb = unpack(sig).float(), unpack(sq).float()
        dist = (qb.sum(1)[:, None] + kb.sum(1)[None] - 2 * qb @ kb.T).round().int()
        z, zq = (x.export(0, n)[0].view(torch.bfloat16).float() for x, n in ((c, N), (cq, B)))
        scores = zq @ z.T
        for radius in (0, bits // 4, bits // 2 - 3 * (N > 5000)):
            idx, score, _, _, n_cand = c.lookup_lsh(q, q, tok[:B], -1.0, 2.0, 1, radius)
            cand = dist <= radius
            assert torch.equal(n_cand.long(), cand.sum(1)), (N, B, radius)
            kept = (cand.sum(1) > 0) & (cand.sum(1) <= 4096)
            best = torch.where(cand, scores, -2.0).max(1).values.clamp(-1, 1)   # reported scores are clamped
            assert torch.all(idx[~(cand.sum(1) > 0)] == -1)
            assert torch.all((score - best)[kept].abs() <= 1e-5), (N, B, radius)
            assert torch.all(cand[torch.arange(B, device="cuda")[kept], idx[kept].long()])
        c.close()
        cq.close()


@pytest.mark.parametrize("bits,B", [(64, 4), (96, 17), (256, 100), (256, 481)])
def test_wide_radius_lists_every_candidate(lc, bits, B):
    """Radii that make half or all of the entries candidates: the counts are exact, the list holds every one of them
    (the winner is the best candidate by the float32 scores), and a list too short for them keeps candidates only."""
    import torch
    d, N, g = 64, 20011, torch.Generator().manual_seed(bits + B)
    keys = torch.randn((N, d), generator=g).to(torch.bfloat16).cuda()
    q = torch.randn((B, d), generator=g).to(torch.bfloat16).cuda()
    hp = torch.randn((bits, d), generator=g).to(torch.bfloat16).cuda()
    tok = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
    c, cq = (lc.LaCache(n, d, 1, lc.BF16, 512, 0) for n in (N, B))
    for x, rows in ((c, keys), (cq, q)):
        x.insert(rows, rows, tok[:rows.shape[0]])
        x.enable_lsh(bits, hp, 32768)
    unpack = lambda x: ((x.view(torch.uint8)[..., None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1).flatten(1)  # noqa: E731
    kb, qb = unpack(c.export_signatures(0, N)).float(), unpack(cq.export_signatures(0, B)).float()
    dist = (qb.sum(1)[:, None] + kb.sum(1)[None] - 2 * qb @ kb.T).round().int()
    z, zq = (x.export(0, n)[0].view(torch.bfloat16).float() for x, n in ((c, N), (cq, B)))
    scores = zq @ z.T
    at = torch.arange(B, device="cuda")
    for max_cand in (32768, 5):
        c.enable_lsh(bits, hp, max_cand)
        for radius in (bits // 2, bits):
            idx, score, _, _, n_cand = c.lookup_lsh(q, q, tok[:B], -1.0, 2.0, 1, radius)
            cand = dist <= radius
            assert torch.equal(n_cand.long(), cand.sum(1))
            assert torch.all(cand[at, idx.long()])
            if max_cand > N:
                best = torch.where(cand, scores, -2.0).max(1).values.clamp(-1, 1)
                assert torch.all((score - best).abs() <= 1e-5)
    c.close()
    cq.close()


def test_wide_radius_scan_time(lc):
    """Counting many candidates costs little beside finding them: 16 queries with every one of 300,000 entries a
    candidate (one kept).  An addition to the query's count per candidate takes 11 ms, one per 64 entries 0.07 ms."""
    import torch
    N, d, bits, B = 300_000, 64, 64, 16
    keys = torch.randn((N, d), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
    tok = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
    c = lc.LaCache(N, d, 1, lc.BF16, 64, 0)
    c.insert(keys, keys, tok)
    c.enable_lsh(bits, to_dev(synth.hyperplanes(bits, d, seed=9)), 1)
    call = lambda: c.lookup_lsh(keys[:B], keys[:B], tok[:B], 0.9, 0.85, 1, bits)  # noqa: E731
    for _ in range(3):
        assert torch.all(call()[4] == N)
    e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
    e0.record()
    for _ in range(5):
        call()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / 5
    say(f"[ok] {B} queries x {N} candidates: {ms:.3f} ms")
    assert ms < 3.0
    c.close()


def test_lsh_recall_full_size_serve(lc):
    """The serving workload at full size (1M x 768, 4096 queries): 256-bit signatures, radius 64.  Against
    the exact lookup every stage-1 hit is found (same entry, same decision) and the candidate lists stay
    short; the exported signatures of all 1M entries and a stratified sample of 48 queries (every class) are
    checked against the oracle's signatures and LSH lookup."""
    sp = synth.spec("serve_small")
    w = synth.generate(sp)
    bits, radius = 256, 64
    hp = synth.hyperplanes(bits, sp.d, seed=77)
    say("[case] lsh full size 1M x 768, B=4096, bits 256, radius 64")
    c = gpu_cache(lc, sp, w.keys, w.emb, w.tokens, insert_chunk=1 << 18)
    ex = gpu_lookup(c, w.queries, w.la_emb, w.la_tok, sp.tau_q, sp.tau_r, sp.k)
    c.enable_lsh(bits, to_dev(hp), 256)
    out = c.lookup_lsh(to_dev(w.queries), to_dev(w.la_emb), to_dev(np.ascontiguousarray(w.la_tok[:, :sp.k])),
                       sp.tau_q, sp.tau_r, sp.k, radius)
    g = [t.cpu().numpy() for t in out]
    gsig = c.export_signatures(0, sp.N).cpu().numpy().view(np.uint32)
    c.close()
    hit = ex["decision"] >= 1                                 # exact stage-1 hits
    found = (g[0] == ex["idx"]) & (g[3] == ex["decision"])
    recall_hits = float(found[hit].mean())
    miss_ok = float(np.mean(g[3][~hit] == 0))
    say(f"[ok] recall of stage-1 hits {recall_hits:.4f} ({int(hit.sum())} hits), misses kept {miss_ok:.4f}, "
        f"mean candidates {g[4].mean():.2f}, max {g[4].max()}")
    assert recall_hits >= 0.999 and miss_ok == 1.0 and g[4].max() <= 256
    # the oracle's LSH lookup on a stratified sample
    rows = sample_rows(w.cls, w.target, 48)
    kq, eq, tok = oracle_store(sp, w.keys, w.emb, w.tokens)
    qq = oracle.quantise(w.queries[rows], sp.in_dtype)
    aq = oracle.quantise(w.la_emb[rows], sp.in_dtype)
    u = np.ascontiguousarray(w.la_tok[rows, :sp.k])
    sk, pk = oracle.simhash(kq, hp, bits)
    flips = _check_signatures(gsig, sk, pk)
    sq, pq = oracle.simhash(qq, hp, bits)
    o = oracle.lookup_lsh(kq, eq, tok, sk, qq, sq, aq, u, radius, sp.tau_q, sp.tau_r, sp.k)
    gs = dict(idx=g[0][rows], score=g[1][rows], resp_score=g[2][rows], decision=g[3][rows], n_cand=g[4][rows])
    exempt = _check_lookup(gs, o, sk, pk, sq, pq, kq, qq, radius, sp)
    say(f"[ok] lsh full size vs oracle: {len(rows)} sampled queries, exempt {exempt}, signature bit flips near "
        f"zero {flips}, hits {int(np.sum(gs['decision'] >= 2))}")
    assert exempt <= 2
