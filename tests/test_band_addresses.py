"""Every address that the band kernels form, over the parts of their matrices, on the host.

The solves and the trailing updates issue their loads unconditionally, from addresses that may
lie outside the band or past the last row of a part, and mask the values afterwards.  Restated
here from paper_1707_04228_amd/csrc/band.hip, for whole matrices and for both parts of split
ones, in sets of several: the storage that the fill kernels write, the forward and backward
sweeps of the one-right-hand-side solve in both segments (stream, blocks in flight, link, the
other part's rows) for up to 16 groups, the chunk fetches of the many-right-hand-side solve, and
the loads of k_chain, k_far, the trailing update, k_merge and k_link.  Band addresses have to lie
in the set's allocation, scratch indexes in the part's own segment or, for the other part's
rows, in its separator; 16-byte loads have to be aligned; what a sweep waits for has to be rows
that this sweep of that part writes.
"""
import os
import re

import numpy as np
import pytest

HIP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1707_04228_amd", "csrc", "band.hip")
NB = SB = 64
GP, CT, T2, U2 = 4, 256, 128, 512
SW, RPW, UB, DL, FL, GMAX = 8, 8, 32, 8, 3, 16
MC, MT, AL = 32, 512, 8
BAND_PAD = 1024
MG = 32
lane = np.arange(64)
wave = np.arange(SW)


def test_constants_are_the_kernels():
    src = open(HIP).read()
    for name, value in dict(GP=GP, CT=CT, T2=T2, U2=U2, GMAX=GMAX, FL=FL, MC=MC, MT=MT, MG=MG,
                            BAND_PAD=BAND_PAD, NB=NB, SB=SB, SOLVE_THREADS=512, UB=UB).items():
        m = re.findall(r"constexpr (?:int|int64_t) %s = (\d+);" % name, src)
        assert m == [str(value)], (name, m)
    for line in ("constexpr int SW = SOLVE_THREADS / 64;", "constexpr int RPW = SB / SW;",
                 "constexpr int DL = SB * SB / SOLVE_THREADS;", "constexpr int AL = SB * SB / MT;",
                 "static constexpr int KC = 32, KS = 34;", "static constexpr int KC = 64, KS = 68;",
                 "static constexpr int KW = 16, KS = 18;", "static constexpr int KW = 64, KS = 68;"):
        assert line in src, line


def split_rows(n, B, n_mat):
    if n < 3 * B or n < 6 * SB or n_mat > 4096:
        return 0, 0
    b = (n - max(B, 1)) // SB
    return b // 2 * SB, (b - b // 2) * SB


class Part:
    pass


class Set:
    """band_layout for matrices of order n and half bandwidth B; A entries to a line."""

    def __init__(self, mats, A, split=True, rng=None):
        self.A = A
        self.part, self.of = [], []
        stored = rows = n_inv = 0
        self.max_B = max((B + A - 1) // A * A for _, B in mats)
        for j, (n, B0) in enumerate(mats):
            n1, n2 = split_rows(n, B0, len(mats)) if split else (0, 0)
            of = []
            for h in range(2 if n2 else 1):
                p = Part()
                p.mat, p.kind = j, "W" if n2 == 0 else "UL"[h]
                p.N, p.B0, p.B = n, B0, (B0 + A - 1) // A * A
                p.rows = n - n2 if h == 0 else n - n1
                p.cols = p.rows if h == 0 else n2
                p.sep = p.rows if n2 == 0 else n1 if h == 0 else n2
                p.ld = p.B + 1
                p.phase = ((0, p.sep), (p.sep, p.cols))
                stored = (stored + A - 1) // A * A
                p.off, p.yoff, p.boff = stored, rows, n_inv
                stored += p.rows * p.ld
                p.al = (p.rows + SB - 1) // SB * SB
                rows += p.al
                p.inv = (p.cols + SB - 1) // SB * SB * SB
                n_inv += p.inv
                self.envelope(p, rng)
                of.append(p)
                self.part.append(p)
            self.of.append(of)
        self.total = stored + BAND_PAD + T2 * (self.max_B + 1)

    @staticmethod
    def envelope(p, rng):
        """fcb and lrb of the band itself, or (rng) of some profile inside it."""
        nbk = (p.rows + SB - 1) // SB
        b0 = np.arange(nbk) * SB
        first = np.maximum(b0 - p.B0, 0)
        if rng is not None:
            first = first + (rng.random(nbk) * (b0 - first)).astype(int)
            if p.kind == "U":
                fill = np.maximum(p.sep, b0 - p.B0)
                first = np.where(b0 >= p.sep, np.minimum(first, np.maximum(fill, 0)), first)
        p.fcb = first
        reach = np.zeros(nbk, int)
        for b in range(nbk):                       # (rows of a block reach at least from its
            f = first[b] // SB                     # first column on)
            reach[f] = max(reach[f], min(p.rows, (b + 1) * SB))
        run = np.maximum.accumulate(reach)
        p.lrb = np.maximum(run, np.minimum(p.rows, b0 + SB))

    def band(self, p, idx, what, width=1):
        idx = np.asarray(idx)
        if idx.size == 0:
            return
        assert idx.min() >= 0 and idx.max() + width < 2 ** 31, (what, p.kind, p.N, p.B0)
        assert p.off + idx.max() + width <= self.total, (what, p.kind, p.N, p.B0)
        if width > 1:
            assert ((p.off + idx) % width == 0).all(), (what, p.kind, p.N, p.B0)

    def other(self, p):
        of = self.of[p.mat]
        return of[1] if p is of[0] else of[0]


def inside(idx, lo, hi, what):
    idx = np.asarray(idx)
    assert idx.size == 0 or (idx.min() >= lo and idx.max() < hi), (what, idx.min(), idx.max(), lo, hi)


def ends(lo, hi, k=4):
    """Blocks whose loads reach the extremes (the address expressions are monotone between)."""
    return sorted(set(range(lo, min(hi, lo + k))) | set(range(max(lo, hi - k), hi)))


def solve_one(S, p, G, V):
    """band_solve_1_mat: the blocks of part p in every segment it is swept in (a split matrix's
    separator: as the upper part's, with the span of both parts' groups)."""
    split = p.kind != "W"
    LA = S.A
    US = 512 // (64 * V)
    n, B, rs, ncb = p.rows, p.B, p.ld - 1, (p.cols + SB - 1) // SB
    GS = 2 * G if 2 * G <= GMAX else G
    segs = [(0, G, 0)]
    if p.kind == "U":
        segs.append((p.sep // SB, GS, 1))
        inside(p.sep - SB + lane, 0, p.sep, "wait for the first segment")
    i_w = (RPW * wave)[:, None] + np.arange(RPW)[None, :]          # rows of the waves
    for kfirst, span, seg in segs:
        nblk = (n + SB - 1) // SB if seg or not split or p.kind == "L" else p.sep // SB
        for k in ends(kfirst, nblk):
            i0 = k * SB
            nb = min(SB, n - i0)
            kc = min(k, ncb)
            kdone = min(max(k - span + 1, kfirst), kc)
            rowb = np.minimum(i0 + i_w, n - 1) * rs + B              # rp[r] of every wave
            cstart = np.maximum(np.maximum(i0 + RPW * wave - B, 0), p.fcb[k]) // LA * LA
            done = kdone * SB - cstart
            for w in range(SW):
                if done[w] <= 0:
                    continue
                last = (done[w] - 1) // 512 * 512
                for c0 in {0, int(last)}:
                    cc = c0 + V * lane[:, None] + 64 * V * np.arange(US)[None, :]
                    S.band(p, rowb[w][:, None, None] + cstart[w] + cc[None], "forward", V)
                    y = cstart[w] + np.minimum(cc[..., None] + np.arange(V), done[w] - 1)
                    inside(y, 0, kdone * SB, "forward, complete")
            linked = k < ncb and kdone < k
            for kin in {kc, kc - 1 if linked else kc}:
                kf = kdone
                while True:
                    rest = kin - kf
                    nfl = (rest - 1) % FL + 1 if rest > FL else rest
                    o = np.minimum(kf + np.arange(FL), max(kc - 1, 0)) * SB
                    S.band(p, rowb[..., None, None] + o[:, None] + lane, "forward, in flight")
                    if nfl > 0:
                        y = np.minimum(kf + np.arange(FL), kf + nfl - 1) * SB
                        # (complete blocks of columns: all of them are written)
                        inside(y[:, None] + lane, kfirst * SB, min(k, ncb) * SB, "polled forward")
                    if rest <= FL:
                        break
                    kf += nfl
            inside(min(k, ncb - 1) * SB * SB + np.arange(512) + 512 * (DL - 1), 0, p.inv, "inverse")
            rows = i0 + np.arange(nb)
            inside(rows, 0, p.al, "forward, written")
            if k < ncb:
                inside(p.N - 1 - rows if p.kind == "L" else rows, 0, p.N, "right-hand side")
            else:
                assert p.kind == "L"
            if i0 >= p.sep and k < ncb and p.kind == "U":
                m = S.other(p)
                inside(p.N - 1 - rows, m.cols, m.rows, "the lower part's share")
            if linked:
                inside(i0 - SB + lane, kfirst * SB, ncb * SB, "forward link")
    if split and p.kind == "L":
        m = S.other(p)
        inside(p.N - 1 - np.arange(p.cols, n), m.sep, m.rows, "the separator's solution")
    for kbeg, span, seg in segs:
        kend = ncb if seg or not split or p.kind == "L" else p.sep // SB
        for kb in ends(kbeg, kend):
            i0 = kb * SB
            nb = min(SB, p.cols - i0)
            rend = min(n, i0 + nb + B, int(p.lrb[kb]))
            assert rend > i0
            kdone = min(kb + span, kend)
            done = min(rend, kdone * SB)

            def solution(rows, what):              # z of the part, or the other part's
                rows = np.asarray(rows)
                inside(rows[rows < p.cols], 0, p.cols, what)
                over = rows[rows >= p.cols]
                if over.size:
                    assert p.kind == "L"
                    m = S.other(p)
                    inside(p.N - 1 - over, m.sep, m.rows, what)
            pr, hf = lane % (64 // V), lane // (64 // V)
            for w in range(SW):
                starts = range(done + w, rend, SW * UB)
                for r0 in {*starts[:1], *starts[-1:]}:
                    left = rend - 1 - r0
                    solution(r0 + np.minimum(SW * (lane % UB), left), "backward, complete")
                    rr = np.minimum(SW * (V * np.arange(UB // V)[:, None] + hf), left)
                    S.band(p, B + (r0 + rr) * rs + i0 + V * pr, "backward", V)
            kin = min(kdone - 1, (rend - 1) // SB)
            linked = kb + 1 < kdone and rend > (kb + 1) * SB
            for kn in {kb, kb + 1 if linked else kb}:
                kl = max(kin, kn)
                while True:
                    rest = kl - kn
                    nfl = (rest - 1) % FL + 1 if rest > FL else rest
                    kf = kl - nfl + 1
                    rr = (kf + np.arange(FL))[:, None] * SB + np.arange(SB)
                    S.band(p, B + np.minimum(rr, n - 1)[..., None] * rs + i0 + lane,
                           "backward, in flight")
                    inside(np.minimum(rr, rend - 1), 0, p.al, "polled backward")
                    need = rr[:nfl][rr[:nfl] < rend]
                    inside(need, (kb + 1) * SB, min(kend * SB, p.cols), "waited for backward")
                    if rest <= FL:
                        break
                    kl -= nfl
            inside(kb * SB * SB + np.arange(512) + 512 * (DL - 1), 0, p.inv, "inverse")
            if linked:
                inside(i0 + SB + lane, 0, p.al, "backward link")
                inside([i0 + SB], 0, min(kend * SB, p.cols), "backward link")


def solve_many(S, p, M):
    """k_band_solve_m: chunk fetches with their prefetches (the last chunk repeated), the
    right-hand sides, the inverse blocks, the lower part's share of the separator's rows."""
    n, B, rs, ncb = p.rows, p.B, p.ld - 1, (p.cols + SB - 1) // SB
    w, ln = np.arange(MT) // 64, np.arange(MT) % 64
    YL = SB * M // MT

    def chunk(bwd, i0, kk):
        r0, c = (kk * SB if bwd else i0) + w, (i0 if bwd else kk * SB) + ln
        S.band(p, B + np.minimum(r0[:, None] + 8 * np.arange(AL), n - 1) * rs + c[:, None], "chunk")
        yend = min(SB, n - kk * SB) * M
        assert yend > 0
        idx = np.minimum(np.arange(MT)[:, None] + MT * np.arange(YL), yend - 1)
        rows = kk * SB + idx // M
        if bwd and kk >= ncb:
            m = S.other(p)
            inside(p.N - 1 - rows, m.sep, m.rows, "chunk of the separator's solution")
        elif bwd:
            inside(rows, 0, p.cols, "chunk of the backward solution")
        else:
            inside(rows, 0, min(ncb * SB, n), "chunk of the forward solution")

    for k in ends(0, (n + SB - 1) // SB):
        i0, nb = k * SB, min(SB, n - k * SB)
        kfirst = max(max(i0 - B, 0), int(p.fcb[k])) // SB
        for kk in ends(kfirst, min(k, ncb)):
            chunk(False, i0, kk)
        inside(min(k, ncb - 1) * SB * SB + np.arange(MT) + MT * (AL - 1), 0, p.inv, "inverse")
        rows = i0 + np.minimum(np.arange(SB), nb - 1)
        if k < ncb:
            inside(p.N - 1 - rows if p.kind == "L" else rows, 0, p.N, "right-hand side")
        if i0 >= p.sep and k < ncb and p.kind == "U":
            m = S.other(p)
            inside(p.N - 1 - rows, m.cols, m.rows, "the lower part's share")
    for kb in ends(0, ncb):
        i0, nb = kb * SB, min(SB, n - kb * SB)
        klast = (min(n, i0 + nb + B, int(p.lrb[kb])) - 1) // SB
        for kk in ends(kb + 1, klast + 1):
            chunk(True, i0, kk)


def factor(S, p, KC, KW):
    """k_chain, k_far and the trailing update (wide_tile) of both phases, KC and KW columns to
    a chunk."""
    VW = 2 if S.A == 16 else 4
    n, B, rs = p.rows, p.B, p.ld - 1
    assert (n + T2) * p.ld + 64 < 2 ** 31          # as band_factor_t requires
    for fb, ce in p.phase:
        starts = list(range(fb, ce, GP * NB))
        for k0 in starts[:2] + starts[-2:]:
            # k_chain: rows of earlier blocks of the group, columns in the band
            for t in range(GP):
                if k0 + NB * t >= n:
                    continue
                np_ = min(t, (ce - k0 + NB - 1) // NB)
                for q in range(np_):
                    for m in range(q + 1, np_):
                        r = k0 + NB * m + np.arange(NB)[:, None]
                        c = k0 + NB * q + lane
                        ok = lane >= NB * (m - q) + np.arange(NB)[:, None] - B
                        inside(r, 0, n, "k_chain rows")
                        S.band(p, np.where(ok, r * rs + B + c, B), "k_chain")
                        assert (r - c)[ok].max(initial=0) <= B and c.max() < ce
            # k_far
            RP, i0 = CT // (KC // VW), np.arange(CT) // (KC // VW)
            kt = np.arange(CT) % (KC // VW) * VW
            NR = (S.max_B + NB - 1) // NB + 1
            for f in ends(0, NR - 1, 2):
                r0 = k0 + NB * (GP + f)
                if r0 >= n:
                    continue
                for q in range(1, GP):
                    c0 = k0 + NB * q
                    if c0 >= ce or r0 > c0 + NB - 1 + B:
                        continue
                    lo = max(r0 - B, int(p.fcb[r0 // NB]))
                    kstart = k0 + (lo - k0) // KC * KC if lo > k0 else k0
                    kcs = range(kstart, c0, KC)
                    for kc in {*kcs[:1], *kcs[-1:]}:
                        for row in (r0, c0):
                            S.band(p, (row + i0[:, None] + RP * np.arange(NB // RP)) * rs + B + kc +
                                   kt[:, None], "k_far", VW)
            # wide_tile
            kj = min(GP * NB, ce - k0)
            t0 = k0 + kj
            W = min(B, n - t0)
            if W <= 0:
                continue
            nt = (W + T2 - 1) // T2
            RP, i0 = U2 // (KW // VW), np.arange(U2) // (KW // VW)
            kt = np.arange(U2) % (KW // VW) * VW
            for tr in ends(0, nt, 2):
                for ts in ends(0, tr + 1, 2):
                    r0, s0 = t0 + tr * T2, t0 + ts * T2
                    inside([r0 // NB], 0, (n + NB - 1) // NB, "wide_tile envelope")
                    lo = max(r0 - B, int(p.fcb[r0 // NB])) - k0
                    kcs = range(lo // KW * KW if lo > 0 else 0, kj, KW)
                    for kc in {*kcs[:1], *kcs[-1:]}:
                        for row in (r0, s0):
                            S.band(p, (row + i0[:, None] + RP * np.arange(T2 // RP)) * rs + B + k0 +
                                   kc + kt[:, None], "wide_tile", VW)


def separator(S, u, low):
    """k_merge and the fill kernels' band_pos."""
    ns = u.rows - u.sep
    assert ns == low.rows - low.cols and ns >= max(u.B0, 1)
    for s in {0, 1, MG - 1, MG, ns // 2, ns - 1} & set(range(ns)):
        t = np.arange(max(0, s - u.B), s + 1)
        S.band(low, (low.cols + ns - 1 - t) * low.ld + (t - s + low.B), "k_merge, lower")
        inside(low.cols + ns - 1 - t, low.cols, low.rows, "k_merge, lower")
        S.band(u, (u.sep + s) * u.ld + (t - s + u.B), "k_merge, upper")
    for r in {u.rows, u.rows + 1, (u.rows + u.N) // 2, u.N - 1}:
        c = np.arange(max(0, r - u.B0), r + 1)     # entries of the matrix in the lower part
        inside(low.N - 1 - c, 0, low.rows, "band_pos rows")
        inside(c - r + low.B, 0, low.ld, "band_pos columns")


def links(S, p):
    n, B, rs = p.rows, p.B, p.ld - 1
    for b in ends(0, (p.cols + SB - 1) // SB):
        i = np.arange(SB)[:, None]
        for r, c, ok in ((b * SB + i, b * SB - SB + lane, b > 0), (b * SB + SB + i, b * SB + lane, True)):
            use = (r < n) & (c < n) & (r - c <= B) & ok
            if use.any():
                S.band(p, (r * rs + B + c)[use], "k_link")
                assert (r >= c)[use].all() and np.broadcast_to(c, use.shape)[use].min() >= 0


SETS = [[(1, 0)], [(2, 1), (63, 5), (64, 63)], [(65, 64), (127, 64), (128, 65)], [(129, 100)],
        [(383, 20), (384, 128), (384, 129)], [(385, 1), (448, 0)], [(639, 192), (705, 235)],
        [(1000, 63), (1000, 333), (1000, 999)], [(2049, 640), (1600, 63), (3000, 90)],
        [(4097, 700)], [(90783, 1899)], [(116493, 2433)]]


@pytest.mark.parametrize("A,V", [(16, 2), (32, 4)], ids=["fp64", "fp32"])
@pytest.mark.parametrize("mats", SETS, ids=str)
@pytest.mark.parametrize("profile", [False, True])
def test_addresses(mats, A, V, profile):
    for split in (True, False):
        S = Set(mats, A, split, np.random.default_rng(7) if profile else None)
        for p in S.part:
            for G in (1, 2, 3, 8, 9, 16):
                solve_one(S, p, G, V)
            for M in (8, 32):
                solve_many(S, p, M)
            factor(S, p, *((32, 16) if A == 16 else (64, 64)))
            links(S, p)
        for of in S.of:
            if len(of) == 2:
                separator(S, *of)


@pytest.mark.parametrize("G", [1, 2, 3, 5, 8, 9, 16])
def test_what_counts_as_complete_is(G):
    """With P <= G groups present, the blocks that a group takes without a poll lie before its
    own last block of the segment, which waited for all of them; for its first block none."""
    for P in range(1, G + 1):
        for span, step in ((G, P),) + (((2 * G, 2 * P),) if 2 * G <= GMAX else ()):
            for kfirst, nblk in ((0, 40), (7, 23)):
                taken = []
                for g in range(step):
                    for k in range(kfirst + g, nblk, step):
                        kdone = max(k - span + 1, kfirst)
                        assert kdone <= (k - step + 1 if k - step >= kfirst else kfirst)
                        taken.append(k)
                    for kb in range(nblk - 1 - g, kfirst - 1, -step):
                        kdone = min(kb + span, nblk)
                        assert kdone >= (kb + step if kb + step < nblk else nblk)
                assert sorted(taken) == list(range(kfirst, nblk))


def test_a_planted_mistake_is_found():
    """An allocation without its padding, and a separator short of a bandwidth."""
    S = Set([(1000, 63)], 16)
    S.total -= BAND_PAD + T2 * (S.max_B + 1)
    with pytest.raises(AssertionError):
        for p in S.part:
            solve_one(S, p, 1, 2)
            factor(S, p, 32, 16)
    S = Set([(1000, 200)], 16)
    S.part[1].cols += SB
    with pytest.raises(AssertionError):
        separator(S, *S.of[0])
