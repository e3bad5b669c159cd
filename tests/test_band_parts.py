"""The two-part elimination of a band matrix and the work-group programs of its solves,
restated on the host.

A matrix of order n >= 3 bw (and six 64-row blocks) is eliminated from both ends towards a
separator.  Checked here: the rule leaves a separator of at least one bandwidth, so the two
parts never couple; eliminating the parts and then the separator gives the same solution as
one sweep from the top; and the one-right-hand-side solve's work-groups (block k of a part to
group k mod G, the separator shared by both parts' groups), each waiting only for what it
polls, all reach the end, with every block they take as complete handed over before.
"""
import numpy as np
import pytest

SB = 64
GMAX = 16


def split_rows(n, B, n_mat):
    if n < 3 * B or n < 6 * SB or n_mat > 4096:
        return 0, 0
    b = (n - max(B, 1)) // SB
    return b // 2 * SB, (b - b // 2) * SB


@pytest.mark.parametrize("n", [1, 383, 384, 385, 448, 511, 640, 705, 1000, 2049, 9001])
def test_parts_do_not_couple(n):
    for B in sorted({0, 1, 15, 63, 64, 127, n // 5, n // 3, n // 3 + 1, n // 2, n - 1}):
        if B >= n:
            continue
        n1, n2 = split_rows(n, B, 3)
        assert split_rows(n, B, 4097) == (0, 0)
        if n2 == 0:
            assert n1 == 0 and (n < 3 * B or n < 6 * SB)
            continue
        assert n1 > 0 and n1 % SB == 0 and n2 % SB == 0
        assert n - n1 - n2 >= max(B, 1)         # the separator holds a bandwidth


@pytest.mark.parametrize("n,B", [(384, 127), (385, 1), (448, 0), (639, 192), (705, 235), (1000, 17)])
def test_two_ends_match_one_sweep(n, B):
    rng = np.random.default_rng(n + B)
    A = np.zeros((n, n))
    for d in range(1, B + 1):
        A += np.diag(rng.uniform(-1, 1, n - d), -d)
    A = A + A.T
    A += np.diag(np.abs(A).sum(1) + 1.0)
    b = rng.standard_normal(n)
    n1, n2 = split_rows(n, B, 1)
    assert n2 > 0
    up, lo, sep = np.arange(n1), np.arange(n - 1, n - 1 - n2, -1), np.arange(n1, n - n2)
    S, rs, part = A[np.ix_(sep, sep)].copy(), b[sep].copy(), []
    for own in (up, lo):                        # L of the part's own columns, its sums
        L = np.linalg.cholesky(A[np.ix_(own, own)])
        W = np.linalg.solve(L, A[np.ix_(own, sep)])
        y = np.linalg.solve(L, b[own])
        S -= W.T @ W
        rs -= W.T @ y
        part.append((own, L, W, y))
    x = np.zeros(n)
    x[sep] = np.linalg.solve(S, rs)
    for own, L, W, y in part:
        x[own] = np.linalg.solve(L.T, y - W @ x[sep])
    ref = np.linalg.solve(A, b)
    # both are backward stable; kappa < 1e3 (diagonally dominant)
    assert np.abs(x - ref).max() <= 1e-11 * np.abs(ref).max()


def parts(n, B0, nm):
    A = 16
    B = (B0 + A - 1) // A * A
    n1, n2 = split_rows(n, B0, nm)
    out = []
    for h in range(2 if n2 else 1):
        rows = n - n2 if h == 0 else n - n1
        cols = rows if h == 0 else n2
        sep = rows if n2 == 0 else (n1 if h == 0 else n2)
        kind = "W" if n2 == 0 else "UL"[h]
        nbk = (rows + 63) // 64
        r = np.arange(rows)
        f = np.minimum(np.maximum(r - B0, 0), r)
        if kind == "U":
            m = r >= sep
            f[m] = np.minimum(f[m], np.maximum(sep, r[m] - B0))
        reach = [0] * nbk
        for rr in range(rows):
            reach[f[rr] // 64] = max(reach[f[rr] // 64], rr + 1)
        run, last = 0, []
        for b in range(nbk):
            run = max(run, reach[b])
            last.append(max(run, min(rows, (b + 1) * 64)))
        out.append(dict(n=rows, cols=cols, sep=sep, N=n, B=B, kind=kind, lrb=last))
    return out


def run_groups(n, B0, nm, G, links):
    """Runs every group of every part as far as its waits allow, in turn; '' when all end."""
    P = parts(n, B0, nm)
    split = len(P) == 2
    Y = [np.zeros((p["n"] + 63) // 64 * 64, bool) for p in P]
    Z = [np.zeros_like(y) for y in Y]

    def forward(h, g):
        low = P[h]["kind"] == "L"
        both = 2 * G <= GMAX
        GS = 2 * G if both else G
        gs = (2 * g + low) if both else (-1 if low else g)
        for seg in range(2 if split else 1):
            h2, kfirst, step, mine = h, 0, G, g
            if seg:
                if gs < 0:
                    return
                s = P[0]["sep"]
                h2, kfirst, step, mine = 0, s // SB, GS, s // SB + gs
                yield Y, 0, np.arange(s - 64, s), False
            p = P[h2]
            n_, cols, sep = p["n"], p["cols"], p["sep"]
            ncb = (cols + 63) // 64
            nblk = (n_ + 63) // 64 if (seg or not split or p["kind"] == "L") else sep // SB
            for k in range(mine, nblk, step):
                i0, nb, kc = k * 64, min(64, n_ - k * 64), min(k, ncb)
                kdone = min(max(k - step + 1, kfirst), kc)
                linked = links and k < ncb and kdone < k
                yield Y, h2, np.arange(0, kdone * 64), True
                yield Y, h2, np.arange(kdone * 64, (kc - 1 if linked else kc) * 64), False
                if k < ncb and i0 >= sep:
                    yield Y, 1, p["N"] - 1 - np.arange(i0, i0 + nb), False
                if linked:
                    yield Y, h2, np.arange(i0 - 64, i0), False
                Y[h2][i0:i0 + nb] = True

    def backward(h, g):
        low = P[h]["kind"] == "L"
        both = 2 * G <= GMAX
        GS = 2 * G if both else G
        gs = (2 * g + low) if both else (-1 if low else g)
        for seg in ([1, 0] if split else [0]):
            if seg and gs < 0:
                continue
            h2 = 0 if seg else h
            p = P[h2]
            lower, n_, cols, sep = p["kind"] == "L", p["n"], p["cols"], p["sep"]

            def rows_of(r):                     # the lower part takes the separator's rows
                own, far = r[r < cols] if lower else r, r[r >= cols] if lower else r[:0]
                return [(Z, h2, own), (Z, 0, p["N"] - 1 - far)]

            if not seg and split:
                for w in rows_of(np.arange(cols if lower else sep, n_)):
                    yield (*w, False)
            kbeg = sep // SB if seg else 0
            kend = (cols + 63) // 64 if (seg or not split or lower) else sep // SB
            step = GS if seg else G
            for kb in range(kend - 1 - (gs if seg else g), kbeg - 1, -step):
                i0, nb = kb * 64, min(64, cols - kb * 64)
                rend = min(min(n_, i0 + nb + p["B"]), p["lrb"][kb])
                kdone = min(kb + step, kend)
                for w in rows_of(np.arange(min(rend, kdone * 64), rend)):
                    yield (*w, True)
                linked = links and kb + 1 < kdone and rend > (kb + 1) * 64
                kn = kb + 1 if linked else kb
                yield Y, h2, np.arange(i0, i0 + nb), False
                kl = max(min(kdone - 1, (rend - 1) // 64), kn)
                yield Z, h2, np.arange((kn + 1) * 64, min((kl + 1) * 64, rend)), False
                if linked:
                    yield Z, h2, np.arange(i0 + 64, min(i0 + 128, n_)), False
                Z[h2][i0:i0 + nb] = True

    def program(h, g):
        yield from forward(h, g)
        yield from backward(h, g)

    progs = [program(h, g) for h in range(len(P)) for g in range(G)]
    at = [next(q, None) for q in progs]
    while any(c is not None for c in at):
        moved = False
        for i, q in enumerate(progs):
            while at[i] is not None:
                V, h, rows, complete = at[i]
                if not V[h][rows].all():
                    if complete:
                        return "not complete: group %d of part %d" % (i % G, i // G)
                    break
                at[i] = next(q, None)
                moved = True
        if not moved:
            return "stuck"
    return "" if all(Z[h][: p["cols"]].all() for h, p in enumerate(P)) else "rows left out"


@pytest.mark.parametrize("n,B", [(383, 20), (384, 128), (384, 129), (385, 1), (448, 0), (639, 192),
                                 (705, 235), (1000, 333), (2049, 640), (1600, 63), (130, 5)])
def test_every_group_ends(n, B):
    for G in (1, 2, 3, 5, 8, 9, 16):
        for links in (False, True):
            assert run_groups(n, B, 14, G, links) == "", (G, links)
