"""The sparse annealer's two ways through a sweep (all at once and repaired;
one accept after another), and the line between them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_13947_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
B = 10


def qb():
    from paper_2502_13947_amd import qb as m
    return m


def sparse_qubo(n, d, lim, seed):
    """Symmetric, with about d couplings a row."""
    rng = np.random.default_rng(seed)
    Q = np.where(rng.random((n, n)) < d / n, rng.integers(-lim, lim + 1, (n, n)), 0)
    Q = np.triu(Q, 1)
    return (Q + Q.T + np.diag(rng.integers(-lim, lim + 1, n))).astype(np.int16)


def jobs(Q, z, m, alpha, seed):
    """One job of m random variables for each of z solutions, extracted, after
    `alpha` Tabu steps."""
    n = Q.shape[0]
    P = qb().Problem.from_csr(*inputs.dense_to_csr(Q), DEV)
    X = torch.as_tensor(inputs.random_solutions(z, n, seed), device=DEV)
    H = torch.zeros((z, n), dtype=torch.int32, device=DEV)
    E = torch.zeros(z, dtype=torch.int64, device=DEV)
    T, LF = torch.zeros_like(H), torch.zeros_like(H)
    qb().field(P, X, H)
    qb().energy(X, H, E)
    if alpha:
        qb().tabu(P, X, H, E, alpha, max(1, n // 150), True, T, LF)
    sol, _, idx = inputs.random_index_sets(z, n, np.full((z, 1), m, np.int32), seed + 1)
    b = qb().Batch(n, z, sol, np.full(z, m))
    b.set_idx(idx)
    tile = torch.zeros(qb().ell_tile_words(b, P.ell_width), dtype=torch.int32, device=DEV)
    F0 = torch.zeros(b.total, dtype=torch.int32, device=DEV)
    y0 = torch.zeros(b.total, dtype=torch.uint8, device=DEV)
    qb().extract_ell(P, b, X, H, tile, F0, y0)
    return P, b, X, H, idx.reshape(z, m), tile, F0, y0


# every block count's remainders; rows of one to several words a lane, wider
# than 64 and than 255; hot starts (all at once), cold ones (one by one) and
# schedules that pass from one to the other
@pytest.mark.parametrize("n,d,lim,m,R,rw,alpha,tmax", [
    (80, 60, 100, 64, 3, 0, 200, 0.5), (40, 30, 100, 33, 16, 16, 0, 0.1), (130, 20, 1000, 65, 2, 1, 300, 0.05),
    (600, 260, 100, 100, 2, 1, 900, 0.3), (300, 110, 100, 128, 5, 2, 600, 0.2), (300, 6, 100, 250, 4, 0, 600, 0.3),
    (500, 40, 100, 300, 3, 2, 1000, 0.2), (700, 25, 1000, 512, 1, 1, 1500, 0.1), (1200, 12, 100, 1000, 9, 0, 0, 0.3),
    (1100, 20, 100, 1024, 2, 0, 3000, 0.05)])
def test_both_ways_match_the_oracle(n, d, lim, m, R, rw, alpha, tmax):
    print("ell ways", n, d, lim, m, R, rw, alpha, tmax, flush=True)
    Q = sparse_qubo(n, d, lim, n + d)
    z, nsw, seed, inst = 2, 30, 77, 5
    P, b, X, H, idx, tile, F0, y0 = jobs(Q, z, m, alpha if d <= 60 else 0, n)
    thr = oracle.threshold_table(nsw, B, tmax * P.sigma, 0.002 * P.sigma)
    Y = torch.zeros(b.total * R, dtype=torch.uint8, device=DEV)
    e = torch.zeros(z * R, dtype=torch.int64, device=DEV)
    acc = torch.zeros(z * R, dtype=torch.int32, device=DEV)
    b.count_accepts(acc)
    qb().anneal_ell(b, P.ell_width, tile, F0, y0, torch.as_tensor(thr, device=DEV), R, seed, inst, Y, e, B, rw=rw)
    b.count_accepts(None)
    Xh, Hh, Yh = X.cpu().numpy(), H.cpu().numpy(), Y.cpu().numpy()
    for q in range(z):
        T, _, F, y = oracle.extract(Q, Xh[q], Hh[q], idx[q])
        Yo, eo, no = oracle.anneal(T, F, y, thr, R, seed, inst + q, B, count=True)
        assert (Yh[q * m * R:(q + 1) * m * R].reshape(R, m) == Yo).all(), q
        assert (e.cpu().numpy()[q * R:(q + 1) * R] == eo).all(), q
        assert (acc.cpu().numpy()[q * R:(q + 1) * R] == no).all(), q


def cliques(m, d, k, seed):
    """k blocks of m variables, each joined with d random others of its block."""
    Q = np.zeros((k * m, k * m), np.int16)
    rng = np.random.default_rng(seed)
    for c in range(k):
        p = rng.permutation(m)
        for s in range(1, d // 2 + 1):
            v = rng.integers(1, 101, m) * rng.choice([-1, 1], m)
            i, j = c * m + p, c * m + np.roll(p, s)
            Q[i, j] = v
            Q[j, i] = v
    return Q


def sweeps_us(m, d, R, nsw=200, z=32, k=4):
    """Microseconds a sweep of z * k jobs of whole blocks after a Tabu run."""
    n = k * m
    P = qb().Problem.from_csr(*inputs.dense_to_csr(cliques(m, d, k, 7)), DEV)
    X = torch.as_tensor(inputs.random_solutions(z, n, 3), device=DEV)
    H = torch.zeros((z, n), dtype=torch.int32, device=DEV)
    E = torch.zeros(z, dtype=torch.int64, device=DEV)
    T, LF = torch.zeros_like(H), torch.zeros_like(H)
    qb().field(P, X, H)
    qb().energy(X, H, E)
    qb().tabu(P, X, H, E, 2 * n, max(1, n // 150), True, T, LF)
    b = qb().Batch(n, z, np.repeat(np.arange(z), k), np.full(z * k, m))
    b.set_idx(np.tile(np.arange(n, dtype=np.int32), z))
    tile = torch.zeros(qb().ell_tile_words(b, P.ell_width), dtype=torch.int32, device=DEV)
    F0 = torch.zeros(b.total, dtype=torch.int32, device=DEV)
    y0 = torch.zeros(b.total, dtype=torch.uint8, device=DEV)
    qb().extract_ell(P, b, X, H, tile, F0, y0)
    thr = torch.as_tensor(qb().threshold_table(nsw, B, 0.25 * P.sigma, 0.002 * P.sigma), device=DEV)
    Y = torch.zeros(b.total * R, dtype=torch.uint8, device=DEV)
    e = torch.zeros(b.J * R, dtype=torch.int64, device=DEV)
    best = float("inf")
    for _ in range(6):
        u, v = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        u.record()
        qb().anneal_ell(b, P.ell_width, tile, F0, y0, thr, R, 5, 0, Y, e, B)
        v.record()
        torch.cuda.synchronize()
        best = min(best, u.elapsed_time(v))
    return 1e3 * best / nsw


@pytest.mark.parametrize("m,d", [(64, 60), (256, 60), (512, 60)])
def test_dense_rows_cost_no_more_than_a_few_sparse_ones(m, d):
    """A sweep that accepts few positions, with rows of 60 within the job and
    with rows of 4 (2.9 to 5.2 times as long where rows were walked entry by
    entry)."""
    us = {w: sweeps_us(m, w, 1) for w in (4, d)}
    print(f"m {m}: rows of 4 {us[4]:.2f} us, of {d} {us[d]:.2f} us", flush=True)
    assert us[d] <= 2.4 * us[4]


def test_one_replica_takes_no_longer_than_many():
    """(It took twice as long where one wave staged the thresholds.)"""
    us = {R: sweeps_us(64, 4, R) for R in (1, 16)}
    print(f"m 64: R = 1 {us[1]:.2f} us, R = 16 {us[16]:.2f} us", flush=True)
    assert us[1] <= 1.25 * us[16]
