"""The dense annealer's kernels that take accepts one by one, by the plans
that name them, and the automatic choice beside them."""
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


class Jobs:
    """z x sizes random jobs of an instance, extracted, with the oracle's runs."""

    def __init__(self, n, z, sizes, int8, seed, nsw):
        Q = inputs.dense_qubo(n, 0.4, seed)
        if not int8:
            Q = (Q.astype(np.int32) * 40).astype(np.int16)
        X = inputs.random_solutions(z, n, seed + 1)
        H = oracle.field(Q, X)
        self.sol, off, self.idx = inputs.random_index_sets(z, n, np.tile(np.asarray(sizes, np.int32), (z, 1)), seed + 2)
        P = self.P = qb().Problem(torch.as_tensor(Q, device=DEV))
        assert P.int8_ok == int8
        b = self.b = qb().Batch(n, z, self.sol, np.tile(sizes, z))
        b.set_idx(self.idx)
        self.tiles = torch.zeros(b.tile_elems, dtype=qb().tile_dtype(P), device=DEV)
        self.F0 = torch.zeros(b.total, dtype=torch.int32, device=DEV)
        self.y0 = torch.zeros(b.total, dtype=torch.uint8, device=DEV)
        qb().extract(P, b, torch.as_tensor(X, device=DEV), torch.as_tensor(H, device=DEV), self.tiles, self.F0, self.y0)
        self.thr = oracle.thresholds(Q, nsw)
        self.thr_d = torch.as_tensor(self.thr, device=DEV)
        self.Q, self.X, self.H = Q, X, H

    def oracle(self, q, R, seed, inst):
        S = self.idx[self.b.off[q]:self.b.off[q + 1]]
        p = self.sol[q]
        T, _, F, y = oracle.extract(self.Q, self.X[p], self.H[p], S)
        return oracle.anneal(T, F, y, self.thr, R, seed, inst + q, B, count=True)

    def run(self, R, seed, inst):
        b = self.b
        Y = torch.full((b.total * R,), 7, dtype=torch.uint8, device=DEV)
        e = torch.full((b.J * R,), 123, dtype=torch.int64, device=DEV)
        n = torch.full((b.J * R,), -1, dtype=torch.int32, device=DEV)
        b.count_accepts(n)
        qb().anneal(b, self.tiles, self.F0, self.y0, self.thr_d, R, seed, inst, Y, e, B)
        b.count_accepts(None)
        Y, off = Y.cpu().numpy(), self.b.off
        return ([Y[off[q] * R:off[q + 1] * R].reshape(R, -1) for q in range(b.J)], e.cpu().numpy().reshape(-1, R),
                n.cpu().numpy().reshape(-1, R))


def test_a_wait_limit_leaves_the_automatic_choice_alone():
    """With a limit other than 0 the automatic choice stays with the kernel
    that has no such waits: no replica gives up."""
    J = Jobs(1500, 2, [512, 256, 100], True, 61, 8)
    want = J.run(1, 3, 0)
    qb().set_anneal_wait_limit(1)
    try:
        got = J.run(1, 3, 0)
    finally:
        qb().set_anneal_wait_limit(qb().DEFAULT_ANNEAL_WAIT_LIMIT)
    assert (got[1] == want[1]).all() and (got[2] == want[2]).all()
    for g, w in zip(got[0], want[0]):
        assert (g == w).all()


def test_autotuner_tries_a_kernel_once():
    """No plan names a kernel by two numbers, and the loads in flight stay as
    they are where no chosen kernel reads them."""
    J = Jobs(1500, 2, [512, 256, 128, 64], True, 71, 5)
    for seed in range(6):
        J.b.set_plan(sleep_after=16, depth=8, kernel=[0] * 5, persistent=0, wgs_per_cu=1, lpt=1)
        plan, _ = qb().autotune_anneal(J.b, J.tiles, J.F0, J.y0, J.thr_d, 1, seed, 0, B, reps=1)
        assert all(k in (0, 1, 2, 3) for k in plan["kernel"]) and plan["depth"] == 8, plan
