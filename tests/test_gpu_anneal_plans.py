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


# every plan kernel on every class: those that take accepts one by one (1, 2,
# 3 and, where it reads rows from memory, 4), the replicas on both sides of
# what the multi-wave kernels fit into a workgroup (1; 4 of mp = 256 and 512;
# 8 of mp = 128), and the fall-backs of 3 and 4
@pytest.mark.parametrize("kernel", [1, 2, 3, 4])
@pytest.mark.parametrize("R", [1, 3, 4, 5, 9, 16])
@pytest.mark.parametrize("int8", [True, False])
def test_plan_kernels_match_the_oracle(int8, R, kernel):
    """Y, e and the accept counts of a plan kernel on jobs of every class."""
    print("plan kernels", int8, R, kernel, flush=True)
    J = Jobs(2200, 1, [1024, 500, 256, 100, 64, 37], int8, 81, 5)
    J.b.set_plan(kernel=[kernel] * 5)
    Y, e, n = J.run(R, 19, 6)
    for q in range(J.b.J):
        Yo, eo, no = J.oracle(q, R, 19, 6)
        assert (Y[q] == Yo).all() and (e[q] == eo).all() and (n[q] == no).all(), (q, J.b.sizes[q])


@pytest.mark.parametrize("int8,m,J,R", [(True, 64, 200, 16), (True, 128, 200, 16), (True, 200, 210, 5),
                                        (True, 300, 130, 4), (True, 520, 140, 4), (False, 64, 400, 4),
                                        (False, 128, 400, 4), (False, 250, 110, 5), (False, 300, 90, 3),
                                        (False, 500, 260, 2)])
def test_automatic_choice_past_its_lines(int8, m, J, R):
    """Enough replicas that the automatic choice is not the kernel with a
    workgroup for each: a sample of the jobs against the oracle."""
    print("past the lines", int8, m, J, R, flush=True)
    per = 4
    z = -(-J // per)
    A = Jobs(per * m + 20, z, [m] * per, int8, 91, 3)
    Y, e, n = A.run(R, 23, 4)
    for q in range(0, A.b.J, 7):
        Yo, eo, no = A.oracle(q, R, 23, 4)
        assert (Y[q] == Yo).all() and (e[q] == eo).all() and (n[q] == no).all(), q
