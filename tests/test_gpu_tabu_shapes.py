"""Dense Tabu at the edges of its workgroups, rows and release ring."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(Q, z, alpha, tenure, asp, seed):
    from paper_2502_13947_amd import qb
    n = Q.shape[0]
    rng = np.random.default_rng(seed)
    X = rng.integers(0, 2, (z, n)).astype(np.uint8)
    H = oracle.field(Q, X)
    E = oracle.energy(X, H)
    P = qb.Problem(torch.as_tensor(Q, device="cuda"))
    Xd, Hd, Ed = (torch.as_tensor(a, device="cuda") for a in (X, H, E))
    T = torch.full((z, n), -7, dtype=torch.int32, device="cuda")
    LF = torch.full((z, n), -7, dtype=torch.int32, device="cuda")
    qb.tabu(P, Xd, Hd, Ed, alpha, tenure, asp, T, LF)
    for p in range(z):
        x, h, ov, To, LFo = oracle.tabu(Q, X[p], H[p], int(E[p]), alpha, tenure, asp)
        assert (Xd[p].cpu().numpy() == x).all(), p
        assert (Hd[p].cpu().numpy() == h).all(), p
        assert int(Ed[p].item()) == ov, p
        assert (T[p].cpu().numpy() == To).all() and (LF[p].cpu().numpy() == LFo).all(), p


def _qubo(n, lim, density, seed):
    rng = np.random.default_rng(seed)
    Q = rng.integers(-lim, lim + 1, (n, n))
    Q[rng.random((n, n)) >= density] = 0
    Q = np.triu(Q)
    return (Q + np.triu(Q, 1).T).astype(np.int16)


@pytest.mark.parametrize("lim", [127, 300])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 384, 385, 512, 513, 640, 641, 768, 769, 896, 897, 1024, 1025, 1280, 1281, 1536,
                               1537, 2048, 2049, 2560, 2561, 3072, 3073,
                               3584, 3585, 4097, 5121, 6145, 7169, 8192, 8193, 10241])
def test_tabu_every_workgroup_and_row(n, lim):
    """Both sides of every variables-per-thread count, one, four and eight
    waves, 8-bit and 16-bit rows; whole numbers, exact."""
    print("tabu shape", n, lim, flush=True)
    _run(_qubo(n, lim, 0.5, n), 2, 300, max(1, n // 100) + 3, True, n + 1)


@pytest.mark.parametrize("n", [40, 700, 1600])
@pytest.mark.parametrize("tenure,alpha", [(0, 200), (1, 200), (2, 300), (3, 301), (1022, 2500), (1023, 2500),
                                          (1024, 2500), (1500, 2500)])
def test_tabu_release_ring(n, tenure, alpha):
    """Tenures at the ring's ends and past it; with n below the tenure every
    variable is tabu and the least bad one is flipped early, so tenure left
    over adds up."""
    print("tabu ring", n, tenure, alpha, flush=True)
    _run(_qubo(n, 100, 1.0, n), 2, alpha, tenure, True, n + 2)
    _run(_qubo(n, 100, 0.3, n), 1, alpha, tenure, False, n + 3)


@pytest.mark.parametrize("n,lim", [(600, 32767), (1500, 32767), (2600, 26000), (4000, 20000)])
def test_tabu_widest_moves(n, lim):
    """Move values that leave the narrow workgroups too few key bits."""
    print("tabu wide", n, lim, flush=True)
    _run(_qubo(n, lim, 1.0, n), 2, 300, 9, True, n + 4)
