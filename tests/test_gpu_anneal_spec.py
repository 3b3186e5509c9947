"""The speculating dense annealer against the oracle (bit-exact), at the edges
of its blocks, phases and size classes and at the extremes of acceptance."""
import numpy as np
import pytest

import oracle
from paper_2502_13947_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# both sides of every block count and size class, one position, full tiles
SIZES = [1, 63, 64, 65, 127, 128, 129, 192, 193, 256, 257, 320, 321, 448, 512, 513, 640, 641, 897, 1023, 1024]


@pytest.mark.parametrize("int8", [True, False])
@pytest.mark.parametrize("accept,nsw,R,B", [("cosine", 13, 1, 10), ("all", 9, 2, 1), ("none", 8, 1, 10),
                                            ("cosine", 9, 5, 16), ("half", 8, 1, 1)])
def test_speculated_sweeps_are_the_sequential_ones(accept, nsw, R, B, int8):
    """`all` and `half` accept whole blocks, so that every row of a phase is
    published and the guesses about later blocks are wrong most of the time."""
    from paper_2502_13947_amd import qb
    print("spec", accept, nsw, R, B, int8, flush=True)
    n = 1100
    lim = 127 if int8 else 900
    Q = inputs.dense_qubo(n, 0.8, 501, lo=-lim, hi=lim)
    sizes = SIZES if R == 1 else [s for s in SIZES if s in (1, 65, 193, 321, 512, 641, 1024)]
    z = len(sizes)
    X = inputs.random_solutions(z, n, 502)
    H = oracle.field(Q, X)
    sol, off, idx = inputs.random_index_sets(z, n, np.asarray(sizes, np.int32)[:, None], 503)
    P = qb.Problem(torch.as_tensor(Q, device="cuda"))
    assert P.int8_ok == int8
    b = qb.Batch(n, z, sol, sizes)
    b.set_idx(idx)
    tiles = torch.zeros(b.tile_elems, dtype=qb.tile_dtype(P), device="cuda")
    F0 = torch.zeros(b.total, dtype=torch.int32, device="cuda")
    y0 = torch.zeros(b.total, dtype=torch.uint8, device="cuda")
    qb.extract(P, b, torch.as_tensor(X, device="cuda"), torch.as_tensor(H, device="cuda"), tiles, F0, y0)
    sig = oracle.sigma(Q)
    if accept == "cosine":
        thr = oracle.threshold_table(nsw, B, 0.5 * sig, 0.002 * sig)
    else:
        thr = np.full((nsw, 1 << B), {"all": 2**31 - 1, "none": -(2**31 - 1), "half": 0}[accept], np.int32)
        if accept == "half":
            thr[:, 0] = int(sig)          # a field's typical size in one of the two buckets, descent in the other
    Y = torch.full((b.total * R,), 7, dtype=torch.uint8, device="cuda")
    e = torch.zeros(b.J * R, dtype=torch.int64, device="cuda")
    qb.anneal(b, tiles, F0, y0, torch.as_tensor(thr, device="cuda"), R, 0x77, 40, Y, e, B)
    Yh, eh = Y.cpu().numpy(), e.cpu().numpy()
    for q, m in enumerate(sizes):
        S = idx[b.off[q]:b.off[q + 1]]
        Tq, _, F, yy = oracle.extract(Q, X[q], H[q], S)
        Yo, eo = oracle.anneal(Tq, F, yy, thr, R, 0x77, 40 + q, B)
        assert (Yh[b.off[q] * R:(b.off[q] + m) * R].reshape(R, m) == Yo).all(), m
        assert (eh[q * R:(q + 1) * R] == eo).all(), m


@pytest.mark.parametrize("density,lim,sizes,R,rw,B,accept", [
    # (rows of some 4, 30 and 300 entries: the last wider than 255, on the kernel that chains accepts)
    (0.005, 3, SIZES, 1, 0, 10, "cosine"),
    (0.005, 100, SIZES, 2, 3, 12, "all"),        # replicas that do not fill the last workgroup; one sweep staged
    (0.03, 100, [1, 64, 65, 130, 257, 511, 512], 9, 8, 16, "cosine"),   # thresholds from memory
    (0.03, 3000, [63, 65, 200, 512], 16, 16, 10, "half"),
    (0.03, 100, [512, 449, 64, 1], 1, 1, 10, "all"),
    (0.3, 100, [64, 33, 1], 2, 2, 10, "cosine"),
])
def test_speculated_sparse_sweeps_are_the_sequential_ones(density, lim, sizes, R, rw, B, accept):
    from paper_2502_13947_amd import qb
    print("spec ell", density, lim, R, rw, B, accept, flush=True)
    n, nsw, z = 1100, 9, len(sizes)
    Q = inputs.dense_qubo(n, density, 511, lo=-lim, hi=lim)
    csr = inputs.dense_to_csr(Q)
    X = inputs.random_solutions(z, n, 512)
    H = oracle.field(Q, X)
    sol, off, idx = inputs.random_index_sets(z, n, np.asarray(sizes, np.int32)[:, None], 513)
    P = qb.Problem.from_csr(*csr, device="cuda")
    b = qb.Batch(n, z, sol, sizes)
    b.set_idx(idx)
    tiles = torch.zeros(qb.ell_tile_words(b, P.ell_width), dtype=torch.int32, device="cuda")
    F0 = torch.zeros(b.total, dtype=torch.int32, device="cuda")
    y0 = torch.zeros(b.total, dtype=torch.uint8, device="cuda")
    qb.extract_ell(P, b, torch.as_tensor(X, device="cuda"), torch.as_tensor(H, device="cuda"), tiles, F0, y0)
    sig = max(oracle.sigma(Q), 1.0)
    if accept == "cosine":
        thr = oracle.threshold_table(nsw, B, 0.5 * sig, 0.002 * sig)
    else:
        thr = np.full((nsw, 1 << B), {"all": 2**31 - 1, "half": 0}[accept], np.int32)
        if accept == "half":
            thr[:, ::2] = int(sig)
    Y = torch.full((b.total * R,), 7, dtype=torch.uint8, device="cuda")
    e = torch.zeros(b.J * R, dtype=torch.int64, device="cuda")
    qb.anneal_ell(b, P.ell_width, tiles, F0, y0, torch.as_tensor(thr, device="cuda"), R, 0x79, 50, Y, e, B, rw=rw)
    Yh, eh = Y.cpu().numpy(), e.cpu().numpy()
    for q, m in enumerate(sizes):
        S = idx[b.off[q]:b.off[q + 1]]
        Tq, _, F, yy = oracle.extract(Q, X[q], H[q], S)
        Yo, eo = oracle.anneal(Tq, F, yy, thr, R, 0x79, 50 + q, B)
        assert (Yh[b.off[q] * R:(b.off[q] + m) * R].reshape(R, m) == Yo).all(), m
        assert (eh[q * R:(q + 1) * R] == eo).all(), m
