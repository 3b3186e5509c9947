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
