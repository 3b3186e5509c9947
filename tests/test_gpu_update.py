"""Field, field update and energy at the edges of their tiles and splits."""
import numpy as np
import pytest

import oracle
from paper_2502_13947_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,z", [(1, 1), (3, 2), (64, 64), (127, 65), (128, 128), (129, 129), (255, 33), (1021, 257),
                                 (1024, 1), (1026, 40), (2049, 4), (4099, 2)])
@pytest.mark.parametrize("variant", [1, 2])
def test_rankk_field_energy_at_the_edges(n, z, variant):
    """Tiles of 64, 128 and 256 solutions, partial columns and rows at every
    alignment, row splits with and without a remainder: whole numbers, exact."""
    from paper_2502_13947_amd import qb
    print("update", n, z, variant, flush=True)
    Q = inputs.dense_qubo(n, 0.7, n)
    P = qb.Problem(torch.as_tensor(Q, device="cuda"))
    rng = np.random.default_rng(n + z)
    X0 = rng.integers(0, 2, (z, n)).astype(np.uint8)
    X1 = rng.integers(0, 2, (z, n)).astype(np.uint8)
    X1[0] = X0[0]                                     # a solution without a change
    dX = (X1.astype(np.int16) - X0).astype(np.int8)
    # rows that start one byte past an aligned address
    raw = torch.zeros(z * n + 1, dtype=torch.int8, device="cuda")
    d = raw[1:].view(z, n)
    d.copy_(torch.as_tensor(dX, device="cuda"))
    H = torch.as_tensor(oracle.field(Q, X0), device="cuda")
    qb.rankk(P, d, H, variant)
    Ho = oracle.field(Q, X1)
    assert (H.cpu().numpy() == Ho).all()
    F = torch.full((z, n), 7, dtype=torch.int32, device="cuda")
    Xd = torch.as_tensor(X1, device="cuda")
    qb.field(P, Xd, F)
    assert (F.cpu().numpy() == Ho).all()
    E = torch.zeros(z, dtype=torch.int64, device="cuda")
    qb.energy(Xd, F, E)
    assert (E.cpu().numpy() == oracle.energy(X1, Ho)).all()


@pytest.mark.parametrize("n,z", [(1, 1), (2, 9), (63, 8), (65, 17), (255, 33), (257, 1), (1023, 3), (1025, 130),
                                 (2047, 5)])
def test_field_of_16_bit_problems(n, z):
    """The least and the largest coefficients, odd numbers of rows, one range
    of rows and several, parts of a group of eight solutions: exact."""
    from paper_2502_13947_amd import qb
    print("field16", n, z, flush=True)
    rng = np.random.default_rng(7 * n + z)
    Q = np.triu(rng.choice(np.array([-32768, -32767, -1, 0, 5, 32767], dtype=np.int16), (n, n)))
    Q = Q + np.triu(Q, 1).T
    P = qb.Problem(torch.as_tensor(Q, device="cuda"))
    X = rng.integers(0, 2, (z, n)).astype(np.uint8)
    X[0] = 1
    raw = torch.zeros(z * n + 1, dtype=torch.uint8, device="cuda")
    Xd = raw[1:].view(z, n)
    Xd.copy_(torch.as_tensor(X, device="cuda"))
    H = torch.full((z, n), -3, dtype=torch.int32, device="cuda")
    qb.field(P, Xd, H)
    assert (H.cpu().numpy() == X.astype(np.int64) @ Q.astype(np.int64)).all()
