"""Ranking, selection and scoring at the edges of their kernels' shapes."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 7168, 7169, 10240, 10241,
                               16384, 16385, 20480, 20481, 32768, 32769])
def test_rank_at_the_edges_of_its_shapes(n):
    """Every elements-per-thread count; keys that need no pass, one pass with
    ties, all six, and the extremes of the allowed range."""
    from paper_2502_13947_amd import qb
    print("rank", n, flush=True)
    rng = np.random.default_rng(n)
    top = 2**47 - 1
    K = np.stack([np.full(n, -5, np.int64), rng.integers(-3, 4, n), rng.integers(-top, top + 1, n),
                  rng.choice(np.array([-top, -1, 0, 1, top], np.int64), n), rng.integers(0, 2**32, n) - 2**31,
                  np.arange(n, dtype=np.int64) * 1000]).astype(np.int64)
    Kd = torch.as_tensor(K, device="cuda")
    order = torch.full(K.shape, -1, dtype=torch.int32, device="cuda")
    qb.rank(Kd, order)
    got = order.cpu().numpy()
    for p in range(K.shape[0]):
        assert (got[p] == np.lexsort((np.arange(n), -K[p]))).all(), p


@pytest.mark.parametrize("n,m", [(1, 1), (64, 64), (1500, 1024), (20000, 1000), (65535, 1024), (65535, 1)])
def test_select_at_the_edges_of_its_shapes(n, m):
    from paper_2502_13947_amd import qb
    print("select", n, m, flush=True)
    rng = np.random.default_rng(n + m)
    order = rng.permutation(n).astype(np.int32)[None]
    b = qb.Batch(n, 1, [0], [m], rank0=[min(7, n - m)])
    qb.select(b, torch.as_tensor(order, device="cuda"))
    assert (b.idx("cuda").cpu().numpy() == np.sort(order[0, min(7, n - m):][:m])).all()


@pytest.mark.parametrize("count", [1, 31, 32, 33, 255, 256, 257, 5000, 70001])
def test_mlp_scores_at_the_edges_of_their_tiles(count):
    """Tiles of 32 rows, more of them than waves, and weights whose sums pass
    through zero and subnormal numbers."""
    from paper_2502_13947_amd import qb
    print("mlp", count, flush=True)
    rng = np.random.default_rng(count)
    for scale in (1.0, 1e-19):
        W = oracle.bf16((rng.normal(0, 0.4, qb.NPARAM) * scale).astype(np.float32))
        W[rng.random(qb.NPARAM) < 0.2] = 0
        F = oracle.bf16(rng.normal(0, 2.0, size=(count, 8)).astype(np.float32)).reshape(count, 8)
        Fd = torch.as_tensor(F.view(np.int16), device="cuda")
        K = torch.zeros(count, dtype=torch.int64, device="cuda")
        s = torch.zeros(count, dtype=torch.float32, device="cuda")
        qb.mlp_score(Fd, torch.as_tensor(W.view(np.int16), device="cuda"), K, score=s)
        so, Ko = oracle.mlp_scores(W, F)
        assert (s.cpu().numpy().view(np.uint32) == so.view(np.uint32)).all()
        assert (K.cpu().numpy() == Ko).all()
