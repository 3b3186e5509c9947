"""A state's borrowed tile buffer: nothing is written past its stated size."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_13947_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("graph", [False, True])
def test_sparse_state_keeps_to_its_tile_words(graph):
    """total * ell_width words of an iteration's ELL rows; the words after
    them, where qb_extract_ell puts its diagonal blocks, stay as they were."""
    from paper_2502_13947_amd import qb
    rp, col, val = inputs.torus_graph_qubo(20, 30, 4.0, 5)
    P = qb.Problem.from_csr(rp, col, val.astype(np.int16), DEV)
    Q = inputs.csr_to_dense(600, rp, col, val)
    z, job_m, R, alpha, ten = 3, np.tile([100, 70], (3, 1)).astype(np.int32), 2, 900, 4
    thr = oracle.thresholds(Q, 12)
    total, words = int(job_m.sum()), int(job_m.sum()) * P.ell_width
    blocks = 1024 * sum(qb.tile_ms(int(m)) for m in job_m.reshape(-1))
    tiles = torch.full((words + blocks,), -1, dtype=torch.int32, device=DEV)
    X = torch.zeros((z, 600), dtype=torch.uint8, device=DEV)
    S = qb.State(P, z=z, job_m=job_m, seed=9, init_m=0, thr_init=None, thr=thr, B=10, R=R, alpha=alpha, tenure=ten,
                 buffers=dict(tiles=tiles, X=X))
    stream = torch.cuda.Stream()
    S.init(stream=stream)
    S.iterate(2, graph=graph, stream=stream)
    stream.synchronize()
    t = tiles.cpu().numpy()
    assert (t[words:] == -1).all()
    assert (t[:words] != -1).all()
    ref = oracle.run(Q, z=z, seed=9, iters=2, alpha=alpha, tenure=ten, job_m=job_m, init_m=0, thr_init=thr, thr=thr,
                     B=10, R=R)
    assert (X.cpu().numpy() == ref["X"]).all() and total == 510
