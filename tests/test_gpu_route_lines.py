"""The lines between two kernels of one call: on either side the call has to
take about as long as the better one.  Each case was measured at least 2
times too long on the wrong side, and is held to 1.6 times."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def qb():
    from paper_2502_13947_amd import qb as m
    return m


def best_ms(f, reps=5):
    """Least time of a call among `reps` (after one to warm up)."""
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def dense_problem(n, lim, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    Q = torch.triu(torch.randint(-lim, lim + 1, (n, n), generator=g, device=DEV, dtype=torch.int16))
    return qb().Problem((Q + torch.triu(Q, 1).T).contiguous())


def solutions(P, z, seed, alpha):
    """z solutions after `alpha` Tabu steps, with their fields and statistics."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    X = torch.randint(0, 2, (z, P.n), generator=g, device=DEV, dtype=torch.uint8)
    H = torch.zeros((z, P.n), dtype=torch.int32, device=DEV)
    E = torch.zeros(z, dtype=torch.int64, device=DEV)
    T, LF = torch.zeros_like(H), torch.zeros_like(H)
    qb().field(P, X, H)
    qb().energy(X, H, E)
    qb().tabu(P, X, H, E, alpha, max(1, P.n // 150), True, T, LF)
    return X, H, E, T, LF


def dense_jobs(lim, m, J):
    """J jobs of m random variables, four of a solution, extracted after a
    Tabu run."""
    n, k = 4 * m + 100, 4
    z = J // k
    P = dense_problem(n, lim, 5)
    X, H, _, _, _ = solutions(P, z, 3, n)
    b = qb().Batch(n, z, np.repeat(np.arange(z), k), np.full(J, m))
    g = torch.Generator(device=DEV)
    g.manual_seed(8)
    order = torch.argsort(torch.rand((z, n), generator=g, device=DEV), dim=1).to(torch.int32).contiguous()
    qb().select(b, order)
    tiles = torch.zeros(b.tile_elems, dtype=qb().tile_dtype(P), device=DEV)
    F0 = torch.zeros(b.total, dtype=torch.int32, device=DEV)
    y0 = torch.zeros(b.total, dtype=torch.uint8, device=DEV)
    qb().extract(P, b, X, H, tiles, F0, y0)
    return P, b, tiles, F0, y0


def two_plans(lim, m, J, R, nsw, kernels):
    """Times of the annealer under two plan kernels; the results are equal."""
    P, b, tiles, F0, y0 = dense_jobs(lim, m, J)
    thr = torch.as_tensor(qb().threshold_table(nsw, 10, 0.25 * P.sigma, 0.002 * P.sigma), device=DEV)
    out, ms = [], []
    for kernel in kernels:
        b.set_plan(kernel=[kernel] * 5)
        Y = torch.zeros(b.total * R, dtype=torch.uint8, device=DEV)
        e = torch.zeros(J * R, dtype=torch.int64, device=DEV)
        ms.append(best_ms(lambda: qb().anneal(b, tiles, F0, y0, thr, R, 5, 0, Y, e, 10)))
        out.append((Y, e))
    print(f"lim {lim} m {m} J {J} R {R} kernels {kernels}: {ms[0]:.3f} and {ms[1]:.3f} ms", flush=True)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    return ms


@pytest.mark.parametrize("lim,m,J,R", [(100, 700, 1024, 2), (100, 1000, 1024, 3), (1000, 400, 1024, 2),
                                       (1000, 512, 1024, 3), (100, 256, 256, 8)])
def test_many_replicas_take_the_packed_annealer(lim, m, J, R):
    """qb_anneal without a plan, against the plan that packs a job's replicas
    into one workgroup (QB_ANNEAL_MULTI_WAVE)."""
    auto, packed = two_plans(lim, m, J, R, 40, (0, 1))
    assert auto <= 1.6 * packed


@pytest.mark.parametrize("lim,m,kernel", [(100, 1000, 3), (1000, 300, 3)])
def test_plan_kernel_without_the_class_is_the_automatic_one(lim, m, kernel):
    """A plan that names a kernel which cannot run the class."""
    named, auto = two_plans(lim, m, 64, 1, 200, (kernel, 0))
    assert named <= 1.6 * auto


def rank_ms(n, z):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    K = torch.randint(-2**46, 2**46, (z, n), generator=g, device=DEV, dtype=torch.int64)
    K[:, ::3] = K[:, :1].clone()                             # ties
    order = torch.full((z, n), -1, dtype=torch.int32, device=DEV)
    ms = best_ms(lambda: qb().rank(K, order), 20)
    want = torch.argsort(K, dim=1, descending=True, stable=True).to(torch.int32)
    assert torch.equal(order, want), n
    return ms


def test_small_ranks_are_cheap():
    """Ranking few variables takes less than ranking a thousand (it took the
    same, three to six times as long as it has to)."""
    ms = {n: rank_ms(n, 2048) for n in (1, 2, 3, 63, 64, 65, 128, 200, 513, 1000, 1023, 1024, 1025)}
    print("rank: " + "  ".join(f"n {n} {v:.4f}" for n, v in ms.items()) + " ms", flush=True)
    assert max(ms[n] for n in (1, 2, 3, 63, 64, 65)) <= 0.5 * ms[1000]
    assert ms[1000] <= 1.2 * ms[1025]


# the matrix product's splits over K: (n, more solutions, fewer, how much longer
# more may take): 1.8 and 3.0 times as long where every workgroup that was
# thought to fit became a split, 1.3 and 1.7 times with fewer
@pytest.mark.parametrize("n,more,fewer,line", [(7000, 128, 64, 1.5), (1000, 2048, 512, 2.3)])
def test_rankk_splits_no_more_than_pays(n, more, fewer, line):
    P = dense_problem(n, 100, 11)
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    ms = {}
    for z in (more, fewer):
        dX = torch.randint(-1, 2, (z, n), generator=g, device=DEV, dtype=torch.int8)
        H = torch.zeros((z, n), dtype=torch.int32, device=DEV)

        def calls():
            for _ in range(50):
                qb().rankk(P, dX, H, 2)
        ms[z] = best_ms(calls) / 50
    print(f"rankk n {n}: " + "  ".join(f"z {z} {v:.4f}" for z, v in ms.items()) + " ms", flush=True)
    assert ms[more] <= line * ms[fewer]


def test_field_of_many_16_bit_solutions():
    """The field takes less than the update of it by two thirds of the
    variables (0.65 of it with two rows a product, 1.1 with a multiplication
    each)."""
    n, z = 2500, 1024
    P = dense_problem(n, 1000, 11)
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    dX = torch.randint(-1, 2, (z, n), generator=g, device=DEV, dtype=torch.int8)
    H = torch.zeros((z, n), dtype=torch.int32, device=DEV)
    X = dX.abs().to(torch.uint8)
    field, update = best_ms(lambda: qb().field(P, X, H)), best_ms(lambda: qb().rankk(P, dX, H, 1))
    print(f"field n {n} z {z}: {field:.4f}  rankk {update:.4f} ms", flush=True)
    assert field <= 0.85 * update


def ell_jobs(n, z, k, m, W, seed):
    """z solutions of k jobs of m random variables on a circulant graph with W
    entries a row: the outputs of qb_extract_ell and its time."""
    i = np.repeat(np.arange(n), W)
    j = (i + np.tile(np.concatenate([np.arange(1, W // 2 + 1), -np.arange(1, W // 2 + 1)]), n)) % n
    o = np.lexsort((j, i))
    v = ((np.minimum(i, j) * 7919 + np.maximum(i, j) * 104729) % 11 - 5)[o]
    v[v == 0] = 6
    P = qb().Problem.from_csr((np.arange(n + 1) * W).astype(np.int32), j[o].astype(np.int32), v.astype(np.int16), DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    X = torch.randint(0, 2, (z, n), generator=g, device=DEV, dtype=torch.uint8)
    H = torch.zeros((z, n), dtype=torch.int32, device=DEV)
    qb().field(P, X, H)
    order = torch.argsort(torch.rand((z, n), generator=g, device=DEV), dim=1).to(torch.int32).contiguous()
    b = qb().Batch(n, z, np.repeat(np.arange(z), k), np.full(z * k, m))
    qb().select(b, order)
    tile = torch.full((qb().ell_tile_words(b, P.ell_width),), -1, dtype=torch.int32, device=DEV)
    F0 = torch.zeros(b.total, dtype=torch.int32, device=DEV)
    y0 = torch.zeros(b.total, dtype=torch.uint8, device=DEV)
    c = torch.zeros(b.total, dtype=torch.int32, device=DEV)
    ms = best_ms(lambda: qb().extract_ell(P, b, X, H, tile, F0, y0, c))
    return P, b, X, H, tile, F0, y0, c, ms


# both ways of finding a column's place (a table over all variables; a search
# in the job's index set), with jobs of one variable, odd sizes and the largest
@pytest.mark.parametrize("n,z,k,m,W", [(5000, 64, 260, 1, 8), (5000, 64, 260, 17, 8), (20001, 64, 256, 33, 10),
                                       (40000, 40, 128, 100, 6), (1000, 4, 3, 33, 8), (65535, 8, 40, 33, 4),
                                       (3001, 2, 2, 1024, 12)])
def test_extract_ell_finds_places_both_ways(n, z, k, m, W):
    """Rows, c, F0 and y0 of a sample of the jobs, rebuilt from the circulant
    rows."""
    P, b, X, H, tile, F0, y0, c, _ = ell_jobs(n, z, k, m, W, n)
    idx = b.idx(DEV).cpu().numpy()
    Xh, Hh = X.cpu().numpy(), H.cpu().numpy()
    Fh, yh, ch = F0.cpu().numpy(), y0.cpu().numpy(), c.cpu().numpy()
    step = np.concatenate([np.arange(1, W // 2 + 1), -np.arange(1, W // 2 + 1)])
    for q in range(0, b.J, max(1, b.J // 50)):
        p, sl = q // k, slice(q * m, (q + 1) * m)
        S = idx[sl]
        I, J = np.repeat(S, W), (np.repeat(S, W) + np.tile(step, m)) % n
        v = (np.minimum(I, J) * 7919 + np.maximum(I, J) * 104729) % 11 - 5
        v[v == 0] = 6
        at = np.searchsorted(S, J)
        hit = (at < m) & (S[np.minimum(at, m - 1)] == J)
        T = np.zeros((m, m), np.int64)
        T[np.repeat(np.arange(m), W)[hit], at[hit]] = v[hit]
        assert (qb().untile_ell(tile, b, q, P.ell_width) == T).all(), q
        assert (yh[sl] == Xh[p, S]).all() and (Fh[sl] == 2 * Hh[p, S]).all(), q
        assert (ch[sl] == 2 * Hh[p, S] - 2 * T @ Xh[p, S].astype(np.int64)).all(), q


def test_small_sparse_jobs_of_many_variables():
    """Extracting many small jobs does not depend on n (it took five times as
    long at n = 65535)."""
    ms = {n: ell_jobs(n, 64, 256, 16, 8, 1)[-1] for n in (5000, 65535)}
    print("extract: " + "  ".join(f"n {n} {v:.4f}" for n, v in ms.items()) + " ms", flush=True)
    assert ms[65535] <= 1.7 * ms[5000]
