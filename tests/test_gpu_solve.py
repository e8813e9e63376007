"""The solve at the edges of its 128-row workgroups, 64-wide blocks, chunks of
16 right-hand sides and launches of 256, in every class, against FP64 products
with the GPU's own factor."""
import numpy as np
import pytest

import synth
from _gpu import M, factor_dense, log, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile,nrhs,pad,mixed", [
    (1, 128, 1, 0, False), (64, 128, 2, 0, False), (65, 128, 1, 3, False), (128, 128, 16, 0, False),
    (129, 128, 17, 1, False), (576, 256, 15, 0, False), (1000, 128, 1, 0, True), (1000, 256, 33, 7, True),
    (3600, 1024, 16, 0, True), (3600, 1024, 1, 0, True), (700, 128, 259, 0, False)])
def test_solve_edges(n, tile, nrhs, pad, mixed):
    """||B - L L^T X||_F <= 4 n u (||L||^2 ||X|| + ||B||): the bound of two
    substitutions (each at most n u relative to |L| |X|), doubled."""
    torch = torch_cuda()
    mod = M()
    h = mod.mpchol_create(n, tile)
    nt = -(-n // tile)
    try:
        if mixed:
            sigma, x = synth.workload(int(np.ceil(np.sqrt(n))))
            mod.mpchol_set_generator(h, sigma[:n], x[:n], 5.0, 1e-8)
            mp = mod.mpchol_precision_map(h, mod.RULE_NORM, 1e-4)
            assert mp.max() > 0
        else:
            L0 = synth.int_lower(n, 11) / (1.0 + np.arange(n))[None, :] + 3.0 * np.eye(n)
            mod.mpchol_set_matrix(h, L0 @ L0.T)
            mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        Lg = factor_dense(h, n)
        B = synth.rhs(n, nrhs)
        Bt = torch.full((nrhs, n + pad), 7.0, dtype=torch.float64, device="cuda")
        Bt[:, :n] = torch.tensor(np.ascontiguousarray(B.T), device="cuda")
        outs = []
        for _ in range(3):  # the same result every time
            X = Bt.clone()
            mod.mpchol_solve(h, X.T, n)
            outs.append(X)
        torch.cuda.synchronize()
    finally:
        mod.mpchol_destroy(h)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert torch.all(outs[0][:, n:] == 7.0)
    X = outs[0][:, :n].T.cpu().numpy()
    R = B - Lg @ (Lg.T @ X)
    scale = np.linalg.norm(Lg) ** 2 * np.linalg.norm(X) + np.linalg.norm(B)
    log(f"  solve n={n} tile={tile} nrhs={nrhs} mixed={mixed}: {np.linalg.norm(R) / scale:.2e}")
    assert np.linalg.norm(R) <= 4 * n * 2.0 ** -53 * scale


@pytest.mark.parametrize("n,tile,exp2,nrhs", [(300, 128, 0, 3), (300, 128, -1010, 16), (300, 128, 980, 17),
                                              (1000, 256, -1004, 1), (1000, 256, 990, 1)])
def test_solve_scaled(n, tile, exp2, nrhs):
    """Diagonals of the factor inside and outside the range in which quotients come
    from reciprocals (2^-500 to 2^500), the bound of test_solve_edges on
    everything scaled back (powers of two: exact)."""
    torch = torch_cuda()
    mod = M()
    S = (synth.int_lower(n, 11) / (1.0 + np.arange(n))[None, :] + 3.0 * np.eye(n)) * 2.0 ** (exp2 // 2)
    B = synth.rhs(n, nrhs)
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, S @ S.T)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        Lg = factor_dense(h, n) * 2.0 ** -(exp2 // 2)
        Bt = torch.tensor(np.ascontiguousarray(B.T), device="cuda") * 2.0 ** (exp2 // 2)
        mod.mpchol_solve(h, Bt.T, n)
        X = Bt.cpu().numpy().T * 2.0 ** (exp2 // 2)
    finally:
        mod.mpchol_destroy(h)
    u = 2.0 ** -53
    res = np.linalg.norm(B - Lg @ (Lg.T @ X))
    assert res <= 4 * n * u * (np.linalg.norm(Lg) ** 2 * np.linalg.norm(X) + np.linalg.norm(B))


def test_solve_hands_on_any_nan():
    """A right-hand side with NaN payloads (the mailbox's own mark among them) ends
    as NaN where it reaches; the other right-hand sides are as without them."""
    torch = torch_cuda()
    mod = M()
    n = 700
    S = synth.int_lower(n, 11) / (1.0 + np.arange(n))[None, :] + 3.0 * np.eye(n)
    h = mod.mpchol_create(n, 128)
    try:
        mod.mpchol_set_matrix(h, S @ S.T)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        B = torch.tensor(np.ascontiguousarray(synth.rhs(n, 5).T), device="cuda")
        clean = B.clone()
        marks = torch.tensor(np.array([0x7FF85EED0BADF00D, 0xFFF85EED0BADF00D], dtype=np.uint64).view(np.float64),
                             device="cuda")
        B[1, 0], B[3, 130], B[3, 131] = marks[0], marks[1], marks[0]
        mod.mpchol_solve(h, B.T, n)
        mod.mpchol_solve(h, clean.T, n)
        torch.cuda.synchronize()
    finally:
        mod.mpchol_destroy(h)
    assert torch.equal(B[[0, 2, 4]], clean[[0, 2, 4]])
    assert torch.isnan(B[1, 0]) and torch.isnan(B[3, 130])


def _int_handle(mod, n, tile, stream=None):
    S = synth.int_lower(n, 11) / (1.0 + np.arange(n))[None, :] + 3.0 * np.eye(n)
    h = mod.mpchol_create(n, tile, stream=stream)
    mod.mpchol_set_matrix(h, S @ S.T)
    mod.mpchol_precision_map(h, mod.RULE_FP64)
    assert mod.mpchol_factor(h) == 0
    return h


@pytest.mark.parametrize("n,tile,nrhs", [(3600, 256, (1, 3)), (2000, 128, (17, 16))])
def test_recorded_solves_replay_side_by_side(n, tile, nrhs):
    """Two solves recorded into graphs, replayed on streams of their own beside
    each other and beside the handle's own draws and solves: every result is the
    one that the call gives alone, bit for bit, in every round."""
    torch = torch_cuda()
    mod = M()
    home, s1, s2 = (torch.cuda.Stream() for _ in range(3))
    h = _int_handle(mod, n, tile, stream=home)
    try:
        rhs = [torch.tensor(np.ascontiguousarray(synth.rhs(n, k + i).T[i:]), device="cuda") for i, k in enumerate((*nrhs, 2))]
        want = [b.clone() for b in rhs]
        Y, Yw = (torch.zeros((64, n), device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        for b in want:
            mod.mpchol_solve(h, b.T, n)
        mod.mpchol_sample(h, 64, 5, Yw.T, n)
        B = [b.clone() for b in rhs]
        graphs = []
        for b in B[:2]:
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=home):
                mod.mpchol_solve(h, b.T, n)
            graphs.append(g)
        for _ in range(8):
            for b, r in zip(B, rhs):
                b.copy_(r)
            Y.zero_()
            torch.cuda.synchronize()
            for g, s in zip(graphs, (s1, s2)):
                with torch.cuda.stream(s):
                    g.replay()
            mod.mpchol_solve(h, B[2].T, n)
            mod.mpchol_sample(h, 64, 5, Y.T, n)
            torch.cuda.synchronize()
            assert all(torch.equal(b, w) for b, w in zip(B, want)) and torch.equal(Y, Yw)
        assert np.isfinite(mod.mpchol_logdet(h))
    finally:
        mod.mpchol_destroy(h)


def test_threads_with_streams_of_their_own():
    """A handle on hipStreamPerThread: solves and draws of two threads run on two
    streams; their shared scratch keeps them apart."""
    import threading

    torch = torch_cuda()
    mod = M()
    n, rounds = 3000, 12
    h = _int_handle(mod, n, 128, stream=2)  # hipStreamPerThread
    try:
        b = torch.tensor(np.ascontiguousarray(synth.rhs(n, 5).T), device="cuda")
        want, B = b.clone(), b.repeat(rounds, 1, 1)
        Yw, Y = torch.zeros((128, n), device="cuda"), torch.zeros((rounds, 128, n), device="cuda")
        torch.cuda.synchronize()
        mod.mpchol_solve(h, want.T, n)
        mod.mpchol_sample(h, 128, 5, Yw.T, n)
        torch.cuda.synchronize()
        # get_stats waits for the solves: the runtime does not, once their thread and its stream are gone
        ts = [threading.Thread(target=lambda: [mod.mpchol_solve(h, B[i].T, n) for i in range(rounds)] + [mod.mpchol_get_stats(h)]),
              threading.Thread(target=lambda: [mod.mpchol_sample(h, 128, 5, Y[i].T, n) for i in range(rounds)])]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        torch.cuda.synchronize()
    finally:
        mod.mpchol_destroy(h)
    assert all(torch.equal(B[i], want) and torch.equal(Y[i], Yw) for i in range(rounds))


def _substitute(L, B):
    """L L^T X = B column by column, in the type of B: terms taken in their natural order."""
    X = B.copy()
    for k in range(len(L)):
        X[k] /= L[k, k]
        X[k + 1:] -= L[k + 1:, k:k + 1] * X[k:k + 1]
    for k in range(len(L) - 1, -1, -1):
        X[k] /= L[k, k]
        X[:k] -= L[k, :k][:, None] * X[k:k + 1]
    return X


@pytest.mark.parametrize("rho", [2.0, 20.0])
@pytest.mark.parametrize("band,tile,nrhs", [(38, 128, 16), (38, 128, 1), (38, 512, 16), (30, 256, 2)])
def test_solve_error_of_neighbours_that_cancel(band, tile, nrhs, rho):
    """Neighbouring terms of a solve with a correlation nearly cancel, so the order
    of the sums decides the error: at most twice that of substitution in natural
    order in FP64 (two draws of rounding errors differ by less), both against long
    double with the GPU's own factor.  Sums over every other term take 4 to 6 times at
    a correlation length of 20."""
    torch = torch_cuda()
    mod = M()
    n = band * band
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_generator(h, *synth.workload(band), rho, 1e-8)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        L = factor_dense(h, n)
        B = synth.rhs(n, nrhs)
        Bt = torch.tensor(np.ascontiguousarray(B.T), device="cuda")
        mod.mpchol_solve(h, Bt.T, n)
        X = Bt.cpu().numpy().T
    finally:
        mod.mpchol_destroy(h)
    exact = _substitute(L.astype(np.longdouble), B.astype(np.longdouble))
    err, ref = (float(np.sqrt((((v - exact) / np.abs(exact).max()) ** 2).sum())) for v in (X, _substitute(L, B)))
    log(f"  n={n} tile={tile} nrhs={nrhs} rho={rho}: {err:.2e}, in natural order {ref:.2e}")
    assert err <= 2.0 * ref
