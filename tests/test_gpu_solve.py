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
