"""The work that users of mpchol have it do, as measurable cases.

Five kinds of calls, each through the Python binding of the C ABI:

* "factor"  -- FP64 tile Cholesky of a covariance: precision map, factor, log-determinant, one solve and the dense
               factor (the small and the middle FP64 workloads of bench.py, band limits 32 and 128);
* "train"   -- the covariance estimated from samples and its FP64 factor (the emulator's training step);
* "emulate" -- the mixed-precision path: map by the norm rule or by the learned selector with randomized
               verification, factor, log-determinant and emulation draws (bench.py's mixed workloads);
* "solve", "sample", "check" -- products on a factor that the program keeps: solves with Sigma, draws L z, and the
               backward error of the factor against a caller's matrix;
* "sht"     -- the spherical harmonic transform of a batch of fields, forward or inverse;
* "selector"-- loss and gradient of the precision selector on a training batch.

Covariances follow the framework's synthetic workload: order N = L^2, coordinates of the (l, m) coefficient order,
scales (1 + l)^-1 with a lognormal(0, 0.1) factor drawn from the seed, exponential correlation over the coordinates and
a nugget of 1e-8.
"""
import math

import numpy as np
import torch

from paper_2408_04440_amd import mpchol as M
from paper_2408_04440_amd import selector as S

NUGGET = 1e-8
DEV = "cuda"


def listed():
    return [
        # one small FP64 covariance from start to end: launches and latencies decide
        dict(name="factor_fp64_1k", kind="factor", L=32, tile=128, rho=5.0, nrhs=1),
        # the FP64 path of a middle-sized workload
        dict(name="factor_fp64_16k", kind="factor", L=128, tile=512, rho=5.0, nrhs=1),
        # training from samples: a ragged order, a matrix without structure
        dict(name="train_4900_m6000", kind="train", L=70, tile=256, m=6000),
        # the mixed path with BF16 under the norm rule and a full set of draws: the largest call
        dict(name="emulate_bf16_65k", kind="emulate", L=256, tile=1024, rho=5.0, rule="norm", lo16="bf16", fp8=False,
             draws=1000),
        # the mixed path with every class, the learned map and its verification, on a ragged order
        dict(name="emulate_learned_32k", kind="emulate", L=180, tile=1024, rho=5.0, rule="learned", lo16="f16", fp8=True,
             draws=100),
        # solves with a kept factor: a block of right-hand sides
        dict(name="solve_16k_16rhs", kind="solve", L=128, tile=512, rho=5.0, nrhs=16),
        # draws from a kept factor
        dict(name="sample_16k_1000", kind="sample", L=128, tile=512, rho=5.0, draws=1000),
        # the acceptance check of a factor against the matrix that it is meant for
        dict(name="check_8100", kind="check", L=90, tile=512, rho=5.0),
        # training data: a batch of fields at the band limit of the factorization workload
        dict(name="sht_forward_360_T512", kind="sht", L=360, ntheta=361, nphi=720, T=512, forward=True),
        # emulated coefficients back to fields on the 0.25 degree grid
        dict(name="sht_inverse_720_T64", kind="sht", L=720, ntheta=721, nphi=1440, T=64, forward=False),
        # one field at a time on a small ragged grid: latency
        dict(name="sht_forward_45_T1", kind="sht", L=45, ntheta=50, nphi=96, T=1, forward=True),
        # a full-batch training step's gradient
        dict(name="selector_grad_8838", kind="selector", nb=8838),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _smooth(n):
    """Smallest product of 2, 3 and 5 that is at least n."""
    while True:
        r = n
        for p in (2, 3, 5):
            while r % p == 0:
                r //= p
        if r == 1:
            return n
        n += 1


def draw(rng):
    kind = rng.choice(["factor", "train", "emulate", "emulate", "solve", "solve", "sample", "sample", "check", "sht", "sht",
                       "sht", "selector"])
    rho = rng.choice([2.0, 5.0, 20.0])
    if kind == "factor":
        return dict(kind=kind, L=_log(rng, 12, 128), tile=rng.choice([128, 256, 512, 1024]), rho=rho, nrhs=rng.randint(1, 4))
    if kind == "train":
        L = _log(rng, 12, 70)
        return dict(kind=kind, L=L, tile=rng.choice([128, 256, 512]), m=int(L * L * rng.uniform(1.2, 1.5)) + 1)
    if kind == "emulate":
        return dict(kind=kind, L=_log(rng, 40, 200), tile=rng.choice([256, 512, 1024]), rho=rho,
                    rule=rng.choice(["norm", "learned"]), lo16=rng.choice(["f16", "bf16"]), fp8=rng.choice([True, False]),
                    draws=_log(rng, 1, 1000))
    if kind == "solve":
        return dict(kind=kind, L=_log(rng, 12, 128), tile=rng.choice([128, 256, 512, 1024]), rho=rho, nrhs=_log(rng, 1, 64))
    if kind == "sample":
        return dict(kind=kind, L=_log(rng, 12, 128), tile=rng.choice([128, 256, 512, 1024]), rho=rho, draws=_log(rng, 1, 1000))
    if kind == "check":
        return dict(kind=kind, L=_log(rng, 12, 100), tile=rng.choice([128, 256, 512, 1024]), rho=rho)
    if kind == "selector":
        return dict(kind=kind, nb=_log(rng, 64, 20000))
    L = _log(rng, 8, 720)
    nt = L + 1 + rng.choice([0, 0, 1, rng.randint(0, L // 4 + 1)])
    T = min(_log(rng, 1, 512), max(1, 512 * 360 * 361 * 720 // (L * nt * 2 * L)))
    return dict(kind=kind, L=L, ntheta=nt, nphi=_smooth(2 * L - 1 + rng.choice([0, 1, 1, rng.randint(0, L)])), T=T,
                forward=rng.choice([True, False]))


# ------------------------------------------------------------------------------------------------------ inputs
def _coords(L):
    l = np.repeat(np.arange(L), 2 * np.arange(L) + 1).astype(np.float64)
    i = np.arange(L * L) - l * l
    return l, l + i / (2.0 * l + 1.0)


def _workload(L, seed):
    l, x = _coords(L)
    g = np.random.RandomState(seed % (1 << 31)).standard_normal(L * L)
    return np.exp(0.1 * g) / (1.0 + l), x


def _cov(sigma, x, rho):
    """Sigma as a dense matrix (FP64, on the GPU)."""
    s, c = torch.from_numpy(sigma).to(DEV), torch.from_numpy(x).to(DEV)
    A = c[:, None] - c[None, :]
    A.abs_().div_(-rho).exp_().mul_(s[:, None]).mul_(s[None, :])
    A.diagonal().add_(NUGGET)
    return A


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 40))


def _normal(shape, seed, dtype=torch.float64):
    return torch.randn(shape, generator=_gen(seed), dtype=dtype, device=DEV)


class _Kept:
    """A library object that is given back with its state."""

    def __init__(self, obj, give_back):
        self.obj, self.give_back = obj, give_back

    def __del__(self):
        try:
            self.give_back(self.obj)
        except Exception:
            pass


def _samples(L, m, seed):
    l = torch.from_numpy(_coords(L)[0]).to(DEV)
    return _normal((m, L * L), seed + 1).div_(1.0 + l[None, :])  # column-major n x m


def _check_matrix(L, rho, seed):
    """The covariance with 1% of its own size added as a smooth low-rank part: what an updated estimate looks like."""
    sigma, x = _workload(L, seed)
    A = _cov(sigma, x, rho)
    U = _normal((L * L, 8), seed + 5).mul_(0.05 * torch.from_numpy(sigma).to(DEV)[:, None])
    return A.addmm_(U, U.T)


def _selector_batch(nb, seed):
    X = _normal((nb, 8), seed + 2, torch.float32).mul_(2.0)
    y = torch.randint(0, 4, (nb,), generator=_gen(seed + 3), device=DEV, dtype=torch.int32)
    return X, y


CW, ALPHA = [0.5, 1.5, 1.0, 0.75], 2.0


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "seed": int(seed)}
    if kind == "sht":
        L, nt, nph, T = case["L"], case["ntheta"], case["nphi"], case["T"]
        st["o"] = _Kept(M.mpchol_sht_create(L, nt, nph, T), M.mpchol_sht_destroy)
        if case["forward"]:
            st["Z"] = _normal((T, nt, nph), seed)
            st["f"] = torch.empty((T, L * L), dtype=torch.float64, device=DEV)
        else:
            st["f"] = _sht_coeffs(L, T, seed)
            st["Z"] = torch.empty((T, nt, nph), dtype=torch.float64, device=DEV)
        return st
    if kind == "selector":
        st["o"] = _Kept(M.mpchol_mlp_create(), M.mpchol_mlp_destroy)
        M.mpchol_mlp_set_params(st["o"].obj, S.load())
        st["X"], st["y"] = _selector_batch(case["nb"], seed)
        st["grad"] = torch.empty(M.MLP_NPARAM, dtype=torch.float32, device=DEV)
        return st
    L = case["L"]
    n = L * L
    opts = {}
    if kind == "emulate":
        opts = dict(lo16=M.LO16_BF16 if case["lo16"] == "bf16" else M.LO16_F16, allowed=0xF if case["fp8"] else 0x7,
                    verify=2 if case["rule"] == "learned" else 0, verify_eps=1e-9)
    h = M.mpchol_create(n, case["tile"], **opts)
    st["o"], st["n"], st["nt"] = _Kept(h, M.mpchol_destroy), n, -(-n // case["tile"])
    if kind == "train":
        st["Xi"] = _samples(L, case["m"], seed)
        st["L"] = torch.empty((n, n), dtype=torch.float64, device=DEV)
        return st
    M.mpchol_set_generator(h, *_workload(L, seed), case["rho"], NUGGET, n)
    if kind == "emulate":
        if case["rule"] == "learned":
            M.mpchol_selector_set(h, S.load())
        st["Y"] = torch.empty((case["draws"], n), dtype=torch.float32, device=DEV)
        return st
    if kind == "factor":
        st["L"] = torch.empty((n, n), dtype=torch.float64, device=DEV)
    else:
        M.mpchol_precision_map(h, M.RULE_FP64, nt=st["nt"])
        assert M.mpchol_factor(h) == 0
    if kind in ("factor", "solve"):
        st["B"] = _normal((case["nrhs"], n), seed + 4)
        st["X"] = torch.empty_like(st["B"])
    elif kind == "sample":
        st["Y"] = torch.empty((case["draws"], n), dtype=torch.float32, device=DEV)
    elif kind == "check":
        st["A"] = _check_matrix(L, case["rho"], seed)
    return st


def run(st):
    case, h = st["case"], st["o"].obj
    kind = case["kind"]
    if kind == "sht":
        if case["forward"]:
            M.mpchol_sht_forward(h, st["Z"], st["f"], case["L"])
            return st["f"]
        M.mpchol_sht_inverse(h, st["f"], st["Z"], case["L"])
        return st["Z"]
    if kind == "selector":
        loss = M.mpchol_mlp_grad(h, st["X"], st["y"], CW, ALPHA, st["grad"])
        return {"grad": st["grad"], "loss": loss}
    n = st["n"]
    if kind == "factor":
        M.mpchol_precision_map(h, M.RULE_FP64, nt=st["nt"])
        assert M.mpchol_factor(h) == 0
        logdet = M.mpchol_logdet(h)
        st["X"].copy_(st["B"])
        M.mpchol_solve(h, st["X"].T, n)
        M.mpchol_get_factor(h, st["L"].T, n)
        return {"L": st["L"], "X": st["X"], "logdet": np.float64(logdet)}
    if kind == "train":
        M.mpchol_set_samples(h, st["Xi"].T, 1.0 / case["m"], NUGGET)
        M.mpchol_precision_map(h, M.RULE_FP64, nt=st["nt"])
        assert M.mpchol_factor(h) == 0
        M.mpchol_get_factor(h, st["L"].T, n)
        return st["L"]
    if kind == "emulate":
        m = M.mpchol_precision_map(h, M.RULE_NORM if case["rule"] == "norm" else M.RULE_LEARNED, 1e-9, nt=st["nt"])
        assert M.mpchol_factor(h) == 0
        logdet = M.mpchol_logdet(h)
        M.mpchol_sample(h, case["draws"], st["seed"], st["Y"].T, n)
        return {"Y": st["Y"], "map": m, "logdet": logdet}
    if kind == "solve":
        st["X"].copy_(st["B"])
        M.mpchol_solve(h, st["X"].T, n)
        return st["X"]
    if kind == "sample":
        M.mpchol_sample(h, case["draws"], st["seed"], st["Y"].T, n)
        return st["Y"]
    berr, tiles = M.mpchol_backward_error_matrix(h, st["A"].T, tiles=True, nt=st["nt"])
    return {"berr": np.float64(berr), "tiles": tiles}


def work(case):
    kind = case["kind"]
    if kind == "sht":
        L, nt, nph, T = case["L"], case["ntheta"], case["nphi"], case["T"]
        # both parities of every order over half the colatitudes, real tables times complex columns; one real FFT a row
        flops = T * (4.0 * (L * (L + 1) / 2) * ((nt + 1) // 2) + nt * 2.5 * nph * math.log2(nph))
        return {"bytes": 8.0 * T * (nt * nph + L * L), "flops": flops}
    if kind == "selector":
        nb, p = case["nb"], 8 * 64 + 64 * 64 + 64 * 4
        return {"bytes": 4.0 * (nb * 9 + 2 * M.MLP_NPARAM), "flops": 6.0 * nb * p}
    n = float(case["L"] ** 2)
    low = n * (n + 1) / 2 * 8
    if kind == "factor":
        return {"bytes": 8 * (2 * n + n * n + 2 * n * case["nrhs"]), "flops": n ** 3 / 3 + 2 * n * n * case["nrhs"]}
    if kind == "train":
        return {"bytes": 8 * (n * case["m"] + n * n), "flops": n * n * case["m"] + n ** 3 / 3}
    if kind == "emulate":
        return {"bytes": 8 * 2 * n + 4 * n * case["draws"], "flops": n ** 3 / 3 + n * n * case["draws"]}
    if kind == "solve":
        return {"bytes": low + 16 * n * case["nrhs"], "flops": 2 * n * n * case["nrhs"]}
    if kind == "sample":
        return {"bytes": low + 4 * n * case["draws"], "flops": n * n * case["draws"]}
    return {"bytes": 2 * low, "flops": n ** 3 / 3}


# ------------------------------------------------------------------------------------------------------ in 64 bits
def _sht_coeffs(L, T, seed):
    l = torch.from_numpy(_coords(L)[0]).to(DEV)
    return _normal((T, L * L), seed).div_(1.0 + l[None, :])


def _legendre(L, m, x):
    """Y_lm(theta, 0), orthonormal with the Condon-Shortley phase, for l = m..L-1 (rows) at x = cos(theta)."""
    s = np.sqrt(np.maximum(0.0, 1.0 - x * x))
    a = np.full_like(x, math.sqrt(1.0 / (4.0 * math.pi)))
    for k in range(1, m + 1):
        a = a * (-math.sqrt((2.0 * k + 1.0) / (2.0 * k))) * s
    P = np.zeros((L - m, len(x)))
    P[0] = a
    if L - m > 1:
        P[1] = math.sqrt(2.0 * m + 3.0) * x * a
    for l in range(m + 2, L):
        c = math.sqrt((4.0 * l * l - 1.0) / (l * l - m * m))
        d = math.sqrt(((l - 1.0) ** 2 - m * m) / (4.0 * (l - 1.0) ** 2 - 1.0))
        P[l - m] = c * (x * P[l - m - 1] - d * P[l - m - 2])
    return P


def _sht_inverse(case, f):
    L, nt, nph, T = case["L"], case["ntheta"], case["nphi"], case["T"]
    x = np.cos(np.pi * np.arange(nt) / (nt - 1))
    l = np.arange(L)
    G = torch.zeros((T, nt, nph // 2 + 1), dtype=torch.complex128, device=DEV)
    for m in range(L):
        P = torch.from_numpy(_legendre(L, m, x)).to(DEV)
        if m % 2:
            P[:, 0] = P[:, -1] = 0.0
        i = torch.from_numpy((l * l + l)[m:]).to(DEV)
        if m == 0:
            G[:, :, 0] = (f[:, i] @ P).to(torch.complex128)
        else:
            G[:, :, m] = torch.complex(f[:, i + m] @ P, f[:, i - m] @ P) / math.sqrt(2.0)
    return torch.fft.irfft(G, n=nph, dim=2, norm="forward")


def _sht_forward(case, Z):
    """The longitude spectrum, its trigonometric interpolant in colatitude cut at |m'| < L, and the integral against
    Y_lm by a Gauss-Legendre rule, which is exact for it."""
    L, nt, nph, T = case["L"], case["ntheta"], case["nphi"], case["T"]
    G = torch.fft.rfft(Z, dim=2)[:, :, :L] * (2.0 * math.pi / nph)
    x, w = np.polynomial.legendre.leggauss(L + 1)
    k, j, mp = np.arccos(x), np.pi * np.arange(nt) / (nt - 1), np.arange(L)
    end = np.where((np.arange(nt) == 0) | (np.arange(nt) == nt - 1), 1.0, 2.0) / (2 * nt - 2)
    even = (np.cos(np.outer(k, mp)) * np.where(mp == 0, 1.0, 2.0)) @ np.cos(np.outer(mp, j)) * end
    odd = 2.0 * np.sin(np.outer(k, mp)) @ np.sin(np.outer(mp, j)) * end
    odd[:, 0] = odd[:, -1] = 0.0
    E = [torch.from_numpy(v * w[:, None]).to(DEV) for v in (even, odd)]
    f = torch.zeros((T, L * L), dtype=torch.float64, device=DEV)
    l = np.arange(L)
    for m in range(L):
        P = torch.from_numpy(_legendre(L, m, x)).to(DEV) @ E[m % 2]
        i = torch.from_numpy((l * l + l)[m:]).to(DEV)
        g = G[:, :, m]
        if m == 0:
            f[:, i] = g.real.contiguous() @ P.T.contiguous()
        else:
            f[:, i + m] = math.sqrt(2.0) * (g.real.contiguous() @ P.T.contiguous())
            f[:, i - m] = math.sqrt(2.0) * (g.imag.contiguous() @ P.T.contiguous())
    return f


def _philox_normals(seed, count):
    """The draw sequence: Philox4x32-10 with counter block e / 4 and key = seed, Box-Muller on output pairs."""
    nb = (count + 3) // 4
    mask = np.uint64(0xFFFFFFFF)
    c = [np.arange(nb, dtype=np.uint64) & mask, np.arange(nb, dtype=np.uint64) >> np.uint64(32),
         np.zeros(nb, np.uint64), np.zeros(nb, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = [torch.from_numpy(((v >> np.uint64(8)) + np.uint64(1)).astype(np.float64)).to(DEV) * 2.0 ** -24 for v in c]
    z = torch.empty((nb, 4), dtype=torch.float64, device=DEV)
    for a in (0, 2):
        r = torch.sqrt(-2.0 * torch.log(u[a]))
        z[:, a], z[:, a + 1] = r * torch.cos(2.0 * math.pi * u[a + 1]), r * torch.sin(2.0 * math.pi * u[a + 1])
    return z.reshape(-1)[:count]


def _logdet(sigma, x, rho):
    """log det of D K D + nugget I with K the exponential kernel on sorted coordinates: K^-1 is tridiagonal."""
    a = np.exp(-np.diff(x) / rho)
    q = 1.0 - a * a
    diag = np.ones(len(x))
    diag[:-1] += a * a / q
    diag[1:] += a * a / q
    off = -a / q / (sigma[:-1] * sigma[1:]) * NUGGET
    diag = 1.0 + NUGGET * diag / (sigma * sigma)
    total, p = 2.0 * np.sum(np.log(sigma)) + np.sum(np.log(q)), 0.0
    for i in range(len(x)):
        p = diag[i] - (off[i - 1] ** 2 / p if i else 0.0)
        total += math.log(p)
    return total


def exact(case, seed):
    kind = case["kind"]
    if kind == "sht":
        L, nt, nph, T = case["L"], case["ntheta"], case["nphi"], case["T"]
        if case["forward"]:
            return _sht_forward(case, _normal((T, nt, nph), seed))
        return _sht_inverse(case, _sht_coeffs(L, T, seed))
    if kind == "selector":
        X, y = _selector_batch(case["nb"], seed)
        p = torch.from_numpy(np.asarray(S.load(), dtype=np.float64)).to(DEV).requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(p, [512, 64, 4096, 64, 256, 4])
        a = torch.relu(X.double() @ W1.view(64, 8).T + b1)
        a = torch.relu(a @ W2.view(64, 64).T + b2)
        q = torch.log_softmax(a @ W3.view(4, 64).T + b3, dim=1)
        y = y.long()
        above = (torch.arange(4, device=DEV)[None, :] > y[:, None]).double()
        cw = torch.tensor(CW, dtype=torch.float64, device=DEV)
        loss = (-cw[y] * q.gather(1, y[:, None])[:, 0] + ALPHA * (q.exp() * above).sum(1)).mean()
        loss.backward()
        return {"grad": p.grad, "loss": np.float64(loss.item())}
    L, n = case["L"], case["L"] ** 2
    if kind == "train":
        Xi = _samples(L, case["m"], seed)
        A = Xi.T.contiguous() @ Xi / case["m"]
        A.diagonal().add_(NUGGET)
        return torch.linalg.cholesky(A).T.contiguous()
    sigma, x = _workload(L, seed)
    if kind == "check":
        A = _check_matrix(L, case["rho"], seed)
        fro, A = torch.linalg.norm(A), A.sub_(_cov(sigma, x, case["rho"])).square_()
        b = case["tile"]
        nt = -(-n // b)
        tiles = np.zeros((nt, nt), order="F")
        for I in range(nt):
            for J in range(I + 1):
                tiles[I, J] = float(A[I * b:(I + 1) * b, J * b:(J + 1) * b].sum())
        return {"berr": np.float64(math.sqrt(float(A.sum())) / float(fro)), "tiles": tiles}
    logdet = np.float64(_logdet(sigma, x, case["rho"])) if kind in ("factor", "emulate") else None
    if n > 33000:  # the dense factor takes too long
        return {"Y": None, "map": None, "logdet": logdet}
    C = torch.linalg.cholesky(_cov(sigma, x, case["rho"]))
    if kind in ("factor", "solve"):
        X = torch.cholesky_solve(_normal((case["nrhs"], n), seed + 4).T.contiguous(), C).T.contiguous()
        return X if kind == "solve" else {"L": C.T.contiguous(), "X": X, "logdet": logdet}
    Z = _philox_normals(int(seed), n * case["draws"]).view(case["draws"], n)
    Y = Z @ C.T.contiguous()
    return Y if kind == "sample" else {"Y": Y, "map": None, "logdet": logdet}
