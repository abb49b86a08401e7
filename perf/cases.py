"""The workloads the library's speed is judged on: data preparation (Q and K from
a Hamiltonian and its dissipation, dense or sparse) and RK4 integration of
dv/dt = Q v + K, each through the entry point a program calls, over the range of
sizes, numbers of states and precisions the benchmark configurations span.

A case is a dict with an "op":
  evolve   dense RK4: N (Hilbert-space dimension, M = N*N - 1 unknowns), R systems
           of B states, steps, fp32 (Q stored in FP32, opt-in)
  prepare  dense Q and K from H (N x N) and a Kossakowski matrix (M x M)
  sparse   CSR Q and K of the bosonic dimer, static or rocked
  csr      sparse RK4 of the dimer, static or under its square-wave drive
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1912_01491_amd as lb
from paper_1912_01491_amd import workloads as wl

DT = 1e-3
PERIOD = 2.0 * math.pi
PERIOD_STEPS = 20000     # steps per period of the rocked dimer
DRIVE = (-1.0, -1.5)     # its drive: eps = E + A on the first half period, E - A on the second
ON_CHIP = 256 << 20      # last-level cache: a matrix beyond it is read again by every stage


def listed():
    return [
        # a qutrit-to-octit toy model, one trajectory: launch and latency bound
        dict(name="evolve-n8-1", op="evolve", N=8, R=1, B=1, steps=1000, fp32=False),
        # the same with a block of initial states
        dict(name="evolve-n8-16", op="evolve", N=8, R=1, B=16, steps=1000, fp32=False),
        # one state of a served request, off the tuned sizes (M = 1368)
        dict(name="evolve-n37-1", op="evolve", N=37, R=1, B=1, steps=100, fp32=False),
        # one state, Q of 134 MB: the middle of the served sizes 16 .. 128
        dict(name="evolve-n64-1", op="evolve", N=64, R=1, B=1, steps=100, fp32=False),
        # realizations of the paper's largest dense model, 16 states each, batched
        dict(name="evolve-n200-16x2", op="evolve", N=200, R=2, B=16, steps=3, fp32=False),
        # 64 initial states on one system: bound by the matrix cores
        dict(name="evolve-n100-64", op="evolve", N=100, R=1, B=64, steps=10, fp32=False),
        # the FP32 opt-in at a ragged size and a partly filled block of states
        dict(name="evolve-n99-50-f32", op="evolve", N=99, R=1, B=50, steps=10, fp32=True),
        # dense preparation: the smallest, a single-node size and the paper's largest
        dict(name="prepare-n8", op="prepare", N=8),
        dict(name="prepare-n100", op="prepare", N=100),
        dict(name="prepare-n200", op="prepare", N=200),
        # sparse preparation of the static dimer at the paper's single-node size
        dict(name="sparse-n1000", op="sparse", N=1000, rocked=False),
        # a stretch of the rocked dimer's period across a switch of the drive
        dict(name="csr-n1000-rocked", op="csr", N=1000, rocked=True, B=1, steps=40),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "one", "block", "block", "block32", "prepare", "prepare", "sparse", "csr"])
    if kind == "prepare":
        return dict(op="prepare", N=_log(rng, 2, 200))
    if kind == "sparse":
        return dict(op="sparse", N=_log(rng, 16, 1000), rocked=rng.random() < 0.3)
    if kind == "csr":
        rocked = rng.random() < 0.5
        return dict(op="csr", N=_log(rng, 16, 1000), rocked=rocked, B=rng.choice([1, 1, 2, 5, 8]),
                    steps=_log(rng, 2, 20))
    R = 1
    if kind == "small":
        N = rng.randint(2, 15)
        B = rng.randint(1, max(1, min(16, 4096 // (N * N - 1))))
        R = rng.choice([1, 1, 4, 16])
        steps = min(_log(rng, 50, 1000), max(20, 1000 * 63 * 63 * 16 // (B * (N * N - 1) ** 2)))
        return dict(op="evolve", N=N, R=R, B=B, steps=steps, fp32=False)
    if kind == "one":
        N, B = _log(rng, 17, 160), 1
    else:
        N, B = _log(rng, 17, 200), _log(rng, 2, 64)
        if N <= 100:
            R = rng.choice([1, 1, 2, 3])
    M = N * N - 1
    steps = int(min(100, max(1, 5e10 // (32 * R * M * M * max(1, B / 16)))))
    return dict(op="evolve", N=N, R=R, B=B, steps=steps, fp32=kind == "block32")


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _states(N, B, g):
    """Coherence vectors of pure states: norm sqrt(1 - 1/N)."""
    V = torch.randn(B, N * N - 1, dtype=torch.float64, device="cuda", generator=g)
    return V * (math.sqrt(1.0 - 1.0 / N) / V.norm(dim=1, keepdim=True))


def _evolve_inputs(case, seed):
    """Q = -1 + noise, the shape of a random Lindbladian's spectrum (a disc around a
    common decay rate), with zero padding columns; K and pure-state vectors."""
    N, M = case["N"], case["N"] ** 2 - 1
    g = _gen(seed)
    ldq = lb.default_ldq(M)
    Qs, Ks, Vs = [], [], []
    for _ in range(case["R"]):
        Q = torch.zeros(M, ldq, dtype=torch.float32 if case["fp32"] else torch.float64, device="cuda")
        for i in range(0, M, 4096):
            n = min(M, i + 4096) - i
            Q[i:i + n, :M] = torch.randn(n, M, dtype=torch.float64, device="cuda", generator=g) * (0.5 / math.sqrt(M))
        Q.diagonal()[:] -= 1.0
        Qs.append(Q)
        Ks.append(torch.randn(M, dtype=torch.float64, device="cuda", generator=g) / M)
        Vs.append(_states(N, case["B"], g))
    return Qs, Ks, Vs


def _prepare_inputs(case, seed):
    """GUE H and a Wishart Kossakowski matrix N W W^H / Tr, exactly Hermitian, from W
    with up to 1024 columns (the full square W of the largest sizes takes minutes)."""
    N, M = case["N"], case["N"] ** 2 - 1
    g = _gen(seed)
    G = torch.randn(N, N, dtype=torch.complex128, device="cuda", generator=g)
    H = ((G + G.mH) / math.sqrt(2.0 * N)).contiguous()
    W = torch.randn(M, min(M, 1024), dtype=torch.complex128, device="cuda", generator=g)
    gamma = W @ W.mH.contiguous()
    n = 4096
    for i in range(0, M, n):
        for j in range(i, M, n):
            X = (gamma[i:i + n, j:j + n] + gamma[j:j + n, i:i + n].mH) * 0.5
            gamma[i:i + n, j:j + n] = X
            gamma[j:j + n, i:i + n] = X.mH
    gamma *= N / gamma.diagonal().real.sum()
    return H, gamma


def _dimer(case, seed):
    """The dimer's operators with parameters near the published ones: (H0, H1, rates, L)."""
    r = np.random.default_rng(seed)
    j, u = r.uniform(0.95, 1.05, 2)
    if case["rocked"]:
        H0, H1, rates, Ls = wl.rocked_dimer_model(case["N"], J=-j, U=2.2 * u)
        return H0, H1, rates, Ls[0]
    H0, rates, Ls = wl.dimer_model(case["N"], J=j, U=0.5 * u)
    return H0, None, rates, Ls[0]


def _csr(A):
    rowptr, col, val = wl.to_csr(A)
    return (torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda())


def _csr_schedule(case):
    """(dt, first step): a rocked run crosses the drive's switch half way."""
    if case["rocked"]:
        return PERIOD / PERIOD_STEPS, PERIOD_STEPS // 2 - case["steps"] // 2
    return DT, 0


def prepare(case, seed):
    st = dict(case=case, ctx=lb.Context(0))
    op = case["op"]
    if op == "evolve":
        Qs, Ks, V0 = _evolve_inputs(case, seed)
        st.update(Q=Qs, K=Ks, V0=V0, V=[v.clone() for v in V0])
    elif op == "prepare":
        H, gamma = _prepare_inputs(case, seed)
        M = gamma.shape[0]
        st.update(H=H, gamma=gamma,
                  Q=torch.empty(M, lb.default_ldq(M), dtype=torch.float64, device="cuda"),
                  K=torch.empty(M, dtype=torch.float64, device="cuda"))
    else:
        H0, H1, rates, L = _dimer(case, seed)
        st.update(H=_csr(H0), rates=rates, L=[_csr(L)])
        if op == "csr":
            N = case["N"]
            *Q0, K = lb.lindblad_prepare_sparse(st["ctx"], N, st["H"], rates, st["L"])
            st.update(Q0=tuple(Q0), K=K, V0=_states(N, case["B"], _gen(seed)))
            st["V"] = st["V0"].clone()
            if case["rocked"]:
                st["Q1"] = lb.lindblad_prepare_sparse(st["ctx"], N, _csr(H1), [], [])[:3]
    torch.cuda.synchronize()
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    op = case["op"]
    if op == "evolve":
        for v, v0 in zip(st["V"], st["V0"]):
            v.copy_(v0)
        prec = lb.FP32 if case["fp32"] else lb.FP64
        Q, Q32 = (None, st["Q"]) if case["fp32"] else (st["Q"], None)
        if case["R"] > 1:
            return lb.lindblad_propagate_batched(ctx, Q, st["K"], st["V"], DT, case["steps"], prec, Q32)
        return lb.lindblad_propagate(ctx, Q and Q[0], st["K"][0], st["V"][0], DT, case["steps"], prec, Q32 and Q32[0])
    if op == "prepare":
        return lb.lindblad_prepare(ctx, st["H"], st["gamma"], Q=st["Q"], K=st["K"])
    if op == "sparse":
        return lb.lindblad_prepare_sparse(ctx, case["N"], st["H"], st["rates"], st["L"])
    st["V"].copy_(st["V0"])
    dt, k0 = _csr_schedule(case)
    if case["rocked"]:
        return lb.lindblad_propagate_csr_drive(ctx, st["Q0"], st["Q1"], st["K"], st["V"], dt, case["steps"], 0.0,
                                               DRIVE[0], DRIVE[1], PERIOD, k0)
    return lb.lindblad_propagate_csr(ctx, *st["Q0"], st["K"], st["V"], dt, case["steps"])


def work(case):
    """Bytes and operations of one pass that no implementation avoids. A stage needs the
    whole result of the one before it, so a matrix too large for the chip is read by
    every stage; a smaller one is read once. A dense preparation reads the independent
    half of the Hermitian Kossakowski matrix and writes Q."""
    N, op = case["N"], case["op"]
    M = N * N - 1
    if op == "prepare":
        return dict(bytes=8.0 * M * M + 8.0 * M * M + 8.0 * M + 16.0 * N * N, flops=16.0 * M * M)
    stages = 4 * case.get("steps", 0)
    if op == "evolve":
        R, B = case["R"], case["B"]
        mat = (4.0 if case["fp32"] else 8.0) * M * M
        times = stages if R * mat > ON_CHIP else 1
        return dict(bytes=R * (mat * times + 8.0 * M * (1 + 2 * B)), flops=R * (2.0 * M * M + 9.0 * M) * B * stages)
    nnz = (20.0 if case["rocked"] and op == "csr" else 18.9 if case["rocked"] else 7.5) * N * N  # stored entries of Q
    if op == "sparse":
        return dict(bytes=16.0 * nnz + 16.0 * M, flops=8.0 * nnz)
    times = stages if 16.0 * nnz > ON_CHIP else 1
    return dict(bytes=16.0 * nnz * times + 8.0 * M * (2 + 2 * case["B"]),
                flops=(2.0 * nnz + 9.0 * M) * case["B"] * stages)


# ---------------------------------------------------------------------------
# the same results from plain torch in 64 bits
# ---------------------------------------------------------------------------

def _rk4(f, x, dt, steps):
    for k in range(steps):
        k1 = f(x, k)
        k2 = f(x + 0.5 * dt * k1, k)
        k3 = f(x + 0.5 * dt * k2, k)
        k4 = f(x + dt * k3, k)
        x = x + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
    return x


def _diag_weights(N):
    """W[l-1, x]: diagonal entry x of the generator D^l."""
    l = torch.arange(1, N, dtype=torch.float64, device="cuda")[:, None]
    x = torch.arange(N, dtype=torch.float64, device="cuda")[None, :]
    return torch.where(x < l, 1.0, torch.where(x == l, -l, 0.0)) / torch.sqrt(l * (l + 1.0))


def _to_basis(A, N, sign):
    """Rows (a, b) of A contracted with the generators: sum_ab (F_s)_ab A_ab, or with
    (F_s)_ab conjugated for sign = +1."""
    j, k = torch.triu_indices(N, N, 1, device="cuda")
    up, lo = A[j * N + k], A[k * N + j]
    d = torch.arange(N, device="cuda") * (N + 1)
    W = _diag_weights(N).to(A.dtype)
    r = math.sqrt(0.5)
    return torch.cat([(up + lo) * r, (up - lo) * (sign * 1j * r), W @ A[d]])


def _from_basis(A, N):
    """Rows s of A expanded over the matrix positions: sum_s (F_s)_ab A_s."""
    P = N * (N - 1) // 2
    j, k = torch.triu_indices(N, N, 1, device="cuda")
    d = torch.arange(N, device="cuda") * (N + 1)
    out = torch.empty((N * N,) + tuple(A.shape[1:]), dtype=A.dtype, device="cuda")
    r = math.sqrt(0.5)
    out[j * N + k] = (A[:P] - 1j * A[P:2 * P]) * r
    out[k * N + j] = (A[:P] + 1j * A[P:2 * P]) * r
    out[d] = _diag_weights(N).T.to(A.dtype).contiguous() @ A[2 * P:]
    return out


def _exact_prepare(case, seed):
    N = case["N"]
    H, gamma = _prepare_inputs(case, seed)
    C = _from_basis(_from_basis(gamma, N).T.contiguous(), N).T.reshape(N, N, N, N)  # [a, b, c, d]
    G = torch.einsum("bcab->ac", C)
    Z = -1j * H - 0.5 * G
    S = C.permute(0, 3, 1, 2).contiguous()  # L(X)_ad = sum_bc S[a, d, b, c] X_bc
    i = torch.arange(N, device="cuda")
    S[:, i, :, i] += Z
    S[i, :, i, :] += Z.conj()
    K = _to_basis(torch.einsum("adbb->ad", S).reshape(N * N, 1), N, +1)[:, 0].real / N
    Q = _to_basis(S.reshape(N * N, N * N), N, +1)
    Q = _to_basis(Q.T.contiguous(), N, -1).T.real
    M = N * N - 1
    out = torch.zeros(M, lb.default_ldq(M), dtype=torch.float64, device="cuda")
    out[:, :M] = Q
    return out, K.contiguous()


def _exact_csr(case, seed):
    """The density matrix itself integrated: RK4 commutes with the change of basis."""
    N = case["N"]
    H0, H1, rates, L = _dimer(case, seed)
    H0, L = torch.from_numpy(H0).cuda(), torch.from_numpy(L).cuda()
    H1 = torch.from_numpy(H1).cuda() if H1 is not None else None
    g, Ld = float(rates[0]), L.mH.contiguous()
    G = Ld @ L
    dt, k0 = _csr_schedule(case)
    out = []
    for v in _states(N, case["B"], _gen(seed)):
        X = _from_basis(v.to(torch.complex128)[:, None], N).reshape(N, N)
        X = X + torch.eye(N, dtype=X.dtype, device="cuda") / N

        def f(x, k):
            H = H0
            if H1 is not None:
                H = H0 + (DRIVE[0] + (DRIVE[1] if (k0 + k) % PERIOD_STEPS < PERIOD_STEPS // 2 else -DRIVE[1])) * H1
            Y = (-1j * H - 0.5 * g * G) @ x
            return Y + Y.mH + g * (L @ x @ Ld)

        X = _rk4(f, X, dt, case["steps"])
        out.append(_to_basis(X.reshape(N * N, 1), N, +1)[:, 0].real)
    return torch.stack(out)


def _exact_sparse_k(case, seed):
    """K_s = Tr(F_s L(1)) / N, L(1) = sum g (L L^H - L^H L)."""
    N = case["N"]
    _, _, rates, L = _dimer(case, seed)
    L = torch.from_numpy(L).cuda()
    Ld = L.mH.contiguous()
    return _to_basis((float(rates[0]) * (L @ Ld - Ld @ L)).reshape(N * N, 1), N, +1)[:, 0].real / N


def exact(case, seed):
    op = case["op"]
    if op == "prepare":
        return _exact_prepare(case, seed) if case["N"] <= 128 else None  # the N^2 x N^2 steps take too long beyond
    if op == "sparse":
        return None, None, None, _exact_sparse_k(case, seed)  # which entries are stored is the library's own choice
    if op == "csr":
        return _exact_csr(case, seed)
    M = case["N"] ** 2 - 1
    Qs, Ks, Vs = _evolve_inputs(case, seed)
    out = []
    for Q, K, V in zip(Qs, Ks, Vs):
        A = Q[:, :M].double() if case["fp32"] else Q[:, :M]
        out.append(_rk4(lambda x, k: A @ x + K[:, None], V.T.contiguous(), DT, case["steps"]).T.contiguous())
    return out if case["R"] > 1 else out[0]
