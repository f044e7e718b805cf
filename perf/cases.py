"""What a user of libqkrylov has it do, as cases for timing and comparison.

A case is one pass through a public entry point on inputs drawn from a seed:
Krylov steps with the survival probability read out after them (`step`),
error-controlled evolution (`evolve`), an ensemble advanced as one graph per
step (`ensemble`), the adjoint gradient (`gradient`) and the bare operator
(`apply`).  The chains are those of the tests, the workloads module and the
benchmark: quasiperiodic XXZ chains of 10 to 30 sites near half filling, open
and periodic, complex128 and complex64, one to 64 disorder phases.

`exact` evaluates the same quantities with torch alone in complex128: index
arrays of the hops, the Taylor series of exp(-iHt) in short substeps, and for
the gradient Gauss-Legendre quadrature of the time-reversed overlap.
"""
import math

import numpy as np
import torch

import paper_1704_02770_amd as qk
from workloads import BETA_GOLDEN

JXY, JZ = 1.0, 1.0
MODES = {"matfree": qk.QK_MATFREE, "csr": qk.QK_CSR}
DTYPES = {"c128": torch.complex128, "c64": torch.complex64}


def _dim(L, n_up):
    return math.comb(L, n_up)


def listed():
    return [
        # the smallest chains of a parity study: a step is all launches and latency
        dict(name="step_L12_open_c128", kind="step", L=12, n_up=6, pbc=False, h=1.5, batch=1, dtype="c128",
             mode="matfree", m=20, reorth=0, dt=0.05),
        # the sixteen-site ring stepped to t = 10
        dict(name="step_L16_ring_c128", kind="step", L=16, n_up=8, pbc=True, h=1.5, batch=1, dtype="c128",
             mode="matfree", m=30, reorth=0, dt=0.1),
        # evolution to a time at a tolerance, the way the paper's runs are done, on an odd chain
        dict(name="evolve_L19_open_c128", kind="evolve", L=19, n_up=9, pbc=False, h=1.0, batch=1, dtype="c128",
             mode="matfree", m=30, reorth=0, t=2.0, tol=1e-7),
        # the gradient workload: 50 steps of 0.1 forward and the sweep backward
        dict(name="gradient_L20_ring", kind="gradient", L=20, n_up=10, pbc=True, h=1.5, batch=1, dtype="c128",
             mode="matfree", m=30, reorth=0, t=5.0, steps=50),
        # the disorder ensemble: 64 phases of the 20-site ring with four single rings, one graph per step
        dict(name="ensemble_L20x64_c64", kind="ensemble", L=20, n_up=10, pbc=True, h=2.0, batch=64, dtype="c64",
             mode="matfree", m=30, reorth=0, dt=0.1, steps=2, also="16,18,20,22"),
        # a few phases at a filling off one half, locally reorthogonalised; a batch that is no power of two
        dict(name="step_L22_x3_open_c128", kind="step", L=22, n_up=10, pbc=False, h=3.0, batch=3, dtype="c128",
             mode="matfree", m=24, reorth=1, dt=0.1),
        # the mid-size open chain
        dict(name="step_L24_open_c128", kind="step", L=24, n_up=12, pbc=False, h=1.0, batch=1, dtype="c128",
             mode="matfree", m=30, reorth=0, dt=0.1),
        # eight phases of a ring, in single precision
        dict(name="step_L26_x8_ring_c64", kind="step", L=26, n_up=13, pbc=True, h=1.5, batch=8, dtype="c64",
             mode="matfree", m=30, reorth=0, dt=0.1),
        # the operator alone, as energies and moments need it, on an odd chain
        dict(name="apply_L27_open_c128", kind="apply", L=27, n_up=13, pbc=False, h=1.5, batch=1, dtype="c128",
             mode="matfree"),
        # the benchmark chain in both precisions
        dict(name="step_L28_ring_c128", kind="step", L=28, n_up=14, pbc=True, h=1.5, batch=1, dtype="c128",
             mode="matfree", m=30, reorth=0, dt=0.1),
        dict(name="step_L28_ring_c64", kind="step", L=28, n_up=14, pbc=True, h=1.5, batch=1, dtype="c64",
             mode="matfree", m=30, reorth=0, dt=0.1),
        # the large ring
        dict(name="step_L30_ring_c64", kind="step", L=30, n_up=15, pbc=True, h=2.0, batch=1, dtype="c64",
             mode="matfree", m=20, reorth=0, dt=0.05),
    ]


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["evolve", "ensemble", "gradient", "apply", "apply"])
    # chain lengths uniform, so dimensions are uniform in their logarithm
    L = rng.randint(10, 28 if kind in ("step", "apply") else 21)
    n_up = L // 2 - rng.choice([0, 0, 0, 1, 2])
    c = dict(kind=kind, L=L, n_up=n_up, pbc=rng.random() < 0.6, h=round(rng.uniform(0.0, 3.0), 3), batch=1,
             dtype=rng.choice(["c128", "c64"]), mode="matfree")
    if kind in ("step", "apply") and rng.random() < 0.4:
        c["batch"] = rng.choice([2, 3, 4, 6, 8, 16])
    if kind == "ensemble":
        c["batch"] = rng.choice([4, 8, 16, 32])
    while _dim(c["L"], c["n_up"]) * c["batch"] > 5e7:
        c["L"] -= 1
        c["n_up"] = c["L"] // 2
    if kind == "apply":
        if _dim(c["L"], c["n_up"]) * c["batch"] < 4e6 and rng.random() < 0.3:
            c["mode"] = "csr"
        return c
    c["m"] = rng.randint(12, 32)
    c["reorth"] = rng.choice([0, 0, 0, 1]) if kind != "gradient" else 0
    if kind == "step":
        if _dim(c["L"], c["n_up"]) * c["batch"] < 1e6 and rng.random() < 0.15:
            c["reorth"] = 2
        c["dt"] = round(rng.uniform(0.02, 0.004 * c["m"]), 4)
    elif kind == "evolve":
        c["t"] = round(rng.uniform(0.5, 3.0), 3)
        c["tol"] = rng.choice([1e-6, 1e-7, 1e-8])
    elif kind == "ensemble":
        c["dt"] = round(rng.uniform(0.02, 0.004 * c["m"]), 4)
        c["steps"] = rng.randint(1, 4)
        c["also"] = ",".join(str(rng.randint(10, 22)) for _ in range(rng.randint(1, 4)))
    else:
        c["dtype"] = "c128"
        c["steps"] = rng.randint(5, 40)
        c["t"] = round(c["steps"] * rng.uniform(0.02, 0.003 * c["m"]), 4)
    return c


# ------------------------------------------------------------------ inputs
def _fields(L, h, batch, seed):
    rng = np.random.default_rng(seed)
    return qk.qk_fields_quasiperiodic(L, h, BETA_GOLDEN, rng.uniform(0.0, 2.0 * math.pi, batch))


def _vector(D, batch, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randn((D, batch) if batch > 1 else (D,), generator=g, dtype=dtype, device="cuda")
    return v.div_(torch.linalg.vector_norm(v, dim=0))


def _chains(case):
    """(L, n_up, batch) of every workspace of a case."""
    out = [(case["L"], case["n_up"], case["batch"])]
    if case["kind"] == "ensemble":
        out += [(int(L), int(L) // 2, 1) for L in case["also"].split(",")]
    return out


def _neel_bits(L, n_up):
    return sum(1 << (2 * i) for i in range(n_up))


def prepare(case, seed):
    s = dict(case=case, items=[])
    for i, (L, n_up, B) in enumerate(_chains(case)):
        basis = qk.qk_basis_build(L, n_up)
        H = qk.qk_ham_create(basis, JXY, JZ, case["pbc"], _fields(L, case["h"], B, seed * 16 + i),
                             MODES[case["mode"]])
        it = dict(basis=basis, H=H, D=qk.qk_basis_dim(basis), r0=int(qk.qk_basis_rank(basis, [_neel_bits(L, n_up)])[0]))
        if case["kind"] != "apply":
            it["k"] = qk.qk_krylov_create(H, case["m"], DTYPES[case["dtype"]], case["reorth"])
        s["items"].append(it)
    one = s["items"][0]
    B, dtype = case["batch"], DTYPES[case["dtype"]]
    if case["kind"] == "ensemble":
        for it, (_, _, Bi) in zip(s["items"], _chains(case)):
            it["psi"] = torch.zeros((it["D"], Bi), dtype=dtype, device="cuda")
            it["psi"][it["r0"]] = 1.0
        s["out"] = torch.empty((case["steps"], sum(Bi for _, _, Bi in _chains(case))), dtype=torch.float64, device="cuda")
        s["batch"] = qk.qk_batch_create([it["k"] for it in s["items"]], [it["psi"] for it in s["items"]],
                                        [it["r0"] for it in s["items"]])
    elif case["kind"] == "apply":
        s["x"] = _vector(one["D"], B, dtype, seed)
        s["y"] = torch.empty_like(s["x"])
    elif case["kind"] != "gradient":
        s["psi"] = _vector(one["D"], B, dtype, seed)
        s["P"] = torch.empty(B, dtype=torch.float64, device="cuda")
    return s


def run(state):
    case, one = state["case"], state["items"][0]
    kind = case["kind"]
    if kind == "step":
        qk.qk_krylov_expm_step(one["k"], state["psi"], case["dt"])
        qk.qk_return_prob(one["basis"], state["psi"], r0=one["r0"], batch=case["batch"], out=state["P"])
        return {"psi": state["psi"], "P": state["P"]}
    if kind == "evolve":
        qk.qk_krylov_evolve(one["k"], state["psi"], case["t"], case["tol"])
        return {"psi": state["psi"]}
    if kind == "ensemble":
        P = qk.qk_batch_run(state["batch"], case["dt"], case["steps"], True, out=state["out"])
        return {"P": P, "psi": [it["psi"] for it in state["items"]]}
    if kind == "gradient":
        F, g = qk.qk_grad_return_prob(one["k"], one["r0"], case["t"], case["steps"])
        return {"F": F, "dF_dh": g}
    return {"y": qk.qk_ham_apply(one["H"], state["x"], state["y"])}


def work(case):
    """Vectors each read or written once per use that the method has: per
    Lanczos iteration two basis vectors in and one out, for the combination the
    basis once more; the gradient reads each step's basis and its mirror's."""
    s = 16 if case["dtype"] == "c128" else 8
    bytes_, flops = 0.0, 0.0
    for L, n_up, B in _chains(case):
        n = float(_dim(L, n_up)) * B
        hop = 2.0 * L * n_up * (L - n_up) / (L * (L - 1.0))   # mean number of hops of a row
        apply_flops = n * (2.0 * hop + 4.0)
        if case["kind"] == "apply":
            bytes_ += 2.0 * s * n
            flops += apply_flops
            continue
        m = case["m"]
        step_bytes = (3.0 * m + (m + 2.0)) * s * n
        step_flops = m * (apply_flops + 20.0 * n) + 8.0 * m * n
        if case["reorth"] == 2:
            step_bytes += m * (m - 1.0) / 2.0 * 2.0 * s * n
            step_flops += m * (m - 1.0) / 2.0 * 32.0 * n
        steps = case.get("steps", 1)
        if case["kind"] == "evolve":
            # about one step of the Krylov dimension's reach per unit of radius
            steps = max(1.0, math.ceil(case["t"] * 0.5 * L / m))
        bytes_ += steps * step_bytes
        flops += steps * step_flops
        if case["kind"] == "gradient":
            bytes_ += steps * 2.0 * m * s * n
            flops += steps * 8.0 * m * m * n
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------- the same in 64 bits
class _Exact:
    """H of one chain as index arrays, applied to complex128 vectors [D, B]."""

    def __init__(self, L, n_up, pbc, fields):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        sub = [[None] * (n_up + 1) for _ in range(L + 1)]
        for l in range(L + 1):
            for k in range(min(l, n_up) + 1):
                if l == 0:
                    sub[l][k] = torch.zeros(1, dtype=torch.int32, device=dev)
                    continue
                parts = [sub[l - 1][k]] if k <= l - 1 else []
                if k > 0:
                    parts.append(sub[l - 1][k - 1] | (1 << (l - 1)))
                sub[l][k] = torch.cat(parts)
            if l > 0:
                sub[l - 1] = None
        st = sub[L][n_up]
        del sub
        self.states, self.L = st, L
        f = torch.tensor(np.atleast_2d(fields), dtype=torch.float64, device=dev)   # [B, L]
        self.diag = torch.zeros((len(st), f.shape[0]), dtype=torch.float64, device=dev)
        for i in range(L):
            self.diag += (((st >> i) & 1).double() - 0.5)[:, None] * f[:, i]
        self.idx, self.anti = [], []
        for a, b in [(i, i + 1) for i in range(L - 1)] + ([(L - 1, 0)] if pbc else []):
            anti = ((st >> a) ^ (st >> b)) & 1
            self.diag += (JZ * (0.25 - 0.5 * anti.double()))[:, None]
            to = torch.where(anti.bool(), st ^ ((1 << a) | (1 << b)), st)
            self.idx.append(torch.searchsorted(st, to, out_int32=True))
            self.anti.append(anti.bool())
        self.radius = float(self.diag.abs().max()) + 0.5 * JXY * len(self.idx)

    def apply(self, x):
        y = torch.zeros_like(x)
        for idx, anti in zip(self.idx, self.anti):
            y += x.index_select(0, idx) * anti[:, None]
        return y.mul_(0.5 * JXY).add_(self.diag * x)

    def propagate(self, x, t):
        n = max(1, math.ceil(abs(t) * self.radius / 4.0))
        tau = t / n
        for _ in range(n):
            term, out = x, x.clone()
            for k in range(1, 60):
                term = self.apply(term).mul_(-1j * tau / k)
                out += term
                if (abs(tau) * self.radius / (k + 1)) < 0.5 and float(term.abs().max()) < 1e-18:
                    break
            x = out
        return x


def _exact_gradient(E, r0, T, steps):
    """F and dF/dh by dA/dh_i = -i int_0^T sum_r psi(T - s)[r] z_i(r) psi(s)[r] ds
    (H and the initial state are real), Gauss-Legendre panels symmetric about T/2."""
    panels = max(2, math.ceil(T / 0.4))
    x, w = np.polynomial.legendre.leggauss(16)
    nodes = np.concatenate([(p + 0.5 + 0.5 * x) * T / panels for p in range(panels)])
    weights = np.tile(0.5 * w * T / panels, panels)
    psi = torch.zeros((len(E.states), 1), dtype=torch.complex128, device=E.states.device)
    psi[r0] = 1.0
    at, kept = 0.0, []
    for s in nodes:
        psi = E.propagate(psi, float(s - at))
        at = float(s)
        kept.append(psi[:, 0])
    A = complex(E.propagate(psi, float(T - at))[r0, 0])
    acc = torch.zeros(len(E.states), dtype=torch.complex128, device=E.states.device)
    for k in range(len(nodes)):
        acc += weights[k] * kept[len(nodes) - 1 - k] * kept[k]
    z = [(acc * (((E.states >> i) & 1).double() - 0.5)).sum() for i in range(E.L)]
    dA = np.array([-1j * complex(v) for v in z])
    return abs(A) ** 2, 2.0 * (np.conj(A) * dA).real


def exact(case, seed):
    if _dim(case["L"], case["n_up"]) * case["batch"] > 9e7:
        return None   # over half a minute of Taylor terms
    results = []
    for i, (L, n_up, B) in enumerate(_chains(case)):
        E = _Exact(L, n_up, case["pbc"], _fields(L, case["h"], B, seed * 16 + i))
        D = len(E.states)
        r0 = int(torch.searchsorted(E.states, torch.tensor([_neel_bits(L, n_up)], dtype=torch.int32,
                                                           device=E.states.device))[0])
        if case["kind"] == "gradient":
            F, g = _exact_gradient(E, r0, case["t"], case["steps"])
            return {"F": float(F), "dF_dh": g}
        if case["kind"] == "ensemble":
            psi = torch.zeros((D, B), dtype=torch.complex128, device=E.states.device)
            psi[r0] = 1.0
            P = []
            for _ in range(case["steps"]):
                psi = E.propagate(psi, case["dt"])
                P.append(psi[r0].abs() ** 2)
            results.append((torch.stack(P), psi))
            continue
        v = _vector(D, B, DTYPES[case["dtype"]], seed)
        x = v.to(torch.complex128).reshape(D, B)
        if case["kind"] == "apply":
            return {"y": E.apply(x).reshape(v.shape)}
        psi = E.propagate(x, case["dt"] if case["kind"] == "step" else case["t"])
        if case["kind"] == "evolve":   # the limit that the tolerance approaches
            return {"psi": psi.reshape(v.shape)}
        return {"psi": psi.reshape(v.shape), "P": psi[r0].abs() ** 2}
    return {"P": torch.cat([p for p, _ in results], dim=1), "psi": [q for _, q in results]}
