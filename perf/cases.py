"""The work that a program has this framework do, as cases that can be timed
and compared.

Five kinds of call, each through a public entry point of the binding:

* ``projection``: G (Eq. 11) of a field that is already on the GPU, the call
  of a host code that runs its own solver around the projection;
* ``bridge``: P and K from a user material's Cauchy stress and Jaumann
  tangent (Appendix A), one call per material evaluation;
* ``forward`` and ``train``: the warm-start network, inference and one Adam
  step with its gradient;
* ``cycle``: one fully reversed load cycle of a polycrystal (Newton-CG
  increments, indicator fields reset at its start), alone or as a batch of
  RVEs of several edges.

FP64 cycles run at the tolerance of parity runs (1e-12) and return the
gradient, the stress and the accumulated slip in float64.  Mixed-precision
cycles return the gradient and the fatigue indicators (Eqs. 23-24) in
float32, as a program stores them, and run at 1e-7, a decade below the
default, so that the stored digits are those of the equilibrium and not of
the iteration's remainder.
"""

import math

import numpy as np
import torch

from paper_1806_10599_amd import binding, warmstart

DEV = "cuda"
# C11, C12, C44, gdot0, g, n, c, d (MPa, s), then E and nu of the particles
PARAMS = (168400.0, 121400.0, 75400.0, 1e-3, 50.0, 20.0, 20000.0, 200.0,
          1.2e6, 0.25)


def listed():
    return [
        # the smallest projection: launches and latency
        dict(name="projection_16", kind="projection", n=16,
             operator="discrete", L0=1.0, L1=1.0, L2=1.0),
        # an edge that is no power of two, a cell that is no cube
        dict(name="projection_40", kind="projection", n=40,
             operator="continuous", L0=1.0, L1=1.5, L2=0.7),
        # the largest edge the allocation-free call takes
        dict(name="projection_64", kind="projection", n=64,
             operator="discrete", L0=1.0, L1=1.0, L2=1.0),
        # a user material on a small odd number of integration points
        dict(name="bridge_4913", kind="bridge", points=17 ** 3),
        # a user material on a 128^3 RVE
        dict(name="bridge_128", kind="bridge", points=128 ** 3),
        # inference on the benchmark's 64^3 grid
        dict(name="forward_64", kind="forward", n=64, scale=0.5),
        # one training step on a sample of the 32^3 histories
        dict(name="train_32", kind="train", n=32, lr=3e-4),
        # the small oracle configuration: FP64 at the parity tolerance
        dict(name="cycle_16_fp64", kind="cycle", n=16, grains=8,
             particles=0.0, operator="continuous", precision="fp64", eps=0.01,
             increments=20, warm=0, forcing=0),
        # the paper's performance case at its smallest edge, extrapolated
        # start
        dict(name="cycle_32_mixed", kind="cycle", n=32, grains=235,
             particles=0.0, operator="discrete", precision="mixed", eps=0.003,
             increments=12, warm=3, forcing=2),
        # the benchmark's 64^3 configuration: particles, learned start
        dict(name="cycle_64_learned", kind="cycle", n=64, grains=200,
             particles=0.08, operator="discrete", precision="mixed",
             eps=0.003, increments=8, warm=2, forcing=2),
        # the 128^3 configuration, learned start
        dict(name="cycle_128_learned", kind="cycle", n=128, grains=1000,
             particles=0.05, operator="discrete", precision="mixed",
             eps=0.002, increments=6, warm=2, forcing=2),
        # statistical volume elements of mixed edges solved together
        dict(name="batch_mixed", kind="batch",
             edges="24,32,40,48,24,32,40,48,24,32,40,48", grains=60,
             operator="discrete", precision="mixed", eps=0.002, increments=6,
             forcing=2),
    ]


def draw(rng):
    kind = rng.choice(("projection", "bridge", "forward", "train", "cycle",
                       "cycle", "batch"))
    operator = rng.choice(("discrete", "continuous"))
    if kind == "projection":
        return dict(kind=kind, n=rng.choice((16, 24, 32, 40, 48, 64)),
                    operator=operator, L0=1.0,
                    L1=round(rng.uniform(0.5, 2.0), 3),
                    L2=round(rng.uniform(0.5, 2.0), 3))
    if kind == "bridge":
        lo, hi = math.log(1000), math.log(128 ** 3)
        return dict(kind=kind, points=int(math.exp(rng.uniform(lo, hi))) | 1)
    if kind == "forward":
        return dict(kind=kind, n=rng.choice((16, 32, 48, 64, 80, 96, 112, 128)),
                    scale=round(rng.uniform(0.2, 1.0), 3))
    if kind == "train":
        return dict(kind=kind, n=rng.choice((16, 32, 48, 64)),
                    lr=round(math.exp(rng.uniform(math.log(1e-5),
                                                  math.log(1e-3))), 7))
    if kind == "batch":
        edges = [rng.choice((16, 24, 32, 40, 48))
                 for _ in range(rng.randint(2, 12))]
        return dict(kind=kind, edges=",".join(map(str, edges)),
                    grains=rng.randint(20, 150), operator=operator,
                    precision="mixed", eps=round(rng.uniform(0.0015, 0.0025), 5),
                    increments=8, forcing=rng.choice((0, 1, 2)))
    fp64 = rng.random() < 0.4
    n = rng.choice((16, 24, 32) if fp64 else (16, 24, 32, 40, 48, 64, 96))
    return dict(kind=kind, n=n, grains=rng.randint(8, 4 * n),
                particles=round(rng.choice((0.0, rng.uniform(0.02, 0.1))), 4),
                operator=operator, precision="fp64" if fp64 else "mixed",
                eps=round(rng.uniform(0.0015, 0.0025), 5),
                increments=rng.choice((8, 12)) if n < 64 else 8,
                warm=rng.choice((0, 3) if n % 16 else (0, 2, 3)),
                forcing=0 if fp64 else rng.choice((0, 1, 2)))


# ------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _micro(n, grains, particles, seed):
    """Labels of a periodic Voronoi polycrystal with spherical particles of
    two to four voxels, orientations uniform on SO(3), and each label's law."""
    g = _gen(seed)
    seeds = torch.rand(grains, 3, generator=g, device=DEV, dtype=torch.float64)
    t = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
    phase = torch.empty(n, n * n, device=DEV, dtype=torch.int32)
    dist = []
    for axis in range(3):
        d = (t[:, None] - seeds[None, :, axis]).abs()
        dist.append(torch.minimum(d, 1.0 - d) ** 2)       # (n, grains)
    yz = (dist[1][:, None, :] + dist[2][None, :, :]).reshape(n * n, grains)
    for a in range(n):
        phase[a] = (yz + dist[0][a]).argmin(dim=1).int()
    phase = phase.reshape(n, n, n)
    quat = _randn(g, grains, 4)
    quat = (quat / quat.norm(dim=1, keepdim=True)).cpu().numpy()
    law = np.zeros(grains, dtype=np.int32)
    if particles > 0:
        rng = np.random.default_rng(seed)
        idx = torch.arange(n, device=DEV, dtype=torch.float64) + 0.5
        mask = torch.zeros(n, n, n, dtype=torch.bool, device=DEV)
        volume = 4.0 / 3.0 * math.pi * 30.0               # mean of r^3: 30
        for _ in range(max(1, round(particles * n ** 3 / volume))):
            c, r = rng.random(3) * n, rng.uniform(2.0, 4.0)
            d = []
            for axis in range(3):
                x = (idx - c[axis]).abs()
                d.append(torch.minimum(x, n - x) ** 2)
            mask |= (d[0][:, None, None] + d[1][None, :, None]
                     + d[2][None, None, :]) <= r * r
        phase = torch.where(mask, torch.full_like(phase, grains), phase)
        quat = np.concatenate([quat, [[1.0, 0.0, 0.0, 0.0]]])
        law = np.append(law, np.int32(1))
    return phase.reshape(-1), np.ascontiguousarray(quat), law


def _cycle_loads(eps, increments):
    """Macroscopic gradients of one fully reversed cycle (Eq. 27), period 4 s."""
    loads = []
    for k in range(1, increments + 1):
        s = k / increments
        e = eps * (4 * s if s <= 0.25 else 2 - 4 * s if s <= 0.75 else 4 * s - 4)
        f = 1.0 + e
        loads.append(np.diag([f, f ** -0.5, f ** -0.5]))
    return loads, 4.0 / increments


def _bridge_inputs(case, seed):
    """Gradients near the identity, a Cauchy stress of some hundred MPa and
    an elastic tangent with a spread of moduli (unsymmetric in its last
    tenth of a percent)."""
    g, m = _gen(seed), case["points"]
    eye = torch.eye(3, device=DEV, dtype=torch.float64).reshape(9, 1)
    F = eye + 0.05 * _randn(g, 9, m)
    sigma = 200.0 * _randn(g, 6, m)
    scale = 1.0 + 0.2 * _randn(g, 1, m).clamp(-3, 3)
    D = torch.zeros(6, 6, 1, device=DEV, dtype=torch.float64)
    D[:3, :3] = PARAMS[1]
    for i in range(6):
        D[i, i] = PARAMS[0] if i < 3 else PARAMS[2]
    ddsdde = D.reshape(36, 1) * scale + 75.0 * _randn(g, 36, m)
    return F.contiguous(), sigma.contiguous(), ddsdde.contiguous()


def _projection_inputs(case, seed):
    """A stress field: a mean of 100 MPa and fluctuations of 30 MPa."""
    g = _gen(seed)
    return (100.0 * _randn(g, 9, 1)
            + 30.0 * _randn(g, 9, case["n"] ** 3)).contiguous()


def _network_inputs(case, seed):
    """Features of the network's 40 channels (bf16, padded to 48), targets of
    its 9 (padded to 16) and random parameters."""
    g, N = _gen(seed), case["n"] ** 3
    X = torch.zeros(N, binding.WS_FEAT, device=DEV, dtype=torch.bfloat16)
    X[:, :40] = (case.get("scale", 0.5)
                 * torch.randn(N, 40, generator=g, device=DEV)).bfloat16()
    T = torch.zeros(N, binding.WS_OUT, device=DEV)
    T[:, :9] = 0.1 * torch.randn(N, 9, generator=g, device=DEV)
    return X, T, warmstart.init_params(seed % (1 << 31), out_scale=1.0)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "projection":
        field = _projection_inputs(case, seed)
        return dict(case=case, field=field, out=torch.empty_like(field),
                    L=(case["L0"], case["L1"], case["L2"]))
    if kind == "bridge":
        return dict(case=case, inputs=_bridge_inputs(case, seed))
    if kind in ("forward", "train"):
        X, T, params = _network_inputs(case, seed)
        net = binding.WarmStartNet()
        net.set_params(params)
        return dict(case=case, X=X.view(torch.int16), T=T, net=net,
                    out=torch.empty(case["n"] ** 3, binding.WS_OUT, device=DEV))
    loads, dt = _cycle_loads(case["eps"], case["increments"])
    params = np.array(PARAMS)
    tol = 1e-12 if case["precision"] == "fp64" else 1e-7
    options = dict(projection=case["operator"], precision=case["precision"],
                   newton_tol=tol, cg_tol=1e-4, cg_forcing=case["forcing"])
    if kind == "batch":
        edges = [int(e) for e in case["edges"].split(",")]
        rves = binding.BatchRve(edges, **options)
        for b, n in enumerate(edges):
            phase, quat, law = _micro(n, case["grains"], 0.0, seed + 1000 * b)
            rves.set_microstructure(b, phase.cpu().numpy(), quat, law, params)
        rves.tune_fft_schedules()
        return dict(case=case, rves=rves, loads=loads, dt=dt)
    n = case["n"]
    rve = binding.Rve(n, warm_start=case["warm"], **options)
    phase, quat, law = _micro(n, case["grains"], case["particles"], seed)
    rve.set_microstructure(phase.cpu().numpy(), quat, law, params)
    if case["warm"] == 2:
        net = binding.WarmStartNet()
        net.set_params(warmstart.trained_params())
        rve.attach_warm_start(net)
    rve.tune_fft_schedule()
    kept = (("P", 9) if case["precision"] == "fp64" else ("wcyc", 12))
    fields = {k: torch.empty(c, n ** 3, device=DEV, dtype=torch.float64)
              for k, c in (("F", 9), ("pcyc", 1), kept)}
    return dict(case=case, rve=rve, loads=loads, dt=dt, fields=fields)


# --------------------------------------------------------------------- runs

def _converged(info):
    if info["status"] != 0:
        raise RuntimeError("increment failed with status %d" % info["status"])
    return info["P_bar"]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "projection":
        return binding.apply_G_noalloc(case["n"], state["field"], state["out"],
                                       L=state["L"],
                                       projection=case["operator"])
    if kind == "bridge":
        return binding.umat_bridge(*state["inputs"])
    if kind == "forward":
        return state["net"].forward(state["X"], case["n"], out=state["out"])
    if kind == "train":
        loss, grad = state["net"].train_step(state["X"], state["T"], case["n"],
                                             case["lr"], want_grad=True)
        return dict(loss=np.float32(loss), grad=grad)
    kept = torch.float64 if case["precision"] == "fp64" else torch.float32
    if kind == "batch":
        rves = state["rves"]
        rves.reset_fips()
        P_bar = [[_converged(i) for i in rves.increment(F_bar, state["dt"])]
                 for F_bar in state["loads"]]
        out = [{k: torch.from_numpy(rves.field(b, k)).to(kept)
                for k in ("F", "wcyc")} for b in range(len(rves))]
        return dict(fields=out, P_bar=torch.from_numpy(np.array(P_bar)).to(kept))
    rve = state["rve"]
    rve.reset_fips()
    P_bar = [_converged(rve.increment(F_bar, state["dt"]))
             for F_bar in state["loads"]]
    out = {k: rve.field_device(k, t).to(kept)
           for k, t in state["fields"].items()}
    out["P_bar"] = torch.from_numpy(np.array(P_bar)).to(kept)
    return out


# --------------------------------------------------------------------- work

def work(case):
    """The least a pass moves and computes.  A cycle is charged, per
    increment, with the committed state in and out, two Newton corrections'
    return mappings and tangents, and twenty CG products each."""
    kind = case["kind"]
    if kind == "projection":
        N = case["n"] ** 3
        fft = 2 * 9 * 2.5 * N * math.log2(N)
        return dict(bytes=2 * 72 * N, flops=fft + 9 * 4 * N)
    if kind == "bridge":
        return dict(bytes=1128 * case["points"], flops=1500 * case["points"])
    if kind in ("forward", "train"):
        N = case["n"] ** 3
        macs = 27 * (40 * 32 + 2 * 32 * 32 + 32 * 9)
        if kind == "forward":
            return dict(bytes=N * (96 + 64), flops=2 * macs * N)
        last = 27 * (2 * 32 * 32 + 32 * 9)
        return dict(bytes=N * (96 + 64) + 4 * 4 * warmstart.param_count(),
                    flops=2 * (2 * macs + last) * N)
    if kind == "batch":
        N = sum(int(e) ** 3 for e in case["edges"].split(","))
        big = max(int(e) for e in case["edges"].split(","))
    else:
        N, big = case["n"] ** 3, case["n"]
    matvec = 162 + 2 * 9 * 2.5 * 3 * math.log2(big)
    point = 2 * (4 * 3600 + 9000)
    state = 8 * 2 * (9 + 9 + 12 + 12 + 1 + 1 + 12)
    return dict(bytes=case["increments"] * N * (state + 72),
                flops=case["increments"] * N * (point + 40 * matvec))


# -------------------------------------------------- the same in plain torch

def _shape9(v):
    return v.reshape(3, 3, -1)


def _mm(A, B):
    """(3, 3, m) products, voxel by voxel."""
    return (A[:, :, None] * B[None]).sum(1)


def _mmt(A, B):
    """A B^T."""
    return (A[:, None] * B[None]).sum(2)


def _tmm(A, B):
    """A^T B."""
    return (A[:, :, None] * B[:, None]).sum(0)


def _sym(A):
    return 0.5 * (A + A.transpose(-3, -2))


def _wave_vectors(n, operator, L, device):
    k = torch.fft.fftfreq(n, 1.0 / n, device=device, dtype=torch.float64)
    q = 2 * math.pi * k / n
    nyquist = k.abs() == n // 2
    q = torch.where(nyquist, torch.zeros_like(q), q)
    v = [(q if operator == "continuous" else torch.tan(q / 2)) * (n / Ld)
         for Ld in L]
    zero = (nyquist[:, None, None] | nyquist[None, :, None]
            | nyquist[None, None, :])
    zero[0, 0, 0] = True
    v = [v[0][:, None, None], v[1][None, :, None], v[2][None, None, :]]
    h = n // 2 + 1
    v[2] = v[2][..., :h]
    zero = zero[..., :h]
    norm = v[0] ** 2 + v[1] ** 2 + v[2] ** 2
    inv = torch.where(zero, torch.zeros_like(norm), 1.0 / norm)
    return v, inv


def _project(A, n, v, inv):
    """Eqs. 11, 19 and 21: B_ij = v_j (A_il v_l) / |v|^2 in Fourier space."""
    Ah = torch.fft.rfftn(A.reshape(3, 3, n, n, n), dim=(2, 3, 4))
    s = (Ah[:, 0] * v[0] + Ah[:, 1] * v[1] + Ah[:, 2] * v[2]) * inv
    B = torch.stack([s * v[0], s * v[1], s * v[2]], dim=1)
    return torch.fft.irfftn(B, s=(n, n, n), dim=(2, 3, 4)).reshape(A.shape)


def _exact_bridge(case, seed):
    """P = J sigma F^-T and Eq. A.16, components in the order 11, 22, 33, 12,
    13, 23."""
    F, sigma, D = _bridge_inputs(case, seed)
    F = _shape9(F)
    pair = [[0, 3, 4], [3, 1, 5], [4, 5, 2]]
    cof = torch.stack([torch.stack([
        F[(i + 1) % 3, (j + 1) % 3] * F[(i + 2) % 3, (j + 2) % 3]
        - F[(i + 1) % 3, (j + 2) % 3] * F[(i + 2) % 3, (j + 1) % 3]
        for j in range(3)]) for i in range(3)])
    J = (F[0] * cof[0]).sum(0)
    Fi = cof.transpose(0, 1) / J
    tau = torch.stack([torch.stack([J * sigma[pair[i][j]] for j in range(3)])
                       for i in range(3)])
    P = _mmt(tau, Fi)
    Fit = _mm(Fi, tau)                                   # F^-1 tau
    K = torch.empty(81, J.numel(), device=DEV, dtype=torch.float64)
    for i in range(3):
        for k in range(3):
            for l in range(3):
                row = []                                 # dtau_ip / dF_kl
                for p in range(3):
                    d = sum(J * D[6 * pair[i][p] + pair[k][m]] * Fi[l, m]
                            for m in range(3))
                    d = d - 0.5 * Fi[l, i] * tau[k, p] - 0.5 * Fi[l, p] * tau[i, k]
                    if i == k:
                        d = d + 0.5 * Fit[l, p]
                    if p == k:
                        d = d + 0.5 * Fit[l, i]
                    row.append(d)
                for j in range(3):
                    K[9 * (3 * i + j) + 3 * k + l] = (
                        sum(row[p] * Fi[j, p] for p in range(3))
                        - Fit[l, i] * Fi[j, k])
    return P.reshape(9, -1), K


def _conv(X, W, b, n):
    """Periodic 3x3x3 convolution of X (N, ci) with W (27, ci, co)."""
    grid = X.reshape(n, n, n, -1)
    Y = b.expand(n ** 3, -1)
    for t in range(27):
        d = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
        S = torch.roll(grid, (-d[0], -d[1], -d[2]), (0, 1, 2))
        Y = Y + S.reshape(n ** 3, -1) @ W[t]
    return Y


def _exact_network(case, seed):
    X, T, params = _network_inputs(case, seed)
    n, h, o = case["n"], X[:, :40].double(), 0
    p = torch.from_numpy(params).to(DEV).double()
    p.requires_grad_(case["kind"] == "train")
    for k, (ci, co) in enumerate(warmstart.LAYERS):
        W = p[o:o + 27 * ci * co].reshape(27, ci, co)
        o += 27 * ci * co
        h = _conv(h, W, p[o:o + co], n)
        o += co
        h = h.relu() if k < 3 else h
    if case["kind"] == "forward":
        out = torch.zeros(n ** 3, binding.WS_OUT, device=DEV,
                          dtype=torch.float64)
        out[:, :9] = h
        return out
    loss = (h - T[:, :9].double()).square().mean()
    loss.backward()
    return dict(loss=float(loss), grad=p.grad)


class _Crystal:
    """The polycrystal of a cycle in 64 bits: the FCC power law with
    Armstrong-Frederick back stress, backward Euler, and St-Venant-Kirchhoff
    particles, on (components, voxels) arrays."""

    def __init__(self, phase, quat, law):
        q = torch.from_numpy(quat).to(DEV)
        w, x, y, z = (q / q.norm(dim=1, keepdim=True)).T
        R = torch.stack([
            torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z),
                         2 * (x * z + w * y)]),
            torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z),
                         2 * (y * z - w * x)]),
            torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x),
                         1 - 2 * (x * x + y * y)])])     # (3, 3, labels)
        normals = ((1, 1, 1), (-1, 1, 1), (1, -1, 1), (1, 1, -1))
        along = ((1, -1, 0), (1, 0, -1), (0, 1, -1), (1, 1, 0), (1, 0, 1),
                 (0, 1, 1))
        pairs = [(s, m) for m in normals for s in along
                 if sum(a * b for a, b in zip(s, m)) == 0]
        s, m = (torch.tensor(v, device=DEV, dtype=torch.float64)
                for v in zip(*pairs))
        s, m = s / math.sqrt(2), m / math.sqrt(3)
        s = torch.tensordot(s, R, dims=([1], [1]))       # (12, 3, labels)
        m = torch.tensordot(m, R, dims=([1], [1]))
        S0 = s[:, :, None] * m[:, None]
        c11, c12, c44 = PARAMS[:3]
        eye = torch.eye(3, device=DEV, dtype=torch.float64)
        cube = torch.zeros(3, 3, 3, 3, device=DEV, dtype=torch.float64)
        cube += c12 * eye[:, :, None, None] * eye[None, None]
        cube += c44 * (eye[:, None, :, None] * eye[None, :, None, :]
                       + eye[:, None, None, :] * eye[None, :, :, None])
        for e in range(3):
            cube[e, e, e, e] += c11 - c12 - 2 * c44
        C = cube[..., None].expand(3, 3, 3, 3, R.shape[2])
        for axis in range(4):                            # rotate every index
            C = (C.movedim(axis, 0)[None] * R.reshape(3, 3, 1, 1, 1, -1)
                 ).sum(1).movedim(0, axis)
        self.cp = torch.from_numpy(law).to(DEV)[phase.long()] == 0
        own = phase[self.cp].long()
        self.S0, self.C = S0[..., own], C[..., own].reshape(9, 9, -1)
        CS = (C.reshape(9, 9, -1)[None] * S0.reshape(12, 1, 9, -1)).sum(2)
        self.CS0 = CS[..., own].reshape(12, 3, 3, -1)    # C : S0_a
        self.law = law
        self.N = phase.numel()
        m = int(self.cp.sum())
        self.Fpi = torch.eye(3, device=DEV, dtype=torch.float64)[
            :, :, None].expand(3, 3, m).contiguous()
        self.chi = torch.zeros(12, m, device=DEV, dtype=torch.float64)
        E, nu = PARAMS[8:]
        self.lam, self.mu = E * nu / ((1 + nu) * (1 - 2 * nu)), E / (2 + 2 * nu)

    def _stress(self, Fes, dg, of):
        A = -(dg[:, None, None] * self.S0[..., of]).sum(0)
        A = A + torch.eye(3, device=DEV, dtype=torch.float64)[:, :, None]
        Fe = _mm(Fes, A)
        E = 0.5 * (_tmm(Fe, Fe)
                   - torch.eye(3, device=DEV, dtype=torch.float64)[:, :, None])
        S = (self.C[..., of] * E.reshape(1, 9, -1)).sum(1).reshape(3, 3, -1)
        return A, Fe, S

    def _local(self, Fes, chi0, dg, dt, of):
        """Residual asinh(dg/a) - asinh(|x|^n sign x) and its Jacobian."""
        gdot0, g, n, c, d = PARAMS[3:8]
        a = dt * gdot0
        _, Fe, S = self._stress(Fes, dg, of)
        tau = (S * self.S0[..., of]).sum((1, 2))
        den = 1 + d * dg.abs()
        chi = (chi0 + c * dg) / den
        x = (tau - chi) / g
        ax = x.abs().clamp_min(1e-300)
        ln = n * ax.log()
        small = torch.exp(-ln.abs())
        big = ln > 0
        root = (1 + small * small).sqrt()
        val = torch.where(big, ln + torch.log1p(root),
                          torch.asinh(small))
        der = torch.where(big, n / (ax * root), n * small / (ax * root))
        R = torch.asinh(dg / a) - x.sign() * val
        Q = _tmm(Fe, Fes)
        V = _sym((Q[None, :, :, None] * self.S0[..., of][:, None]).sum(2))
        dx = -(self.CS0[..., of].reshape(12, 1, 9, -1)
               * V.reshape(1, 12, 9, -1)).sum(2)
        dchi = (c - d * dg.sign() * chi) / den
        J = -(der / g)[:, None] * dx
        k = torch.arange(12, device=DEV)
        J[k, k] += 1.0 / (a * a + dg * dg).sqrt() + der / g * dchi
        return R, J, der / g, V

    @staticmethod
    def _eliminate(J, B):
        """J^-1 B for (12, 12, m) and (12, r, m); J has a dominant positive
        part, no pivoting."""
        J, B = J.clone(), B.clone()
        for k in range(12):
            f = J[k + 1:, k] / J[k, k]
            J[k + 1:] -= f[:, None] * J[k][None]
            B[k + 1:] -= f[:, None] * B[k][None]
        for k in range(11, -1, -1):
            B[k] = (B[k] - (J[k, k + 1:][:, None] * B[k + 1:]).sum(0)) / J[k, k]
        return B

    def _slips(self, Fes, dg, dt):
        """Damped Newton of the twelve slips, voxels leaving as they end."""
        dg = dg.clone()
        of = torch.arange(dg.shape[1], device=DEV)
        for _ in range(60):
            F, chi0, at = Fes[..., of], self.chi[:, of], dg[:, of]
            R, J, _, _ = self._local(F, chi0, at, dt, of)
            step = -self._eliminate(J, R[:, None])[:, 0]
            merit = R.square().sum(0)
            lam = torch.ones_like(merit)
            for _ in range(30):
                Rt = self._local(F, chi0, at + lam * step, dt, of)[0]
                bad = ~(Rt.square().sum(0) <= (1 - 2e-4 * lam) * merit)
                bad &= R.abs().amax(0) > 1e-11
                if not bool(bad.any()):
                    break
                lam = torch.where(bad, 0.5 * lam, lam)
            dg[:, of] = at + lam * step
            size = step.abs().amax(0)
            going = ~(size <= 1e-18 + 1e-13 * dg[:, of].abs().amax(0))
            going &= ~((R.abs().amax(0) <= 1e-13) & (lam == 1))
            of = of[going]
            if not of.numel():
                break
        return dg

    def update(self, F, dg0, dt, tangent):
        """P (9, N), dP/dF (81, N) and the trial state at the gradient F."""
        P = torch.empty(9, self.N, device=DEV, dtype=torch.float64)
        K = torch.empty(81, self.N, device=DEV, dtype=torch.float64)
        eye = torch.eye(3, device=DEV, dtype=torch.float64)
        Fc = _shape9(F[:, self.cp])
        Fes = _mm(Fc, self.Fpi)
        dg = self._slips(Fes, dg0, dt)
        every = slice(None)
        A, Fe, Sc = self._stress(Fes, dg, every)
        Fpi = _mm(self.Fpi, A)
        FeS = _mm(Fe, Sc)
        P[:, self.cp] = _mmt(FeS, Fpi).reshape(9, -1)
        if tangent:
            _, J, h, V = self._local(Fes, self.chi, dg, dt, every)
            # dR/dF_kl = -h (Fe C:S0_a Fp^-T)_kl at fixed slips
            b = torch.stack([_mmt(_mm(Fe, self.CS0[a]), Fpi)
                             for a in range(12)])
            D = self._eliminate(J, (h[:, None] * b.reshape(12, 9, -1)))
            Kc = torch.zeros(3, 3, 9, Fe.shape[-1], device=DEV,
                             dtype=torch.float64)
            for k in range(3):
                for l in range(3):
                    g = D[:, 3 * k + l]                  # d dg / d F_kl
                    dFpi = -_mm(self.Fpi, (g[:, None, None] * self.S0).sum(0))
                    dFe = _mm(Fc, dFpi)
                    dFe[k] += Fpi[l]
                    dE = _sym(_tmm(Fe, dFe))
                    dS = (self.C * dE.reshape(1, 9, -1)).sum(1)
                    dS = dS.reshape(3, 3, -1)
                    Kc[:, :, 3 * k + l] = (
                        _mmt(_mm(dFe, Sc) + _mm(Fe, dS), Fpi)
                        + _mmt(FeS, dFpi))
            K[:, self.cp] = Kc.reshape(81, -1)
        el = ~self.cp
        if bool(el.any()):
            Fp = _shape9(F[:, el])
            E = 0.5 * (_tmm(Fp, Fp) - eye[:, :, None])
            trE = E[0, 0] + E[1, 1] + E[2, 2]
            S = self.lam * trE * eye[:, :, None] + 2 * self.mu * E
            P[:, el] = _mm(Fp, S).reshape(9, -1)
            B = _mmt(Fp, Fp)
            Kc = (self.lam * Fp[:, :, None, None] * Fp[None, None]
                  + self.mu * Fp[:, None, None]
                  * Fp.transpose(0, 1)[None, :, :, None])
            for i in range(3):
                for j in range(3):
                    Kc[i, j, i] += S[:, j]
                    for k in range(3):
                        Kc[i, j, k, j] += self.mu * B[i, k]
            K[:, el] = Kc.reshape(81, -1)
        return P, K, (Fpi, dg, Sc)

    def commit(self, trial):
        Fpi, dg, S = trial
        c, d = PARAMS[6:8]
        self.Fpi = Fpi
        self.chi = (self.chi + c * dg) / (1 + d * dg.abs())
        slip = (dg[:, None, None] * self.S0).sum(0)
        pcyc = torch.zeros(1, self.N, device=DEV, dtype=torch.float64)
        pcyc[0, self.cp] = (2.0 / 3.0 * slip.square().sum((0, 1))).sqrt()
        wcyc = torch.zeros(12, self.N, device=DEV, dtype=torch.float64)
        wcyc[:, self.cp] = (S * self.S0).sum((1, 2)) * dg
        return pcyc, wcyc


def _exact_cycle(case, n, phase, quat, law):
    """Newton-CG (Eqs. 12-16) of one cycle to a residual of 1e-11; None where
    it is not reached."""
    rve = _Crystal(phase, quat, law)
    v, inv = _wave_vectors(n, case["operator"], (1.0, 1.0, 1.0), DEV)
    loads, dt = _cycle_loads(case["eps"], case["increments"])
    eye = torch.eye(3, device=DEV, dtype=torch.float64).reshape(9, 1)
    F, before = eye.expand(9, n ** 3).clone(), np.eye(3)
    m = int(rve.cp.sum())
    pcyc, wcyc, P_bar = 0.0, 0.0, []
    dg = torch.zeros(12, m, device=DEV, dtype=torch.float64)
    for F_bar in loads:
        F = F + torch.from_numpy((F_bar - before).reshape(9, 1)).to(DEV)
        before = F_bar
        for _ in range(25):
            P, K, trial = rve.update(F, dg, dt, True)
            dg = trial[1]
            r = -_project(P, n, v, inv)
            rr = (r * r).sum()
            if float(rr.sqrt()) <= 1e-11 * float(P.norm()):
                break
            K = K.reshape(9, 9, -1)
            x, p, stop = torch.zeros_like(r), r.clone(), 1e-10 * float(rr)
            for k in range(2000):
                Ap = _project((K * p[None]).sum(1), n, v, inv)
                alpha = rr / (p * Ap).sum()
                x += alpha * p
                r -= alpha * Ap
                new = (r * r).sum()
                if k % 4 == 3 and float(new) <= stop:
                    break
                p = r + (new / rr) * p
                rr = new
            F = F + x
        else:
            return None
        slip, energy = rve.commit(trial)
        pcyc, wcyc = pcyc + slip, wcyc + energy
        P_bar.append(P.mean(1).reshape(3, 3).cpu())
    return dict(F=F, P=P, pcyc=pcyc, wcyc=wcyc), torch.stack(P_bar)


def exact(case, seed):
    kind = case["kind"]
    if kind == "projection":
        field = _projection_inputs(case, seed)
        v, inv = _wave_vectors(case["n"], case["operator"],
                               (case["L0"], case["L1"], case["L2"]), DEV)
        return _project(field, case["n"], v, inv)
    if kind == "bridge":
        return _exact_bridge(case, seed)
    if kind in ("forward", "train"):
        return _exact_network(case, seed)
    if kind == "batch":
        edges = [int(e) for e in case["edges"].split(",")]
        if sum(e ** 3 for e in edges) > 500000:
            return None                       # minutes in plain torch
        fields, P_bar = [], []
        for b, n in enumerate(edges):
            solved = _exact_cycle(case, n, *_micro(n, case["grains"], 0.0,
                                                   seed + 1000 * b))
            if solved is None:
                return None
            out, P = solved
            fields.append(dict(F=out["F"], wcyc=out["wcyc"]))
            P_bar.append(P)
        return dict(fields=fields, P_bar=torch.stack(P_bar, dim=1))
    n = case["n"]
    if n > 64:
        return None                           # minutes in plain torch
    solved = _exact_cycle(case, n, *_micro(n, case["grains"],
                                           case["particles"], seed))
    if solved is None:
        return None
    out, P_bar = solved
    del out["wcyc" if case["precision"] == "fp64" else "P"]
    return dict(out, P_bar=P_bar)
