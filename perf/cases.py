"""The work this library does for its users, as cases with inputs, one pass each, and FP64 values.

A pass is one call of a public entry point:
  saliency   `Saliency.saliency(V)`: the map of a resident volume (FP32 or a 16-bit form, windows at
             every voxel or on a stride lattice, axis or oriented comparisons);
  maps       `Saliency.saliency_maps(V)`: the same with every intermediate map returned;
  box        `Saliency.raw_box`: the raw maps of one region of interest of a resident volume;
  stream     `stream.plain_streamed`: a volume in pinned host memory, slab by slab;
  surrogate  `surrogate.infer_with_fallback`: the trained network, its tile checks and Eq. (6);
  train      `Net.train_step`: one optimiser step of the network on a batch of 16^3 windows.

Volumes are layered reflectivity with a regional dip and faults, convolved with a Ricker
wavelet, with a chaotic body and white noise (the character of the seeded survey volumes of
`synth.py`), made on the GPU from the seed.
"""
import math

import numpy as np
import torch

from paper_1901_11095_amd import sal, stream, surrogate

DEV = "cuda"

RAYS = {
    "axis": sal.RAYS_AXIS,  # the default: every map along its own axis
    # the oriented set of the paper's Fig. 3: +-t and the t-x diagonals for S_t
    "fig3": (sal.RAY_PT | sal.RAY_MT | sal.RAY_DIAG_TX, sal.RAYS_AXIS[1], sal.RAYS_AXIS[2]),
    "all_axis": sal.RAYS_ALL,  # the six axis rays for every map
}
PRECISIONS = {"fp32": sal.FP32, "bf16": sal.BF16, "bf16_split": sal.BF16_SPLIT, "fp16": sal.FP16,
              "fp16_split": sal.FP16_SPLIT}


def _vol(op, L, n, stride=1, precision="fp32", rays="axis"):
    return {"op": op, "L": L, "n0": n[0], "n1": n[1], "n2": n[2], "stride": stride, "precision": precision,
            "rays": rays}


def listed():
    return [
        # an interactive probe of a few traces: launches and latency
        dict(_vol("maps", 8, (32, 32, 32)), name="probe_cube8_32"),
        # one small block at the survey cube (the parity volume's size)
        dict(_vol("saliency", 16, (64, 64, 64)), name="block_cube16_64"),
        # a survey block at the headline cube and precision
        dict(_vol("saliency", 16, (512, 512, 512)), name="survey_cube16_512"),
        # the same method at the finer cube, the second benchmark volume
        dict(_vol("saliency", 8, (256, 512, 512)), name="survey_cube8"),
        # the paper's own 5 x 5 x 5 cube on that volume
        dict(_vol("saliency", 5, (256, 512, 512)), name="survey_cube5"),
        # a cube side chosen for the resolution, on a cut-out with odd sides
        dict(_vol("saliency", 12, (131, 187, 253)), name="cutout_cube12"),
        # a quick look: windows on a stride lattice
        dict(_vol("saliency", 16, (512, 512, 512), stride=4), name="quicklook_cube16_s4"),
        # dipping structure: the paper's t-x diagonal comparisons
        dict(_vol("saliency", 8, (201, 255, 319), rays="fig3"), name="oriented_cube8"),
        # the 16-bit split form
        dict(_vol("saliency", 16, (128, 256, 256), precision="bf16_split"), name="split16_cube16"),
        # a volume kept on the host
        dict(_vol("stream", 16, (192, 256, 320)), name="streamed_cube16", slab=64),
        # the learned surrogate with its checks
        dict(_vol("surrogate", 16, (256, 256, 256)), name="surrogate_256"),
        # one training step of the surrogate (batch of the training configuration)
        {"name": "train_step_64", "op": "train", "batch": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["saliency"] * 9 + ["maps", "box", "box", "stream", "surrogate", "train"])
    if op == "train":
        return {"op": "train", "batch": _log(rng, 4, 128)}
    if op == "surrogate":
        return _vol("surrogate", 16, [rng.randint(96, 256) for _ in range(3)])
    L = rng.choice([16, 16, 8, 8, 5, rng.randint(2, 20), rng.randint(9, 20)])
    stride, precision, rays = 1, "fp32", "axis"
    if op == "saliency":
        kind = rng.choice(["plain", "plain", "stride", "precision", "rays"])
        if kind == "stride":
            wide = [s for s in range(2, L) if 2 * s < L] + [L]
            stride = rng.choice(wide)
        elif kind == "precision":
            L = rng.choice([8, 16])
            precision = rng.choice(["bf16", "bf16_split", "fp16", "fp16_split"])
        elif kind == "rays":
            rays = rng.choice(["fig3", "all_axis"])
    # voxels of the volume, over the logarithm: a few traces to a survey block
    most = 3.2e7 if L in (8, 16) or L <= 7 else 6e6
    if op in ("stream", "box"):
        most = 1.6e7 if L <= 8 or L == 16 else 4e6
    n = math.exp(rng.uniform(math.log(4e4), math.log(most)))
    side = n ** (1 / 3)
    a, b = math.exp(rng.uniform(-0.5, 0.5)), math.exp(rng.uniform(-0.5, 0.5))
    dims = [max(24, int(side * a)), max(24, int(side * b)), max(24, int(side / (a * b)))]
    c = _vol(op, L, dims, stride, precision, rays)
    if op == "stream":
        c["slab"] = rng.choice([32, 64, 128])
    if op == "box":
        for k in range(3):
            d = rng.randint(max(8, dims[k] // 4), dims[k])
            c["b%d" % k], c["d%d" % k] = rng.randint(0, dims[k] - d), d
    return c


# --------------------------------------------------------------------------- inputs

def _volume(n, seed):
    """Layered, dipping, faulted reflectivity convolved with a Ricker wavelet, plus noise."""
    n0, n1, n2 = n
    r = np.random.default_rng([seed, n0, n1, n2])
    over = 4                                     # trace samples per row
    span = n0 + n1 + n2 + 256                    # rows the shifts can reach
    refl = np.zeros(span * over)
    pos = np.cumsum(1 + r.geometric(0.2, size=span)) * over
    pos = pos[pos < len(refl)]
    refl[pos] = r.normal(0.0, 0.1, size=len(pos))
    tt = np.arange(-32 * over, 32 * over + 1) / over * 0.004
    u = (math.pi * 30.0 * tt) ** 2
    trace = np.convolve(refl, (1 - 2 * u) * np.exp(-u), mode="same")
    trace /= trace.std()
    trace = torch.from_numpy(trace.astype(np.float32)).to(DEV)
    t = torch.arange(n0, device=DEV, dtype=torch.float32).view(-1, 1, 1)
    x = torch.arange(n1, device=DEV, dtype=torch.float32).view(1, -1, 1)
    y = torch.arange(n2, device=DEV, dtype=torch.float32).view(1, 1, -1)
    dip = r.uniform(-0.09, 0.09, size=2)
    row = t + (float(dip[0]) * x + float(dip[1]) * y)
    for _ in range(3):
        th, off = r.uniform(0, math.pi), r.uniform(0.2, 0.8)
        side = (x * math.cos(th) + y * math.sin(th) + 0.4 * t) > off * (n1 + n2) / 2
        row = row + float(r.uniform(4, 12)) * side
    idx = ((row + 96.0 + 0.1 * (n1 + n2)) * over).to(torch.int64).clamp_(0, trace.numel() - 1)
    del row
    V = trace[idx]
    del idx
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 13)
    k = max(4, min(n) // 4)                      # a chaotic body
    lo = [int(r.integers(0, m - k + 1)) for m in n]
    V[lo[0]:lo[0] + k, lo[1]:lo[1] + k, lo[2]:lo[2] + k] = torch.randn((k, k, k), generator=g, device=DEV)
    V.add_(torch.randn(tuple(n), generator=g, device=DEV), alpha=0.3)
    V.sub_(V.mean()).div_(V.std())
    return V.contiguous()


def _windows(case, seed):
    """A batch of 16^3 training windows with their raw maps (scaled as the training driver scales)."""
    V = _volume((64, 96, 96), seed)
    lab = surrogate.exact_raw_maps(sal.Saliency(L=16), V)
    scale = lab.flatten(1).std(dim=1)
    r = np.random.default_rng([seed, 5])
    X, T = [], []
    for _ in range(case["batch"]):
        at = tuple(slice(a, a + surrogate.WINDOW) for a in
                   (int(r.integers(0, m - surrogate.WINDOW + 1)) for m in V.shape))
        X.append(V[at])
        T.append(lab[(slice(None),) + at].permute(1, 2, 3, 0) / scale)
    return torch.stack(X).contiguous(), torch.stack(T).contiguous()


def _ctx(case):
    return sal.Saliency(L=case["L"], stride=case["stride"], precision=PRECISIONS[case["precision"]],
                        rays=RAYS[case["rays"]])


def prepare(case, seed):
    if case["op"] == "train":
        X, T = _windows(case, seed)
        net = surrogate.load()
        return {"case": case, "X": X, "T": T, "net": net,
                "loss": torch.zeros(1, dtype=torch.float32, device=DEV)}
    V = _volume((case["n0"], case["n1"], case["n2"]), seed)
    s = {"case": case, "V": V}
    if case["op"] == "surrogate":
        s["net"] = surrogate.load()
        s["ctx"] = sal.Saliency(L=16, precision=sal.BF16_SPLIT)
    else:
        s["ctx"] = _ctx(case)
    if case["op"] == "stream":
        s["V"] = torch.empty(V.shape, dtype=torch.float32, pin_memory=True).copy_(V)
    return s


def run(state):
    case, op = state["case"], state["case"]["op"]
    if op == "saliency":
        return state["ctx"].saliency(state["V"])
    if op == "maps":
        S, E, S_raw, stats = state["ctx"].saliency_maps(state["V"])
        return {"S": S, "E": E, "S_raw": S_raw, "stats": stats}
    if op == "box":
        return state["ctx"].raw_box(state["V"], (case["b0"], case["b1"], case["b2"]),
                                    (case["d0"], case["d1"], case["d2"]))
    if op == "stream":
        S, S_raw, stats = stream.plain_streamed(state["ctx"], state["V"], slab=case["slab"])
        return {"S": S, "S_raw": S_raw, "stats": stats[:7]}
    if op == "surrogate":
        out = surrogate.infer_with_fallback(state["net"], state["ctx"], state["V"])
        return {"S": out["S"], "S_raw": out["S_raw"], "stats": out["stats"][:7]}
    state["net"].train_step(state["X"], state["T"], surrogate.MARGIN, 1e-3, loss_out=state["loss"])
    return {"loss": state["loss"], "params": state["net"].get_params()}


# ----------------------------------------------------------------- what a pass cannot do without

def work(case):
    if case["op"] == "train":
        n = case["batch"] * 16 ** 3
        # forward, input gradient, weight gradient: 95,904 flops a voxel each
        return {"bytes": float(n * 16), "flops": float(n) * 3 * 95904}
    N = case["n0"] * case["n1"] * case["n2"]
    if case["op"] == "surrogate":
        return {"bytes": float(N * 20), "flops": float(N) * (95904 + 60)}
    L, r = case["L"], case["L"] // 2
    nw, nout, vals = N, N, 1
    if case["op"] == "box":
        nout = case["d0"] * case["d1"] * case["d2"]
        nw = 1
        for k in range(3):
            nw *= min(case["n%d" % k], case["d%d" % k] + 2 * r)
        vals = 3
    elif case["op"] == "stream":
        vals = 4
    elif case["op"] == "maps":
        vals = 7
    lat = 1
    for k in range(3):
        lat *= -(-case["n%d" % k] // case["stride"])
    if case["stride"] > 1:
        nw = lat
    # a window: half of its L^3 bins enter once, give one magnitude and one weighted sum per
    # component; its plane's 2-D transform.  Eq. (5): 4 flops a neighbour
    win = L ** 3 // 2 * (2 + 4 + 2) + 5 * L * L * math.log2(L)
    nbr = 4 * r * sum(bin(m).count("1") for m in RAYS[case["rays"]])
    return {"bytes": 4.0 * (N if case["op"] != "box" else nw) + 4.0 * vals * nout,
            "flops": float(nw) * win + float(nout) * (nbr + 10)}


# --------------------------------------------------------------------------- values in 64 bits

def _energies(V, L, pos):
    """[3, k0, k1, k2] mean projected magnitudes of the windows centred on the given positions."""
    H, dims = L // 2, V.shape
    f = torch.arange(L, device=DEV, dtype=torch.float64)
    sf = torch.where(f > L // 2, f - L, f)
    W = torch.polar(torch.ones((L, L), dtype=torch.float64, device=DEV), -2 * math.pi / L * torch.outer(f, f))
    out = torch.zeros([3] + [len(p) for p in pos], dtype=torch.float64, device=DEV)
    tap = torch.arange(L, device=DEV) - H
    refl = []
    for p, n in zip(pos, dims):
        i = (torch.tensor(p, device=DEV).view(-1, 1) + tap).abs()
        refl.append(torch.where(i >= n, 2 * (n - 1) - i, i))  # [k, L]
    k1, k2 = len(pos[1]), len(pos[2])
    rows = max(1, int(1.5e9 / (16.0 * max(k1 * k2 * L, dims[1] * dims[2]))))
    for a in range(0, len(pos[0]), rows):
        src = V[refl[0][a:a + rows]]                           # [m, L, n1, n2]
        m = src.shape[0]
        for mu in range(L // 2 + 1):
            mult = 1.0 if mu == 0 or 2 * mu == L else 2.0
            A = torch.zeros((m,) + tuple(dims[1:]), dtype=torch.complex128, device=DEV)
            for p in range(L):
                A.add_(src[:, p], alpha=complex(W[mu, p].item()))
            for nu in range(L):
                B = torch.zeros((m, k1, dims[2]), dtype=torch.complex128, device=DEV)
                for q in range(L):
                    B.add_(A[:, refl[1][:, q]], alpha=complex(W[nu, q].item()))
                F = torch.matmul(B[:, :, refl[2]].reshape(-1, L), W).abs()
                i2, j2, l2 = sf[mu] ** 2, sf[nu] ** 2, sf ** 2
                rho = torch.sqrt(i2 + j2 + l2)
                w = torch.stack([torch.sqrt(j2 + l2), torch.sqrt(i2 + l2), torch.sqrt(i2 + j2).expand(L)])
                w = torch.where(rho > 0, w / torch.where(rho > 0, rho, 1.0), 0.0) * mult
                out[:, a:a + m] += (F @ w.T).T.reshape(3, m, k1, k2)
    return out / (L ** 3 * (L ** 3 - 1.0))


def _interpolate(E, stride, n):
    for ax in range(3):
        u = torch.arange(n[ax], device=DEV, dtype=torch.float64)
        k = torch.clamp((u / stride).floor().long(), max=E.shape[ax + 1] - 1)
        k1 = torch.clamp(k + 1, max=E.shape[ax + 1] - 1)
        shape = [1, 1, 1, 1]
        shape[ax + 1] = -1
        f = ((u - k * stride) / stride).view(shape)
        a, b = E.index_select(ax + 1, k), E.index_select(ax + 1, k1)
        E = a + f * (b - a)
    return E


def _steps(mask):
    """(t, x, y) steps of the ray bits of a mask."""
    out = []
    for b in range(6):
        if mask >> b & 1:
            e = [0, 0, 0]
            e[b // 2] = -1 if b & 1 else 1
            out.append(tuple(e))
    for b, (s0, s1) in zip(range(6, 10), ((1, 1), (-1, -1), (1, -1), (-1, 1))):
        if mask >> b & 1:
            out.append((s0, s1, 0))
    return out


def _compare(E, L, rays):
    r, sigma, n = L // 2, L / 4.0, E.shape[1:]
    S = torch.zeros_like(E)
    for m in range(3):
        steps = _steps(rays[m])
        for e in steps:
            for s in range(1, r + 1):
                N = E[m]
                for ax in range(3):
                    if e[ax]:
                        i = (torch.arange(n[ax], device=DEV) + s * e[ax]).abs()
                        N = N.index_select(ax, torch.where(i >= n[ax], 2 * (n[ax] - 1) - i, i))
                w = math.exp(-(s * s) * sum(v * v for v in e) / (2 * sigma * sigma))
                S[m] += (E[m] - w * N).abs()
        S[m] /= len(steps) * r
    return S


def _cost(case):
    lat = 1
    for k in range(3):
        lat *= -(-case["n%d" % k] // case["stride"])
    return lat * float(case["L"]) ** 3


def exact(case, seed):
    if case["op"] in ("train", "surrogate") or _cost(case) > 1.5e11:
        return None
    V = _volume((case["n0"], case["n1"], case["n2"]), seed).double()
    n, L, st = tuple(V.shape), case["L"], case["stride"]
    E = _energies(V, L, [list(range(0, m, st)) for m in n])
    if st > 1:
        E = _interpolate(E, st, n)
    S_raw = _compare(E, L, RAYS[case["rays"]])
    if case["op"] == "box":
        sl = tuple(slice(case["b%d" % k], case["b%d" % k] + case["d%d" % k]) for k in range(3))
        return S_raw[(slice(None),) + sl].contiguous()
    vmax = float(V.abs().max())
    S, stats = torch.zeros_like(V), []
    for m in range(3):
        lo, hi = float(S_raw[m].min()), float(S_raw[m].max())
        stats += [lo, hi]
        if hi - lo > 1e-6 * vmax:
            S += (S_raw[m] - lo) / (hi - lo) / 3.0
    stats = torch.tensor(stats + [vmax], dtype=torch.float64, device=DEV)
    if case["op"] == "saliency":
        return S
    if case["op"] == "maps":
        return {"S": S, "E": E, "S_raw": S_raw, "stats": stats}
    return {"S": S, "S_raw": S_raw, "stats": stats}
