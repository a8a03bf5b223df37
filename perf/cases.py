"""Workloads of the local-FFT PSATD field push that its speed is measured on.

A case is a grid cut into boxes ("x", "y", "z": the owned lengths along each
axis, comma separated, the boxes being their product), guard widths dealt to
the boxes in turn ("g"), the order p of the modified wavenumbers, the precision
form, and the call that one pass makes:

  run    Plan.run, `steps` steps with the current held (a field-only stretch)
  step   Plan.step, one step with a new current (the field push of a PIC loop);
         with deposited currents the pass first puts the freshly deposited
         partial currents into J, as the deposition of such a loop does
  heat   Plan.heat_run, `steps` steps of the diffusion equation

Fields are smooth, as resolved fields are: a few plane waves polarised across
the order-p wave vector, and a Gaussian current pulse.  A pass advances the
state in place and returns it.
"""
import math

import numpy as np
import torch

from paper_1707_08500_amd import psatd

DT, C, DIFFUSIVITY = 0.5, 1.0, 0.3
D = (1.0, 1.0, 1.0)


def _case(name, x, y, z, g, p, prec, call, steps=1, jmode="replicated"):
    c = {"x": x, "y": y, "z": z, "g": g, "p": p, "prec": prec, "call": call, "steps": steps, "jmode": jmode}
    return {"name": name, **c} if name else c


def _even(n, count):
    return ",".join([str(n)] * count)


def listed():
    b64, b128 = _even(64, 4), _even(128, 4)
    return [
        # one small periodic box, double precision: a dispersion check, step by
        # step; launches and latency are all of it
        _case("step_32_f64_global", "32", "32", "32", "0", 16, "f64", "step"),
        # eight small boxes, two held-current steps: a first run on a new machine
        _case("run2_32_f64", "16,16", "16,16", "16,16", "4", 16, "f64", "run", 2),
        # a small PIC-like step with uneven boxes, odd lengths and deposited currents
        _case("step_odd_f32_deposited", "22,26", "25,35", "11,15,23", "5", 16, "f32", "step", 1, "deposited"),
        # the workhorse: 256^3 in 64 boxes of 64^3 with 16 guards, held current
        _case("run4_256_f32", b64, b64, b64, "16", 32, "f32", "run", 4),
        # the same boxes inside a PIC loop: new deposited currents each step
        _case("step_256_f32_deposited", b64, b64, b64, "16", 32, "f32", "step", 1, "deposited"),
        # the same boxes in double precision
        _case("run2_256_f64", b64, b64, b64, "16", 32, "f64", "run", 2),
        # the matrix-core form on a grid of eight such boxes
        _case("run4_128_bf16x6", "64,64", "64,64", "64,64", "16", 32, "bf16x6", "run", 4),
        # load-balanced decomposition: 126 uneven boxes, guard widths of their own
        _case("run2_uneven_f32", "96,96,64,96,96,64", "96,96,64,80,48,80,48", "80,96,80", "8,16,32,16,8,32,32", 64,
              "f32", "run", 2),
        # large boxes at very high order: 512^3 in 64 boxes of 128^3 with 24 guards
        _case("run2_512_f32", b128, b128, b128, "24", 100, "f32", "run", 2),
        # large boxes in double precision (their planes exceed the LDS)
        _case("step_256_f64_128", "128,128", "128,128", "128,128", "24", 100, "f64", "step"),
        # the global method on one device: one 256^3 box, no guards
        _case("run4_256_f32_global", "256", "256", "256", "0", 32, "f32", "run", 4),
        # the diffusion equation on the workhorse's boxes
        _case("heat4_256_f32", b64, b64, b64, "16", 32, "f32", "heat", 4),
    ]


def _ints(text):
    return [int(v) for v in text.split(",")]


def _boxes(case):
    """lo, n, g (each (boxes, 3), axes x, y, z; boxes x fastest) and the grid."""
    cuts = [_ints(case[a]) for a in "xyz"]
    guards = _ints(case["g"])
    lo, n, g = [], [], []
    oz = 0
    for nz in cuts[2]:
        oy = 0
        for ny in cuts[1]:
            ox = 0
            for nx in cuts[0]:
                lo.append((ox, oy, oz))
                n.append((nx, ny, nz))
                g.append((guards[len(g) % len(guards)],) * 3)
                ox += nx
            oy += ny
        oz += nz
    return np.array(lo, np.int64), np.array(n, np.int64), np.array(g, np.int64), tuple(sum(c) for c in cuts)


def _smooth(n):
    for p in (2, 3, 5, 7, 11):
        while n % p == 0:
            n //= p
    return n == 1


def _cost(case):
    """Padded cells x steps (double precision counts twice)."""
    _, n, g, _ = _boxes(case)
    cells = int(np.prod(n + 2 * g, axis=1).sum())
    return cells * case["steps"] * (2 if case["prec"] == "f64" else 1)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        call = rng.choice(("run", "run", "run", "step", "step", "heat"))
        prec = rng.choice(("f32", "f32", "f32", "f64", "f64", "bf16x6"))
        # one guard width, or a few dealt over the boxes; none only for a single box
        counts = [rng.choice((1, 2, 2, 3, 4)) for _ in range(3)]
        single = counts == [1, 1, 1] and rng.random() < 0.7
        widths = [0] if single else [rng.choice((4, 5, 8, 12, 16, 24)) for _ in range(rng.choice((1, 1, 1, 2, 3)))]
        size = math.exp(rng.uniform(math.log(20), math.log(300 if single else 150)))
        cuts = []
        for a in range(3):
            uneven = rng.random() < 0.4
            fits = [v for v in range(max(8, int(0.6 * size)), int(1.4 * size) + 1)
                    if all(_smooth(v + 2 * w) and (a or (v + 2 * w) % 2 == 0) for w in widths)]
            if not fits:
                break
            cuts.append(",".join(str(rng.choice(fits)) for _ in range(counts[a])) if uneven
                        else _even(rng.choice(fits), counts[a]))
        if len(cuts) < 3:
            continue
        case = _case(None, *cuts, ",".join(map(str, widths)), rng.choice((8, 16, 32, 64, 100)), prec, call,
                     rng.choice((1, 2, 4)) if call != "step" else 1,
                     rng.choice(("replicated", "deposited")) if call == "step" else "replicated")
        _, n, g, _ = _boxes(case)
        P = n + 2 * g
        sb = 8 if prec == "f64" else 4
        if P[:, 2].max() > 270:
            continue
        if call == "heat" and int((P[:, 0] * P[:, 1]).max()) * sb > 130 * 1024:
            continue  # the heat step takes planes that fit the LDS
        if 20_000 <= _cost(case) <= most // 2:
            return case


# ------------------------------------------------------------------ inputs
def _modified_k(N, p, device="cpu"):
    """Order-p modified wavenumbers over the FFT index, 64 bits (unit spacing)."""
    m = np.arange(N)
    mt = np.where(m <= (N - 1) // 2, m, m - N)
    M = p // 2
    w, acc = M / (M + 1.0), np.zeros(N)
    for j in range(1, M + 1):
        acc += w * np.sin(2.0 * np.pi * ((j * mt) % N) / N)
        w = -w * (j / (j + 1.0)) * ((M - j) / (M + j + 1.0))
    if N % 2 == 0:
        acc[N // 2] = 0.0
    return torch.from_numpy(2.0 * acc).to(device)


def _outer(ax):
    return ax[2][:, None, None] * ax[1][None, :, None] * ax[0][None, None, :]


def _globals(case, seed):
    """Global E, B, J (or, for heat, u), [z][y][x], in the case's element type."""
    N = _boxes(case)[3]
    r = np.random.default_rng([1707, int(seed) & 0x7FFFFFFF])
    dev, f64 = "cuda", torch.float64
    typ = f64 if case["prec"] == "f64" else torch.float32
    shape = (N[2], N[1], N[0])
    idx = [torch.arange(n, dtype=f64, device=dev) for n in N]
    mmax = [max(1, min(8, n // 4)) for n in N]
    kt = [_modified_k(n, case["p"]).numpy() for n in N]

    def wave(m, phase):
        ax = [torch.polar(torch.ones_like(idx[u]), (2 * math.pi * m[u] / N[u]) * idx[u]) for u in range(3)]
        ax[0] = ax[0] * complex(math.cos(phase), math.sin(phase))
        return _outer(ax).real

    def blob(centre, sigma):
        ax = []
        for u in range(3):
            d = idx[u] - centre[u]
            d = d - N[u] * torch.round(d / N[u])
            ax.append(torch.exp(-d * d / (2 * sigma * sigma)))
        return _outer(ax)

    sigma = min(8.0, min(N) / 6.0)
    if case["call"] == "heat":
        u = blob([r.uniform(0, n) for n in N], sigma)
        for _ in range(8):
            m = [int(r.integers(-q, q + 1)) for q in mmax]
            u.add_(wave(m, r.uniform(0, 2 * math.pi)), alpha=0.1)
        return [u.to(typ)]
    E, B = [[torch.zeros(shape, dtype=f64, device=dev) for _ in range(3)] for _ in range(2)]
    for _ in range(8):
        while True:
            m = [int(r.integers(-q, q + 1)) for q in mmax]
            kv = np.array([kt[u][m[u] % N[u]] for u in range(3)])
            if np.linalg.norm(kv) > 1e-3:
                break
        kh = kv / np.linalg.norm(kv)
        a = r.normal(size=3)
        a -= (a @ kh) * kh
        a *= 0.1 / np.linalg.norm(a)
        b = np.cross(kh, a)
        w = wave(m, r.uniform(0, 2 * math.pi))
        for u in range(3):
            E[u].add_(w, alpha=float(a[u]))
            B[u].add_(w, alpha=float(b[u]))
        del w
    v = r.normal(size=3)
    v *= r.uniform(0.5, 1.0) / np.linalg.norm(v)
    pulse = blob([r.uniform(0, n) for n in N], sigma)
    E, B = [t.to(typ) for t in E], [t.to(typ) for t in B]
    return E + B + [(pulse * float(a)).to(typ) for a in v]


def _shares(elems, typ, seed):
    """What part of a cell's current each padded copy of it was given (0 to 1)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)
    return torch.rand(elems, generator=gen, device="cuda", dtype=typ)


def prepare(case, seed):
    lo, n, g, N = _boxes(case)
    plan = psatd.Plan(N, D, lo, n, g, case["p"], DT, C, precision=case["prec"], jmode=case["jmode"])
    glob = [t.reshape(-1) for t in _globals(case, seed)]
    state = {"case": case, "plan": plan}
    if case["call"] == "heat":
        u = plan.empty_fields()
        plan.scatter(glob * 3, u)
        state["u"] = u[0]
        return state
    for k, name in enumerate("EBJ"):
        state[name] = plan.empty_fields()
        plan.scatter(glob[3 * k:3 * k + 3], state[name])
    if case["jmode"] == "deposited":
        w = _shares(plan.field_elems, plan.dtype, seed)
        state["parts"] = [j * w for j in state["J"]]
    return state


def run(state):
    case, plan = state["case"], state["plan"]
    if case["call"] == "heat":
        plan.heat_run(state["u"], DIFFUSIVITY, case["steps"])
        return {"u": state["u"]}
    E, B, J = state["E"], state["B"], state["J"]
    if case["call"] == "run":
        plan.run(E, B, J, case["steps"])
    else:
        if case["jmode"] == "deposited":
            for j, part in zip(J, state["parts"]):
                j.copy_(part)
        plan.step(E, B, J)
    out = {"E": E, "B": B}
    if case["jmode"] == "deposited":
        out["J"] = J
    return out


def work(case):
    """Per step: E, B and J read and E and B written once over the padded cells
    (u read and written for heat), the transforms of the nine fields and back of
    six (one and one), and the update at every point of the half spectra."""
    _, n, g, _ = _boxes(case)
    sb = 8 if case["prec"] == "f64" else 4
    moved = transforms = points = 0.0
    heat = case["call"] == "heat"
    for P in (n + 2 * g).tolist():
        V = float(P[0] * P[1] * P[2])
        moved += (2 if heat else 15) * V * sb
        transforms += (2 if heat else 15) * 2.5 * V * math.log2(V)
        points += (P[0] // 2 + 1) * P[1] * P[2]
    return {"bytes": case["steps"] * moved, "flops": case["steps"] * (transforms + (20 if heat else 150) * points)}


# ------------------------------------------------------- 64-bit reference
def _dft(N, sign):
    e = torch.arange(N, device="cuda")
    a = (sign * 2.0 * math.pi / N) * ((e[:, None] * e[None, :]) % N).to(torch.float64)
    return torch.polar(torch.ones_like(a), a)


def _transform(F, W):
    F = F.to(torch.complex128)
    nz, ny, nx = F.shape
    F = torch.matmul(F.reshape(nz * ny, nx), W[0]).reshape(nz, ny, nx)
    F = torch.matmul(W[1].expand(nz, ny, ny), F)
    return torch.matmul(W[2], F.reshape(nz, ny * nx)).reshape(nz, ny, nx)


def _push(E, B, J, k, W, Wi):
    """One padded box: Eqs. PSATD_1 and PSATD_2 at c = 1 in k-space."""
    E, B, J = ([_transform(f, W) for f in F] for F in (E, B, J))
    kx, ky, kz = k
    k2 = kx * kx + ky * ky + kz * kz
    kk = torch.sqrt(k2)
    safe = torch.where(kk > 0, kk, torch.ones_like(kk))
    th = kk * DT
    S = torch.where(kk > 0, torch.sin(th) / safe, torch.full_like(kk, DT))
    Cc = torch.cos(th)
    X1 = torch.where(kk > 0, 2 * torch.sin(th / 2) ** 2 / safe ** 2, torch.full_like(kk, 0.5 * DT * DT))
    t2 = th * th
    series = -DT ** 3 * (1 / 6 - t2 * (1 / 120 - t2 * (1 / 5040 - t2 * (1 / 362880 - t2 / 39916800))))
    X2 = torch.where(th < 0.1, series, (S - DT) / safe ** 2)

    def cross(F):
        return ky * F[2] - kz * F[1], kz * F[0] - kx * F[2], kx * F[1] - ky * F[0]

    def dot(F):
        return kx * F[0] + ky * F[1] + kz * F[2]

    kB, kE, kJ, dE, dJ = cross(B), cross(E), cross(J), dot(E), dot(J)
    V = E[0].numel()
    out = []
    for a in range(3):
        out.append(Cc * E[a] + 1j * S * kB[a] - S * J[a] + k[a] * (X1 * dE + X2 * dJ))
    for a in range(3):
        out.append(Cc * B[a] - 1j * S * kE[a] + 1j * X1 * kJ[a])
    return [_transform(f, Wi).real / V for f in out]


def exact(case, seed):
    lo, n, g, N = _boxes(case)
    dev = "cuda"
    glob = [t.to(torch.float64) for t in _globals(case, seed)]
    sb = 8 if case["prec"] == "f64" else 4
    # element offset of each padded box: its first interior x cell begins a
    # 128-byte line, to within the 16 bytes of a vector access
    line, vec, offs, elems = 128 // sb, 16 // sb, [], 0
    for s in range(len(lo)):
        want = -(-((-int(g[s][0])) % line) // vec) * vec % line
        elems += (want - elems) % line
        offs.append(elems)
        elems += int(np.prod(n[s] + 2 * g[s]))
    idx = [[(torch.arange(int(n[s][u] + 2 * g[s][u]), device=dev) + int(lo[s][u] - g[s][u])) % N[u] for u in range(3)]
           for s in range(len(lo))]

    def padded(F, s):
        i = idx[s]
        return F[i[2]][:, i[1]][:, :, i[0]]

    def buffers(F):
        out = torch.zeros(elems, dtype=torch.float64, device=dev)
        for s in range(len(lo)):
            v = padded(F, s)
            out[offs[s]:offs[s] + v.numel()] = v.reshape(-1)
        return out

    if case["jmode"] == "deposited":
        typ = torch.float32 if sb == 4 else torch.float64
        w = _shares(elems, typ, seed)
        for c in range(6, 9):
            total = torch.zeros(N[::-1], dtype=torch.float64, device=dev)
            for s in range(len(lo)):
                v = padded(glob[c], s).to(typ)
                v = (v * w[offs[s]:offs[s] + v.numel()].view(v.shape)).to(torch.float64)
                for u, d in ((2, 0), (1, 1), (0, 2)):  # fold each axis onto the grid
                    f = torch.zeros(v.shape[:d] + (N[u],) + v.shape[d + 1:], dtype=torch.float64, device=dev)
                    v = f.index_add_(d, idx[s][u], v)
                total += v
            glob[c] = total
    tables = {}

    def table(P):
        if P not in tables:
            tables[P] = (_dft(P, -1), _dft(P, 1), _modified_k(P, case["p"], dev))
        return tables[P]

    heat = case["call"] == "heat"
    for _ in range(case["steps"]):
        new = [torch.empty_like(f) for f in glob[:1 if heat else 6]]
        for s in range(len(lo)):
            t = [table(int(n[s][u] + 2 * g[s][u])) for u in range(3)]
            W, Wi = [v[0] for v in t], [v[1] for v in t]
            k = (t[0][2][None, None, :], t[1][2][None, :, None], t[2][2][:, None, None])
            F = [padded(f, s) for f in glob]
            if heat:
                u = _transform(F[0], W) * torch.exp(-DIFFUSIVITY * DT * (k[0] ** 2 + k[1] ** 2 + k[2] ** 2))
                got = [_transform(u, Wi).real / u.numel()]
            else:
                got = _push(F[:3], F[3:6], F[6:], k, W, Wi)
            own = tuple(slice(int(g[s][u]), int(g[s][u] + n[s][u])) for u in (2, 1, 0))
            at = tuple(slice(int(lo[s][u]), int(lo[s][u] + n[s][u])) for u in (2, 1, 0))
            for f, v in zip(new, got):
                f[at] = v[own]
        glob[:len(new)] = new
    if heat:
        return {"u": buffers(glob[0])}
    out = {"E": [buffers(f) for f in glob[:3]], "B": [buffers(f) for f in glob[3:6]]}
    if case["jmode"] == "deposited":
        out["J"] = [buffers(f) for f in glob[6:]]
    return out
