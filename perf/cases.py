"""The work that users of this framework have it do, as measurable cases.

A case is a dict of plain values:
  what       "modes" (mode-amplitude Langevin steps), "euler" (bead-space
             Euler steps), "mc" (Metropolis sweeps), "wlc" (inextensible
             limit) or "static" (the allocation-free FP64 mode step)
  precision  "fp64", "fp32" or "bf16x3" (how the mode step computes)
  chains     chains in the ensemble
  beads      beads per chain, or a text "64,96,128": every chain's length is
             drawn uniformly from these
  steps      steps (sweeps) of one pass
  every      observables are sampled every this many steps (0 = never)
  wi         Weissenberg number of a simple shear flow (0 = no flow)
  tuned      True: autotuned tile shapes and replayed sampling blocks, as the
             benchmark runs; False: the defaults of set_params
  read       "device": the frame of positions stays on the GPU (an analysis
             there); "host": mode amplitudes as a NumPy array

One pass advances the ensemble and reads it out: the frame of every chain and,
where observables are sampled, the accumulators.  The reduced-precision paths
hold their state in 32 bits, so their frames and sums are kept as float32.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_1411_3487_amd import Context, load, DM_OBS_ACCUM, NU_DSDNA, T_STAR_DSDNA

T_WLC = 1.0 / 114.4     # reduced bending temperature of dsDNA
WLC_CYCLES = 8          # fixed tension cycles of one inextensible step
EULER_DT = 0.1          # the bead-space scheme's safe time step
WLC_DT = 1e-4
SEEDS = 1 << 40


def _case(name, what, precision, chains, beads, steps, every=0, wi=0.0, tuned=False,
          read="device"):
    return {"name": name, "what": what, "precision": precision, "chains": chains,
            "beads": beads, "steps": steps, "every": every, "wi": wi, "tuned": tuned,
            "read": read}


def listed():
    return [
        # the headline: 4096 dsDNA chains of 256 bp, the report interval of a
        # production run with observables every 100 steps
        _case("bf16x3 4096x256", "modes", "bf16x3", 4096, 256, 500, every=100, tuned=True),
        # long chains, few of them: a batch that does not fill the chip
        _case("bf16x3 1024x512", "modes", "bf16x3", 1024, 512, 200, every=100, tuned=True),
        # an uneven ensemble of the lengths the paper and the benchmark name
        _case("bf16x3 uneven 8192", "modes", "bf16x3", 8192, "64,96,128,192,256,384,512", 100,
              every=100, tuned=True),
        # a handful of short chains, interactive use: latency counts
        _case("bf16x3 6x64", "modes", "bf16x3", 6, 64, 50),
        # shear flow in single precision (mean extension and tumbling)
        _case("fp32 2048x256 shear", "modes", "fp32", 2048, 256, 200, every=100, wi=10.0,
              tuned=True),
        # one chain in double precision, as the paper simulates
        _case("fp64 1x64", "modes", "fp64", 1, 64, 200, every=100, tuned=True, read="host"),
        # the double-precision reference run beside the headline
        _case("fp64 4096x256", "modes", "fp64", 4096, 256, 100, every=100, tuned=True),
        # double precision, ragged: even and odd bead counts (N = 64, 128, 256
        # bonds as in the coarse-graining check), no sampling
        _case("fp64 uneven 700", "modes", "fp64", 700, "65,96,129,200,257", 40),
        # the bead-space baseline scheme
        _case("euler 4096x256", "euler", "fp64", 4096, 256, 100),
        # equilibrium values by Monte Carlo
        _case("mc 1024x128", "mc", "fp64", 1024, 128, 10, every=5),
        # the inextensible wormlike chain
        _case("wlc 8192x64", "wlc", "fp64", 8192, 64, 20),
        # a serving loop on caller-owned amplitudes that may not allocate
        _case("static 512x128", "static", "fp64", 512, 128, 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: any path, sizes over their logarithm."""
    what = rng.choice(["modes", "modes", "modes", "modes", "euler", "mc", "wlc", "static"])
    if what == "modes":
        precision = rng.choice(["bf16x3", "bf16x3", "fp32", "fp64", "fp64"])
        chains = _log_int(rng, 1, 6000)
        if rng.random() < 0.25:
            pool = ([64, 96, 128, 192, 256, 384, 512] if precision != "fp64" else
                    [48, 65, 96, 129, 200, 257, 320])
            beads = ",".join(str(m) for m in sorted(rng.sample(pool, 3)))
            longest = max(int(m) for m in beads.split(","))
        else:
            beads = _log_int(rng, 32, 512)
            if precision != "fp64":
                beads += beads % 2          # these paths need an even number of beads
            longest = beads
        # no more work than the largest listed case
        cap = 5.0e8 if precision == "bf16x3" else 1.0e8
        steps = max(10, min(200, int(cap / (chains * longest * max(1.0, longest / 256.0)))))
        chains = max(1, min(chains, int(cap / (steps * longest * max(1.0, longest / 256.0)))))
        every = rng.choice([0, 0, steps // 2, steps])
        return _case("drawn", what, precision, chains, beads, steps, every=every,
                     wi=rng.choice([0.0, 0.0, 1.0, 10.0]),
                     tuned=every > 0 and rng.random() < 0.7,
                     read=rng.choice(["device", "device", "host"]))
    if what == "euler":
        beads, chains = _log_int(rng, 32, 512), _log_int(rng, 1, 4096)
        steps = max(10, min(100, int(1.0e8 / (beads * chains))))
    elif what == "mc":
        beads, chains, steps = _log_int(rng, 32, 256), _log_int(rng, 1, 2048), 4
        steps = max(1, min(10, int(1.7e8 / (beads * beads * chains))))
    elif what == "wlc":
        beads, chains = _log_int(rng, 16, 128), _log_int(rng, 1, 8192)
        steps = max(2, min(40, int(1.0e7 / (beads * chains))))
    else:
        beads, chains, steps = _log_int(rng, 33, 256), _log_int(rng, 1, 1024), 20
    return _case("drawn", what, "fp64", chains, beads, steps,
                 every=rng.choice([0, steps]) if what == "mc" else 0,
                 wi=rng.choice([0.0, 10.0]) if what == "static" else 0.0)


# ------------------------------------------------------------------- inputs
def _dtau(M):
    """The paper's largest time step of a chain of M beads (its Table 1)."""
    return 10.0 if M < 120 else 50.0 if M < 240 else 100.0


def _shear(case, M):
    """Shear rate in units of the relaxation rate of the slowest mode."""
    return case["wi"] * 16 * NU_DSDNA * math.sin(math.pi / (2 * M)) ** 4


def _lengths(case):
    """The ensemble's chain lengths: part of the case, not of its inputs."""
    if isinstance(case["beads"], str):
        rng = np.random.default_rng(2)
        pool = np.array([int(m) for m in case["beads"].split(",")], dtype=np.int32)
        return pool[rng.integers(0, len(pool), case["chains"])]
    return np.full(case["chains"], case["beads"], dtype=np.int32)


def _directions(rng, n):
    v = rng.standard_normal((n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def _chain_block(rng, n, M, wlc):
    """(n, 3, M): straight chains of bond length 1/(1 - 2 nu) along uniform
    directions with one per cent of jitter; the inextensible limit starts from
    wormlike chains of unit bonds in equilibrium."""
    if not wlc:
        b = 1.0 / (1.0 - 2.0 * NU_DSDNA)
        x = _directions(rng, n)[:, :, None] * (b * np.arange(M))
        return x + 0.01 * b * rng.standard_normal((n, 3, M), dtype=np.float32)
    u = np.zeros((n, 3, M))
    p = _directions(rng, n)
    u[:, :, 1] = p
    for k in range(2, M):
        y = rng.random(n)[:, None]
        c = 1 + T_WLC * np.log(y + (1 - y) * math.exp(-2 / T_WLC))
        q = np.cross(p, _directions(rng, n))
        q /= np.linalg.norm(q, axis=1, keepdims=True)
        p = c * p + np.sqrt(np.maximum(0, 1 - c * c)) * q
        p /= np.linalg.norm(p, axis=1, keepdims=True)
        u[:, :, k] = p
    return np.cumsum(u, axis=2)


def _inputs(case, seed):
    """Lengths, one (3, M) array per chain (ordered) and the Philox seed."""
    rng = np.random.default_rng(seed)
    beads = _lengths(case)
    pos = [None] * len(beads)
    for M in np.unique(beads):
        at = np.flatnonzero(beads == M)
        block = _chain_block(rng, len(at), int(M), case["what"] == "wlc")
        for j, c in enumerate(at):
            pos[c] = block[j]
    return beads, pos, int(rng.integers(0, SEEDS))


def prepare(case, seed):
    beads, pos, key = _inputs(case, seed)
    if case["what"] == "static":
        M = int(beads[0])
        phi = _phi(M, "cpu")
        R = torch.from_numpy(np.stack(pos)) @ phi
        return {"case": case, "M": M, "key": key, "R": R.cuda().contiguous(), "step": 0,
                "lib": load()}
    stream = torch.cuda.current_stream()
    ctx = Context(pos, seed=key, precision=case["precision"], stream=stream)
    state = {"case": case, "ctx": ctx,
             "frame": torch.empty(int(3 * beads.sum()), dtype=torch.float64, device="cuda")}
    if case["what"] != "wlc":
        lens = sorted(set(int(m) for m in beads))
        ctx.set_params(lens, [_dtau(m) for m in lens], T_star=T_STAR_DSDNA, nu=NU_DSDNA,
                       gamma_dot=_shear(case, lens[-1]), sample_every=case["every"],
                       use_graphs=case["tuned"],
                       autotune=case["tuned"] and case["precision"] != "fp64")
    return state


# --------------------------------------------------------------------- pass
def run(state):
    case = state["case"]
    n = case["steps"]
    if case["what"] == "static":
        M, lib = state["M"], state["lib"]
        rc = lib.dm_step_modes_f64_static(
            state["R"].data_ptr(), case["chains"], M, T_STAR_DSDNA, NU_DSDNA, _dtau(M),
            _shear(case, M), 1, state["key"], 0, state["step"], n,
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        if rc:
            raise RuntimeError(lib.dm_last_error(None).decode())
        state["step"] += n
        return [state["R"]]
    ctx, out = state["ctx"], []
    if case["what"] == "modes":
        ctx.step_modes(n)
    elif case["what"] == "euler":
        ctx.step_euler(n, EULER_DT)
    elif case["what"] == "mc":
        out.append(ctx.step_mc(n))
    else:
        ctx.step_wlc(n, WLC_DT, T_WLC, iters=WLC_CYCLES)
    single = case["precision"] != "fp64"
    if case["read"] == "host":
        R = ctx.modes()
        R = np.concatenate([r.ravel() for r in R]) if isinstance(R, list) else R.ravel()
        out.append(R.astype(np.float32) if single else R)
    else:
        ctx.positions_to_device(state["frame"].data_ptr())
        out.append(state["frame"].float() if single else state["frame"])
    if case["every"]:
        acc = ctx.observables(DM_OBS_ACCUM)
        out.append(acc.astype(np.float32) if single else acc)
    return out


# --------------------------------------------------------------------- work
def work(case):
    """State read and written once, the frame written once; the transforms as
    dense products of the two mirror halves, normals at 25 operations each."""
    beads = case["beads"]
    pool = [int(m) for m in beads.split(",")] if isinstance(beads, str) else [beads]
    word = 8 if case["precision"] == "fp64" else 4
    nbytes = flops = 0.0
    for M in pool:
        chains, n = case["chains"] / len(pool), case["steps"]
        nbytes += chains * 3 * M * (2 * word + (0 if case["what"] == "static" else 8))
        if case["what"] in ("modes", "static"):
            per = 6.0 * M * M + 3 * M * 35 + 15 * M
        elif case["what"] == "euler":
            per = M * (3 * 25 + 60.0)
        elif case["what"] == "mc":
            per = 3.0 * (M - 1) * (M - 1) * 18
        else:
            per = M * (3 * 25 + 70.0 * WLC_CYCLES)
        flops += chains * n * per
    return {"bytes": nbytes, "flops": flops}


# -------------------------------------------------------- the same in 64 bits
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _phi(M, dev):
    n = torch.arange(M, dtype=torch.float64, device=dev)
    m = torch.remainder(torch.outer(2 * n + 1, n), 4 * M)
    phi = math.sqrt(2.0 / M) * torch.cos(m * (math.pi / (2 * M)))
    phi[:, 0] = math.sqrt(1.0 / M)
    return phi


def _mulhilo(a, c):
    lo, hi = a * (c & 0xFFFF), a * (c >> 16)
    t = hi + (lo >> 16)
    return t >> 16, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)


def _philox(c, key):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    k0, k1 = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    c0, c1, c2, c3 = c
    for _ in range(10):
        ah, al = _mulhilo(c0, 0xD2511F53)
        bh, bl = _mulhilo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = bh ^ c1 ^ k0, bl, ah ^ c3 ^ k1, al
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _uniform(x):
    return (x.double() + 0.5) * 2.0 ** -32


def _normals(ids, M, step, key, tag):
    """(n, 3, M) standard normals of one step (Box-Muller on Philox blocks)."""
    dev = ids.device
    q = torch.arange((M + 3) // 4, device=dev)
    a = torch.arange(3, device=dev)
    c0 = q[None, None, :] + 0 * ids[:, None, None] + 0 * a[None, :, None]
    c1 = ids[:, None, None] + 0 * c0
    c3 = ((step >> 32) << 8) + (a[None, :, None] << 4) + tag + 0 * c0
    w = _philox((c0, c1, 0 * c0 + (step & 0xFFFFFFFF), c3), key)
    z = []
    for i in (0, 2):
        r, t = torch.sqrt(-2 * torch.log(_uniform(w[i]))), 2 * math.pi * _uniform(w[i + 1])
        z += [r * torch.cos(t), r * torch.sin(t)]
    return torch.stack(z, dim=-1).reshape(len(ids), 3, -1)[:, :, :M]


class _Sums:
    """The accumulators of one length bucket, 109 + M values (no time correlations)."""

    def __init__(self, x0):
        n, _, self.M = x0.shape
        self.cm0 = x0.mean(dim=2)
        self.s = torch.zeros(13 + self.M + 32 + 64, dtype=torch.float64)
        self.s[0], self.s[1] = self.M, n
        self.state, self.last = torch.zeros(n), torch.zeros(n)

    def add(self, x, R, step):
        s, M = self.s, self.M
        u = x.diff(dim=2)
        l2 = u.square().sum(dim=1)
        L, cm = x[:, :, -1] - x[:, :, 0], x.mean(dim=2)
        s[2] += 1
        s[3] += float(l2.sqrt().mean(dim=1).sum())
        s[4] += float(l2.mean(dim=1).sum())
        s[5] += float(L.square().sum())
        s[6] += float((cm - self.cm0).square().sum())
        s[7] += float((x[:, :, (M - 1) // 2] - cm).square().sum())
        s[8] += float((x[:, 0].amax(dim=1) - x[:, 0].amin(dim=1)).sum())
        s[13:13 + M] += R.square().sum(dim=(0, 1)).cpu()
        half = 0.5 * torch.hypot(L[:, 0], L[:, 1]).cpu()
        Lx, old = L[:, 0].cpu(), self.state
        new = torch.where(Lx > half, 1.0, torch.where(Lx < -half, -1.0, old.double())).float()
        flip = (old != 0) & (new != old)
        s[9] += int(flip.sum())
        for tau in (step + 1 - self.last[flip & (self.last > 0)]).tolist():
            s[10] += tau
            s[11] += tau * tau
            s[12] += 1
            s[13 + M + min(31, max(0, int(math.floor(math.log2(tau)))))] += 1
        self.last[flip] = step + 1
        self.state = new


def _mode_steps(R, M, ids, key, first, n, gdot, sums, every):
    dev = R.device
    dt, nu, T = _dtau(M), NU_DSDNA, T_STAR_DSDNA
    phi = _phi(M, dev)
    chi = phi.diff(dim=0)
    chi[:, 0] = 0
    s2 = torch.sin(math.pi * torch.arange(M, dtype=torch.float64, device=dev) / (2 * M)) ** 2
    zeta, dz = 16 * nu * s2 * s2, (1 - 2 * nu) * 4 * s2
    E = torch.exp(-zeta * dt)
    C = -E * torch.expm1(-dz * dt) / dz
    W = torch.sqrt(-T * torch.expm1(-2 * zeta * dt) / zeta)
    C[0], W[0] = 0.0, math.sqrt(2 * T * dt)
    for k in range(first, first + n):
        u = R @ chi.T
        g = u * (u.square().sum(dim=1, keepdim=True).rsqrt() - (1 - 2 * nu))
        new = E * R + C * (g @ chi) + W * _normals(ids, M, k, key, 0)
        if gdot:
            new[:, 0] += gdot * dt * E * R[:, 1]
        R = new
        if every and (k + 1) % every == 0:
            sums.add(R @ phi.T, R, k + 1)
    return R


def _euler_steps(x, ids, key, n):
    nu, dt = NU_DSDNA, EULER_DT
    amp = math.sqrt(2 * T_STAR_DSDNA * dt)
    pad = torch.nn.functional.pad
    for k in range(n):
        u = x.diff(dim=2)
        l = u.square().sum(dim=1, keepdim=True).sqrt()
        h = (l - 1) * u / l - nu * (pad(u, (1, 0))[:, :, :-1] + pad(u, (0, 1))[:, :, 1:])
        x = x + dt * pad(h, (1, 1)).diff(dim=2) + amp * _normals(ids, x.shape[2], k, key, 1)
    return x


def _mc_sweeps(x, ids, key, n, sums, every):
    nu, T, M, dev = NU_DSDNA, T_STAR_DSDNA, x.shape[2], x.device
    phi = _phi(M, dev)
    chi = phi.diff(dim=0).T.contiguous()
    R, u = x @ phi, x.diff(dim=2)
    taken = 0
    p = torch.arange(1, M, device=dev)
    zl = [4 * math.sin(math.pi * q / (2 * M)) ** 2 * (1 - 2 * nu * math.cos(math.pi * q / M))
          for q in range(1, M)]
    width = 3.0 * torch.sqrt(T / torch.tensor(zl, dtype=torch.float64, device=dev))
    for k in range(n):
        a = torch.arange(3, device=dev)
        c0 = p[:, None, None] + 0 * a[None, :, None] + 0 * ids
        w = _philox((c0, ids + 0 * c0, 0 * c0 + k, (a[None, :, None] << 4) + 2 + 0 * c0), key)
        delta = width[:, None, None] * (2 * _uniform(w[0]) - 1)
        bar = -T * torch.log(_uniform(w[1]))
        l2 = u.square().sum(dim=1)
        for i in range(M - 1):
            c = chi[i + 1]
            for b in range(3):
                d = delta[i, b][:, None]
                ua, step = u[:, b], c * d
                l2n = l2 + step * (2 * ua + step)
                dh = (0.5 * (l2n - l2) - (l2n.sqrt() - l2.sqrt())).sum(dim=1)
                dh -= nu * (step[:, :-1] * ua[:, 1:] + step[:, 1:] * ua[:, :-1]
                            + step[:, :-1] * step[:, 1:]).sum(dim=1)
                ok = dh < bar[i, b]
                taken += ok
                step = torch.where(ok[:, None], step, 0.0)
                ua += step
                l2 = torch.where(ok[:, None], l2n, l2)
                R[:, b, i + 1] += torch.where(ok, d[:, 0], 0.0)
        if every and (k + 1) % every == 0:
            sums.add(R @ phi.T, R, k + 1)
    return int(taken.sum()), R @ phi.T


def _wlc_steps(x, ids, key, n):
    dt, M = WLC_DT, x.shape[2]
    amp = math.sqrt(2 * T_WLC * dt)
    pad = torch.nn.functional.pad
    u = x.diff(dim=2)
    u = u / u.square().sum(dim=1, keepdim=True).sqrt()
    r0, N = x[:, :, 0].clone(), M - 1
    for k in range(n):
        noise = amp * _normals(ids, M, k, key, 3)
        un = u
        for _ in range(WLC_CYCLES):
            w = u + un
            um = w / w.square().sum(dim=1, keepdim=True).sqrt()
            left, right = pad(um, (1, 0))[:, :, :-1], pad(um, (0, 1))[:, :, 1:]
            d = pad(-(left + right), (1, 1)).diff(dim=2) * dt + noise
            dd = d.diff(dim=2)
            A = ((w * left).sum(dim=1) * dt).T.contiguous()
            B = ((w * um).sum(dim=1) * (-2 * dt)).T.contiguous()
            C = ((w * right).sum(dim=1) * dt).T.contiguous()
            r = (-(w * dd).sum(dim=1)).T.contiguous()
            cs, ds = [C[0] / B[0]], [r[0] / B[0]]
            for i in range(1, N):
                m = B[i] - A[i] * cs[-1]
                cs.append(C[i] / m)
                ds.append((r[i] - A[i] * ds[-1]) / m)
            f = [ds[-1]]
            for i in range(N - 2, -1, -1):
                f.append(ds[i] - cs[i] * f[-1])
            f = torch.stack(f[::-1], dim=1)[:, None, :]
            fu = f * um
            un = u + dd + (f.roll(1, 2) * left - 2 * fu + f.roll(-1, 2) * right) * dt
        r0 = r0 + d[:, :, 0] + f[:, :, 0] * um[:, :, 0] * dt
        u = un
    return r0[:, :, None] + pad(u, (1, 0)).cumsum(dim=2)


def exact(case, seed):
    """What run() returns on the first pass, in plain 64-bit torch."""
    dev = _device()
    beads, pos, key = _inputs(case, seed)
    start = np.concatenate([[0], np.cumsum(3 * beads.astype(np.int64))])
    flat, taken, accs = np.empty(int(start[-1])), 0, []
    longest = int(beads.max())
    for M in sorted(set(int(m) for m in beads)):
        at = np.flatnonzero(beads == M)
        ids = torch.from_numpy(at).to(dev)
        x = torch.from_numpy(np.stack([pos[c] for c in at])).double().to(dev)
        sums = _Sums(x) if case["every"] else None
        if case["what"] in ("modes", "static"):
            phi = _phi(M, dev)
            R = _mode_steps(x @ phi, M, ids, key, 0, case["steps"], _shear(case, longest), sums,
                            case["every"])
            x = R if case["what"] == "static" or case["read"] == "host" else R @ phi.T
        elif case["what"] == "euler":
            x = _euler_steps(x, ids, key, case["steps"])
        elif case["what"] == "mc":
            n, x = _mc_sweeps(x, ids, key, case["steps"], sums, case["every"])
            taken += n
        else:
            x = _wlc_steps(x, ids, key, case["steps"])
        x = x.cpu().numpy()
        for j, c in enumerate(at):
            flat[start[c]:start[c + 1]] = x[j].ravel()
        if sums:
            accs.append(sums.s.numpy())
    if case["what"] == "static":
        return [torch.from_numpy(flat).reshape(case["chains"], 3, -1)]
    out = [taken] if case["what"] == "mc" else []
    out.append(torch.from_numpy(flat) if case["read"] == "device" else flat)
    if case["every"]:
        out.append(np.concatenate(accs))
    return out
