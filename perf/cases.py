"""Workloads for timing the short-range MD step through its public entry points.

listed() names the fixed cases, draw() makes further ones of the same ranges,
prepare() builds a case's handle and buffers from a seed, run() is one pass,
work() the bytes and operations a pass cannot do without, and exact() the
results of the first pass in plain FP64 torch.

A pass is what a program does between two frames of its trajectory: md_step
for a few steps, then md_get_state into its own buffers (or one force
evaluation, or one training step).  Frames, forces and energies of the FP32
pair path are handed on in FP32, as trajectory files hold them; forces of the
FP64 path in FP64.  A handle is not reset between passes: its trajectory goes
on.
"""
import math
import os

import numpy as np
import torch

from paper_2608_14911_amd import inputs, md
from paper_2608_14911_amd.system import Batch, System, lj_pair

WCA = 2.0 ** (1.0 / 6.0)
ADAM_EPS = 1e-3      # far above the rounding of a gradient component, far below a typical one
DATA = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_14911_amd", "data")
DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest everyday system: a 20 x 50 Kremer-Grest melt sampled every 50 steps with its
        # energies (integrator.run(50); computeEnergy()); latency and launches count
        dict(name="melt_1k", kind="kg", chains=20, chain_len=50, k_bend=1.5, gamma=1.0, skin=0.3, steps=50, energies=True),
        # the paper's example script: 10,000 random positions, capped warm-up at a small time step
        dict(name="warmup_10k", kind="warmup", n=10000, steps=50, energies=True),
        # a mid-size fluid of a ragged particle number, between two analysis frames
        dict(name="fluid_33k", kind="lj", n=33333, density=0.8, temperature=1.0, skin=0.3, steps=40),
        # the headline fluid
        dict(name="fluid_1m", kind="lj", n=1048576, density=0.8442, temperature=0.72, skin=0.3, steps=20),
        # the headline melt size: bonded forces, Langevin noise
        dict(name="melt_2m", kind="kg", chains=2000, chain_len=1000, k_bend=1.5, gamma=0.5, skin=0.4, steps=20, energies=False),
        # a parameter study: uneven replicas, fluids and melts, advanced together
        dict(name="replicas_48", kind="batch", systems=48, n_min=2048, n_max=65536, steps=40),
        # inference with the trained network on a large melt
        dict(name="surrogate_1m", kind="sur", chains=1000, chain_len=1000, precision="bf16", skin=0.3, steps=10),
        # one force evaluation with the FP32 network (labels, error estimates)
        dict(name="surrogate_forces_100k", kind="sur_forces", chains=100, chain_len=1000, precision="fp32", skin=0.4),
        # one training step: loss and gradient over a minibatch of four frames, then Adam
        dict(name="train_100k", kind="train", chains=100, chain_len=1000, frames=4, precision="fp32", skin=0.4),
        # a dissipative-particle-dynamics fluid under Lees-Edwards shear, soft tabulated repulsion
        dict(name="dpd_shear_1m", kind="dpd", n=1048576, density=3.0, shear=0.1, steps=10),
        # adaptive resolution on the fluid: an atomistic slab (capped, so that particles that overlapped in
        # the soft bath can enter it) in a tabulated coarse-grained bath, Langevin
        dict(name="adress_300k", kind="adress", n=299997, density=0.8442, steps=20),
        # reference forces in FP64 of a two-component mixture in a non-cubic box, with a fresh list
        dict(name="mixture_forces_fp64", kind="mixture", n=131000, density=0.8442),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["kg", "kg", "warmup", "lj", "lj", "batch", "sur", "sur_forces", "train", "dpd", "adress", "mixture"])
    if kind in ("kg", "sur", "sur_forces", "train"):
        n = _log(rng, 1000, 2000000) if kind == "kg" else _log(rng, 10000, 1000000 if kind == "sur" else 200000)
        length = rng.randint(10, 200) if n < 100000 else rng.randint(50, 1000)
        c = dict(kind=kind, chains=max(1, n // length), chain_len=length)
        if kind == "kg":
            c.update(k_bend=rng.choice([0.0, 1.5]), gamma=rng.choice([0.5, 1.0]), skin=rng.choice([0.3, 0.4, 0.5]),
                     steps=rng.randint(10, 50) if n < 100000 else rng.randint(10, 20), energies=n < 20000)
        else:
            c.update(precision=rng.choice(["bf16", "fp32"]) if n < 300000 else "bf16", skin=rng.choice([0.3, 0.4]))
            if kind == "sur":
                c.update(steps=rng.randint(2, 10))
            if kind == "train":
                c.update(frames=rng.randint(1, 4))
        return c
    if kind == "warmup":
        return dict(kind=kind, n=_log(rng, 2000, 40000), steps=rng.randint(20, 60), energies=True)
    if kind == "batch":
        return dict(kind=kind, systems=rng.randint(5, 48), n_min=2048, n_max=rng.choice([8192, 32768, 65536]), steps=rng.randint(10, 40))
    if kind == "dpd":
        return dict(kind=kind, n=_log(rng, 6000, 1048576), density=3.0, shear=rng.choice([0.05, 0.1, 0.3]), steps=rng.randint(5, 10))
    if kind == "mixture":
        return dict(kind=kind, n=_log(rng, 3000, 500000), density=rng.uniform(0.7, 0.9))
    if kind == "adress":
        return dict(kind=kind, n=_log(rng, 5000, 1048576), density=rng.uniform(0.7, 0.85), steps=rng.randint(10, 20))
    n = _log(rng, 2048, 1048576)
    return dict(kind=kind, n=n, density=rng.uniform(0.70, 0.90), temperature=rng.uniform(0.7, 1.2), skin=rng.choice([0.3, 0.4]),
                steps=rng.randint(10, 40) if n < 100000 else rng.randint(10, 20))


# ------------------------------------------------------------------ inputs
def _fluid(n, density, temperature, seed):
    """n of the sites of the smallest FCC lattice that holds them, at the
    density, jittered; Maxwell-Boltzmann velocities (as in the batch sampler)."""
    nc = int(math.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9))
    L = (n / density) ** (1.0 / 3.0)
    sites, _ = inputs.fcc_lattice(nc, 4.0 * nc ** 3 / L ** 3)
    g = inputs.rng(seed, inputs.STREAM_POS)
    if n < sites.shape[0]:
        sites = sites[np.sort(g.permutation(sites.shape[0])[:n])]
    box = np.array([L, L, L])
    pos = inputs.wrap_into_box(sites + g.uniform(-0.05, 0.05, size=sites.shape), box)
    return pos, box, inputs.maxwell_boltzmann(n, temperature, seed=seed)


def _melt(chains, chain_len, density, seed):
    """Chains laid through a simple cubic lattice (no push-off needed)."""
    w = inputs.lattice_melt(chains, chain_len, density, jitter=0.05, seed=seed)
    w["vel"] = inputs.maxwell_boltzmann(w["pos"].shape[0], 1.0, seed=seed, zero_momentum=False, exact=False)
    return w


def _members(case, seed):
    """The sampler's replicas (sizes, densities, temperatures and chain lengths
    of one study), with positions and velocities of their own."""
    out = []
    for k, r in enumerate(inputs.batch_replicas(case["systems"], seed=1003, n_min=case["n_min"], n_max=case["n_max"])):
        sub, n = 1000 * (int(seed) % 10 ** 9) + k, r["pos"].shape[0]
        if r["kind"] == "kg":
            w = inputs.lattice_melt(n // r["chain_len"], r["chain_len"], r["density"], jitter=0.05, seed=sub)
            r.update(pos=w["pos"], box=w["box"], bonds=w["bonds"], angles=w["angles"], skin=0.5,
                     vel=inputs.maxwell_boltzmann(n, r["temperature"], seed=sub, zero_momentum=False, exact=False))
        else:
            r["pos"], r["box"], r["vel"] = _fluid(n, r["density"], r["temperature"], sub)
        r["seed"] = sub
        out.append(r)
    return out


def _soft_table(a, rc, points):
    r = np.linspace(0.0, rc, points)
    return 0.5 * a * (1.0 - r / rc) ** 2, a * (1.0 - r / rc) / rc


MIX = {(0, 0): (1.0, 1.0, 2.5, math.nan, 0.0), (0, 1): (1.5, 0.9, 2.25, math.nan, 0.0), (1, 1): (0.5, 0.88, 2.2, math.nan, 0.0)}


def _setup(case, seed):
    """What defines the run, as plain host values: the System's arguments."""
    kind = case["kind"]
    seed = int(seed) % 10 ** 9
    if kind == "lj":
        pos, box, vel = _fluid(case["n"], case["density"], case["temperature"], seed)
        return dict(pos=pos, box=box, vel=vel, pair={(0, 0): lj_pair(rc=2.5)}, dt=0.005, skin=case["skin"], seed=seed)
    if kind == "kg":
        w = _melt(case["chains"], case["chain_len"], 0.85, seed)
        return dict(pos=w["pos"], box=w["box"], vel=w["vel"], bonds=w["bonds"], angles=w["angles"], pair={(0, 0): lj_pair(rc=WCA)},
                    k_bend=case["k_bend"], dt=0.01, skin=case["skin"], integrator="langevin", temperature=1.0, gamma=case["gamma"], seed=seed)
    if kind in ("sur", "sur_forces", "train"):
        w = _melt(case["chains"], case["chain_len"], 0.85, seed)
        return dict(pos=w["pos"], box=w["box"], vel=w["vel"], bonds=w["bonds"], angles=w["angles"], pair={(0, 0): lj_pair(rc=WCA)},
                    k_bend=1.5, dt=0.01, skin=case["skin"], integrator="langevin", temperature=1.0, gamma=0.5, seed=seed,
                    list_cutoff=md.MD_SUR_RCUT, surrogate=True)
    if kind == "warmup":
        L = (case["n"] / 1.25) ** (1.0 / 3.0)
        box = np.array([L, L, L])
        pos = inputs.random_positions(case["n"], box, seed=seed)
        return dict(pos=pos, box=box, vel=np.zeros_like(pos), pair={(0, 0): lj_pair(rc=1.12246, caprad=0.8)}, dt=0.0001, skin=0.3,
                    integrator="langevin", temperature=1.0, gamma=1.0, seed=seed)
    if kind == "dpd":
        L = (case["n"] / case["density"]) ** (1.0 / 3.0)
        box = np.array([L, L, L])
        pos = inputs.random_positions(case["n"], box, seed=seed)
        vel = inputs.maxwell_boltzmann(case["n"], 1.0, seed=seed)
        vel[:, 0] += case["shear"] * (pos[:, 1] - 0.5 * L)
        return dict(pos=pos, box=box, vel=vel, pair={(0, 0): lj_pair(rc=1.0)}, skin=0.3, dt=0.01, integrator="dpd", temperature=1.0,
                    gamma=4.5, seed=seed, dpd_rc=1.0, shear_rate=case["shear"], table_points=256)
    if kind == "adress":
        pos, box, vel = _fluid(case["n"], case["density"], 0.72, seed)
        L = box[0]
        return dict(pos=pos, box=box, vel=vel, pair={(0, 0): lj_pair(rc=2.5, caprad=0.8)}, skin=0.3, dt=0.005, integrator="langevin",
                    temperature=0.72, gamma=0.5, table_points=512, adress=(0.5 * L, L / 8.0, L / 8.0), seed=seed)
    pos, box, _ = _fluid(case["n"], case["density"], 1.0, seed)
    stretch = np.array([1.0, 1.1, 1.0 / 1.1])
    types = inputs.rng(seed, inputs.STREAM_BATCH).integers(0, 2, size=case["n"]).astype(np.int32)
    return dict(pos=pos * stretch, box=box * stretch, pair=MIX, n_types=2, types=types, masses=(1.0, 1.0), skin=0.3, dt=0.005,
                precision="fp64", seed=seed)


def _network(case, seed):
    """(theta, mean, istd): the trained weights, or the initial ones of a training run."""
    d = np.load(os.path.join(DATA, "surrogate_kg.npz"))
    theta = inputs.mlp_init(seed=int(seed) % 10 ** 9) if case["kind"] == "train" else d["theta_" + case["precision"]]
    return theta.astype(np.float32), d["g_mean"].astype(np.float32), d["g_istd"].astype(np.float32)


def _frames(case, seed, a):
    """Training frames: displaced copies of the melt, and their plain pair forces."""
    g = inputs.rng(int(seed) % 10 ** 9, inputs.STREAM_MINIBATCH)
    box = torch.as_tensor(a["box"], dtype=F64, device=DEVICE)
    pos = torch.as_tensor(a["pos"], dtype=F64, device=DEVICE)
    frames = []
    for _ in range(case["frames"]):
        d = torch.as_tensor(g.uniform(-0.06, 0.06, size=a["pos"].shape), dtype=F64, device=DEVICE)
        frames.append(torch.remainder(pos + d, box))
    frames = torch.stack(frames)
    model = _Model(case, a)
    f_ref = torch.stack([model.pair_terms(f, _pairs(f, box, WCA))[0] for f in frames])
    return frames, f_ref


def prepare(case, seed):
    if case["kind"] == "batch":
        members = _members(case, seed)
        b = Batch(members)
        ends = np.concatenate([[0], np.cumsum(b.n)])
        pos = torch.zeros((int(ends[-1]), 3), dtype=F64, device="cuda")
        return dict(case=case, b=b, pos=pos, vel=torch.zeros_like(pos), at=[int(e) for e in ends])
    a = _setup(case, seed)
    s = System(**a)
    n = s.n
    st = dict(case=case, s=s, pos=torch.zeros((n, 3), dtype=F64, device="cuda"), vel=torch.zeros((n, 3), dtype=F64, device="cuda"))
    if case["kind"] == "dpd":
        s.set_pair_table(0, 0, *_soft_table(25.0, 1.0, 256), 0.0)
    if case["kind"] == "adress":
        s.set_cg_table(0, 0, *_soft_table(20.0, 2.0, 512), 0.0, 2.0)
    if case["kind"] in ("sur", "sur_forces", "train"):
        s.sur_set(*_network(case, seed), case["precision"])
        if case["kind"] == "train":
            st["frames"], st["f_ref"] = _frames(case, seed, a)
            st["grad"] = torch.zeros(md.MD_SUR_NPARAM, dtype=torch.float32, device="cuda")
            st["theta"] = torch.zeros(md.MD_SUR_NPARAM, dtype=torch.float32, device="cuda")
            st["t"] = 0
        else:
            s.set_pair_mode("surrogate")
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "batch":
        b = st["b"]
        b.step(case["steps"])
        row = 3 * st["pos"].element_size()
        for k in range(b.nsys):
            off = st["at"][k] * row
            md.md_batch_get_state(b.h, k, st["pos"].data_ptr() + off, st["vel"].data_ptr() + off)
        return dict(pos=st["pos"].float(), vel=st["vel"].float())
    s = st["s"]
    if kind == "mixture":
        md.md_build_neighbors(s.h)
        md.md_forces(s.h, st["vel"])
        return st["vel"]
    if kind == "sur_forces":
        md.md_forces(s.h, st["vel"])
        return st["vel"].float()
    if kind == "train":
        st["t"] += 1
        loss = md.md_sur_loss_grad(s.h, st["frames"], st["f_ref"], case["frames"], st["grad"])
        md.md_sur_adam(s.h, st["t"], 3e-3, eps=ADAM_EPS)
        md.md_sur_get(s.h, st["theta"])
        return dict(loss=np.float32(loss), grad=st["grad"], theta=st["theta"])
    md.md_step(s.h, case["steps"])
    md.md_get_state(s.h, st["pos"], st["vel"])
    out = dict(pos=st["pos"].float(), vel=st["vel"].float())
    if case.get("energies"):
        o = md.md_observables(s.h)
        out["energies"] = np.array([o[k] for k in ("e_pair", "e_bond", "e_angle", "e_kin", "virial")], dtype=np.float32)
    return out


# ------------------------------------------------------------------ what a pass needs
def _count(case):
    return case["n"] if "n" in case else case["chains"] * case["chain_len"]


def work(case):
    """Positions and velocities read and written once per step (FP64), half a
    neighbour list (int32) and the topology read once per step, and about 30
    operations per pair inside the cutoff (the network's own for the surrogate)."""
    kind = case["kind"]

    def half(density, r):
        return density * 2.0 / 3.0 * math.pi * r ** 3

    if kind == "batch":
        n = case["systems"] * (case["n_max"] - case["n_min"]) / math.log(case["n_max"] / case["n_min"])
        per, flops = 96 + 4 * 0.5 * (half(0.8, 2.8) + half(0.8, WCA + 0.5)), 30 * 0.5 * (half(0.8, 2.5) + half(0.8, WCA))
        return {"bytes": n * per * case["steps"], "flops": n * flops * case["steps"]}
    n, steps = _count(case), case.get("steps", 1)
    if kind in ("lj", "adress"):
        skin = case.get("skin", 0.3)
        return {"bytes": n * steps * (96 + 4 * half(case["density"], 2.5 + skin)), "flops": n * steps * 30 * half(case["density"], 2.5)}
    if kind == "kg":
        return {"bytes": n * steps * (96 + 16 + 4 * half(0.85, WCA + case["skin"])), "flops": n * steps * (200 + 30 * half(0.85, WCA))}
    if kind == "warmup":
        return {"bytes": n * steps * (96 + 4 * half(1.25, 1.12246 + 0.3)), "flops": n * steps * 30 * half(1.25, 1.12246)}
    if kind == "dpd":
        return {"bytes": n * steps * (96 + 4 * half(3.0, 1.3)), "flops": n * steps * 120 * half(3.0, 1.0)}
    if kind == "mixture":
        return {"bytes": n * (48 + 4 * half(case["density"], 2.8)), "flops": n * (30 + 9) * half(case["density"], 2.5)}
    net = 2 * 2 * (32 * 64 + 64 * 64)
    flops = (134 + 262) * half(0.85, 2.5) + net
    data = 96 + 4 * half(0.85, 2.5 + case["skin"]) + 2 * 128
    if kind == "train":
        return {"bytes": n * case["frames"] * (48 + 4 * half(0.85, 2.5) + 4 * 128), "flops": n * case["frames"] * (2 * flops + 2 * net)}
    return {"bytes": n * steps * data, "flops": n * steps * flops}


# ------------------------------------------------------------------ the same in plain FP64
def _pairs(pos, box, r):
    """(i, j) of all pairs closer than r (each once), minimum image, through a
    cell grid; brute force when the box holds fewer than 3 cells."""
    n, dev = pos.shape[0], pos.device
    nc = [max(1, int(float(box[d]) / r)) for d in range(3)]
    found_i, found_j = [], []

    def keep(i, j):
        d = pos[j] - pos[i]
        d = d - box * torch.round(d / box)
        m = (d * d).sum(1) < r * r
        found_i.append(i[m])
        found_j.append(j[m])

    if min(nc) < 3:
        for a in range(0, n, 512):
            i = torch.arange(a, min(n, a + 512), device=dev)
            ii, jj = i.repeat_interleave(n), torch.arange(n, device=dev).repeat(len(i))
            m = jj > ii
            keep(ii[m], jj[m])
        return torch.cat(found_i), torch.cat(found_j)
    ncd = torch.tensor(nc, device=dev)
    c = torch.minimum((pos / box * ncd).long(), ncd - 1)
    cid = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
    order = torch.argsort(cid, stable=True)
    count = torch.bincount(cid, minlength=nc[0] * nc[1] * nc[2])
    start = torch.cumsum(count, 0) - count
    offsets = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dz, dy, dx) >= (0, 0, 0)]
    for o in offsets:
        m = torch.remainder(c + torch.tensor(o, device=dev), ncd)
        nb = (m[:, 2] * nc[1] + m[:, 1]) * nc[0] + m[:, 0]
        for part in torch.arange(n, device=dev).split(1 << 18):
            k = count[nb[part]]
            i = part.repeat_interleave(k)
            first = (torch.cumsum(k, 0) - k).repeat_interleave(k)
            j = order[start[nb[part]].repeat_interleave(k) + torch.arange(i.numel(), device=dev) - first]
            if o == (0, 0, 0):
                m0 = j > i
                i, j = i[m0], j[m0]
            keep(i, j)
    return torch.cat(found_i), torch.cat(found_j)


_M64 = 0xFFFFFFFF


def _mulhi64(a, b):
    """High 64 bits of the unsigned product of int64 bit patterns (b a Python int)."""
    a0, a1 = a & _M64, (a >> 32) & _M64
    b0, b1 = b & _M64, b >> 32

    def mul(x, y):  # 32 x 32 -> (high, low) without overflowing int64
        lo, hi = x * (y & 0xFFFF), x * (y >> 16)
        t = lo + ((hi & 0xFFFF) << 16)
        return (hi >> 16) + (t >> 32), t & _M64

    h00, _ = mul(a0, b0)
    h01, l01 = mul(a0, b1)
    h10, l10 = mul(a1, b0)
    h11, l11 = mul(a1, b1)
    mid = h00 + l01 + l10
    low = h01 + h10 + l11 + (mid >> 32)
    return ((h11 + (low >> 32)) << 32) | (low & _M64)


def _signed(k):
    k &= (1 << 64) - 1
    return k - (1 << 64) if k >> 63 else k


def _noise(seed, step, n):
    """Three N(0,1) draws per particle: Philox4x64-10 at counter (step, id, 0, 0), key (seed, 0)."""
    x = [torch.full((n,), step, dtype=torch.int64, device=DEVICE), torch.arange(n, device=DEVICE),
         torch.zeros(n, dtype=torch.int64, device=DEVICE), torch.zeros(n, dtype=torch.int64, device=DEVICE)]
    k0, k1 = seed, 0
    m0, m1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    for _ in range(10):
        h0, l0 = _mulhi64(x[0], m0), x[0] * _signed(m0)
        h1, l1 = _mulhi64(x[2], m1), x[2] * _signed(m1)
        x = [h1 ^ x[1] ^ _signed(k0), l1, h0 ^ x[3] ^ _signed(k1), l0]
        k0 += 0x9E3779B97F4A7C15
        k1 += 0xBB67AE8584CAA73B
    u = [(((w >> 11) & ((1 << 53) - 1)).to(F64) + 0.5) * 2.0 ** -53 for w in x]
    r0, r1 = torch.sqrt(-2.0 * torch.log(u[0])), torch.sqrt(-2.0 * torch.log(u[2]))
    return torch.stack([r0 * torch.cos(2 * math.pi * u[1]), r0 * torch.sin(2 * math.pi * u[1]), r1 * torch.cos(2 * math.pi * u[3])], 1)


def _theta(seed, step, i, j):
    """The DPD pair draw: Philox4x32-10 at (step words, min id, max id), key (seed words, high ^ 6)."""
    x = [torch.full_like(i, step & _M64), torch.full_like(i, step >> 32), torch.minimum(i, j), torch.maximum(i, j)]
    k0, k1 = seed & _M64, (seed >> 32) ^ 6

    def mul(v, m):  # 32 x 32 -> (high, low) words
        lo, hi = v * (m & 0xFFFF), v * (m >> 16)
        t = lo + ((hi & 0xFFFF) << 16)
        return ((hi >> 16) + (t >> 32)) & _M64, t & _M64

    for _ in range(10):
        h0, l0 = mul(x[0], 0xD2511F53)
        h1, l1 = mul(x[2], 0xCD9E8D57)
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & _M64, (k1 + 0xBB67AE85) & _M64
    u0, u1 = ((w.to(F64) + 0.5) * 2.0 ** -32 for w in x[:2])
    return torch.sqrt(-2.0 * torch.log(u0)) * torch.cos(2 * math.pi * u1)


def _linear(table, r, rc):
    """A uniform table from 0 to rc, interpolated linearly (stored in FP32)."""
    t = torch.as_tensor(table.astype(np.float32).astype(np.float64), device=r.device)
    q = r * (len(table) - 1) / rc
    k = q.long().clamp(0, len(table) - 2)
    w = q - k
    return (1 - w) * t[k] + w * t[k + 1]


class _Model:
    """The forces of a case, written from their definitions."""

    def __init__(self, case, a, net=None):
        self.case, self.a = case, a
        self.box = torch.as_tensor(np.asarray(a["box"]), dtype=F64, device=DEVICE)
        self.bonds, self.angles = ([torch.as_tensor(np.asarray(a[k]), dtype=torch.int64, device=DEVICE) if a.get(k) is not None else None
                                    for k in ("bonds", "angles")])
        self.types = torch.as_tensor(a["types"], dtype=torch.int64, device=DEVICE) if a.get("types") is not None else None
        self.net = net
        self.delta = 0.0     # Lees-Edwards offset

    def image(self, d):
        L = self.box
        if self.a.get("shear_rate"):
            s = (d[:, 1] > 0.5 * L[1]).to(F64) - (d[:, 1] < -0.5 * L[1]).to(F64)
            x = d[:, 0] - L[0] * torch.round(d[:, 0] / L[0]) - s * self.delta
            d = torch.stack([x, d[:, 1], d[:, 2]], 1)
        return d - L * torch.round(d / L)

    def reach(self):
        return max([p[2] for p in self.a["pair"].values()] + [self.a.get("list_cutoff", 0.0)])

    def plain(self, i, j, r2):
        """(u, f / r) of the pair table."""
        u, fr = torch.zeros_like(r2), torch.zeros_like(r2)
        for (p, q), (eps, sig, rc, _, cap) in self.a["pair"].items():
            m = r2 < rc * rc
            if self.types is not None:
                lo, hi = torch.minimum(self.types[i], self.types[j]), torch.maximum(self.types[i], self.types[j])
                m = m & (lo == p) & (hi == q)
            rr = torch.clamp(r2, min=cap * cap) if cap > 0 else r2
            s6 = (sig * sig / rr) ** 3
            c6 = (sig * sig / (rc * rc)) ** 3
            u = u + m * 4 * eps * ((s6 * s6 - s6) - (c6 * c6 - c6))
            f = 24 * eps * (2 * s6 * s6 - s6) / rr
            if cap > 0:
                f = f * torch.sqrt(rr / r2)
            fr = fr + m * f
        return u, fr

    def weight(self, x):
        x0, dat, dhy = self.a["adress"]
        d = x - x0
        d = (d - self.box[0] * torch.round(d / self.box[0])).abs()
        w = torch.cos(0.5 * math.pi * (d - dat) / dhy) ** 2
        return torch.where(d < dat, torch.ones_like(d), torch.where(d >= dat + dhy, torch.zeros_like(d), w))

    def pair_terms(self, x, ij, v=None, step=0):
        """(F, e_pair, W) of the non-bonded pairs; v: the DPD thermostat's velocities."""
        F, e, W = torch.zeros_like(x), 0.0, 0.0
        for i, j in zip(ij[0].split(1 << 24), ij[1].split(1 << 24)):
            raw = x[j] - x[i]
            d = self.image(raw)
            r2 = (d * d).sum(1)
            m = r2 < self.reach() ** 2
            i, j, d, r2, raw = i[m], j[m], d[m], r2[m], raw[m]
            if self.case["kind"] == "dpd":
                r = torch.sqrt(r2)
                tab = _soft_table(25.0, 1.0, 256)
                u, fr = _linear(tab[0], r, 1.0), _linear(tab[1], r, 1.0) / r
            else:
                u, fr = self.plain(i, j, r2)
            if self.case["kind"] == "adress":
                r = torch.sqrt(r2)
                tab = _soft_table(20.0, 2.0, 512)
                lam, in_cg = self.weight(x[i, 0]) * self.weight(x[j, 0]), r < 2.0
                u = lam * u + (1 - lam) * in_cg * _linear(tab[0], r, 2.0)
                fr = lam * fr + (1 - lam) * in_cg * _linear(tab[1], r, 2.0) / r
            e = e + u.sum()
            W = W + (fr * r2).sum()
            if v is not None:
                r = torch.sqrt(r2)
                ev = -d / r[:, None]
                s = (raw[:, 1] > 0.5 * self.box[1]).to(F64) - (raw[:, 1] < -0.5 * self.box[1]).to(F64)
                vij = v[i] - v[j]
                vij[:, 0] += s * self.a["shear_rate"] * float(self.box[1])
                w = 1 - r
                A = -self.a["gamma"] * w * w * (ev * vij).sum(1)
                A = A + math.sqrt(2 * self.a["gamma"] * self.a["temperature"] / self.a["dt"]) * w * _theta(self.a["seed"], step, i, j)
                fr = fr + A / r
            f = -fr[:, None] * d
            F.index_add_(0, i, f)
            F.index_add_(0, j, -f)
        return F, e, W

    def energy(self, x, ij, theta=None):
        """Total energy of the network (differentiable)."""
        th = self.net[0] if theta is None else theta
        mean, istd = self.net[1:]
        W1, b1, W2, b2, w3, b3 = th[:2048].view(64, 32), th[2048:2112], th[2112:6208].view(64, 64), th[6208:6272], th[6272:6336], th[6336]
        mu = md.MD_SUR_MU0 + torch.arange(32, dtype=F64, device=DEVICE) * (md.MD_SUR_MU1 - md.MD_SUR_MU0) / 31
        d = self.image(x[ij[1]] - x[ij[0]])
        r = torch.sqrt((d * d).sum(1))
        g = torch.exp(-(r[:, None] - mu) ** 2 / (2 * md.MD_SUR_WIDTH ** 2)) * (0.5 * torch.cos(math.pi * r / md.MD_SUR_RCUT) + 0.5)[:, None]
        G = torch.zeros((x.shape[0], 32), dtype=F64, device=DEVICE).index_add(0, ij[0], g).index_add(0, ij[1], g)
        h = torch.nn.functional.silu((G - mean) * istd @ W1.T + b1)
        return (torch.nn.functional.silu(h @ W2.T + b2) @ w3 + b3).sum()

    def network(self, x, ij):
        d = self.image(x[ij[1]] - x[ij[0]])
        m = (d * d).sum(1) < md.MD_SUR_RCUT ** 2
        y = x.detach().requires_grad_(True)
        with torch.enable_grad():
            e = self.energy(y, (ij[0][m], ij[1][m]))
            g, = torch.autograd.grad(e, y)
        return -g, e.detach(), 0.0

    def bonded(self, x):
        F, eb, ea, W = torch.zeros_like(x), 0.0, 0.0, 0.0
        if self.bonds is not None and len(self.bonds):
            i, j = self.bonds[:, 0], self.bonds[:, 1]
            d = self.image(x[i] - x[j])
            r2 = (d * d).sum(1)
            fr = -30.0 / (1 - r2 / 2.25)
            F.index_add_(0, i, fr[:, None] * d)
            F.index_add_(0, j, -fr[:, None] * d)
            eb, W = (-0.5 * 30.0 * 2.25 * torch.log(1 - r2 / 2.25)).sum(), W + (fr * r2).sum()
        if self.angles is not None and len(self.angles) and self.a["k_bend"]:
            p, q, s = self.angles.unbind(1)
            b1, b2 = self.image(x[q] - x[p]), self.image(x[s] - x[q])
            l1, l2 = (b1 * b1).sum(1), (b2 * b2).sum(1)
            il = 1 / torch.sqrt(l1 * l2)
            c = (b1 * b2).sum(1) * il
            k = self.a["k_bend"]
            fp = -k * (b2 * il[:, None] - b1 * (c / l1)[:, None])
            fs = k * (b1 * il[:, None] - b2 * (c / l2)[:, None])
            F.index_add_(0, p, fp)
            F.index_add_(0, s, fs)
            F.index_add_(0, q, -fp - fs)
            ea, W = (k * (1 - c)).sum(), W + (b2 * fs).sum() - (b1 * fp).sum()
        return F, eb, ea, W


def _trajectory(case, a, steps, net=None):
    """x_n, v_{n-1/2} and the energies of step n after `steps` steps of velocity Verlet."""
    model = _Model(case, a, net)
    x, v = (torch.as_tensor(np.asarray(a[k]), dtype=F64, device=DEVICE) for k in ("pos", "vel"))
    n, dt, box = x.shape[0], a["dt"], model.box
    x = torch.remainder(x, box)
    langevin, dpd = a.get("integrator") == "langevin", a.get("integrator") == "dpd"
    rate = a.get("shear_rate", 0.0) * float(box[1])
    # one pair list, wide enough for several steps; the sheared image moves too
    slack = 0.6 + abs(rate) * dt * steps
    ij, x0 = _pairs(x, box, model.reach() + slack), x.clone()
    half = False
    for step in range(steps + 1):
        if not rate:
            d = model.image(x - x0)
            if 2 * float(torch.sqrt((d * d).sum(1).max())) > 0.55:
                ij, x0 = _pairs(x, box, model.reach() + slack), x.clone()
        model.delta = math.fmod(rate * step * dt, float(box[0]))
        if net is not None:
            F, ep, W = model.network(x, ij)
        else:
            F, ep, W = model.pair_terms(x, ij, v if dpd and step < steps else None, step)
        Fb, eb, ea, Wb = model.bonded(x)
        F = F + Fb
        if langevin:
            F = F - a["gamma"] * v + math.sqrt(2 * a["gamma"] * a["temperature"] / dt) * _noise(a["seed"], step, n)
        on = v + 0.5 * dt * F if half else v
        if step == steps:
            return x, v, torch.stack([torch.as_tensor(t, dtype=F64, device=DEVICE) for t in (ep, eb, ea, 0.5 * (on * on).sum(), W + Wb)])
        v = on + 0.5 * dt * F
        x = x + dt * v
        half = True
        if rate:
            nxt = math.fmod(rate * (step + 1) * dt, float(box[0]))
            s = (x[:, 1] >= box[1]).to(F64) - (x[:, 1] < 0).to(F64)
            x[:, 0] -= s * nxt
            v[:, 0] -= s * rate
        x = torch.remainder(x, box)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        got = []
        for m in _members(case, seed):
            got.append(_trajectory(dict(kind=m["kind"]), m, case["steps"])[:2])
        return dict(pos=torch.cat([g[0] for g in got]), vel=torch.cat([g[1] for g in got]))
    a = _setup(case, seed)
    net = None
    if kind in ("sur", "sur_forces", "train"):
        net = [torch.as_tensor(t, dtype=F64, device=DEVICE) for t in _network(case, seed)]
    if kind in ("mixture", "sur_forces"):
        model = _Model(case, a, net)
        x = torch.remainder(torch.as_tensor(a["pos"], dtype=F64, device=DEVICE), model.box)
        ij = _pairs(x, model.box, model.reach())
        return model.pair_terms(x, ij)[0] if kind == "mixture" else model.network(x, ij)[0] + model.bonded(x)[0]
    if kind == "train":
        model = _Model(case, a, net)
        frames, f_ref = _frames(case, seed, a)
        theta = net[0].clone().requires_grad_(True)
        loss = 0.0
        for x, f in zip(frames, f_ref):
            y = x.clone().requires_grad_(True)
            ij = _pairs(x, model.box, md.MD_SUR_RCUT)
            e = model.energy(y, ij, theta)
            g, = torch.autograd.grad(e, y, create_graph=True)
            part = ((-g - f) ** 2).sum() / frames.numel()
            part.backward()
            loss = loss + float(part.detach())
        g = theta.grad
        moved = net[0] - 3e-3 * g / (g.abs() + ADAM_EPS)     # the first Adam step from zero moments
        return dict(loss=loss, grad=g, theta=moved)
    x, v, e = _trajectory(case, a, case["steps"], net)
    out = dict(pos=x, vel=v)
    if case.get("energies"):
        out["energies"] = e
    return out
