"""The work a program has this library do, as measurable cases.

Each case names an entry point ("do"), a kind of system, its size and its
options; listed() holds the ones that stand for everyday use, draw() gives
others of the same ranges, prepare() builds what a program holds before the
call, run() is one pass through the public entry points, and exact() is the
same answer in 64 bits from plain torch.

Systems: rigid-water boxes at 1.0 g/cm^3, organic-like periodic boxes at 0.1
atoms/A^3 (H/C/O/N/S/F/Cl mix, no two atoms closer than 0.9 A), and open
chain-grown molecules of 8 to 150 atoms.  The model has the ANI-2x shape
(7 species, 1008 features, 1008-256-192-160-1 CELU networks) with random
weights that do not depend on the seed, as a program loads one model and
evaluates many geometries.  Random weights hold no repulsion: dynamics runs on
a copy whose energies are scaled down to a fraction of k_B T, so that the
fluid keeps its density however long a trajectory is continued.

Structure energies come back as float64 sums of float32 atomic energies; the
cases return the atomic energies themselves, or the sum as the float32 (or
Python) number that carries all of its accuracy.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2405_01491_amd as nnp
from paper_2405_01491_amd import md as nmd
from paper_2405_01491_amd.server import Server, nnp_poll, nnp_submit

H, C, N, O, F, S, CL = range(7)
MASSES = np.array([1.008, 12.011, 14.007, 15.999, 18.998, 32.06, 35.45])
MIX = ((H, 0.50), (C, 0.25), (O, 0.12), (N, 0.08), (S, 0.03), (F, 0.01), (CL, 0.01))
WIDTHS = (1008, 256, 192, 160, 1)


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one small molecule, list, energy and forces, results on the host: an
        # optimiser's or a scan's single call, where latency and launches count
        dict(name="molecule_host", do="host", system="molecule", n=19),
        # requests of many users in one go through the batching server
        dict(name="serve_48", do="serve", system="molecule", n=48),
        # a batch of molecules with the energy differentiated through autograd
        # (fitting to energies, batched relaxation): forward and backward
        dict(name="batch_grad_96", do="grad", system="molecule", n=96),
        # Langevin dynamics of the smallest benchmark box (216 waters, 2 A skin, rebuild every 80 steps)
        dict(name="md_648", do="md", system="water", n=216, steps=10, skin=2.0, every=80),
        # 1,500 waters with the list rebuilt on every step
        dict(name="md_4500", do="md", system="water", n=1500, steps=10, skin=0.0, every=1),
        # the largest box: 33,333 waters, 0.5 A skin
        dict(name="md_99999", do="md", system="water", n=33333, steps=5, skin=0.5, every=20),
        # an organic box of the size of a solvated protein, where every species is near every atom
        dict(name="organic_23000", do="forces", system="organic", n=23000),
        # forces with virials per structure and per atom: constant-pressure dynamics
        dict(name="virial_6000", do="virial", system="water", n=2000),
        # eight networks on one feature vector: mean, spread and forces
        dict(name="ensemble8_99999", do="ensemble", system="water", n=33333, nets=8),
        # the networks alone, forward and adjoint, float32, an odd number of atoms
        dict(name="mlp_6001", do="mlp", system="organic", n=6001, precision="fp32"),
        # the same in the form with bfloat16 matrix products.  (That form is
        # measured here, where its inputs are given: behind other layers one
        # rounding of a feature travels through all bfloat16 roundings after it.)
        dict(name="mlp_23000_bf16", do="mlp", system="organic", n=23000, precision="bf16"),
        # the neighbour list alone
        dict(name="neighbors_99999", do="neighbors", system="water", n=33333),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    do = rng.choice(["host", "serve", "grad", "md", "md", "forces", "forces", "virial", "ensemble", "mlp", "mlp",
                     "neighbors", "aev"])
    if do == "host":
        return dict(do=do, system="molecule", n=size(8, 150))
    if do == "serve":
        return dict(do=do, system="molecule", n=size(4, 56))
    if do == "grad":
        return dict(do=do, system="molecule", n=size(2, 128))
    if do == "md":
        skin, every = rng.choice([(0.0, 1), (0.5, 20), (2.0, 80)])
        return dict(do=do, system="water", n=size(150, 20000), steps=rng.randint(3, 6), skin=skin, every=every)
    system = rng.choice(["water", "organic"])
    per = 3 if system == "water" else 1
    if do == "neighbors":
        return dict(do=do, system=system, n=size(1500, 90000) // per)
    if do == "mlp":
        return dict(do=do, system=system, n=size(450, 24000) // per, precision=rng.choice(["fp32", "bf16"]))
    if do == "ensemble":
        return dict(do=do, system=system, n=size(450, 24000) // per, nets=rng.choice([2, 3, 5, 8]))
    return dict(do=do, system=system, n=size(450, 40000) // per)


# ---------------------------------------------------------------- systems

def rotations(rng, n):
    q = rng.normal(size=(n, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                     2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                     2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], -1).reshape(n, 3, 3)


def lattice_sites(rng, n, side):
    """n of the sites of the smallest simple cubic lattice that has n."""
    m = math.ceil(n ** (1 / 3) - 1e-9)
    pick = np.sort(rng.choice(m ** 3, size=n, replace=False))
    return (np.stack(np.unravel_index(pick, (m, m, m)), -1) + 0.5) * (side / m), side / m


def wrap(x, side):
    y = np.mod(x, side).astype(np.float32)
    return np.where(y >= np.float32(side), np.float32(0), y)


def water(rng, n_mol):
    side = max((n_mol * 18.01528 / 0.602214076) ** (1 / 3), 15.0)
    r, th = 0.9572, math.radians(104.52)
    local = np.array([[0, 0, 0], [r * math.sin(th / 2), 0, r * math.cos(th / 2)],
                      [-r * math.sin(th / 2), 0, r * math.cos(th / 2)]])
    xyz = lattice_sites(rng, n_mol, side)[0][:, None, :] + local @ rotations(rng, n_mol).transpose(0, 2, 1)
    species = np.tile(np.array([O, H, H], np.int32), n_mol)
    return wrap(xyz.reshape(-1, 3), side), species, np.full(3, side, np.float32)


def organic(rng, n):
    side = max((n / 0.1) ** (1 / 3), 15.0)
    sites, a = lattice_sites(rng, n, side)
    half = max(0.0, (a - 0.9) / 2)
    species = rng.choice(np.array([s for s, _ in MIX], np.int32), size=n, p=[p for _, p in MIX])
    return wrap(sites + rng.uniform(-half, half, size=(n, 3)), side), species, np.full(3, side, np.float32)


def molecule(rng, n):
    """Grown atom by atom: 0.95 to 1.6 A from one of the last four atoms, 1.5 A from every other."""
    x = np.zeros((n, 3))
    k = 1
    while k < n:
        parent = k - 1 - rng.integers(0, min(4, k), size=24)
        d = rng.normal(size=(24, 3))
        c = x[parent] + d * (rng.uniform(0.95, 1.6, size=24) / np.linalg.norm(d, axis=1))[:, None]
        d2 = ((c[:, None] - x[None, :k]) ** 2).sum(-1)
        d2[np.arange(24), parent] = np.inf
        ok = np.nonzero((d2 >= 2.25).all(1))[0]
        if len(ok):
            x[k] = c[ok[0]]
            k += 1
        else:
            k = 1   # a crowded tail: grow it again
    species = rng.choice(np.array([s for s, _ in MIX], np.int32), size=n, p=[p for _, p in MIX])
    return (x - x.mean(0)).astype(np.float32), species


def molecules(rng, count):
    # sizes spread evenly over the logarithm of 8 to 150, in an order of the seed's
    sizes = rng.permutation(np.exp(np.linspace(math.log(8), math.log(150.9), count)).astype(int))
    return [molecule(rng, int(n)) for n in sizes]


def system_of(case, seed):
    """(pos, species, box, mol, n_mol) as host arrays."""
    rng = np.random.default_rng(1_000_003 * (seed + 1))
    if case["system"] == "molecule":
        if case["do"] == "host":
            pos, species = molecule(rng, case["n"])
            return pos, species, None, None, 1
        mols = molecules(rng, case["n"])
        mol = np.repeat(np.arange(len(mols), dtype=np.int32), [len(s) for _, s in mols])
        return np.concatenate([p for p, _ in mols]), np.concatenate([s for _, s in mols]), None, mol, len(mols)
    pos, species, box = (water if case["system"] == "water" else organic)(rng, case["n"])
    return pos, species, box, None, 1


# ---------------------------------------------------------------- the model

@functools.lru_cache(maxsize=None)
def spec_of(nets, scale=1.0):
    f = np.float32

    def weights(seed):
        rng = np.random.default_rng(seed)
        out = []
        for _ in range(7):
            layers = []
            for a, b in zip(WIDTHS, WIDTHS[1:]):
                lim = math.sqrt(6 / (a + b))
                layers.append((rng.uniform(-lim, lim, size=(b, a)).astype(f),
                               rng.uniform(-0.05, 0.05, size=b).astype(f)))
            layers[-1] = tuple(v * f(scale) for v in layers[-1])
            out.append(layers)
        return out

    every = [weights(123456 + k) for k in range(nets)]
    return SimpleNamespace(
        n_species=7, rc_r=5.1, eta_r=19.7, shf_r=np.array([0.8 + 0.26875 * k for k in range(16)], f), rc_a=3.5,
        eta_a=12.5, zeta=14.1, shf_a=np.array([0.8 + 0.3375 * k for k in range(4)], f),
        shf_z=np.array([(2 * k + 1) * math.pi / 16 for k in range(8)], f), radial_prefactor=0.25, cos_scale=0.95,
        widths=WIDTHS, celu_alpha=0.1, weights=every[0], self_energy=np.zeros(7),
        ensemble=every if nets > 1 else None)


@functools.lru_cache(maxsize=None)
def model_of(precision, nets, scale):
    return nnp.Model(spec_of(nets, scale), precision)


# ---------------------------------------------------------------- one pass

def prepare(case, seed):
    do = case["do"]
    m = model_of(case.get("precision", "fp32"), case.get("nets", 1), 1 / 1024 if do == "md" else 1.0)
    pos, species, box, mol, n_mol = system_of(case, seed)
    st = SimpleNamespace(do=do, model=m, box=box, n_mol=n_mol, nl=None)
    if do == "serve":
        cut = np.searchsorted(mol, np.arange(n_mol + 1))
        st.requests = [(species[a:b], pos[a:b]) for a, b in zip(cut, cut[1:])]
        st.server = Server(m)
        return st
    st.pos = torch.from_numpy(pos).cuda()
    st.species = torch.from_numpy(species).cuda()
    st.mol = None if mol is None else torch.from_numpy(mol).cuda()
    if do == "md":
        masses = MASSES[species]
        vel = torch.from_numpy(nmd.maxwell_boltzmann(masses, 300.0, seed)).cuda()
        st.engine = nmd.MDEngine(m, st.pos, vel, st.species, masses, box, dt=0.5, integrator="langevin",
                                 temperature=300.0, friction=1.0, seed=seed, skin=case["skin"],
                                 rebuild_every=case["every"])
        st.steps = case["steps"]
    elif do == "neighbors":
        # the list's buffers, held across builds: entries past the last pair stay as they are
        st.nl = nnp.NeighborList(len(species), 80 * len(species), st.pos.device)
        for t in (st.nl.col, st.nl.shift, st.nl.rev):
            t.zero_()
    elif do == "mlp":
        st.aev = torch.zeros((len(species), m.aev_stride), dtype=torch.float32, device="cuda")
        for rows, feats in aev_chunks(torch.from_numpy(pos).cuda().double(), st.species.long(), box):
            st.aev[rows, :feats.shape[1]] = feats.float()
    elif do == "grad":
        st.target = torch.from_numpy(np.random.default_rng(seed).normal(size=n_mol).astype(np.float32)).cuda()
    return st


def run(st):
    m, do = st.model, st.do
    if do == "host":
        nl = nnp.nnp_neighbors(m, st.pos)
        e, _, forces = nnp.nnp_energy_forces(m, st.pos, st.species, nl=nl)
        return float(e), forces.cpu().numpy()
    if do == "serve":
        tickets = [nnp_submit(st.server, species, pos) for species, pos in st.requests]
        got = {}
        while len(got) < len(tickets):
            for t in tickets:
                if t not in got:
                    r = nnp_poll(st.server, t)
                    if r is not None:
                        got[t] = r
        return np.array([got[t][0] for t in tickets], np.float32), np.concatenate([got[t][1] for t in tickets])
    if do == "grad":
        x = st.pos.detach().requires_grad_(True)
        e = nnp.energy(m, x, st.species, st.mol, st.n_mol).float()
        ((e - st.target) ** 2).mean().backward()
        return e.detach(), x.grad
    if do == "md":
        st.engine.run(st.steps)
        pos, vel, forces, e = st.engine.state()
        return pos, vel, forces, e.float()
    if do == "mlp":
        return nnp.nnp_mlp(m, st.species, st.aev)
    # a program that evaluates one geometry after another keeps its list's buffers
    st.nl = nnp.nnp_neighbors(m, st.pos, st.mol, st.n_mol, st.box, nl=st.nl)
    if do == "neighbors":
        return st.nl.row_ptr, st.nl.col, st.nl.shift, st.nl.rev
    if do == "aev":
        return nnp.nnp_aev(m, st.pos, st.species, st.box, st.nl)
    if do == "ensemble":
        _, e_net, e_atom, forces = nnp.nnp_energy_forces_ensemble(m, st.pos, st.species, st.mol, st.n_mol, st.box,
                                                                  st.nl, e_atom=True)
        return e_net.float(), e_atom, forces
    out = {}
    _, e_atom, forces = nnp.nnp_energy_forces(m, st.pos, st.species, st.mol, st.n_mol, st.box, st.nl, e_atom=True,
                                              out=out, virial=do == "virial", atom_virial=do == "virial")
    if do == "virial":
        return e_atom, forces, out["virial"].float(), out["atom_virial"]
    return e_atom, forces


# ---------------------------------------------------------------- what a pass cannot do without

# per atom: pairs within 5.1 A, unordered pairs of neighbours within 3.5 A, features that can be non-zero
DENSITY = {"water": (55.6, 143, 128), "organic": (55.6, 150, 1008), "molecule": (28, 60, 560)}


def work(case):
    do, nets = case["do"], case.get("nets", 1)
    pairs, triples, feats = DENSITY[case["system"]]
    atoms = case["n"] * {"water": 3, "organic": 1, "molecule": 1 if do == "host" else 48.6}[case["system"]]
    if do == "neighbors":
        # each pair is tested once from each side; positions in, rows, columns, shifts and reverse indices out
        return {"bytes": atoms * (12 + 4 + 11 * pairs), "flops": atoms * pairs * 10}
    if do == "mlp":
        feats = 1008
    per_net = feats * 256 + 256 * 192 + 192 * 160 + 160
    net = 2 * 2 * per_net                                               # forward and adjoint
    weights = 4 * {"water": 2, "organic": 7, "molecule": 7}[case["system"]] * per_net
    features = pairs * 16 * 5 + triples * (8 * 6 + 4 * 4 + 32 * 2)
    if do == "mlp":
        return {"bytes": atoms * (2 * 4 * 1024 + 8) + weights, "flops": atoms * net}
    if do == "aev":
        return {"bytes": atoms * (16 + 11 * pairs + 4 * 1024), "flops": atoms * features}
    steps = case.get("steps", 1)
    per_atom = 16 + 12 + 4 + (24 if do == "md" else 0) + (36 if do == "virial" else 0)
    return {"bytes": steps * (atoms * per_atom + nets * weights), "flops": steps * atoms * (3 * features + nets * net)}


# ---------------------------------------------------------------- the same in 64 bits

def f64(x):
    return torch.as_tensor(np.asarray(x, np.float32).astype(np.float64)).cuda()


def rows_near(x, box, mol, rows, cut):
    """(row position, neighbour, image vector) of every pair within cut of the atoms `rows`."""
    d = x[None] - x[rows, None]
    n = torch.zeros_like(d) if box is None else -torch.round(d / f64(box))
    if box is not None:
        d = d + n * f64(box)
    near = (d * d).sum(-1) < float(np.float32(cut)) ** 2
    near[torch.arange(len(rows), device=x.device), rows] = False
    if mol is not None:
        near &= mol[None] == mol[rows, None]
    i, j = near.nonzero(as_tuple=True)
    return i, j, n[i, j] if box is None else n[i, j] * f64(box)


def slots(i, count):
    """Position of each entry of the sorted rows i within its row, and the longest row."""
    per = torch.bincount(i, minlength=count)
    return torch.arange(len(i), device=i.device) - (per.cumsum(0) - per)[i], int(per.max()) if len(i) else 0


def aev_rows(x, species, box, mol, rows):
    p = spec_of(1)
    dev, n = x.device, len(rows)
    with torch.no_grad():
        i, j, image = rows_near(x, box, mol, rows, p.rc_r)
    v = x[j] - x[rows[i]] + image
    r = (v * v).sum(-1).sqrt()
    fc = 0.5 * torch.cos(math.pi * r / f64(p.rc_r)) + 0.5
    g = f64(p.radial_prefactor) * torch.exp(-f64(p.eta_r) * (r[:, None] - f64(p.shf_r)) ** 2) * fc[:, None]
    radial = torch.zeros((n * 7, 16), dtype=x.dtype, device=dev).index_add(0, i * 7 + species[j], g).reshape(n, -1)
    # angular: the rows of the closer neighbours, padded, and every pair of their entries
    a = (r.detach() < f64(p.rc_a)).nonzero()[:, 0]
    at, most = slots(i[a], n)
    out = torch.zeros((n * 28, 32), dtype=x.dtype, device=dev)
    if most > 1:
        pad = torch.full((n, most), -1, dtype=torch.long, device=dev)
        pad[i[a], at] = a
        ja, ka = torch.triu_indices(most, most, 1, device=dev)
        e1, e2 = pad[:, ja].reshape(-1), pad[:, ka].reshape(-1)
        both = ((e1 >= 0) & (e2 >= 0)).nonzero()[:, 0]
        e1, e2 = e1[both], e2[both]
        u = f64(p.cos_scale) * ((v[e1] * v[e2]).sum(-1) / (r[e1] * r[e2])).clamp(-1, 1)
        w = u[:, None] * torch.cos(f64(p.shf_z)) + (1 - u * u).sqrt()[:, None] * torch.sin(f64(p.shf_z))
        f1 = (0.5 * (1 + w)).clamp(min=1e-300) ** f64(p.zeta)
        f2 = torch.exp(-f64(p.eta_a) * (0.5 * (r[e1] + r[e2])[:, None] - f64(p.shf_a)) ** 2)
        fca = 0.5 * torch.cos(math.pi * r / f64(p.rc_a)) + 0.5
        t = (2 * fca[e1] * fca[e2])[:, None, None] * f2[:, :, None] * f1[:, None, :]
        s = torch.minimum(species[j[e1]], species[j[e2]])
        q = torch.maximum(species[j[e1]], species[j[e2]])
        bins = s * 7 - s * (s - 1) // 2 + (q - s)
        out = out.index_add(0, i[e1] * 28 + bins, t.reshape(-1, 32))
    return torch.cat([radial, out.reshape(n, -1)], 1), (i, j, v)


def chunks_of(n):
    step = max(64, min(3000, 200_000_000 // max(n, 1)))
    for a in range(0, n, step):
        yield torch.arange(a, min(n, a + step), device="cuda")


def aev_chunks(x, species, box):
    with torch.no_grad():
        for rows in chunks_of(len(x)):
            yield rows, aev_rows(x, species, box, None, rows)[0]


def networks(feats, species, nets):
    """Atomic energies [nets, rows] of the rows' features."""
    p = spec_of(nets)
    e = torch.zeros((nets, len(species)), dtype=torch.float64, device=feats.device)
    for s in species.unique().tolist():
        at = (species == s).nonzero()[:, 0]
        for k, weights in enumerate(p.ensemble or [p.weights]):
            h = feats[at]
            for layer, (w, b) in enumerate(weights[s]):
                h = h @ f64(w).t() + f64(b)
                if layer < 3:
                    h = torch.nn.functional.celu(h, float(np.float32(p.celu_alpha)))
            e = e.index_put((torch.full_like(at, k), at), h[:, 0])
    return e


def exact(case, seed):
    do, nets = case["do"], case.get("nets", 1)
    if do in ("md", "neighbors"):
        return None
    pos, species, box, mol, n_mol = system_of(case, seed)
    if do == "mlp":
        st = prepare(case, seed)
        e, g = [], []
        for rows in chunks_of(len(species)):
            a = st.aev[rows].double().requires_grad_(True)
            with torch.enable_grad():
                ek = networks(a[:, :WIDTHS[0]], st.species[rows].long(), 1)[0]
                g.append(torch.autograd.grad(ek.sum(), a)[0])
            e.append(ek.detach())
        return torch.cat(e), torch.cat(g)
    x = torch.from_numpy(pos).cuda().double()
    z = torch.from_numpy(species).cuda().long()
    m = None if mol is None else torch.from_numpy(mol).cuda()
    n = len(species)
    if do == "aev":
        out = torch.zeros((n, 1024), dtype=torch.float64, device="cuda")
        for rows, feats in aev_chunks(x, z, box):
            out[rows, :feats.shape[1]] = feats
        return out
    e = torch.zeros((nets, n), dtype=torch.float64, device="cuda")
    forces = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    virial = torch.zeros((n, 9), dtype=torch.float64, device="cuda")
    for rows in chunks_of(n):
        y = x.detach().requires_grad_(True)
        with torch.enable_grad():
            feats, (i, _, v) = aev_rows(y, z, box, m, rows)
            ek = networks(feats, z[rows], nets)
            gx, gv = torch.autograd.grad(ek.mean(0).sum(), (y, v), allow_unused=True)
        e[:, rows] = ek.detach()
        if gv is not None:
            forces -= gx
            virial.index_add_(0, rows[i], -(v.detach()[:, :, None] * gv[:, None, :]).reshape(-1, 9))
    whole = torch.zeros((nets, n_mol), dtype=torch.float64, device="cuda")
    whole.index_add_(1, torch.zeros(n, dtype=torch.long, device="cuda") if m is None else m.long(), e)
    if do == "host":
        return float(whole[0, 0]), forces
    if do == "serve":
        return whole[0], forces
    if do == "grad":
        target = torch.from_numpy(np.random.default_rng(seed).normal(size=n_mol).astype(np.float32)).cuda().double()
        return whole[0], -forces * (2 * (whole[0] - target) / n_mol)[m.long()][:, None]
    if do == "ensemble":
        return whole, e.mean(0), forces
    if do == "virial":
        return e[0], forces, virial.sum(0).reshape(1, 3, 3), virial.reshape(n, 3, 3)
    return e[0], forces
