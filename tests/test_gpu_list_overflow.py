"""Search bins that overflow on the way: a cluster of atoms moves into one bin
while a call runs, so the list rebuild decided on the device finds more atoms
than the bin has slots.  The call has to grow the bins and go on as if nothing
had happened: NVE and NVT restore the call's start and redo it, NPT repeats the
step's evaluation before anything is kicked, a relaxation its trial point.
Everything is compared with the oracle bit for bit; that the overflow happens
is asserted on the oracle's own positions.
"""
import numpy as np
import pytest

from paper_1012_5082_amd import inputs as I
from parity_utils import gpu_context

pytestmark = pytest.mark.gpu

SKIN, SLOTS = 0.3, 16
NAMES = ("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz")


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _grid(box, pot):
    return np.floor(box / (pot.rc + SKIN)).astype(int)


def _fullest_bin(x, y, z, box, pot):
    nb = _grid(box, pot)
    c = [np.clip((a / L * n).astype(int), 0, n - 1) for a, L, n in zip((x, y, z), box, nb)]
    return int(np.bincount(c[0] + nb[0] * (c[1] + nb[1] * c[2])).max())


def _cluster(dims, pot, atoms, xs, seed):
    """A bcc block with a vacancy of radius 6 A around the middle of a face
    between two search bins (normal along x), `atoms` atoms within 0.4 A of it,
    at x between xs[0] and xs[1] from the face."""
    rng = np.random.default_rng(seed)
    x, y, z, box = I.bcc(*dims)
    nb = _grid(box, pot)
    m = nb // 2
    c = box / nb * (m + [0.0, 0.5, 0.5])
    keep = np.sqrt((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2) > 6.0
    off = np.stack([rng.uniform(*xs, atoms), *rng.uniform(-0.4, 0.4, (2, atoms))], axis=1)
    x, y, z = (np.concatenate([a[keep], c[k] + off[:, k]]) for k, a in enumerate((x, y, z)))
    sp = I.initial_species(x.size, 0.2, seed + 1)
    return dict(x=x, y=y, z=z, box=np.asarray(box, dtype=np.float64), species=sp,
                moving=np.arange(x.size) >= x.size - atoms)


def _moving_cluster(dims, pot, seed=71):
    """20 atoms, most of them left of the face, all moving right by 0.1 A per
    step of 0.5 fs: after two steps they have moved by more than half the
    skin, and all are right of the face."""
    d = _cluster(dims, pot, 20, (-0.15, 0.05), seed)
    d["vx"], d["vy"], d["vz"] = I.mb_velocities(d["species"], 300.0, seed + 2)
    d["vx"] = d["vx"] + np.where(d["moving"], 0.2, 0.0)
    assert _fullest_bin(d["x"], d["y"], d["z"], d["box"], pot) <= SLOTS
    return d


def _first_rebuild_overflows(d, pot, steps, at):
    """at(k): the oracle's positions and box after k steps.  The first step
    after which an atom is farther than half the skin from its start finds a
    bin over its slots."""
    for k in range(1, steps + 1):
        (x, y, z), box = at(k)
        far = max(float(np.abs(a - b)[d["moving"]].max()) for a, b in
                  zip((x, y, z), (d["x"], d["y"], d["z"])))
        if far > 0.5 * SKIN:
            return _fullest_bin(x, y, z, box, pot) > SLOTS
    return False


# 2,000 atoms: the drift bins its atoms and one kernel builds the list; 50,400: a
# kernel bins them
@pytest.mark.parametrize("dims", [(10, 10, 10), (30, 28, 30)])
@pytest.mark.parametrize("ensemble", ["nve", "nvt", "npt"])
def test_steps_with_a_bin_that_overflows(torch_cuda, oracle_mod, dims, ensemble):
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _moving_cluster(dims, pot)
    dt, steps, T, tau, p_ext, tau_p = 0.5, 6, 300.0, 100.0, -0.01, 200.0
    start = (d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"])

    def oracle(n_steps):
        if ensemble == "nve":
            return O.md(*start, d["species"], d["box"], pot, dt, n_steps), d["box"], None
        if ensemble == "nvt":
            out, state = O.md_nvt(*start, d["species"], d["box"], pot, dt, n_steps, T, tau)
            return out, d["box"], state
        out, box, state, _ = O.md_npt(*start, d["species"], d["box"], pot, dt, n_steps, T, tau,
                                      p_ext, tau_p)
        return out, box, state

    assert _first_rebuild_overflows(d, pot, steps,
                                    lambda k: (lambda o: (o[0][:3], o[1]))(oracle(k)))
    g = gpu_context(d, pot, velocities=True, forces=True, skin=SKIN)
    if ensemble != "nve":
        g.set_thermostat(T, tau)
    if ensemble == "npt":
        g.set_barostat(p_ext, tau_p)
    print(f"[overflow] {ensemble} {dims}", flush=True)
    g.md(dt, steps)
    assert g.info()["md_rebuilds"] > 1
    out, box, state = oracle(steps)
    for nm, want in zip(NAMES, out[:9]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    if ensemble != "nve":
        assert g.thermostat() == (state[0], state[1])
    if ensemble == "npt":
        pe, gbox, _ = g.barostat()
        assert pe == state[2] and np.array_equal(gbox, box)
    # the context goes on: the grown bins serve the next call
    g.md(dt, 2)
    print("[overflow] next call done", flush=True)
    now = g.barostat()[1]
    rows = O.neighbors(*[getattr(g, nm).cpu().numpy() for nm in "xyz"], now, pot.rc, vectors=False)
    assert np.array_equal(g.rho().cpu().numpy(), O.density(rows, d["species"], pot))
    g.close()


@pytest.mark.parametrize("dims", [(10, 10, 10), (30, 28, 30)])
def test_relaxation_with_a_bin_that_overflows(torch_cuda, oracle_mod, dims):
    """32 atoms, 16 on either side of the face, driven apart: the first trial
    point of the line search (the largest move is 0.2 A) leaves more than 16 on
    one side."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _cluster(dims, pot, 32, (-0.3, 0.3), 84)
    nb = _grid(d["box"], pot)
    face = d["box"][0] / nb[0] * (nb[0] // 2)
    # the face at the median: the cluster moved, not the lattice
    xs = np.sort(d["x"][d["moving"]])
    d["x"] = d["x"] + np.where(d["moving"], face - 0.5 * (xs[15] + xs[16]), 0.0)
    assert _fullest_bin(d["x"], d["y"], d["z"], d["box"], pot) <= SLOTS
    nl = O.neighbors(d["x"], d["y"], d["z"], d["box"], pot.rc)
    f = np.stack(O.forces(nl, d["species"], pot, O.density(nl, d["species"], pot)))
    a = 0.2 / np.sqrt((f ** 2).sum(axis=0).max())
    trial = [np.mod(p + a * q, L) for p, q, L in
             zip((d["x"], d["y"], d["z"]), f, d["box"])]
    assert _fullest_bin(*trial, d["box"], pot) > SLOTS
    g = gpu_context(d, pot, forces=True, skin=SKIN)
    print(f"[overflow] cg {dims}", flush=True)
    rg = g.minimize(max_iter=8, ftol=1e-6, dmax=0.2)
    out, ro, _ = O.cg(d["x"], d["y"], d["z"], d["species"], d["box"], pot, max_iter=8, ftol=1e-6,
                      dmax=0.2)
    for k in ("iterations", "evaluations", "reason", "energy", "fnorm"):
        assert rg[k] == ro[k], (k, rg[k], ro[k])
    for nm, want in zip(("x", "y", "z", "fx", "fy", "fz"), out[:6]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    assert g.info()["md_rebuilds"] > 1
    g.close()
