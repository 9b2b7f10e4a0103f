"""GPU (HIP, through the C ABI) against the oracle on identical seeded inputs.

Bar: integer state (species, n_B, site choices, decisions, counters) bit
for bit; FP64 dU within 1e-12 relative, forces within 1e-10 relative of the
sum of term magnitudes, energies/densities/positions bit for bit where the
arithmetic is the same (both sides evaluate the same expressions in the same
order without contraction); decisions may differ only at near ties
(|ln u + x| < 1e-9), where the oracle adopts the GPU's decision.
"""
import math

import numpy as np
import pytest

from paper_1012_5082_amd import inputs as I
from paper_1012_5082_amd import workloads as W
from parity_utils import compare_logs, gpu_context, oracle_state, tie_overrides

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_device_sqrt_correctly_rounded(torch_cuda):
    torch = torch_cuda
    from paper_1012_5082_amd.binding import selftest_sqrt
    rng = np.random.default_rng(1)
    bits = rng.integers(0, 0x7FEFFFFFFFFFFFFF, size=4_000_000, dtype=np.int64)
    vals = np.concatenate([bits.view(np.float64),
                           rng.uniform(0.0, 40.0, 2_000_000),
                           rng.uniform(0.0, 1e-3, 500_000),
                           np.array([0.0, 1.0, 2.0, 4.0, 13.134408449586, 5e-324, 1e300])])
    x = torch.tensor(vals, dtype=torch.float64, device="cuda")
    got = selftest_sqrt(x).cpu().numpy()
    assert np.array_equal(got.view(np.int64), np.sqrt(vals).view(np.int64))


def _md_math_inputs(torch, gen, n):
    """n square-root arguments a and divisor pairs (a2, b) on the GPU: a third
    each of random bit patterns over [2^-767, 2^1023), uniform r^2 in
    (1e-6, 64) and arguments just above the squares of random numbers
    (where the rounding of the root is hardest); quotients of signed
    uniform and random-exponent numerators by uniform and random-exponent
    divisors."""
    k = n // 3
    dev = "cuda"
    lo, hi = 256, 2047  # biased exponents of 2^-767 and of the largest finite binade
    bits = (torch.randint(lo, hi, (k,), device=dev, generator=gen, dtype=torch.int64) << 52) | \
        torch.randint(0, 1 << 52, (k,), device=dev, generator=gen, dtype=torch.int64)
    a1 = bits.view(torch.float64)
    a2 = 1e-6 + 64.0 * torch.rand(k, device=dev, generator=gen, dtype=torch.float64)
    y = 1e-2 + 8.0 * torch.rand(n - 2 * k, device=dev, generator=gen, dtype=torch.float64)
    u = torch.nextafter(y, torch.full_like(y, float("inf"))) - y
    a3 = y * y + y * u
    a = torch.cat([a1, a2, a3])
    num = torch.cat([200.0 * torch.rand(n - k, device=dev, generator=gen, dtype=torch.float64) - 100.0,
                     torch.ldexp(torch.rand(k, device=dev, generator=gen, dtype=torch.float64) + 0.5,
                                 torch.randint(-900, 900, (k,), device=dev, generator=gen))])
    den = torch.cat([1e-3 + 10.0 * torch.rand(n - k, device=dev, generator=gen, dtype=torch.float64),
                     torch.ldexp(torch.rand(k, device=dev, generator=gen, dtype=torch.float64) + 0.5,
                                 torch.randint(-60, 60, (k,), device=dev, generator=gen))])
    return a, num, den


def test_md_math_correctly_rounded(torch_cuda):
    """The MD passes' square root and quotient are correctly rounded over the
    ranges they serve: 10^9 arguments of each against the library's sqrt and
    the device's IEEE division, and 2 x 10^7 of each against the host's."""
    torch = torch_cuda
    from paper_1012_5082_amd.binding import selftest_md_math, selftest_sqrt
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    for chunk in range(10):
        a, num, den = _md_math_inputs(torch, gen, 100_000_000)
        sq, _ = selftest_md_math(a, den)
        assert torch.equal(sq.view(torch.int64), selftest_sqrt(a).view(torch.int64)), chunk
        _, q = selftest_md_math(num, den)
        assert torch.equal(q.view(torch.int64), (num / den).view(torch.int64)), chunk
        if chunk < 2:  # host references on every tenth argument
            an, nn, dn = a[::10].cpu().numpy(), num[::10].cpu().numpy(), den[::10].cpu().numpy()
            assert np.array_equal(sq[::10].cpu().numpy().view(np.int64), np.sqrt(an).view(np.int64))
            assert np.array_equal(q[::10].cpu().numpy().view(np.int64), (nn / dn).view(np.int64))
        del a, num, den, sq, q


def test_create_rejects_bad_input(torch_cuda):
    from paper_1012_5082_amd.binding import VCSGC, VcsgcError
    pot = I.params("FS-P1")
    x, y, z, box = I.bcc(10, 10, 10)
    sp = np.zeros(x.size, np.uint8)
    xb = x.copy()
    xb[5] = box[0] + 1.0
    with pytest.raises(VcsgcError) as e:
        VCSGC(xb, y, z, box, sp, pot)
    assert e.value.code == -1
    sp2 = sp.copy()
    sp2[3] = 2
    with pytest.raises(VcsgcError) as e:
        VCSGC(x, y, z, box, sp2, pot)
    assert e.value.code == -1
    xs, ys, zs, bs = I.bcc(4, 4, 4)
    with pytest.raises(VcsgcError) as e:
        VCSGC(xs, ys, zs, bs, np.zeros(xs.size, np.uint8), pot)
    assert e.value.code == -2
    g = VCSGC(x, y, z, box, sp, pot)
    with pytest.raises(VcsgcError) as e:
        g.sweep(0.0, -1.0, 0.05, 600.0, 1, 1)
    assert e.value.code == -1
    with pytest.raises(VcsgcError):
        g.md(1.0, 1)   # MC-only context
    g.close()


def _eam_parity(O, d, pot):
    g = gpu_context(d, pot, forces=True)
    st = oracle_state(O, d, pot)
    rho_g = g.rho().cpu().numpy()
    assert np.array_equal(rho_g, st.rho)
    e_o = O.energy_atoms(st.nl, st.species, pot, st.rho)
    e_g = g.atom_energies().cpu().numpy()
    assert np.array_equal(e_g, e_o)
    U = g.energy(forces=True)
    assert abs(U - math.fsum(e_o)) <= 1e-12 * abs(U)
    nlv = O.neighbors(d["x"], d["y"], d["z"], d["box"], pot.rc)
    fo = O.forces(nlv, st.species, pot, st.rho)
    for a, b in zip((g.fx, g.fy, g.fz), fo):
        a = a.cpu().numpy()
        assert np.array_equal(a, b)
    g.close()


def test_eam_parity_c1_thermal(torch_cuda, oracle_mod):
    d = W.c1(c_init=0.3)
    d["x"], d["y"], d["z"] = I.thermalize(d["x"], d["y"], d["z"], d["box"], 0.05, 5)
    _eam_parity(oracle_mod, d, I.params("FS-P1"))


def test_eam_parity_c2(torch_cuda, oracle_mod):
    _eam_parity(oracle_mod, W.c2(cbar=0.10), I.params("FS-P1"))


def _dense_bins_system(kind):
    """Systems whose search bins need the larger bin capacity.  "cluster": a
    10^3 bcc block with a vacancy of radius 6 A holding a cluster of 20
    atoms within 0.4 A (20 atoms in one bin: more than its 16 slots).
    "clusters": 16 atoms within 0.05 A of every bin centre of a 7^3 grid of
    4.2 A bins (no bin over 16, but more staged atoms around a region than
    the 16-slot search stages; clusters 4.1 A apart, beyond rc + skin)."""
    rng = np.random.default_rng(61 if kind == "cluster" else 62)
    if kind == "cluster":
        x, y, z, box = I.bcc(10, 10, 10)
        c = 0.5 * box
        keep = np.sqrt((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2) > 6.0
        off = rng.uniform(-0.4, 0.4, size=(20, 3)) / np.sqrt(3.0)
        x = np.concatenate([x[keep], c[0] + off[:, 0]])
        y = np.concatenate([y[keep], c[1] + off[:, 1]])
        z = np.concatenate([z[keep], c[2] + off[:, 2]])
    else:
        b = 4.2
        box = np.full(3, 7 * b)
        g = (np.arange(7) + 0.5) * b
        cx, cy, cz = [a.ravel() for a in np.meshgrid(g, g, g, indexing="ij")]
        k = np.arange(16)
        grid = 0.025 * np.stack([k % 2, (k // 2) % 2, k // 4], axis=1) - [0.0125, 0.0125, 0.0375]
        off = grid[None] + rng.uniform(-0.003, 0.003, size=(cx.size, 16, 3))
        x = (cx[:, None] + off[..., 0]).ravel()
        y = (cy[:, None] + off[..., 1]).ravel()
        z = (cz[:, None] + off[..., 2]).ravel()
    sp = I.initial_species(x.size, 0.2, 63)
    return dict(x=x, y=y, z=z, box=np.asarray(box, dtype=np.float64), species=sp)


@pytest.mark.parametrize("kind", ["cluster", "clusters"])
def test_eam_parity_dense_bins(torch_cuda, oracle_mod, kind):
    """Bins grown on the way (the 32-slot search): densities, energies and
    forces still equal the oracle's bit for bit, and the MD list holds every
    pair within rc + skin."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _dense_bins_system(kind)
    _eam_parity(O, d, pot)
    g = gpu_context(d, pot, forces=True)
    g.energy(forces=True)
    nl = O.neighbors(d["x"], d["y"], d["z"], d["box"], pot.rc + 0.3, vectors=False)
    assert g.info()["md_pairs"] == nl.j.size
    g.close()


def _full_rows_system(cells=24):
    """A simple-cubic lattice of edge 1.7 A (0.005 A of noise): every atom
    has exactly 32 neighbours within rc + 0.1 A, all of them within rc
    (shells at 1.7, 2.40, 2.94 and 3.4 A; the next at 3.80 A)."""
    a = 1.7
    k = (np.arange(cells) + 0.5) * a
    x, y, z = [v.ravel().copy() for v in np.meshgrid(k, k, k, indexing="ij")]
    rng = np.random.default_rng(71 + cells)
    for v in (x, y, z):
        v += rng.uniform(-0.005, 0.005, v.size)
    box = np.full(3, cells * a)
    sp = I.initial_species(x.size, 0.2, 72)
    return dict(x=x, y=y, z=z, box=box, species=sp, dmu0=0.0, kappa=1000.0, cbar=0.2, T=600.0,
                seed=73)


def test_eam_parity_full_rows(torch_cuda, oracle_mod):
    """Every row of the MD list full (the lattice above with an MD-list skin
    of 0.1 A).  The lists come from the region search (eleven search bins
    per axis, grown to 32 slots).  A row holding the largest count must keep
    every neighbour: energies and forces equal the oracle's bit for bit."""
    O = oracle_mod
    pot = I.params("FS-P1")
    s = _full_rows_system()
    x, y, z, box, sp = s["x"], s["y"], s["z"], s["box"], s["species"]
    wide = O.neighbors(x, y, z, box, pot.rc + 0.1 + 1e-3, vectors=False)
    near = O.neighbors(x, y, z, box, pot.rc, vectors=False)
    assert np.all(np.diff(wide.start) == 32) and np.all(np.diff(near.start) == 32)
    zero = np.zeros(x.size)
    d = dict(x=x, y=y, z=z, vx=zero, vy=zero, vz=zero, box=box, species=sp)
    g = gpu_context(d, pot, velocities=True, skin=0.1)
    U = g.energy(forces=True)
    st = O.SweepState(x, y, z, box, sp, pot)
    e_o = O.energy_atoms(st.nl, st.species, pot, st.rho)
    assert np.array_equal(g.atom_energies().cpu().numpy(), e_o)
    assert abs(U - math.fsum(e_o)) <= 1e-12 * abs(U)
    fo = O.forces(O.neighbors(x, y, z, box, pot.rc), sp, pot, st.rho)
    for got, want in zip((g.fx, g.fy, g.fz), fo):
        assert np.array_equal(got.cpu().numpy(), want)
    info = g.info()
    assert info["md_pairs"] == 32 * x.size
    # two MD steps of 0.1 fs (no rebuild), then a sweep on the r < rc rows
    # filtered out of the full MD rows
    g.md(0.1, 2)
    out = O.md(x, y, z, zero, zero, zero, sp, box, pot, 0.1, 2)
    for nm, want in zip(("x", "y", "z", "vx", "vy", "vz"), out[:6]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    s_g = g.sweep(0.0, 1000.0, 0.2, 600.0, 1, 73)
    st2 = O.SweepState(out[0], out[1], out[2], box, sp, pot, vx=out[3], vy=out[4], vz=out[5])
    s_o, _, _ = O.sweep(st2, 0.0, 1000.0, 0.2, 600.0, 1, 73)
    assert g.info()["mc_pairs"] == 32 * x.size
    for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert s_g[k] == s_o[k], k
    assert np.array_equal(g.species.cpu().numpy(), st2.species)
    assert np.array_equal(g.rho().cpu().numpy(), st2.rho)
    g.close()


@pytest.mark.parametrize("strategy,tpg", [("graph", 1), ("stage", 1), ("persistent", 1),
                                          ("batch", 3)])
def test_sweep_full_rows(torch_cuda, oracle_mod, strategy, tpg):
    """Every MC row full (32 neighbours within rc for every atom): each sweep
    strategy reproduces the oracle's chain over two sweeps."""
    r = _sweep_parity(oracle_mod, _full_rows_system(), I.params("FS-P1"), 2,
                      log=strategy != "batch", strategy=strategy, trials_per_group=tpg)
    assert r["flips"] > 0


def test_local_chain_full_rows(torch_cuda, oracle_mod):
    """Local chains of 2 trials per cell and stage on full MC rows: the chain
    (statistics, species and densities) equals the oracle's."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _full_rows_system()
    args = (d["dmu0"], 5.0, d["cbar"], d["T"])
    g = gpu_context(d, pot)
    g.set_local_steps(2)
    sg = g.sweep(*args, 2, d["seed"])
    st = oracle_state(O, d, pot)
    so, _, _ = O.sweep(st, *args, 2, d["seed"], local_steps=2)
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert sg[key] == so[key], key
    assert sg["flips"] > 0
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


def _sweep_parity(O, d, pot, n_sweeps, kappa=None, cbar=None, log=True, chunks=None,
                  strategy="graph", trials_per_group=1):
    kappa = d["kappa"] if kappa is None else kappa
    cbar = d["cbar"] if cbar is None else cbar
    args = (d["dmu0"], kappa, cbar, d["T"])
    g = gpu_context(d, pot)
    g.set_tuning(strategy, trials_per_group)
    info = g.info()
    S = info["stages_per_sweep"]
    ncpc = int(np.prod(info["n_cells"])) // 8
    st0 = oracle_state(O, d, pot)
    if log:
        g.enable_log(n_sweeps * S * ncpc, n_sweeps * S)
    chunks = chunks or [n_sweeps]
    gs = None
    for k in chunks:
        s = g.sweep(*args, k, d["seed"])
        gs = s if gs is None else {key: gs[key] + s[key] if key not in ("n_final",) else s[key]
                                   for key in s}
    sp_g = g.species.cpu().numpy()
    rho_g = g.rho().cpu().numpy()
    res = {}
    tl_g = sl_g = None
    if log:
        tl_g, sl_g, nt, ns = g.logs()
        assert nt == tl_g.shape[0] and ns == sl_g.shape[0]
    over = tie_overrides(tl_g, sl_g) if log else None
    so, tl_o, sl_o = O.sweep(st0, *args, n_sweeps, d["seed"], log_trials=10 ** 8 if log else 0,
                             log_stages=10 ** 8 if log else 0, overrides=over)
    if log:
        res = compare_logs(tl_g, sl_g, tl_o, sl_o)
    for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert gs[k] == so[k], (k, gs[k], so[k])
    assert gs["sum_n"] == so["sum_n"] and gs["sum_n2"] == so["sum_n2"]
    assert np.array_equal(sp_g, st0.species)
    assert np.array_equal(rho_g, st0.rho)
    g.close()
    res.update(gs)
    return res


@pytest.mark.parametrize("kappa", [1000.0, 10.0, 0.0])
def test_sweep_parity_c1(torch_cuda, oracle_mod, kappa):
    d = W.c1()
    r = _sweep_parity(oracle_mod, d, I.params("FS-P1"), 100, kappa=kappa)
    assert r["trials"] == 100 * 2000
    if kappa <= 10.0:
        assert r["flips"] > 0


@pytest.mark.parametrize("cbar", [0.02, 0.05, 0.10])
def test_sweep_parity_c2(torch_cuda, oracle_mod, cbar):
    d = W.c2(cbar=cbar)
    r = _sweep_parity(oracle_mod, d, I.params("FS-P1"), 10)
    assert r["flips"] > 0


@pytest.mark.parametrize("strategy,tpg", [("stage", 1), ("persistent", 1), ("graph", 3)])
def test_sweep_strategies_agree(torch_cuda, oracle_mod, strategy, tpg):
    """Per-stage launches, the direct persistent launch and other tilings of
    the graph-captured persistent launch all reproduce the oracle."""
    d = W.c2(cbar=0.05)
    r = _sweep_parity(oracle_mod, d, I.params("FS-P1"), 4, strategy=strategy,
                      trials_per_group=tpg)
    assert r["flips"] > 0
    r1 = _sweep_parity(oracle_mod, W.c1(), I.params("FS-P1"), 20, kappa=10.0,
                       strategy=strategy, trials_per_group=tpg)
    assert r1["trials"] == 20 * 2000


def _replica_set(n_rep=6, seed=55):
    """Uneven rigid bcc replicas on a T x kappa x cbar grid (small sizes)."""
    rng = np.random.default_rng(seed)
    reps = []
    for r in range(n_rep):
        nx, ny, nz = (int(v) for v in rng.integers(10, 19, size=3))
        x, y, z, box = I.bcc(nx, ny, nz)
        T = [400.0, 600.0, 800.0][r % 3]
        kappa = [100.0, 1000.0][(r // 3) % 2]
        cbar = float(np.exp(rng.uniform(np.log(0.01), np.log(0.2))))
        sp = I.initial_species(x.size, cbar, seed + r)
        reps.append(dict(x=x, y=y, z=z, box=box, species=sp, T=T, kappa=kappa, cbar=cbar,
                         dmu0=W.dmu_s(T, cbar)))
    return reps


def test_batch_replicas_match_oracle(torch_cuda, oracle_mod):
    """Each replica of a batch equals an independent oracle chain keyed
    (seed, replica index), with its own parameters and stage count."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGCBatch
    pot = I.params("FS-P1")
    reps = _replica_set()
    b = VCSGCBatch(reps, pot)
    args = [np.array([r[k] for r in reps]) for k in ("dmu0", "kappa", "cbar", "T")]
    seed = 777
    s1 = b.sweep_batch(*args, 3, seed)
    s2 = b.sweep_batch(*args, 2, seed)
    for k, r in enumerate(reps):
        st = O.SweepState(r["x"], r["y"], r["z"], r["box"], r["species"], pot)
        so, _, _ = O.sweep(st, r["dmu0"], r["kappa"], r["cbar"], r["T"], 5, seed, replica=k)
        assert s1[k]["trials"] + s2[k]["trials"] == so["trials"]
        assert s1[k]["flips"] + s2[k]["flips"] == so["flips"]
        assert s2[k]["n_final"] == so["n_final"]
        assert np.array_equal(b.replica_species(k), st.species), k
        assert np.array_equal(b.replica_rho(k), st.rho), k
    b.close()


@pytest.mark.parametrize("n,batch,persistent", [
    (76, 8, 3),   # 8,000 active cells: two stages in one pass of 16,000 trial groups
    (80, 16, 3),  # 9,261: one stage, and the rest of the grid for the next ones
    (92, 8, 3),   # 13,824
    (92, 16, 1),  # the pipeline once a call has accepted next to nothing
])
def test_sweeps_at_rest_and_with_accepted_stages(torch_cuda, oracle_mod, n, batch, persistent):
    """27 colours, nothing accepted, on the whole grid: the number of the three
    calls that run persistently; then every stage accepted, the next calls on
    fewer workgroups; the chain is the oracle's throughout."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGC
    pot = I.params("FS-P1")
    x, y, z, box = I.bcc(n, n, n)
    sp = I.initial_species(x.size, 0.02, 6)
    g = VCSGC(x, y, z, box, sp, pot, colours=27)
    print(f"[rest] {n} {batch} {g.info()['n_cells']}", flush=True)
    g.set_tuning("batch", batch)
    assert g.tuning()["workgroups"] >= 248
    g.kernel_timing(["persist"])
    args = (3.0, 1000.0, 0.02, 300.0)
    for _ in range(3):
        s = g.sweep(*args, 1, 31)
    assert s["stage_accepts"] == 0
    assert g.kernel_times()["persist"][2] == persistent
    st = O.SweepState(x, y, z, box, sp, pot)
    so, _, _ = O.sweep(st, *args, 3, 31, colour_period=3)
    assert (s["n_final"], so["flips"]) == (so["n_final"], 0)
    for kappa in (0.0, 0.0, 0.5):
        a = g.sweep(-0.2, kappa, 0.02, 600.0, 1, 31)
        b, _, _ = O.sweep(st, -0.2, kappa, 0.02, 600.0, 1, 31, colour_period=3)
        for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
            assert a[k] == b[k], (kappa, k)
        assert kappa or a["stage_accepts"] == a["stages"]
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


@pytest.mark.parametrize("strategy,tpg", [("stage", 1), ("batch", 4)])
def test_pipeline_strategies_never_time_out(torch_cuda, oracle_mod, strategy, tpg):
    """With a wait limit of one poll the workgroups of a persistent launch give up
    before they wait: the launch ends without effect and the call runs with
    kernels per stage, then persistently again with the default limit; the chain
    is the oracle's."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    args = (d["dmu0"], 10.0, d["cbar"], d["T"])
    g = gpu_context(d, pot)
    g.set_tuning(strategy, tpg)
    assert g.tuning()["workgroups"] > 1
    st = oracle_state(O, d, pot)
    for limit, n_sw in ((1, 1), (1 << 24, 1), (1, 2), (3, 1)):
        print(f"[limit] {strategy} {limit}", flush=True)
        g.set_wait_limit(limit)
        a = g.sweep(*args, n_sw, d["seed"])
        b, _, _ = O.sweep(st, *args, n_sw, d["seed"])
        for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final",
                  "sum_n", "sum_n2"):
            assert a[k] == b[k], (limit, k)
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


def _sparse_system(cells, pot):
    """A 12^3 bcc block and 20,000 scattered atoms in a box of cells^3 link
    cells, most of them empty."""
    rng = np.random.default_rng(5)
    box = np.full(3, cells * 2.0 * pot.rc + 1.0)
    x, y, z, _ = I.bcc(12, 12, 12)
    p = rng.uniform(0.0, 1.0, (20000, 3)) * box
    p = p[~np.all(p < 45.0, axis=1)]
    x, y, z = (np.concatenate([a + 5.0, p[:, k]]) for k, a in enumerate((x, y, z)))
    return dict(x=x, y=y, z=z, box=box, species=I.initial_species(x.size, 0.5, 6))


@pytest.mark.parametrize("cells,strategy", [
    (204, "graph"),       # 1,061,208 active cells: more than 2^20
    (204, "batch"),
    (254, "persistent"),  # 2,048,383: more per workgroup than the LDS draws at once
    (254, "graph"),
])
def test_many_active_cells(torch_cuda, oracle_mod, cells, strategy):
    """Boxes of over a million active cells per stage: created, and every
    strategy gives the oracle's chain (logs included where they are kept)."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _sparse_system(cells, pot)
    print(f"[cells] {cells} {strategy}", flush=True)
    g = gpu_context(d, pot, skin=3.6)
    g.set_tuning(strategy, 1)
    log = (cells, strategy) == (254, "graph")
    if log:
        g.enable_log(100000, 100)
    a = [g.sweep(0.0, 3e-3, 0.5, 600.0, k, 31) for k in (1, 2)]
    st = O.SweepState(d["x"], d["y"], d["z"], d["box"], d["species"], pot)
    so, tl_o, sl_o = O.sweep(st, 0.0, 3e-3, 0.5, 600.0, 3, 31, log_trials=100000 if log else 0,
                             log_stages=100 if log else 0)
    for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips"):
        assert a[0][k] + a[1][k] == so[k], k
    assert a[1]["n_final"] == so["n_final"]
    if log:
        tl_g, sl_g, _, _ = g.logs()
        compare_logs(tl_g, sl_g, tl_o, sl_o)
        g.disable_log()
    assert so["stage_accepts"] == so["stages"]  # then a stiffer reservoir, with rejected stages
    a = g.sweep(0.0, 30.0, 0.5, 600.0, 2, 31)
    so, _, _ = O.sweep(st, 0.0, 30.0, 0.5, 600.0, 2, 31)
    assert so["stage_accepts"] < so["stages"]
    for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert a[k] == so[k], k
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


def test_batch_with_many_active_cells(torch_cuda, oracle_mod):
    """The same box in a batch with a replica that fits the LDS."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGCBatch
    pot = I.params("FS-P1")
    reps = [_sparse_system(254, pot), dict(zip(("x", "y", "z", "box"), I.bcc(6, 6, 6)))]
    reps[1]["species"] = I.initial_species(reps[1]["x"].size, 0.5, 8)
    print("[cells] batch", flush=True)
    b = VCSGCBatch(reps, pot)
    s = b.sweep_batch(0.0, 3e-3, 0.5, 600.0, 2, 31)
    for k, r in enumerate(reps):
        st = O.SweepState(r["x"], r["y"], r["z"], r["box"], r["species"], pot)
        so, _, _ = O.sweep(st, 0.0, 3e-3, 0.5, 600.0, 2, 31, replica=k)
        for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
            assert s[k][key] == so[key], (k, key)
        assert np.array_equal(b.replica_species(k), st.species), k
        assert np.array_equal(b.replica_rho(k), st.rho), k
    b.close()


def test_log_capacity_of_the_last_set_log(torch_cuda):
    """A log set again on the same buffers with smaller capacities: the sweep
    (graph-captured, as built for the first ones) writes no row beyond them."""
    torch = torch_cuda
    import ctypes as C
    from paper_1012_5082_amd import binding as B
    d = W.c1()
    g = gpu_context(d, I.params("FS-P1"))
    t = torch.zeros((4000, 8), dtype=torch.float64, device="cuda")
    s = torch.zeros((4000, 8), dtype=torch.float64, device="cuda")
    P = C.c_void_p
    for cap in (4000, 7):
        t.fill_(-1.0)
        s.fill_(-1.0)
        g._check(B.lib().vcsgc_set_log(g._h, P(t.data_ptr()), cap, P(s.data_ptr()), cap), "set_log")
        n = g.sweep(d["dmu0"], 10.0, d["cbar"], d["T"], 1, d["seed"])["trials"]
        assert n == 2000
        torch.cuda.synchronize()
        written = min(cap, n)
        for a in (t, s):
            assert bool((a[:written, 0] >= 0.0).all()) and bool((a[written:] == -1.0).all()), cap
    g.close()


@pytest.mark.parametrize("pot,n_rep,strategy", [
    ("FS-P1", 257, "graph"),        # one more than compute units
    ("FS-P1", 1024, "persistent"),  # the most
    ("TAB-X", 768, "graph"),
])
def test_batch_of_more_replicas_than_compute_units(torch_cuda, oracle_mod, pot, n_rep, strategy):
    """Small replicas with some among them whose state does not fit the LDS, one
    workgroup each: the chains of the first, the last and every 37th replica
    are the oracle's; one replica more than the most is refused."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGCBatch, VcsgcError
    print(f"[batch] {pot} {n_rep} {strategy}", flush=True)
    limit = {"FS-P1": 1024, "TAB-X": 768}[pot]
    p = I.params(pot) if pot == "FS-P1" else I.table(pot)
    small, large = I.bcc(6, 6, 7), I.bcc(19, 18, 19)
    reps = []
    for k in range(n_rep):
        x, y, z, box = large if k in (3, n_rep - 2) else small
        reps.append(dict(x=x, y=y, z=z, box=box,
                         species=I.initial_species(x.size, 0.05 + 0.1 * (k % 3), 900 + k),
                         T=500.0 + k, kappa=1.0 + k % 2, cbar=0.1, dmu0=-0.2 + 0.01 * (k % 5)))
    b = VCSGCBatch(reps, p)
    b.set_tuning(strategy, 1)
    assert b.tuning()["workgroups"] == n_rep
    args = [np.array([r[k] for r in reps]) for k in ("dmu0", "kappa", "cbar", "T")]
    s1 = b.sweep_batch(*args, 1, 12)
    s2 = b.sweep_batch(*args, 2, 12)
    species, rho = b.species.cpu().numpy(), b.rho().cpu().numpy()
    for k in sorted({0, 3, n_rep - 2, n_rep - 1, *range(0, n_rep, 37)}):
        r = reps[k]
        st = O.SweepState(r["x"], r["y"], r["z"], r["box"], r["species"], p)
        so, _, _ = O.sweep(st, r["dmu0"], r["kappa"], r["cbar"], r["T"], 3, 12, replica=k)
        for key in ("trials", "stages", "stage_accepts", "flips"):
            assert s1[k][key] + s2[k][key] == so[key], (k, key)
        assert s2[k]["n_final"] == so["n_final"], k
        own = slice(b.offsets[k], b.offsets[k + 1])
        assert np.array_equal(species[own], st.species), k
        assert np.array_equal(rho[own], st.rho), k
    b.close()
    if n_rep == limit:
        with pytest.raises(VcsgcError) as e:
            VCSGCBatch(reps + reps[:1], p)
        assert e.value.code == -1


def test_batch_get_state(torch_cuda):
    """get_state on a batch of replicas: the sweep counter, the seed, n_B of the
    first replica and the density cache, and nothing beyond the state it was
    given is written."""
    import ctypes as C
    from paper_1012_5082_amd import binding as B
    reps = _replica_set()
    b = B.VCSGCBatch(reps, I.params("FS-P1"))
    args = [np.array([r[k] for r in reps]) for k in ("dmu0", "kappa", "cbar", "T")]
    b.sweep_batch(*args, 2, 777)
    states = (B.State * 3)()
    C.memset(C.byref(states), 0x5A, C.sizeof(states))
    guard = bytes(states[0]), bytes(states[2])
    states[1].rho_dev = None
    b._check(B.lib().vcsgc_get_state(b._h, C.byref(states[1])), "get_state")
    assert (states[1].sweeps_done, states[1].seed) == (2, 777)
    assert states[1].n_b == int(b.replica_species(0).sum())
    assert (bytes(states[0]), bytes(states[2])) == guard
    st = b.get_state(with_rho=True)
    assert st["n_b"] == states[1].n_b
    assert np.array_equal(st["rho"].cpu().numpy(), b.rho().cpu().numpy())
    b.close()


def test_sweep_chunking_and_determinism(torch_cuda, oracle_mod):
    d = W.c2(cbar=0.05)
    pot = I.params("FS-P1")
    _sweep_parity(oracle_mod, d, pot, 6, log=False, chunks=[2, 1, 3])
    a = gpu_context(d, pot)
    b = gpu_context(d, pot)
    a.sweep(d["dmu0"], d["kappa"], d["cbar"], d["T"], 5, 9)
    b.sweep(d["dmu0"], d["kappa"], d["cbar"], d["T"], 5, 9)
    assert np.array_equal(a.species.cpu().numpy(), b.species.cpu().numpy())
    assert np.array_equal(a.rho().cpu().numpy(), b.rho().cpu().numpy())
    a.close()
    b.close()


def test_stage_graph_replay(torch_cuda, oracle_mod):
    """Per-stage sweeps without logs run as a replayed graph of one sweep
    (sweep counter on the device, rebuilt when the parameters change): the
    chain equals the oracle's across calls, chunks and parameter changes."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    _sweep_parity(O, d, pot, 6, log=False, chunks=[2, 1, 3], strategy="stage")
    g = gpu_context(d, pot)
    g.set_tuning("stage", 1)
    st = oracle_state(O, d, pot)
    plan = [((d["dmu0"], d["kappa"], 0.05, d["T"]), 2), ((d["dmu0"] + 0.02, 10.0, 0.04, 650.0), 3),
            ((d["dmu0"], d["kappa"], 0.05, d["T"]), 1)]
    for args, k in plan:
        sg = g.sweep(*args, k, d["seed"])
        so, _, _ = O.sweep(st, *args, k, d["seed"])
        for key in ("trials", "local_accepts", "stage_accepts", "flips", "n_final"):
            assert sg[key] == so[key], key
        assert sg["sum_n"] == so["sum_n"]
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


@pytest.mark.parametrize("log", [True, False])
@pytest.mark.parametrize("kappa", [0.0, 10.0])
def test_stage_pipeline_accepting_stages(torch_cuda, oracle_mod, kappa, log):
    """The fused stage pipeline with many accepted stages (kappa = 0 accepts
    every stage with a local accept): the extra trial kernels after accepted
    stages, the host's top-up launches when its estimate falls short, direct
    launches (logs) and graph replays all give the oracle's chain."""
    d = W.c2(cbar=0.05)
    r = _sweep_parity(oracle_mod, d, I.params("FS-P1"), 3, kappa=kappa, log=log,
                      chunks=[1, 2], strategy="stage")
    assert r["stage_accepts"] > 0
    if kappa == 0.0:
        assert r["stage_accepts"] * 2 > r["stages"]


@pytest.mark.parametrize("D,kappa", [(1, 10.0), (4, 0.0), (8, 1000.0), (16, 10.0)])
def test_batched_pipeline_parity(torch_cuda, oracle_mod, D, kappa):
    """Batches of D stages tried on the state as it is and tested in order up
    to the first accepted stage (whose commit drops the trials after it): the
    chain equals the oracle's, across calls, with few and with most stages
    accepted (kappa = 0)."""
    d = W.c2(cbar=0.05)
    r = _sweep_parity(oracle_mod, d, I.params("FS-P1"), 3, kappa=kappa, log=False,
                      chunks=[1, 2], strategy="batch", trials_per_group=D)
    assert r["stage_accepts"] > 0


def test_batched_pipeline_timed_and_retuned(torch_cuda, oracle_mod):
    """The batched pipeline with per-kernel timing (event nodes in its graphs),
    a change of batch length between calls and a call of zero sweeps."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    g = gpu_context(d, pot)
    g.set_tuning("batch", 8)
    st = oracle_state(O, d, pot)
    args = (d["dmu0"], 10.0, d["cbar"], d["T"])
    g.kernel_timing(["stage"])
    s0 = g.sweep(*args, 0, d["seed"])
    assert s0["trials"] == 0 and s0["stages"] == 0
    for D, n_sw in ((8, 2), (3, 1)):
        g.set_tuning("batch", D)
        sg = g.sweep(*args, n_sw, d["seed"])
        so, _, _ = O.sweep(st, *args, n_sw, d["seed"])
        for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
            assert sg[key] == so[key], key
        assert sg["sum_n"] == so["sum_n"] and sg["sum_n2"] == so["sum_n2"]
    kt = g.kernel_times()
    assert kt["stage"][1] > 0 and kt["stage"][0] > 0
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


def test_stage_pipeline_timed_and_empty(torch_cuda, oracle_mod):
    """Per-kernel timing of the pipeline (event nodes in its graphs) and a
    call of zero sweeps leave the chain equal to the oracle's."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    g = gpu_context(d, pot)
    g.set_tuning("stage", 1)
    st = oracle_state(O, d, pot)
    args = (d["dmu0"], 10.0, d["cbar"], d["T"])
    g.kernel_timing(["stage"])
    s0 = g.sweep(*args, 0, d["seed"])
    assert s0["trials"] == 0 and s0["stages"] == 0
    sg = g.sweep(*args, 2, d["seed"])
    kt = g.kernel_times()
    assert kt["stage"][2] >= sg["stages"] and kt["stage"][1] > 0
    so, _, _ = O.sweep(st, *args, 2, d["seed"])
    for key in ("trials", "local_accepts", "stage_accepts", "flips", "n_final"):
        assert sg[key] == so[key], key
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


@pytest.mark.parametrize("k", [2, 5])
def test_local_chain_parity(torch_cuda, oracle_mod, k):
    """k trials per active cell per stage: every trial (its dU, decision and
    margin), every stage and the final state equal the oracle's."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    args = (d["dmu0"], 5.0, d["cbar"], d["T"])
    g = gpu_context(d, pot)
    g.set_local_steps(k)
    info = g.info()
    S = info["stages_per_sweep"]
    ncpc = int(np.prod(info["n_cells"])) // 8
    n_sw = 3
    g.enable_log(n_sw * S * ncpc * k, n_sw * S)
    sg = g.sweep(*args, n_sw, d["seed"])
    tl_g, sl_g, nt, ns = g.logs()
    st = oracle_state(O, d, pot)
    so, tl_o, sl_o = O.sweep(st, *args, n_sw, d["seed"], log_trials=10 ** 8, log_stages=10 ** 8,
                             overrides=tie_overrides(tl_g, sl_g), local_steps=k)
    compare_logs(tl_g, sl_g, tl_o, sl_o)
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert sg[key] == so[key], key
    assert 0 < sg["stage_accepts"] < sg["stages"]
    assert sg["local_accepts"] > sg["flips"]  # some stages were undone
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    # the same chain without logs (replayed graph), from a fresh context
    g2 = gpu_context(d, pot)
    g2.set_tuning("stage", 1)
    g2.set_local_steps(k)
    s2 = g2.sweep(*args, n_sw, d["seed"])
    assert s2["flips"] == so["flips"] and s2["n_final"] == so["n_final"]
    assert np.array_equal(g2.species.cpu().numpy(), st.species)
    g.close()
    g2.close()


def test_local_chain_undo_restores_velocities(torch_cuda, oracle_mod):
    """With velocities, trials of undone stages restore them exactly."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _md_system(n=16, c=0.1, seed=43)
    g = gpu_context(d, pot, velocities=True)
    g.set_local_steps(3)
    sg = g.sweep(d["dmu0"], 1.0, d["cbar"], d["T"], 2, d["seed"])
    st = O.SweepState(d["x"], d["y"], d["z"], d["box"], d["species"], pot, vx=d["vx"], vy=d["vy"],
                      vz=d["vz"])
    so, _, _ = O.sweep(st, d["dmu0"], 1.0, d["cbar"], d["T"], 2, d["seed"], local_steps=3)
    assert sg["flips"] == so["flips"] and sg["stage_accepts"] < sg["stages"]
    for nm in ("vx", "vy", "vz"):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), getattr(st, nm)), nm
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    g.close()


def _md_system(n=10, T=700.0, seed=31, c=0.05):
    x, y, z, box = I.bcc(n, n, n)
    x, y, z = I.thermalize(x, y, z, box, 0.05, seed)
    sp = I.initial_species(x.size, c, seed + 1)
    vx, vy, vz = I.mb_velocities(sp, T, seed + 2)
    return dict(x=x, y=y, z=z, box=box, species=sp, vx=vx, vy=vy, vz=vz, T=T, kappa=1000.0,
                cbar=c, dmu0=W.dmu_s(T, c), seed=4001)


def test_md_parity(torch_cuda, oracle_mod):
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _md_system()
    g = gpu_context(d, pot, velocities=True)
    g.md(1.0, 40)
    out = O.md(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"], d["species"], d["box"], pot,
               1.0, 40)
    names = ("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz")
    for nm, want in zip(names, out[:9]):
        got = getattr(g, nm).cpu().numpy()
        assert np.array_equal(got, want), nm
    g.close()


@pytest.mark.parametrize("n,skin", [(6, 0.75), (7, 0.3)])
def test_md_parity_build_paths(torch_cuda, oracle_mod, n, skin):
    """MD lists from both builders: a 6^3 box with a 0.75 A skin has three
    search bins per axis (one lane per atom), a 7^3 box with the default skin
    five (super-bins, odd count: the last super-bin is half empty).
    Device-decided rebuilds happen in the 60 steps at 1000 K; positions,
    velocities and forces stay bit for bit those of the oracle, and the
    list statistics equal a fresh build at the final positions."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _md_system(n=n, T=1000.0, seed=53 + n)
    g = gpu_context(d, pot, velocities=True, skin=skin)
    g.md(1.0, 60)
    out = O.md(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"], d["species"], d["box"], pot,
               1.0, 60)
    names = ("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz")
    for nm, want in zip(names, out[:9]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    info = g.info()
    assert info["md_rebuilds"] >= 1
    x, y, z = out[0], out[1], out[2]
    nl = O.neighbors(x, y, z, d["box"], pot.rc, vectors=False)
    # the r < rc list filtered out of the MD list and the density cache from
    # the last MD density pass
    g.sweep(d["dmu0"], 0.0, d["cbar"], d["T"], 0, d["seed"])
    assert g.info()["mc_pairs"] == nl.j.size
    assert g.info()["mc_kmax_used"] == int(np.diff(nl.start).max())
    assert np.array_equal(g.rho().cpu().numpy(), O.density(nl, d["species"], pot))
    g.close()


@pytest.mark.parametrize("dims,pot", [
    ((29, 29, 29), "FS-P1"),  # 48,778 atoms: the largest cube with four lanes per atom
    ((30, 28, 30), "FS-P1"),  # 50,400: one lane
    ((30, 28, 30), "TAB-X"),  # two lanes
    ((6, 7, 9), "TAB-X"),     # four lanes, a row is one to two rounds, every wave wraps
])
def test_md_lanes_per_atom(torch_cuda, oracle_mod, dims, pot):
    """Energies, forces and three steps on both sides of the sizes at which the
    MD passes change their lanes per atom, bit for bit."""
    O = oracle_mod
    pot = I.params(pot) if pot == "FS-P1" else I.table(pot)
    x, y, z, box = I.bcc(*dims)
    x, y, z = I.thermalize(x, y, z, box, 0.08, 21)
    sp = I.initial_species(x.size, 0.2, 22)
    vx, vy, vz = I.mb_velocities(sp, 900.0, 23)
    d = dict(x=x, y=y, z=z, box=box, species=sp, vx=vx, vy=vy, vz=vz)
    _eam_parity(O, d, pot)
    g = gpu_context(d, pot, velocities=True)
    g.md(2.0, 3)
    out = O.md(x, y, z, vx, vy, vz, sp, box, pot, 2.0, 3)
    for nm, want in zip(("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz"), out[:9]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    g.close()


@pytest.mark.parametrize("dims", [(6, 8, 11), (29, 29, 29), (30, 28, 30)])
def test_md_list_statistics_after_rebuild(torch_cuda, oracle_mod, dims):
    """The list the steps rebuild, with the drift's own binning (up to 48k
    atoms) and without: after the step that rebuilds it holds every pair
    within rc + skin and none beyond the float margin of the search; the
    trajectory is the oracle's."""
    O = oracle_mod
    pot = I.params("FS-P1")
    skin = 0.3
    x, y, z, box = I.bcc(*dims)
    x, y, z = I.thermalize(x, y, z, box, 0.05, 41)
    sp = I.initial_species(x.size, 0.1, 42)
    vx, vy, vz = I.mb_velocities(sp, 1500.0, 43)
    d = dict(x=x, y=y, z=z, box=box, species=sp, vx=vx, vy=vy, vz=vz)
    g = gpu_context(d, pot, velocities=True, skin=skin)
    g.md(1.0, 1)
    base, steps = g.info()["md_rebuilds"], 1
    while g.info()["md_rebuilds"] == base:
        g.md(1.0, 1)
        steps += 1
        assert steps < 60
    pos = [v.cpu().numpy() for v in (g.x, g.y, g.z)]
    lo = O.neighbors(*pos, box, pot.rc + skin, vectors=False).j.size
    hi = O.neighbors(*pos, box, pot.rc + skin + 2e-3, vectors=False).j.size
    assert lo <= g.info()["md_pairs"] <= hi
    g.close()
    g = gpu_context(d, pot, velocities=True, skin=skin)
    g.md(1.0, steps + 2)
    assert g.info()["md_rebuilds"] > base
    out = O.md(x, y, z, vx, vy, vz, sp, box, pot, 1.0, steps + 2)
    for nm, want in zip(("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz"), out[:9]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    g.close()


def test_md_list_statistics_of_an_empty_list(torch_cuda, oracle_mod):
    """Two atoms that fly apart: the list rebuilt on the way has no entry, and
    says so."""
    O = oracle_mod
    pot = I.params("FS-P1")
    x, y, z = np.array([8.0, 11.85]), np.array([9.0, 9.0]), np.array([10.0, 10.0])
    v, zero = np.array([-0.05, 0.05]), np.zeros(2)
    box, sp = np.full(3, 20.0), np.array([0, 1], np.uint8)
    d = dict(x=x, y=y, z=z, box=box, species=sp, vx=v, vy=zero, vz=zero)
    g = gpu_context(d, pot, velocities=True)
    g.md(1.0, 1)
    assert g.info()["md_pairs"] == 2
    g.md(1.0, 11)
    assert g.info()["md_rebuilds"] > 1
    assert g.info()["md_pairs"] == 0
    out = O.md(x, y, z, v, zero, zero, sp, box, pot, 1.0, 12)
    assert np.array_equal(g.x.cpu().numpy(), out[0])
    g.close()


@pytest.mark.parametrize("path", ["pipeline", "da_perfect", "chain3", "persistent", "batch",
                                  "da_batch"])
def test_sweep_paths_after_md(torch_cuda, oracle_mod, path):
    """Sweeps right after MD run on the r < rc list filtered out of the MD
    rows and on the last MD density pass: every sweep kernel family (fused
    pipeline, delayed acceptance with a perfect surrogate, local chains with
    their undo log, the persistent kernel) gives the oracle's chain bit for
    bit, velocities included."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _md_system(n=16, c=0.1, seed=47)
    kappa, n_sw, k = 1.0, 2, 3 if path == "chain3" else 1
    x, y, z, vx, vy, vz, *_ = O.md(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"],
                                   d["species"], d["box"], pot, 1.0, 20)
    g = gpu_context(d, pot, velocities=True)
    g.md(1.0, 20)
    if path in ("da_perfect", "da_batch"):
        g.set_surrogate("perfect")
    if path in ("batch", "da_batch"):
        g.set_tuning("batch", 4)
    elif path == "chain3":
        g.set_local_steps(k)
    elif path == "persistent":
        g.set_tuning("graph", 1)
    nl = O.neighbors(x, y, z, d["box"], pot.rc, vectors=False)
    assert np.array_equal(g.rho().cpu().numpy(), O.density(nl, d["species"], pot))
    info = g.info()
    S = info["stages_per_sweep"]
    ncpc = int(np.prod(info["n_cells"])) // 8
    assert info["mc_pairs"] == nl.j.size
    log = path in ("pipeline", "chain3")
    if log:
        g.enable_log(n_sw * S * ncpc * k, n_sw * S)
    sg = g.sweep(d["dmu0"], kappa, d["cbar"], d["T"], n_sw, d["seed"])
    st = O.SweepState(x, y, z, d["box"], d["species"], pot, vx=vx, vy=vy, vz=vz)
    over = None
    if log:
        tl_g, sl_g, _, _ = g.logs()
        over = tie_overrides(tl_g, sl_g)
    so, tl_o, sl_o = O.sweep(st, d["dmu0"], kappa, d["cbar"], d["T"], n_sw, d["seed"],
                             log_trials=10 ** 8 if log else 0, log_stages=10 ** 8 if log else 0,
                             overrides=over, local_steps=k)
    if log:
        compare_logs(tl_g, sl_g, tl_o, sl_o)
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert sg[key] == so[key], key
    assert sg["flips"] > 0
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    for nm in ("vx", "vy", "vz"):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), getattr(st, nm)), nm
    g.close()


def test_hybrid_cycle_parity(torch_cuda, oracle_mod):
    """[1 sweep; 20 MD steps] x 3 with velocity rescaling on transmutation."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = _md_system(n=16, c=0.1, seed=41)
    g = gpu_context(d, pot, velocities=True)
    x, y, z = d["x"], d["y"], d["z"]
    vx, vy, vz = d["vx"], d["vy"], d["vz"]
    sp = d["species"]
    w = 0
    for cyc in range(3):
        g.sweep(d["dmu0"], 1.0, d["cbar"], d["T"], 1, d["seed"])
        st = O.SweepState(x, y, z, d["box"], sp, pot, vx=vx, vy=vy, vz=vz)
        st.w = w
        O.sweep(st, d["dmu0"], 1.0, d["cbar"], d["T"], 1, d["seed"])
        w += 1
        sp = st.species
        assert np.array_equal(g.rho().cpu().numpy(), st.rho)
        g.md(1.0, 20)
        x, y, z, vx, vy, vz, *_ = O.md(x, y, z, st.vx, st.vy, st.vz, sp, d["box"], pot, 1.0, 20)
        # the sweep's lists and density cache after MD come from the MD list and
        # the last MD density pass: equal to a fresh r < rc build at the new positions
        nl = O.neighbors(x, y, z, d["box"], pot.rc, vectors=False)
        assert np.array_equal(g.rho().cpu().numpy(), O.density(nl, sp, pot))
        assert g.info()["mc_pairs"] == nl.j.size
    assert np.array_equal(g.species.cpu().numpy(), sp)
    for nm, want in zip(("x", "y", "z", "vx", "vy", "vz"), (x, y, z, vx, vy, vz)):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    g.close()


@pytest.fixture(scope="module")
def c3_data():
    return W.c3()


def test_full_size_c3_sweep_and_md(torch_cuda, oracle_mod, c3_data):
    """The 1.96M-site polycrystal: one full sweep (species and density cache
    bit for bit, every counter equal) and two MD steps (positions and
    velocities bit for bit)."""
    O = oracle_mod
    pot = I.params("FS-P1")
    d = c3_data
    g = gpu_context(d, pot, velocities=True)
    s = g.sweep(d["dmu0"], d["kappa"], d["cbar"], d["T"], 1, d["seed"])
    st = oracle_state(O, d, pot, velocities=True)
    so, _, _ = O.sweep(st, d["dmu0"], d["kappa"], d["cbar"], d["T"], 1, d["seed"])
    for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert s[k] == so[k], k
    assert s["trials"] >= 0.9 * x_size(d)
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.md(1.0, 2)
    out = O.md(d["x"], d["y"], d["z"], st.vx, st.vy, st.vz, st.species, d["box"], pot, 1.0, 2)
    for nm, want in zip(("x", "y", "z", "vx", "vy", "vz"), out[:6]):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), want), nm
    g.close()


def x_size(d):
    return d["x"].size


@pytest.mark.parametrize("path", ["stage_logged", "batch", "graph", "chain3", "da_perfect"])
def test_colours27_parity(torch_cuda, oracle_mod, path):
    """The 27-colour scheme (cells of edge >= r_dep / 2, colours by indices
    modulo 3) on every sweep kernel family: the chain equals the oracle's
    chain with the same colouring, bit for bit (trial and stage logs too on
    the logged path)."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGC
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    k = 3 if path == "chain3" else 1
    args = (d["dmu0"], 10.0, d["cbar"], d["T"])
    g = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot, colours=27)
    info = g.info()
    nc = np.array(info["n_cells"])
    assert np.all(nc % 3 == 0) and np.array_equal(nc, O.cell_grid(d["box"], 2 * pot.rc, 3))
    ncells = int(np.prod(nc))
    assert info["stages_per_sweep"] == 27 * -(-d["x"].size // ncells)
    if path == "stage_logged":
        g.set_tuning("stage", 1)
        g.enable_log(3 * info["stages_per_sweep"] * (ncells // 27), 3 * info["stages_per_sweep"])
    elif path == "batch":
        g.set_tuning("batch", 4)
    elif path == "graph":
        g.set_tuning("graph", 1)
    elif path == "chain3":
        g.set_local_steps(k)
    elif path == "da_perfect":
        g.set_surrogate("perfect")
    sg = g.sweep(*args, 2, d["seed"])
    sg2 = g.sweep(*args, 1, d["seed"])
    st = oracle_state(O, d, pot)
    log = path == "stage_logged"
    over = None
    if log:
        tl_g, sl_g, _, _ = g.logs()
        over = tie_overrides(tl_g, sl_g)
    so, tl_o, sl_o = O.sweep(st, *args, 3, d["seed"], log_trials=10 ** 8 if log else 0,
                             log_stages=10 ** 8 if log else 0, overrides=over, local_steps=k,
                             colour_period=3)
    if log:
        compare_logs(tl_g, sl_g, tl_o, sl_o)
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips"):
        assert sg[key] + sg2[key] == so[key], key
    assert sg2["n_final"] == so["n_final"]
    assert so["stage_accepts"] > 0
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


def test_colours27_after_md_and_replicas(torch_cuda, oracle_mod):
    """27 colours after MD with velocities (batched pipeline), and in a
    replica batch (persistent launch): both equal the oracle."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGC, VCSGCBatch
    pot = I.params("FS-P1")
    d = _md_system(n=16, c=0.1, seed=49)
    x, y, z, vx, vy, vz, *_ = O.md(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"],
                                   d["species"], d["box"], pot, 1.0, 20)
    g = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot, vx=d["vx"], vy=d["vy"],
              vz=d["vz"], colours=27)
    g.md(1.0, 20)
    g.set_tuning("batch", 4)
    sg = g.sweep(d["dmu0"], 1.0, d["cbar"], d["T"], 2, d["seed"])
    st = O.SweepState(x, y, z, d["box"], d["species"], pot, vx=vx, vy=vy, vz=vz)
    so, _, _ = O.sweep(st, d["dmu0"], 1.0, d["cbar"], d["T"], 2, d["seed"], colour_period=3)
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final"):
        assert sg[key] == so[key], key
    assert sg["flips"] > 0
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    for nm in ("vx", "vy", "vz"):
        assert np.array_equal(getattr(g, nm).cpu().numpy(), getattr(st, nm)), nm
    g.close()
    reps = _replica_set(n_rep=4, seed=57)
    b = VCSGCBatch(reps, pot, colours=27)
    par = [np.array([r[k] for r in reps]) for k in ("dmu0", "kappa", "cbar", "T")]
    s1 = b.sweep_batch(*par, 2, 888)
    for k, r in enumerate(reps):
        stk = O.SweepState(r["x"], r["y"], r["z"], r["box"], r["species"], pot)
        sok, _, _ = O.sweep(stk, r["dmu0"], r["kappa"], r["cbar"], r["T"], 2, 888, replica=k,
                            colour_period=3)
        assert s1[k]["flips"] == sok["flips"] and s1[k]["n_final"] == sok["n_final"], k
        assert np.array_equal(b.replica_species(k), stk.species), k
    b.close()


@pytest.mark.parametrize("nx,colours,kappa,tpg", [
    ((6, 6, 6), 8, 0.0, 1),        # state in LDS, one cell per stage, accepted stages
    ((10, 10, 10), 27, 1.0, 1),    # resident, 8 cells per stage
    ((17, 18, 19), 8, 1.0, 1),     # the last sizes that stay resident
    ((18, 18, 19), 8, 0.0, 1),     # the first that do not: several workgroups, commits at every stage
    ((23, 31, 17), 27, 10.0, 4),   # uneven shares of the cells
    ((33, 26, 29), 8, 1000.0, 16),  # more cells per workgroup than trial groups
])
def test_persistent_batches(torch_cuda, oracle_mod, nx, colours, kappa, tpg):
    """The persistent sweep tries batches of stages: on both sides of its
    choices (state in LDS or in memory, one or several workgroups, one or
    several passes over the cells) three calls give the oracle's chain bit for
    bit, with the statistics of decided stages only."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGC
    pot = I.params("FS-P1")
    x, y, z, box = I.bcc(*nx)
    x, y, z = I.thermalize(x, y, z, box, 0.04, 5)
    sp = I.initial_species(x.size, 0.1, 6)
    g = VCSGC(x, y, z, box, sp, pot, colours=colours)
    g.set_tuning("graph", 2)
    g.set_tuning("graph", tpg)
    st = O.SweepState(x, y, z, box, sp, pot)
    for n_sw in (1, 2, 1):
        a = g.sweep(-0.2, kappa, 0.1, 600.0, n_sw, 31)
        b, _, _ = O.sweep(st, -0.2, kappa, 0.1, 600.0, n_sw, 31,
                          colour_period=3 if colours == 27 else 2)
        for k in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final",
                  "sum_n", "sum_n2"):
            assert a[k] == b[k], (k, a[k], b[k])
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()


@pytest.mark.parametrize("k", [2, 5])
def test_local_chains_odd_stages(torch_cuda, oracle_mod, k):
    """Local chains over sweeps of an odd number of stages (27 colours): n_B
    after the last stage of a sweep is the one that the next sweep starts
    from, also between the sweeps of one call."""
    O = oracle_mod
    from paper_1012_5082_amd.binding import VCSGC
    pot = I.params("FS-P1")
    x, y, z, box = I.bcc(12, 12, 12)
    x, y, z = I.thermalize(x, y, z, box, 0.05, 5)
    sp = I.initial_species(x.size, 0.1, 6)
    args = (-0.3, 1.0, 0.1, 600.0)
    g = VCSGC(x, y, z, box, sp, pot, colours=27)
    g.set_local_steps(k)
    S = g.info()["stages_per_sweep"]
    assert S % 2 == 1
    sg = g.sweep(*args, 4, 313)
    st = O.SweepState(x, y, z, box, sp, pot)
    so, _, sl = O.sweep(st, *args, 4, 313, local_steps=k, colour_period=3, log_stages=4 * S)
    last = [sl[S * (q + 1) - 1] for q in range(3)]
    assert any(r[5] == 1.0 and r[3] != 0.0 for r in last)  # n_B changes in a last stage
    for key in ("trials", "local_accepts", "stages", "stage_accepts", "flips", "n_final",
                "sum_n", "sum_n2"):
        assert sg[key] == so[key], key
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()
