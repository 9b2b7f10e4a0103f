"""GPU surrogate pieces against the oracle.

* network forward (BF16 MFMA, FP32 accumulation) vs the oracle's FP64
  evaluation with BF16 rounding of the same operands;
* gradients of the hand-written backward kernels vs the oracle's emulated
  gradient, norm-wise per parameter tensor;
* descriptors (current and flipped state) bit for bit;
* delayed acceptance: a perfect surrogate reproduces the plain chain bit for
  bit; with the network, the oracle replays the chain from the GPU's logged
  surrogate values (compare mode) and must agree bit for bit;
* sample logging and training on samples of the method itself.
"""
import numpy as np
import pytest

from paper_1012_5082_amd import inputs as I
from paper_1012_5082_amd import workloads as W
from parity_utils import compare_logs

pytestmark = pytest.mark.gpu

# Tolerances of the network against the oracle's emulation (BF16 operands,
# FP64 sums), set from measured errors: the GPU sums in FP32 in the MFMA
# units' order and evaluates SiLU in FP32, so now and then a hidden
# activation rounds to the neighbouring BF16 value.  Measured on MI355X:
# forward max 1.9e-7 / median 9.6e-9 (1,000 samples), in-sweep block max
# 1.5e-4 / median 9.6e-9 (390,295 values), gradient at most 7.5e-6 per
# tensor.
FWD_MAX, FWD_MEDIAN = 1e-3, 1e-7   # of (max |dE| + out_sd)
GRAD_REL = 1e-4                    # per parameter tensor, norm-wise

TENSORS = [("w1", 0, 640), ("b1", 640, 704), ("w2", 704, 4800), ("b2", 4800, 4864),
           ("w3", 4864, 4928), ("b3", 4928, 4929)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _samples(n=512, seed=1):
    rng = np.random.default_rng(seed)
    d = np.column_stack([rng.integers(0, 2, n), rng.integers(0, 4, (n, 3)),
                         rng.integers(6, 13, (n, 3)), rng.normal(13.0, 0.3, (n, 3))])
    t = rng.normal(0.4, 0.2, n)
    return d.astype(np.float64), t


def _params(seed=3):
    from oracle.oracle import MlpParams
    mu = np.array([0.5, 1, 1, 1, 8, 6, 12, 13, 13, 13], dtype=np.float64)
    sd = np.array([0.5, 1, 1, 1, 1, 1, 1, 0.5, 0.5, 0.5], dtype=np.float64)
    return MlpParams.random(seed, mu=mu, sd=sd, out_mu=0.4, out_sd=0.2)


def _gpu_mlp(m):
    from paper_1012_5082_amd.binding import Mlp
    g = Mlp(seed=0)
    g.set_params(m.flat(), m.mu, m.sd, m.out_mu, m.out_sd)
    return g


def test_mlp_forward_matches_oracle(torch_cuda, oracle_mod):
    torch = torch_cuda
    m = _params()
    d, _ = _samples(1000)
    g = _gpu_mlp(m)
    got = g.forward(torch.tensor(d, device="cuda")).cpu().numpy()
    _, want = oracle_mod.mlp_forward(m, d, bf16_emul=True)
    err = np.abs(got - want)
    scale = np.abs(want).max() + m.out_sd
    print(f"network forward vs oracle: max err {err.max() / scale:.3e}, "
          f"median {np.median(err) / scale:.3e} of scale {scale:.4f} eV")
    assert err.max() <= FWD_MAX * scale, (err.max(), scale)
    assert np.median(err) <= FWD_MEDIAN * scale, np.median(err)
    g.close()


def test_mlp_gradient_matches_oracle(torch_cuda, oracle_mod):
    torch = torch_cuda
    m = _params(5)
    d, t = _samples(2048, seed=2)
    g = _gpu_mlp(m)
    loss_g, grad_g = g.grad(torch.tensor(d, device="cuda"), torch.tensor(t, device="cuda"))
    loss_o, grad_o = oracle_mod.mlp_grad(m, d, t, bf16_emul=True)
    assert abs(loss_g - loss_o) <= 1e-3 * loss_o
    rels = {}
    for name, a, b in TENSORS:
        rels[name] = float(np.linalg.norm(grad_g[a:b] - grad_o[a:b]) / np.linalg.norm(grad_o[a:b]))
    print("gradient rel. norm error per tensor: " +
          ", ".join(f"{k} {v:.2e}" for k, v in rels.items()) + f"; loss {loss_g:.6e} vs {loss_o:.6e}")
    for name, rel in rels.items():
        assert rel <= GRAD_REL, (name, rel)
    g.close()


def _c2_state(O, pot, sweeps=3, cbar=0.1, r_dep=0.0):
    from paper_1012_5082_amd.binding import VCSGC
    d = W.c2(cbar=cbar)
    g = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot, descriptor=True, r_dep=r_dep)
    if sweeps:
        g.sweep(d["dmu0"], 5.0, cbar, d["T"], sweeps, 11)
    return d, g


def test_descriptors_match_oracle(torch_cuda, oracle_mod):
    O = oracle_mod
    pot = I.params("FS-P1")
    d, g = _c2_state(O, pot)
    sp = g.species.cpu().numpy()
    rho = g.rho().cpu().numpy()
    dnl = O.neighbors(d["x"], d["y"], d["z"], d["box"], O.DESC_CUTOFF, vectors=False)
    sites = np.random.default_rng(0).choice(d["x"].size, 600, replace=False).astype(np.int32)
    for flip in (False, True):
        got = g.descriptors(sites, flip=flip)
        want = np.stack([O.descriptor(dnl, i, sp, rho, pot, flip=flip) for i in sites])
        assert np.array_equal(got, want), flip
    g.close()


@pytest.mark.parametrize("desc,batch", [(False, 0), (True, 0), (True, 8)])
def test_da_perfect_surrogate_equals_plain(torch_cuda, oracle_mod, desc, batch):
    """With the exact dU as surrogate the chain is the plain one, bit for bit;
    with the descriptor list present dU comes from that list's r < rc
    entries instead of the r < rc list, and must be the same number.  Also
    through the batched pipeline (batch > 0 stages per kernel)."""
    pot = I.params("FS-P1")
    d = W.c2(cbar=0.05)
    from paper_1012_5082_amd.binding import VCSGC
    a = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot)
    b = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot, descriptor=desc,
              r_dep=8.01 if desc else 0.0)
    if desc:
        a.close()
        a = VCSGC(d["x"], d["y"], d["z"], d["box"], d["species"], pot, r_dep=8.01)
    b.set_surrogate("perfect")
    if batch:
        b.set_tuning("batch", batch)
    args = (d["dmu0"], 5.0, 0.05, d["T"], 5, d["seed"])
    sa, sb = a.sweep(*args), b.sweep(*args)
    for k in ("trials", "local_accepts", "stage_accepts", "flips", "n_final"):
        assert sa[k] == sb[k], k
    assert sb["stage1_pass"] == sa["local_accepts"]
    assert np.array_equal(a.species.cpu().numpy(), b.species.cpu().numpy())
    assert np.array_equal(a.rho().cpu().numpy(), b.rho().cpu().numpy())
    a.close()
    b.close()


def test_da_network_chain_matches_oracle_replay(torch_cuda, oracle_mod):
    """DA with the network: the oracle consumes the GPU's logged surrogate
    values (forward and reverse) and must reproduce the whole chain."""
    O = oracle_mod
    pot = I.params("FS-P1")
    r_dep = 8.01
    d, g = _c2_state(O, pot, sweeps=0, cbar=0.05, r_dep=r_dep)
    m = _params(7)
    m.out_mu, m.out_sd = float(np.float32(0.45)), float(np.float32(0.2))
    net = _gpu_mlp(m)
    g.set_surrogate("mlp", net)
    info = g.info()
    S, ncpc = info["stages_per_sweep"], int(np.prod(info["n_cells"])) // 8
    n_sw = 3
    g.enable_log(n_sw * S * ncpc, n_sw * S)
    g.enable_surrogate_log(n_sw * S * ncpc)
    args = (d["dmu0"], d["kappa"], d["cbar"], d["T"])
    sg = g.sweep(*args, n_sw, d["seed"])
    tl_g, sl_g, nt, ns = g.logs()
    table = g.surrogate_log()
    assert table.shape[0] == nt
    assert 0 < sg["stage1_pass"] < sg["trials"]
    st = O.SweepState(d["x"], d["y"], d["z"], d["box"], d["species"], pot)
    dnl = O.neighbors(d["x"], d["y"], d["z"], d["box"], O.DESC_CUTOFF, vectors=False)
    so, p1, tl_o, sl_o, dlog = O.sweep_da(st, *args, n_sw, d["seed"], "table", r_dep=r_dep,
                                          table=table, desc_nl=dnl, log_trials=10 ** 8,
                                          log_stages=10 ** 8, log_desc=nt + 1)
    assert p1 == sg["stage1_pass"]
    # the values the in-sweep network block produced, against the oracle's
    # network (BF16 operand rounding, FP64 sums) on the oracle's own
    # descriptors of the same trials at the same states
    assert dlog.shape[0] == table.shape[0]
    assert np.array_equal(dlog[:, :3], table[:, :3])
    _, want_f = O.mlp_forward(m, dlog[:, 3:13], bf16_emul=True)
    _, want_r = O.mlp_forward(m, dlog[:, 13:23], bf16_emul=True)
    surv = ~np.isnan(table[:, 4])
    assert surv.sum() == sg["stage1_pass"]
    err = np.concatenate([np.abs(table[:, 3] - want_f), np.abs(table[surv, 4] - want_r[surv])])
    scale = max(np.abs(want_f).max(), np.abs(want_r[surv]).max()) + m.out_sd
    print(f"in-sweep network vs oracle: {err.size} values, max err {err.max() / scale:.3e}, "
          f"median {np.median(err) / scale:.3e} of scale {scale:.4f} eV")
    assert err.max() <= FWD_MAX * scale, (err.max(), scale)
    assert np.median(err) <= FWD_MEDIAN * scale, (np.median(err), scale)
    for k in ("trials", "local_accepts", "stage_accepts", "flips", "n_final"):
        assert sg[k] == so[k], k
    # dU is logged (and compared) for survivors only
    keep = ~np.isnan(tl_o[:, 6])
    assert np.array_equal(np.isnan(tl_g[:, 6]), ~keep)
    compare_logs(tl_g[keep], sl_g, tl_o[keep], sl_o)
    assert np.array_equal(g.species.cpu().numpy(), st.species)
    assert np.array_equal(g.rho().cpu().numpy(), st.rho)
    g.close()
    net.close()


@pytest.mark.parametrize("batch", [0, 8])
def test_da_network_graph_replay_matches_direct(torch_cuda, oracle_mod, batch):
    """DA with the network, replayed as a graph (no logs; stage by stage, or
    batches of stages when batch > 0) and launched stage by stage (the
    surrogate log forces that path): the same chain bit for bit, over calls
    that change the parameters in between."""
    O = oracle_mod
    pot = I.params("FS-P1")
    r_dep = 8.01
    m = _params(7)
    m.out_mu, m.out_sd = float(np.float32(0.45)), float(np.float32(0.2))
    net = _gpu_mlp(m)
    runs = []
    for logged in (True, False):
        d, g = _c2_state(O, pot, sweeps=0, cbar=0.05, r_dep=r_dep)
        g.set_surrogate("mlp", net)
        if batch:
            g.set_tuning("batch", batch)
        if logged:
            g.enable_surrogate_log(2 * 10 ** 6)
        out = []
        for cb, n_sw in ((0.05, 2), (0.10, 3), (0.05, 2)):
            s = g.sweep(d["dmu0"], d["kappa"], cb, d["T"], n_sw, d["seed"])
            out.append({k: s[k] for k in ("trials", "stage1_pass", "local_accepts",
                                           "stage_accepts", "flips", "n_final")})
        out.append(g.species.cpu().numpy().copy())
        out.append(g.rho().cpu().numpy().copy())
        runs.append(out)
        g.close()
    a, b = runs
    for k in range(3):
        assert a[k] == b[k], k
    assert a[0]["stage1_pass"] < a[0]["trials"]
    assert np.array_equal(a[3], b[3])
    assert np.array_equal(a[4], b[4])
    net.close()


@pytest.mark.parametrize("dims,colours,pot,kappa", [
    ((6, 6, 6), 8, "FS-P1", 0.0),       # one workgroup, one cell per stage
    ((17, 13, 19), 8, "TAB-X", 1.0),    # tables, several workgroups
    ((23, 31, 17), 27, "FS-P1", 10.0),  # 27 colours, uneven shares of the cells
    ((62, 60, 64), 8, "FS-P1", 1000.0),  # more than one pass of the trial groups
])
def test_da_network_persistent_matches_stages(torch_cuda, dims, colours, pot, kappa):
    """The network's delayed acceptance in the persistent sweep against the
    kernels per stage (the surrogate log takes that path): the same chain and
    statistics bit for bit."""
    from paper_1012_5082_amd.binding import VCSGC
    pot = I.params(pot) if pot == "FS-P1" else I.table(pot)
    x, y, z, box = I.bcc(*dims)
    x, y, z = I.thermalize(x, y, z, box, 0.04, 5)
    sp = I.initial_species(x.size, 0.1, 6)
    m = _params(7)
    m.out_mu, m.out_sd = float(np.float32(0.45)), float(np.float32(0.2))
    net = _gpu_mlp(m)
    runs = []
    for logged in (True, False):
        g = VCSGC(x, y, z, box, sp, pot, descriptor=True, r_dep=8.01, colours=colours)
        g.set_surrogate("mlp", net)
        if logged:
            g.enable_surrogate_log(10 ** 6)
        out = []
        for n_sw in (1, 2):
            s = g.sweep(-0.2, kappa, 0.1, 600.0, n_sw, 31)
            out.append({k: s[k] for k in ("trials", "stage1_pass", "local_accepts", "stages",
                                           "stage_accepts", "flips", "n_final", "sum_n", "sum_n2")})
        runs.append((out, g.species.cpu().numpy().copy(), g.rho().cpu().numpy().copy()))
        g.close()
    net.close()
    assert runs[0][0] == runs[1][0]
    assert 0 < runs[0][0][0]["stage1_pass"] < runs[0][0][0]["trials"]
    assert np.array_equal(runs[0][1], runs[1][1])
    assert np.array_equal(runs[0][2], runs[1][2])


@pytest.mark.parametrize("strategy,tpg", [("graph", 1), ("batch", 4)])
def test_da_network_never_times_out(torch_cuda, strategy, tpg):
    """With a wait limit of one poll the network's persistent sweep ends before
    it has changed anything and the call runs with kernels per stage: the chain
    of the default limit, with a network trained on the system's own samples."""
    from paper_1012_5082_amd.binding import VCSGC, Mlp
    pot = I.params("FS-P1")
    x, y, z, box = I.bcc(23, 31, 17)
    x, y, z = I.thermalize(x, y, z, box, 0.04, 5)
    sp = I.initial_species(x.size, 0.1, 6)
    dmu0 = W.dmu_s(600.0, 0.1)

    def context():
        return VCSGC(x, y, z, box, sp, pot, descriptor=True, r_dep=8.01)

    g = context()
    g.enable_sample_log(60000, 1)
    g.sweep(dmu0, 5.0, 0.1, 600.0, 2, 3)
    desc, dE = g.samples()
    net = Mlp(seed=1)
    net.fit_normalization(desc, dE)
    net.train(desc, dE, epochs=4, batch=4096, lr=2e-3, seed=5)
    g.close()
    runs = []
    for limits in ((1 << 24, 1 << 24, 1 << 24), (1, 1 << 24, 1)):
        g = context()
        g.set_surrogate("mlp", net)
        g.set_tuning(strategy, tpg)
        out = []
        for limit in limits:
            g.set_wait_limit(limit)
            for kappa in (1000.0, 0.0):
                print(f"[limit] {strategy} {limit} {kappa}", flush=True)
                s = g.sweep(dmu0, kappa, 0.1, 600.0, 2, 31)
                out.append({k: s[k] for k in ("trials", "stage1_pass", "local_accepts", "stages",
                                               "stage_accepts", "flips", "n_final", "sum_n",
                                               "sum_n2")})
        runs.append((out, g.species.cpu().numpy().copy(), g.rho().cpu().numpy().copy()))
        g.close()
    net.close()
    assert runs[0][0] == runs[1][0]
    assert 0 < runs[0][0][1]["stage_accepts"]
    assert np.array_equal(runs[0][1], runs[1][1])
    assert np.array_equal(runs[0][2], runs[1][2])


def test_contexts_on_threads_and_streams(torch_cuda):
    """Sweeps whose workgroups wait for each other, from six contexts on
    threads and streams of their own (more workgroups together than compute
    units; two of them screened by a network, one a batch of replicas), beside
    a long run of a system in one workgroup: every chain is the one it makes
    alone."""
    import threading
    from paper_1012_5082_amd.binding import VCSGC, VCSGCBatch
    torch = torch_cuda
    pot = I.params("FS-P1")
    m = _params(7)
    m.out_mu, m.out_sd = float(np.float32(0.45)), float(np.float32(0.2))
    net = _gpu_mlp(m)
    torch.cuda.synchronize()
    sizes = [(20, 20, 20), (40, 40, 40), (23, 31, 17), (40, 38, 42), (62, 60, 64), None,
             (10, 10, 10)]

    def make(k, stream):
        if k == 5:
            reps = []
            for r in range(6):
                x, y, z, box = I.bcc(20 + r, 21, 24)
                reps.append(dict(x=x, y=y, z=z, box=box,
                                 species=I.initial_species(x.size, 0.1, 80 + r)))
            return VCSGCBatch(reps, pot, stream=stream)
        x, y, z, box = I.bcc(*sizes[k])
        x, y, z = I.thermalize(x, y, z, box, 0.04, 5 + k)
        g = VCSGC(x, y, z, box, I.initial_species(x.size, 0.1, 60 + k), pot, stream=stream,
                  descriptor=k in (2, 3), r_dep=8.01 if k in (2, 3) else 0.0)
        if k in (2, 3):
            g.set_surrogate("mlp", net)
        g.set_tuning(*(("batch", 4) if k == 1 else ("graph", 1)))
        return g

    def chain(k, g, out):
        stats = []
        for n_sw in (1, 2, 1, 1) if k < 6 else (200,):
            for kappa in (1.0, 0.0):
                stats.append(g.sweep_batch(-0.2, kappa, 0.1, 600.0, n_sw, 31) if k == 5
                             else g.sweep(-0.2, kappa, 0.1, 600.0, n_sw, 31))
        out[k] = (stats, g.species.cpu().numpy().copy())

    def contexts():
        gs = []
        for k in range(7):
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                gs.append(make(k, s))
        torch.cuda.synchronize()
        return gs

    alone, together = {}, {}
    gs = contexts()
    assert sum(g.tuning()["workgroups"] for g in gs) > 256
    for k, g in enumerate(gs):
        print(f"[threads] {k} alone", flush=True)
        chain(k, g, alone)
        g.close()
    gs = contexts()
    threads = [threading.Thread(target=chain, args=(k, g, together)) for k, g in enumerate(gs)]
    print("[threads] together", flush=True)
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, g in enumerate(gs):
        g.close()
        assert together[k][0] == alone[k][0], k
        assert np.array_equal(together[k][1], alone[k][1]), k
    net.close()


def test_sample_log_and_training(torch_cuda, oracle_mod):
    torch = torch_cuda
    pot = I.params("FS-P1")
    from paper_1012_5082_amd.binding import Mlp
    d, g = _c2_state(oracle_mod, pot, sweeps=0, cbar=0.05)
    g.enable_sample_log(200000, 7)
    g.sweep(d["dmu0"], 5.0, 0.05, d["T"], 6, 3)
    desc, dE = g.samples()
    n = desc.shape[0]
    assert n > 50000
    D = desc.cpu().numpy()
    assert np.all((D[:, 0] == 0) | (D[:, 0] == 1))
    # thermal bcc (sigma 0.05 A): a few first/second-shell neighbours cross the
    # 2.68 A edge, none crosses 3.46 A (0.6 A away from both shells)
    assert np.all(D[:, 4] + D[:, 5] == 14)
    assert np.median(D[:, 4]) == 8 and np.median(D[:, 5]) == 6
    assert np.all(np.abs(D[:, 6] - 12) <= 2)
    assert np.all(D[:, 1:4] <= D[:, 4:7])
    E = dE.cpu().numpy()
    assert np.all(np.isfinite(E)) and 0.2 < np.median(np.abs(E)) < 1.5
    net = Mlp(seed=1)
    net.fit_normalization(desc, dE)
    rep = net.train(desc, dE, epochs=4, batch=4096, lr=2e-3, seed=5)
    assert rep["loss_last"] < 0.5 * rep["loss_first"], rep
    pred = net.forward(desc).cpu().numpy()
    rmse = float(np.sqrt(np.mean((pred - E) ** 2)))
    assert rmse < 0.5 * float(np.std(E)), (rmse, float(np.std(E)))
    g.close()
    net.close()


@pytest.mark.parametrize("n", [1, 15, 17, 33, 255, 257, 511, 1025])
def test_gradient_batch_edges(torch_cuda, oracle_mod, n):
    """Batches around the kernels' tiles (16 samples per block, 32 per MFMA
    step, 256 rows per column-sum tile): gradient and loss against the oracle,
    with the tolerance of the gradient test."""
    torch = torch_cuda
    m = _params(5)
    net = _gpu_mlp(m)
    d, t = _samples(n, 40 + n)
    loss, g = net.grad(torch.tensor(d, device="cuda"), torch.tensor(t, device="cuda"))
    want_loss, want = oracle_mod.mlp_grad(m, d, t, bf16_emul=True)
    assert abs(loss - want_loss) <= GRAD_REL * max(abs(want_loss), 1e-12)
    for name, a, b in TENSORS:
        err = np.linalg.norm(g[a:b] - want[a:b])
        assert err <= GRAD_REL * max(np.linalg.norm(want[a:b]), 1e-12), (name, err)
    net.close()


@pytest.mark.parametrize("n", [2, 24, 25, 26, 6399, 6401, 100003])
def test_normalization_edges(torch_cuda, n):
    """Mean and standard deviation per column around the row groups of a block
    (25 rows) and of the grid (6,400), against numpy in 64 bits: FP64 sums
    rounded once to FP32 (the variance as E[x^2] - mean^2: its cancellation
    costs at most 2^-52 mean^2 n^(1/2) / var relative, below 1e-6 here)."""
    torch = torch_cuda
    from paper_1012_5082_amd.binding import Mlp
    d, t = _samples(n, 60)
    net = Mlp(seed=1)
    net.fit_normalization(torch.tensor(d, device="cuda"), torch.tensor(t, device="cuda"))
    _, mu, sd, om, osd = net.get_params()
    want = d.std(0)
    want[want <= 1e-6] = 1.0
    assert np.allclose(mu, d.mean(0), rtol=1e-6, atol=1e-7)
    assert np.allclose(sd, want, rtol=2e-6, atol=1e-7)
    assert abs(om - t.mean()) <= 1e-6 and abs(osd - t.std()) <= 1e-6
    net.close()
