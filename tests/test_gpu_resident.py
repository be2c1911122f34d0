"""GPU parity of the resident driver (ESP_MODE_RESIDENT, and ESP_MODE_AUTO where
the table fits): tiles kept on chip for the whole launch, every iteration
completed inside the launch; with several workgroups per cluster their exact
sums meet in counted words, as 45-bit limbs when one word does not hold them.
Every iterate against the free-running oracle (bitwise), over
one and many workgroups, dense and CSR tables, one to three limbs, several
clusters, penalties, staggered stops, and solves longer than one launch."""
import dataclasses
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2608_07971_amd as esp
import workloads

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-case] {msg}", flush=True)


def _wide(inst, seed, span):
    rng = np.random.default_rng(seed)
    inst.demand = (inst.demand.astype(np.float64) *
                   np.exp2(rng.integers(-span, span + 1, inst.demand.shape))).astype(np.float32)
    inst.eta0 = np.full(inst.B, 1e-12)
    return inst


CASES = {
    # name: (instance, blocks_per_cluster (0 = library default), T)
    "tiny_1wg": (lambda: workloads.make("tiny"), 0, 200),
    "small_128wg": (lambda: workloads.make("small"), 0, 500),
    "small_64wg_2tiles": (lambda: workloads.make("small"), 64, 120),
    "small_3wg_ragged_tail": (lambda: workloads.make("small", n_jobs=190), 3, 80),   # 24 tiles, last partial
    "ragged_3000_csr": (lambda: workloads.make("ragged", n_jobs=3000), 0, 120),
    "ragged_150_csr_1wg": (lambda: workloads.make("ragged", n_jobs=150), 1, 60),
    "batched_3x515": (lambda: workloads.make("batched", n_jobs=515, n_clusters=3), 0, 100),
    "k64_r8_dyadic": (lambda: workloads.random_small(7, 130, 64, 8, dense=True, dyadic=True, iters=80,
                                                     rule=workloads.STEP_CONST), 0, 80),
    "r1_k4": (lambda: workloads.random_small(5, 301, 4, 1, dense=True, iters=80), 0, 80),
    "wide_2limbs_k16": (lambda: _wide(workloads.random_small(90, 3000, 16, 5, dense=True, iters=60), 5, 12), 0, 60),
    "wide_3limbs_k16": (lambda: _wide(workloads.random_small(90, 3000, 16, 5, dense=True, iters=60), 5, 36), 0, 60),
    "wide_3limbs_csr_r8": (lambda: _wide(workloads.random_small(94, 1200, 40, 8, iters=60), 5, 36), 0, 60),
    "penalties_small": (lambda: workloads.with_penalties(workloads.make("small", n_jobs=2000), 9), 0, 100),
    "penalties_csr": (lambda: workloads.with_penalties(workloads.make("ragged", n_jobs=2500), 8), 0, 100),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_resident_every_iterate_matches_oracle(name):
    make, blocks, T = CASES[name]
    inst = make()
    _say(f"resident {name} B={inst.B} N={inst.N} R={inst.R} T={T} blocks={blocks}")
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT, blocks_per_cluster=blocks)
    assert s.loop_driver() == esp.ESP_MODE_RESIDENT
    g = s.solve(s.prices(inst.lam0), T, trace=True, trace_choice=True)
    torch.cuda.synchronize()
    assert s.device_status() == 0
    ref = oracle.Oracle(inst).solve(iters=T, trace_choice=True)
    for t in range(T):
        assert np.array_equal(g["tr_choice"][t].cpu().numpy(), ref["tr_choice"][t]), f"choices at t={t + 1}"
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    assert np.array_equal(g["U"].cpu().numpy(), ref["U"])
    assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
    assert (g["iters_done"].cpu().numpy() == T).all()
    s.close()


def test_auto_takes_the_resident_driver_for_small_tables():
    for name in ("tiny", "small"):
        inst = workloads.make(name)
        s = esp.Solver(inst)
        assert s.loop_driver() == esp.ESP_MODE_RESIDENT, name
        s.close()
    # 256 workgroups of 32 tiles at R = 8: 8,192 tiles of 4 jobs
    for n_jobs, want in ((20000, esp.ESP_MODE_RESIDENT), (32768, esp.ESP_MODE_RESIDENT),
                         (32769, esp.ESP_MODE_PERSISTENT)):
        s = esp.Solver(workloads.make("large", n_jobs=n_jobs))
        assert s.loop_driver() == want, n_jobs
        s.close()


def _staggered():
    """Four clusters (94 tiles each) stopping after 1, 3, 108 and all 120
    updates under tol = 1e-3."""
    inst = workloads.random_small(31, 1500, 16, 3, dense=True, n_clusters=4, iters=120, eta0=0.02)
    inst.eta0 = np.array([1e-5, 4e-5, 1e-3, 0.05], dtype=np.float64)
    return inst


def _tiny_tol():
    inst = workloads.make("tiny")
    inst.eta0 = np.array([0.05])
    return inst


@pytest.mark.parametrize("case,blocks", [("staggered", 12), ("staggered", 24), ("tiny", 1)])
def test_resident_stops_under_tol(case, blocks):
    inst = _staggered() if case == "staggered" else _tiny_tol()
    ref = oracle.Oracle(inst).solve(tol=1e-3, trace=True)
    n = [int(x) for x in ref["iters_done"]]
    if case == "staggered":
        assert n == [1, 3, 108, 120]
    _say(f"resident stops under tol: {case} blocks={blocks} stops={n}")
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT, blocks_per_cluster=blocks)
    g = s.solve(s.prices(inst.lam0), inst.iters, tol=1e-3, trace=True)
    torch.cuda.synchronize()
    assert s.device_status() == 0
    tl, tu = g["tr_lam"].cpu().numpy(), g["tr_U"].cpu().numpy()
    for b, k in enumerate(n):
        assert np.array_equal(tl[:k, b], ref["tr_lam"][:k, b]), b
        assert np.array_equal(tu[:k, b], ref["tr_U"][:k, b]), b
        assert np.isnan(tl[k:, b]).all(), b
    assert np.array_equal(g["iters_done"].cpu().numpy(), ref["iters_done"])
    assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    s.close()


def test_resident_solve_longer_than_one_launch_and_warm_start():
    """1,100 iterations on Small: two resident launches (1,024 + 76), the
    second starting from the prices the first wrote; and the same solve split
    in two esp_solve calls (t_start)."""
    inst = workloads.make("small")
    T = 1100
    _say(f"resident T={T} small, and split at 600")
    ref = oracle.Oracle(inst).solve(iters=T, trace=True)
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT)
    g = s.solve(s.prices(inst.lam0), T, trace=True)
    torch.cuda.synchronize()
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    lam = s.prices(inst.lam0)
    a = s.solve(lam, 600, trace=True)
    b = s.solve(lam, 500, t_start=601, trace=True)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat([a["tr_lam"], b["tr_lam"]]), g["tr_lam"])
    assert torch.equal(b["choice"], g["choice"])
    assert s.device_status() == 0
    s.close()


def test_resident_under_capture_is_refused():
    inst = workloads.make("tiny")
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT)
    lam = s.prices(inst.lam0)
    graph = torch.cuda.CUDAGraph()
    codes = []
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        lam.mul_(1.0)
        try:
            esp.esp_solve(s.ctx, lam, 10, 1, 0.0, None, None, None, None, torch.cuda.current_stream())
        except esp.EspError as e:
            codes.append(e.code)
    assert codes == [esp.ESP_ERR_INVALID_ARG]
    s.close()


def _dense(seed, n_jobs, k, r, **kw):
    return workloads.random_small(seed, n_jobs, k, r, dense=True, **kw)


# AUTO keeps dense tables beyond two tiles per wavefront on chip (8 wavefronts
# per workgroup: 16 tiles in registers, the rest in LDS): tables around those
# sizes and around the LDS limit (at R = 8: 32 tiles per workgroup, 33 are
# streamed; with a penalty column 24 and 25), last tiles partial, one to three limbs, 1 to 17 workgroups (the
# exchange's 16 copies) and the whole device.
ON_CHIP = {
    # name: (instance, blocks_per_cluster (0 = library default), T)
    "k64_r8_15tiles": (lambda: _dense(1, 60, 64, 8), 0, 40),
    "k64_r8_16tiles": (lambda: _dense(2, 61, 64, 8), 0, 40),
    "k64_r8_17tiles_1wg": (lambda: _dense(3, 65, 64, 8), 1, 40),
    "k64_r8_32tiles_1wg": (lambda: _dense(4, 127, 64, 8), 1, 40),
    "k64_r8_33tiles_1wg": (lambda: _dense(5, 129, 64, 8), 1, 40),
    "k64_r8_2wg": (lambda: _dense(6, 230, 64, 8), 2, 40),
    "k16_r5_3wg_2limbs": (lambda: _wide(_dense(7, 1700, 16, 5), 5, 14), 3, 30),
    "k16_r7_3wg_3limbs": (lambda: _wide(_dense(8, 1300, 16, 7), 6, 36), 3, 30),
    "k8_r8_9wg_3limbs": (lambda: _wide(_dense(9, 2500, 8, 8), 7, 36), 9, 30),
    "k4_r1_2wg": (lambda: _dense(10, 3100, 4, 1), 2, 40),
    "k32_r6_17wg": (lambda: _dense(11, 2611, 32, 6), 17, 40),
    "k32_r3_3clusters": (lambda: _dense(12, 900, 32, 3, n_clusters=3), 4, 40),
    "k8_r2_penalties": (lambda: workloads.with_penalties(_dense(13, 1500, 8, 2), 9), 2, 40),
    "k64_r8_penalties_24tiles_1wg": (lambda: workloads.with_penalties(_dense(14, 95, 64, 8), 9), 1, 40),
    "k64_r8_penalties_25tiles_1wg": (lambda: workloads.with_penalties(_dense(14, 100, 64, 8), 9), 1, 40),
    "k64_r8_9000jobs": (lambda: workloads.make("large", n_jobs=9000), 0, 12),
    "300clusters": (lambda: _dense(15, 65, 64, 4, n_clusters=300), 0, 8),
}


@pytest.mark.parametrize("name", sorted(ON_CHIP))
def test_auto_keeps_tables_on_chip(name):
    make, blocks, T = ON_CHIP[name]
    inst = make()
    _say(f"on chip {name} B={inst.B} N={inst.N} R={inst.R} T={T} blocks={blocks}")
    s = esp.Solver(inst, blocks_per_cluster=blocks)
    ref = oracle.Oracle(inst).solve(iters=T, trace_choice=True)
    for _ in range(2):                               # the second solve reuses the exchange words
        g = s.solve(s.prices(inst.lam0), T, trace=True, trace_choice=True)
        torch.cuda.synchronize()
        assert s.device_status() == 0
        assert np.array_equal(g["tr_choice"].cpu().numpy(), ref["tr_choice"])
        assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
        assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
        assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
        assert np.array_equal(g["U"].cpu().numpy(), ref["U"])
        assert (g["iters_done"].cpu().numpy() == T).all()
    streamed = name in ("k64_r8_33tiles_1wg", "k64_r8_penalties_25tiles_1wg")
    assert s.loop_driver() == (esp.ESP_MODE_PERSISTENT if streamed else esp.ESP_MODE_RESIDENT)
    s.close()


def test_on_chip_long_solve_and_stops():
    """Two launches (1,024 + 76 iterations) over LDS tiles with an exchange,
    and clusters that stop at different iterations."""
    inst = _dense(20, 230, 64, 8)
    _say("on chip, T=1100 on 2 workgroups; staggered stops on 2 workgroups")
    ref = oracle.Oracle(inst).solve(iters=1100, trace=True)
    s = esp.Solver(inst, blocks_per_cluster=2)
    g = s.solve(s.prices(inst.lam0), 1100, trace=True)
    torch.cuda.synchronize()
    assert s.device_status() == 0
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    s.close()
    inst = _staggered()                              # 94 tiles per cluster
    ref = oracle.Oracle(inst).solve(tol=1e-3, trace=True)
    s = esp.Solver(inst, blocks_per_cluster=2)
    g = s.solve(s.prices(inst.lam0), inst.iters, tol=1e-3)
    torch.cuda.synchronize()
    assert s.device_status() == 0
    assert np.array_equal(g["iters_done"].cpu().numpy(), ref["iters_done"])
    assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    s.close()


@pytest.mark.parametrize("mode", ["resident", "persistent"])
def test_limbs_of_512_workgroups(mode):
    """128-bit sums of 512 workgroups: the low limbs are arbitrary, so their
    total nears 512 times the largest limb and must not reach the count."""
    inst = workloads.random_small(12, 80000, 7, 1, dense=True, iters=6)
    rng = np.random.default_rng(3)
    inst.demand = (inst.demand.astype(np.float64) *
                   np.exp2(rng.integers(-36, 37, inst.demand.shape))).astype(np.float32)
    inst.eta0 = np.full(inst.B, 1e-14)
    print(f"[gpu-case] 512 workgroups {mode}", flush=True)
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT if mode == "resident" else esp.ESP_MODE_PERSISTENT)
    g = s.solve(s.prices(inst.lam0), 6, trace=True)
    torch.cuda.synchronize()
    ref = oracle.Oracle(inst).solve(iters=6, trace=True)
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert s.device_status() == 0
    s.close()


# The whole sum's bits (span + 9 for 500 jobs, + 13 for 5,000) on both sides of the
# 53 that binary64 holds and of the 56 that one exchanged word holds.
@pytest.mark.parametrize("n_jobs,log_jobs", [(500, 9), (5000, 13)])
@pytest.mark.parametrize("need", [52, 53, 54, 56, 57, 63])
def test_sums_at_the_accumulators_edges(n_jobs, log_jobs, need):
    inst = workloads.random_small(n_jobs + need, n_jobs, 16, 5, dense=True, iters=15)
    low = 2.0 ** (2 - (need - log_jobs))                   # values below 4: `need - log_jobs` bits
    d = np.floor(inst.demand.astype(np.float64) * 2.0 ** 20) / 2.0 ** 20
    small = np.random.default_rng(need).random(d.shape) < 0.5
    d = np.where(small, np.floor(d * 2.0 ** 20) * low, d)
    d[:, 0, :] = 3.75
    d[:, 1, :] = low
    inst.demand = d.astype(np.float32)
    print(f"[gpu-case] need {need} bits, {n_jobs} jobs", flush=True)
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT)
    g = s.solve(s.prices(inst.lam0), 15, trace=True)
    torch.cuda.synchronize()
    ref = oracle.Oracle(inst).solve(iters=15, trace=True)
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert s.device_status() == 0
    s.close()


# Ragged tables around one workgroup's 16 tiles (36 families of 7 in a tile),
# the most that 85 workgroups hold for each of 3 clusters (1,360 tiles; above,
# the table is streamed), and more clusters than compute units.
@pytest.mark.parametrize("clusters,n_jobs", [(1, 576), (1, 577), (3, 48960), (3, 48961), (3, 49000), (300, 40)])
def test_ragged_resident_shapes(clusters, n_jobs):
    inst = workloads.random_small(5, n_jobs, 7, 2, dense=True, n_clusters=clusters, iters=4)
    print(f"[gpu-case] ragged resident B={clusters} N={n_jobs}", flush=True)
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT)
    streamed = clusters == 3 and n_jobs > 48960
    assert s.loop_driver() == (esp.ESP_MODE_PERSISTENT if streamed else esp.ESP_MODE_RESIDENT)
    g = s.solve(s.prices(inst.lam0), 4, trace=True, trace_choice=True)
    torch.cuda.synchronize()
    ref = oracle.Oracle(inst).solve(iters=4, trace=True, trace_choice=True)
    assert np.array_equal(g["tr_choice"].cpu().numpy(), ref["tr_choice"])
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert s.device_status() == 0
    s.close()


# Clusters whose planned workgroups (192 over the clusters, rounded up) are more
# than one for each of 256 compute units: 86..95 x 3 and 129..191 x 2.  Tables of 20
# tiles per cluster, of 33 and 60 (LDS tiles, or more than fit), and a tolerance.
@pytest.mark.parametrize("clusters", [86, 90, 95, 129, 150, 191])
@pytest.mark.parametrize("tiles,r", [(20, 4), (33, 6), (60, 2), (60, 6)])
def test_dense_batches_keep_their_driver(clusters, tiles, r):
    inst = _dense(clusters + tiles, tiles * 8 - 3, 32, r, n_clusters=clusters)
    _say(f"dense batch B={clusters} tiles={tiles} R={r}")
    for tol in (0.0, 1e-3):
        s = esp.Solver(inst)
        g = s.solve(s.prices(inst.lam0), 5, tol=tol, trace=True)
        torch.cuda.synchronize()
        assert s.device_status() == 0
        # no grid was refused: 256 / clusters workgroups of 8 wavefronts hold the table (two tiles of a
        # wavefront in registers, and in LDS 160 KB / 8 / (R + 1) KB = 6, 3 or 2), or it is streamed
        fits = -(-tiles // (8 * (256 // clusters))) - 2 <= {2: 6, 4: 3, 6: 2}[r]
        assert s.loop_driver() == (esp.ESP_MODE_RESIDENT if fits else esp.ESP_MODE_PERSISTENT)
        ref = oracle.Oracle(inst).solve(iters=5, tol=tol)
        assert np.array_equal(g["iters_done"].cpu().numpy(), ref["iters_done"])
        assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
        assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
        s.close()


# Grids of more than one workgroup per compute unit that ESP_MODE_RESIDENT
# accepts: the plan's own (90 x 3) and a caller's (one cluster on 400 workgroups,
# 40 on 8, 3 on 170 with tables that fewer workgroups hold, 130 on 3 with one that they do not).
@pytest.mark.parametrize("clusters,tiles,r,blocks", [
    (90, 20, 4, 0), (95, 24, 2, 0), (1, 2001, 2, 400), (40, 50, 3, 8), (3, 1350, 2, 170), (130, 24, 4, 3)])
def test_explicit_resident_grids_beyond_the_device(clusters, tiles, r, blocks):
    inst = _dense(tiles, tiles * 8 - 5, 32, r, n_clusters=clusters)
    _say(f"explicit resident B={clusters} tiles={tiles} R={r} blocks={blocks}")
    s = esp.Solver(inst, mode=esp.ESP_MODE_RESIDENT, blocks_per_cluster=blocks)
    g = s.solve(s.prices(inst.lam0), 4, trace=True)
    torch.cuda.synchronize()
    assert s.device_status() == 0
    assert s.loop_driver() == (esp.ESP_MODE_PERSISTENT if clusters == 130 else esp.ESP_MODE_RESIDENT)
    ref = oracle.Oracle(inst).solve(iters=4, trace=True)
    assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    s.close()


def _one_packing_per_unit():
    """A solver of 250 equal clusters and a model whose packing takes a compute
    unit each for some hundred microseconds."""
    one = workloads.make("small", n_jobs=1000)
    rep = {k: np.repeat(getattr(one, k), 250, axis=0) for k in ("utility", "demand", "capacity", "eta0", "lam0")}
    many = workloads.with_penalties(dataclasses.replace(one, **rep), 3)
    model = workloads.iac_model(many, gpus=[2048] * 250)
    for k in ("sensitivity", "pressure", "tau_base"):
        setattr(model, k, torch.as_tensor(getattr(model, k), device="cuda"))
    return esp.Solver(many), model


@pytest.mark.parametrize("case", ["resident", "on_chip", "csr", "persistent", "persistent_csr"])
@pytest.mark.parametrize("error", ["bad_price", "earlier_call"])
def test_waits_outlast_errors_of_others(case, error):
    """A bad price in another cluster, or an error of an earlier call that nobody
    has read, does not end the solve of a healthy cluster, however long its
    workgroups wait for each other: here for the last of them to get a compute
    unit, which first-fit packings on another stream hold."""
    if case.endswith("csr"):
        inst = workloads.random_small(50, 3000, 40, 4, n_clusters=3, iters=30)
    else:
        inst = _dense(51, 2500 if case == "on_chip" else 600, 32, 4, n_clusters=3)
    T = 30
    mode = esp.ESP_MODE_AUTO if case == "on_chip" else esp.ESP_MODE_PERSISTENT if case.startswith("p") else esp.ESP_MODE_RESIDENT
    _say(f"waits outlast errors: {case} {error}")
    s = esp.Solver(inst, mode=mode)
    lam0 = np.array(inst.lam0, dtype=np.float64).reshape(3, 4).copy()
    if error == "bad_price":
        lam0[1, 2] = np.nan
    else:
        s.reduce_demand(torch.full((3, inst.N), 1000, dtype=torch.int32, device="cuda"))
    healthy = [0, 2] if error == "bad_price" else [0, 1, 2]
    ref = oracle.Oracle(inst).solve(iters=T)
    busy, model = _one_packing_per_unit()
    side = torch.cuda.Stream()
    lam = s.prices(lam0)
    blam = busy.prices(np.zeros((busy.B, busy.R)))
    torch.cuda.synchronize()
    got = []
    for _ in range(4):
        # (one round without iterations: returns while the packing runs, whose outputs
        # must then not be freed for this stream's tensors)
        packed = busy.schedule(model, blam, 1, 0, stream=side)
        lam.copy_(torch.as_tensor(lam0))
        got.append({k: v.clone() for k, v in s.solve(lam, T).items()})
        torch.cuda.synchronize()
        del packed
    busy.close()
    assert s.device_status() == (esp.ESP_ERR_NONFINITE if error == "bad_price" else esp.ESP_ERR_INVALID_ARG)
    for g in got:
        for b in healthy:
            assert g["iters_done"].cpu().numpy()[b] == T, b
            assert np.array_equal(g["lam"].cpu().numpy()[b], ref["lam"][b]), b
            assert np.array_equal(g["choice"].cpu().numpy()[b], ref["choice"][b]), b
    s.close()


@pytest.mark.parametrize("n_jobs,k,r,shortest", [(40000, 64, 8, 16), (30000, 64, 8, 5), (220000, 12, 8, 9)])
def test_short_solves_of_large_tables_take_no_cooperative_launch(n_jobs, k, r, shortest):
    """Above 64 MiB a one-iteration solve of AUTO takes about as long as with one
    launch per iteration (a cooperative launch makes it 1.3 to 1.6 times as
    long), and both sides of the shortest cooperative solve match it bit for bit."""
    inst = _dense(n_jobs, n_jobs, k, r)
    assert 4 * inst.utility.size * (r + 1) > 64 << 20
    auto, stream = esp.Solver(inst), esp.Solver(inst, mode=esp.ESP_MODE_STREAM)
    for T in (1, shortest - 1, shortest):
        _say(f"short solves N={n_jobs} K={k} R={r} T={T}")
        a = auto.solve(auto.prices(inst.lam0), T, trace=True)
        b = stream.solve(stream.prices(inst.lam0), T, trace=True)
        torch.cuda.synchronize()
        for key in ("choice", "U", "lam", "tr_lam", "tr_U", "iters_done"):
            assert torch.equal(a[key], b[key]), (T, key)
    lam = auto.prices(inst.lam0)
    us = {id(auto): [], id(stream): []}
    for i in range(31):
        for s in (auto, stream):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                s.solve(lam, 1)
            e1.record()
            torch.cuda.synchronize()
            us[id(s)].append(e0.elapsed_time(e1) * 100.0)
    a, b = (sorted(us[id(s)])[15] for s in (auto, stream))
    print(f"[gpu-case] us a solve of one iteration: AUTO {a:.1f}, one launch each {b:.1f}", flush=True)
    assert a < 1.2 * b
    auto.close()
    stream.close()


def test_contexts_of_one_kernel_in_two_threads():
    """Two threads solve on contexts of the same kernel instance with 1 and 2 LDS
    tiles a wavefront: neither changes what the other's launches may use."""
    _say("two threads, 17 and 32 tiles on one workgroup")
    insts = [_dense(3, 65, 64, 8), _dense(4, 127, 64, 8)]
    refs = [oracle.Oracle(i).solve(iters=3) for i in insts]
    solvers = [esp.Solver(i, blocks_per_cluster=1) for i in insts]
    start, errors = threading.Barrier(2), []

    def work(i):
        try:
            s, stream = solvers[i], torch.cuda.Stream()
            with torch.cuda.stream(stream):
                lam0 = s.prices(insts[i].lam0)
                start.wait()
                for _ in range(400):
                    lam = lam0.clone()
                    g = s.solve(lam, 3)
            stream.synchronize()
            assert s.device_status() == 0 and s.loop_driver() == esp.ESP_MODE_RESIDENT
            assert np.array_equal(g["lam"].cpu().numpy(), refs[i]["lam"])
            assert np.array_equal(g["choice"].cpu().numpy(), refs[i]["choice"])
        except BaseException as e:                   # noqa: BLE001 (reported below)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
    for s in solvers:
        s.close()


# More clusters than compute units, one workgroup each: of four wavefronts with up
# to 8 tiles (two per wavefront), of eight above; both sides of 256 clusters and of 8
# tiles; binary64, 64- and 128-bit sums; ragged tiles; penalties; a tolerance.
@pytest.mark.parametrize("clusters,tiles,r,k,span", [
    (256, 8, 4, 32, 0), (257, 8, 4, 32, 0), (257, 9, 4, 32, 0), (600, 1, 8, 64, 0), (300, 5, 1, 4, 0), (300, 7, 6, 16, 12),
    (300, 3, 5, 8, 36), (260, 8, 8, 12, 0), (260, 9, 3, 12, 0), (520, 2, 7, 40, 0), (300, 6, 8, 12, 12), (300, 4, 4, 7, 36)])
def test_more_clusters_than_compute_units(clusters, tiles, r, k, span):
    inst = _dense(clusters + tiles, max(1, tiles * (256 // k) - 1), k, r, n_clusters=clusters)
    if span:
        inst = _wide(inst, 3, span)
    if tiles == 7:
        inst = workloads.with_penalties(inst, 5)
    _say(f"many clusters B={clusters} tiles={tiles} R={r} K={k} span={span}")
    s = esp.Solver(inst)
    assert s.loop_driver() == esp.ESP_MODE_RESIDENT
    o = oracle.Oracle(inst)
    for tol in (0.0, 1e-3):
        ref = o.solve(iters=12, tol=tol, trace=True)
        g = s.solve(s.prices(inst.lam0), 12, tol=tol, trace=True)
        torch.cuda.synchronize()
        assert s.device_status() == 0
        assert np.array_equal(g["iters_done"].cpu().numpy(), ref["iters_done"])
        assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
        assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
        if tol == 0.0:
            assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
    s.close()


def test_small_clusters_share_a_compute_unit():
    """512 clusters of 4 tiles take hardly longer than 256 (in workgroups that fill
    a compute unit 1.8 times as long)."""
    us = []
    for clusters in (512, 256):
        inst = _dense(1, 32, 32, 4, n_clusters=clusters)
        s = esp.Solver(inst)
        lam = s.prices(inst.lam0)
        t = []
        for _ in range(21):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                s.solve(lam, 200)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1) * 200.0)
        us.append(sorted(t)[10])
        s.close()
    _say(f"200 iterations: {us[0]:.0f} us of 512 clusters, {us[1]:.0f} of 256")
    assert us[0] < 1.4 * us[1]
