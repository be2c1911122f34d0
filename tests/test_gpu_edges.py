"""GPU parity on the edges of the input space: every resource count, a
single job, zero iterations, and demand columns whose bit span needs the
128-bit accumulators.  All results bitwise equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_07971_amd as esp
import workloads

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-case] {msg}", flush=True)


def _parity(inst, T, mode=esp.ESP_MODE_AUTO):
    s = esp.Solver(inst, mode=mode)
    g = s.solve(s.prices(inst.lam0), T, trace=T > 0, trace_choice=T > 0)
    torch.cuda.synchronize()
    ref = oracle.Oracle(inst).solve(iters=T, trace_choice=T > 0, trace=T > 0)
    if T > 0:
        assert np.array_equal(g["tr_choice"].cpu().numpy(), ref["tr_choice"])
        assert np.array_equal(g["tr_U"].cpu().numpy(), ref["tr_U"])
        assert np.array_equal(g["tr_lam"].cpu().numpy(), ref["tr_lam"])
    assert np.array_equal(g["choice"].cpu().numpy(), ref["choice"])
    assert np.array_equal(g["U"].cpu().numpy(), ref["U"])
    assert np.array_equal(g["lam"].cpu().numpy(), ref["lam"])
    assert s.device_status() == 0
    s.close()


@pytest.mark.parametrize("R", list(range(1, 9)))
@pytest.mark.parametrize("layout", ["dense_k8", "csr"])
def test_every_resource_count(R, layout):
    inst = (workloads.random_small(60 + R, 900, 8, R, dense=True, iters=40) if layout == "dense_k8"
            else workloads.random_small(70 + R, 700, 23, R, iters=40))
    _say(f"R={R} {layout}")
    # both drivers explicitly: the persistent one is a cooperative launch of
    # the whole grid, which the kernel's registers must let the device hold
    for mode in (esp.ESP_MODE_STREAM, esp.ESP_MODE_PERSISTENT):
        _parity(inst, 40, mode)


@pytest.mark.parametrize("layout", ["dense", "csr"])
def test_single_job(layout):
    # K = 16 takes the dense kernel; K = 7 (no dense variant) the CSR kernel
    inst = workloads.random_small(80 if layout == "dense" else 81, 1, 16 if layout == "dense" else 7, 3,
                                  dense=True, iters=30)
    _say(f"single job {layout}")
    for mode in (esp.ESP_MODE_STREAM, esp.ESP_MODE_PERSISTENT):
        _parity(inst, 30, mode)


def test_zero_iterations_reselects_at_the_given_prices():
    inst = workloads.make("small", n_jobs=1000)
    inst.lam0 = np.full((1, inst.R), 0.01)
    _say("T = 0")
    _parity(inst, 0)


def _wide(inst, seed, span=36):
    """Demands multiplied by 2^U{-span..span} per entry: a column spans more
    than 63 bits with log2(N + 1), so the packer picks 128-bit sums."""
    rng = np.random.default_rng(seed)
    inst.demand = (inst.demand.astype(np.float64) *
                   np.exp2(rng.integers(-span, span + 1, inst.demand.shape))).astype(np.float32)
    return inst


@pytest.mark.parametrize("layout", ["dense_k16", "dense_k64_r8", "csr", "csr_batched", "csr_r8"])
def test_wide_spans_use_128_bit_sums(layout):
    inst = {
        "dense_k16": lambda: workloads.random_small(90, 3000, 16, 5, dense=True, iters=60),
        "dense_k64_r8": lambda: workloads.random_small(91, 700, 64, 8, dense=True, iters=60),
        "csr": lambda: workloads.random_small(92, 2500, 30, 6, iters=60),
        "csr_batched": lambda: workloads.random_small(93, 800, 30, 4, n_clusters=3, iters=60),
        "csr_r8": lambda: workloads.random_small(94, 1200, 40, 8, iters=60),
    }[layout]()
    _wide(inst, 5)
    inst.eta0 = np.full(inst.B, 1e-12)                   # prices stay in a useful range for 2^36 demands
    _say(f"128-bit sums {layout}")
    for mode in (esp.ESP_MODE_STREAM, esp.ESP_MODE_PERSISTENT):
        _parity(inst, 60, mode)


# CSR scans: one-entry families (256 winners in a tile), families that end with
# a tile, families over many lanes, equal scores (dyadic), and demands whose
# lanes' sums fit 53 bits (22 bits + the 3 of 8 additions) or need the 64-bit
# fixed point (52 + 3 bits; 52 + 11 bits for the whole sum of up to 2,047 jobs).
@pytest.mark.parametrize("sizes", ["ones", "k2", "k3", "k5", "k128", "k255", "k256", "mixed", "mixed_dyadic"])
@pytest.mark.parametrize("bits", [22, 52])
def test_csr_scan_edges(sizes, bits):
    if sizes.startswith("mixed"):
        inst = workloads.random_small(21, 900, 256, 6, iters=25, dyadic=sizes == "mixed_dyadic")
    else:
        k = 1 if sizes == "ones" else int(sizes[1:])
        inst = workloads.random_small(k, 40 if k > 100 else 1500, k, 1 + k % 8, dense=True, iters=25, dyadic=k == 5)
    d = np.floor(inst.demand.astype(np.float64) * 2.0 ** 20) / 2.0 ** 20
    small = np.random.default_rng(9).random(d.shape) < 0.5
    inst.demand = np.where(small, d * 2.0 ** (22 - bits), d).astype(np.float32)
    for mode in (esp.ESP_MODE_STREAM, esp.ESP_MODE_PERSISTENT, esp.ESP_MODE_RESIDENT):
        _say(f"csr {sizes} bits={bits} mode={mode}")
        _parity(inst, 25, mode)


# Around the gather kernel's 256 threads (1,024 from 2,500 jobs per workgroup at up
# to 4 resources), 4 jobs per thread and the plan's workgroups, dense and CSR, 64- and
# 128-bit sums, several clusters.
@pytest.mark.parametrize("n_jobs,k,r,clusters,blocks", [
    (1, 4, 1, 1, 0), (63, 8, 3, 1, 1), (1023, 16, 8, 1, 1), (1024, 16, 5, 1, 1), (1025, 5, 7, 1, 1),
    (4095, 4, 2, 1, 1), (4097, 12, 6, 1, 1), (5000, 32, 4, 3, 2), (9001, 7, 8, 2, 3), (3000, 64, 8, 1, 0),
    (255, 4, 2, 1, 1), (257, 12, 6, 1, 1), (2499, 4, 4, 1, 1), (2500, 12, 3, 1, 1), (4999, 8, 1, 2, 2),
    (5000, 4, 4, 2, 2), (8193, 16, 3, 1, 2), (40, 8, 6, 300, 0), (56, 16, 5, 300, 0),
    (100, 12, 8, 600, 0), (33, 5, 7, 600, 0), (70, 8, 4, 520, 0), (64, 4, 3, 520, 0), (90, 16, 2, 520, 0)])
@pytest.mark.parametrize("wide", [False, True])
def test_reduce_demand_edges(n_jobs, k, r, clusters, blocks, wide):
    inst = workloads.random_small(n_jobs + k, n_jobs, k, r, dense=k != 12, n_clusters=clusters)
    rng = np.random.default_rng(n_jobs)
    if wide:
        inst.demand = (inst.demand.astype(np.float64) *
                       np.exp2(rng.integers(-30, 31, inst.demand.shape))).astype(np.float32)
    _say(f"reduce_demand N={n_jobs} K={k} R={r} B={clusters} blocks={blocks} wide={wide}")
    s = esp.Solver(inst, blocks_per_cluster=blocks)
    sizes = np.diff(inst.offsets)
    choice = (rng.random((clusters, n_jobs)) * sizes).astype(np.int32)
    o = oracle.Oracle(inst)
    for _ in range(2):
        U = s.reduce_demand(torch.as_tensor(choice, device="cuda"))
        torch.cuda.synchronize()
        for b in range(clusters):
            assert np.array_equal(U.cpu().numpy()[b], o.demand_sum(b, choice[b])), b
    choice[-1, -1] = sizes[-1]                         # outside the last job's family
    U = s.reduce_demand(torch.as_tensor(choice, device="cuda"))
    torch.cuda.synchronize()
    assert np.isnan(U.cpu().numpy()[-1]).all() and not np.isnan(U.cpu().numpy()[:-1]).any()
    assert s.device_status() == esp.ESP_ERR_INVALID_ARG
    s.close()


def test_score_select_checks_prices_per_cluster():
    """A selection validates its own prices: clusters with a bad price keep
    their choices untouched and are reported; the others are selected."""
    inst = workloads.random_small(3, 700, 16, 3, dense=True, n_clusters=5)
    csr = workloads.random_small(4, 700, 40, 3, n_clusters=5)
    for prob in (inst, csr):
        s = esp.Solver(prob)
        o = oracle.Oracle(prob)
        lam = np.full((5, 3), 0.25)
        for bad in (np.nan, np.inf, -1.0, 2.0 ** 401):
            _say(f"select with a bad price {bad}")
            lam[1, 2] = lam[4, 0] = bad
            ch = torch.full((5, 700), -7, dtype=torch.int32, device="cuda")
            esp.esp_score_select(s.ctx, s.prices(lam), ch)
            assert s.device_status() == esp.ESP_ERR_NONFINITE
            for b in range(5):
                got = ch[b].cpu().numpy()
                assert (got == -7).all() if b in (1, 4) else np.array_equal(got, o.select(b, lam[b])), b
        lam[1, 2] = lam[4, 0] = -0.0
        ch = s.score_select(s.prices(lam))
        assert s.device_status() == 0
        for b in range(5):
            assert np.array_equal(ch[b].cpu().numpy(), o.select(b, lam[b]))
        s.close()


def test_default_stream_is_the_callers():
    side = torch.cuda.Stream()
    assert esp._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert esp._stream(None) == side.cuda_stream != torch.cuda.default_stream().cuda_stream
    assert esp._stream(side) == side.cuda_stream


def test_demand_of_many_clusters_takes_no_longer_than_of_one():
    """128,000 ragged jobs as 64 clusters or as one: the same loads.  512 workgroups
    are on the device at once when they have 4 wavefronts (0.8 times as long);
    with 16 they took 1.6 times as long."""
    us = []
    for clusters in (64, 1):
        inst = workloads.random_small(3, 128000 // clusters, 12, 6, dense=True, n_clusters=clusters)
        s = esp.Solver(inst)
        choice = torch.randint(0, 12, (clusters, inst.N), dtype=torch.int32, device="cuda")
        U = s.reduce_demand(choice)
        t = []
        for _ in range(31):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(50):
                esp.esp_reduce_demand(s.ctx, choice, U)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1) * 20.0)
        us.append(sorted(t)[15])
        s.close()
    _say(f"demand of 128,000 jobs: {us[0]:.1f} us as 64 clusters, {us[1]:.1f} as one")
    assert us[0] < 1.2 * us[1]
