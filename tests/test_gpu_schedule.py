"""GPU parity of the outer ESP-IAC rounds (Sec. 3.4, Alg. 1) through the
C-ABI against the oracle: rounds run, violating pairs, prices, choices,
the GPU occupancy lists and the final penalties, all bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_07971_amd as esp
import workloads
from tests._helpers import schedule_fixture

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-case] {msg}", flush=True)


def _with_penalty_inputs(inst):
    """A context needs the penalty column for Alg. 1: zero interference
    penalties (Alg. 1 resets them anyway), no switching cost."""
    if inst.penalty is None:
        inst.penalty = np.zeros((inst.B, inst.nnz), np.float32)
    return inst


def _compare(inst, model, M, T, tol=0.0, clusters=None):
    s = esp.Solver(_with_penalty_inputs(inst))
    lam = s.prices(inst.lam0)
    g = s.schedule(model, lam, M, T, tol)
    torch.cuda.synchronize()
    pen = s.read_penalties()
    assert s.device_status() == 0
    o = oracle.Oracle(inst)
    gj = g["gpu_jobs"].cpu().numpy()
    for b in (range(inst.B) if clusters is None else clusters):
        r = o.schedule(b, model, M, T, tol)
        G = int(model.gpus[b])
        assert int(g["rounds"][b]) == r["rounds"], b
        assert int(g["violations"][b]) == r["violations"], b
        assert np.array_equal(g["choice"][b].cpu().numpy(), r["choice"]), b
        assert np.array_equal(g["lam"][b].cpu().numpy(), r["lam"]), b
        assert np.array_equal(gj[b, :G], r["occ"]), b
        assert (gj[b, G:] == -1).all()
        assert np.array_equal(pen[b], r["penalty"]), b
    s.close()
    return g


def test_hand_example_on_gpu():
    inst, m, results = schedule_fixture()
    _say("schedule hand example")
    for M, nr, V, ch, g0, g1, pen in results:
        g = _compare(inst, m, int(M[0]), inst.iters)
        assert int(g["rounds"][0]) == int(nr[0]) and int(g["violations"][0]) == int(V[0])


CASES = {
    "tiny": lambda: workloads.make("tiny"),
    "small_600": lambda: workloads.make("small", n_jobs=600),
    "small_2000": lambda: workloads.make("small", n_jobs=2000),
    "batched_3x700": lambda: workloads.make("batched", n_jobs=700, n_clusters=3),
    "ragged_shape_r6": lambda: workloads.make("ragged", n_jobs=1500),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_schedule_matches_oracle(name):
    inst = CASES[name]()
    model = workloads.iac_model(inst, gpus=None if name != "ragged_shape_r6" else [600])
    _say(f"schedule {name}: B={inst.B} N={inst.N} R={inst.R} G={list(model.gpus)}")
    for M, T in ((1, 40), (3, 60)):
        _compare(inst, model, M, T)


# GPUs around the 4 slots of a lane and the 256-GPU groups of the packing
# kernel (one group in registers, up to 8 in all); jobs around its batches of
# 64 and chunks of 14 batches; T = 0 takes every job's favourite configuration
# (8 whole GPUs, shares split over groups, many failures), T = 3 small shares.
@pytest.mark.parametrize("gpus,n_jobs", [(1, 1), (3, 63), (64, 65), (65, 128), (255, 300), (256, 895), (257, 896),
                                         (300, 897), (512, 1793), (513, 700), (1024, 1500), (1025, 2700),
                                         (2047, 3000), (2048, 2048)])
def test_packing_edges(gpus, n_jobs):
    _say(f"packing edges: {gpus} GPUs, {n_jobs} jobs")
    dense = workloads.make("small", n_jobs=n_jobs)
    ragged = workloads.make("ragged", n_jobs=n_jobs)
    for inst, mem, T in ((dense, 80.0, 0), (dense, 80.0, 3), (dense, 40.0, 3), (ragged, 60.0, 1)):
        model = workloads.iac_model(inst, gpus=[gpus], gpu_memory=mem, gpu_compute=2.0 if mem == 40.0 else 1.0)
        _compare(inst, model, 2, T)


def test_packing_mixed_cluster_sizes():
    """One launch over clusters of one to all eight groups."""
    inst = workloads.make("batched", n_jobs=500, n_clusters=4)
    _say("packing of clusters with 1, 64, 700 and 2048 GPUs")
    _compare(inst, workloads.iac_model(inst, gpus=[1, 64, 700, 2048]), 2, 2)


def test_schedule_with_switching_cost_and_tolerance():
    """Switching costs stay through Gamma's reset; rounds use a stop
    tolerance (the persistent driver)."""
    inst = workloads.with_penalties(workloads.make("small", n_jobs=800), 3)
    model = workloads.iac_model(inst)
    _say("schedule small_800 with switching cost, tol")
    _compare(inst, model, 3, 200, tol=1e-3)


def test_schedule_errors():
    inst = workloads.make("tiny")
    _say("schedule errors")
    s = esp.Solver(inst)                             # no penalty column
    model = workloads.iac_model(inst)
    with pytest.raises(esp.EspError) as e:
        s.schedule(model, s.prices(inst.lam0), 2, 10)
    assert e.value.code == esp.ESP_ERR_STATE
    s2 = esp.Solver(_with_penalty_inputs(workloads.make("tiny")))
    for field, value in (("gpus", np.array([0])), ("gpus", np.array([5000])), ("r_sm", 7), ("kappa", -1.0),
                         ("u_target", 0.0)):
        bad = workloads.iac_model(inst)
        setattr(bad, field, value)
        with pytest.raises(esp.EspError) as e:
            s2.schedule(bad, s2.prices(inst.lam0), 2, 10)
        assert e.value.code == esp.ESP_ERR_INVALID_ARG, field
    bad = workloads.iac_model(inst)
    bad.beta = float("nan")
    with pytest.raises(esp.EspError) as e:
        s2.schedule(bad, s2.prices(inst.lam0), 2, 10)
    assert e.value.code == esp.ESP_ERR_NONFINITE
    torch.cuda.synchronize()
    assert s2.device_status() == 0


def test_fullsize_batched_rounds():
    """The Batched workload (256 clusters x 16,384 jobs x 64 configurations,
    256..1024 GPUs each) with 3 rounds of 20 iterations, in the launch
    configuration bench.py uses; four clusters checked against the oracle."""
    inst = workloads.make("batched")
    model = workloads.iac_model(inst)
    _say("schedule full-size batched, M=3, T=20")
    _compare(inst, model, 3, 20, clusters=(0, 1, 131, inst.B - 1))


def _jobs_of_several_gpus(n_jobs, lo, hi, seed=1):
    """Every job's favourite configuration takes lo..hi GPUs, 15 to 45% of the
    compute and 5 to 30 GB of each."""
    inst = workloads.make("small", n_jobs=n_jobs)
    rng = np.random.default_rng(seed)
    d = inst.demand.copy().reshape(1, n_jobs, -1, inst.R)
    shape = d.shape[:2] + (1,)
    g = rng.integers(lo, hi + 1, shape)
    d[..., 0] = g
    d[..., 1] = g * rng.uniform(5.0, 30.0, shape)
    d[..., 2] = g * rng.uniform(0.15, 0.45, shape)
    inst.demand = d.reshape(inst.demand.shape).astype(np.float32)
    return inst


# Jobs that take several GPUs of a group at once: all and parts of a lane's four
# GPUs, the last of a group and the first of the next, GPUs that become full.
@pytest.mark.parametrize("gpus,n_jobs,lo,hi", [(5, 30, 2, 5), (9, 60, 8, 8), (63, 100, 1, 8), (255, 300, 2, 3),
                                               (259, 400, 7, 8), (600, 900, 1, 8), (2048, 1500, 3, 8)])
def test_packing_jobs_of_several_gpus(gpus, n_jobs, lo, hi):
    _say(f"packing jobs of {lo}..{hi} GPUs: {gpus} GPUs, {n_jobs} jobs")
    inst = _jobs_of_several_gpus(n_jobs, lo, hi, gpus)
    _compare(inst, workloads.iac_model(inst, gpus=[gpus]), 2, 0)


def test_jobs_of_several_gpus_are_placed_at_once():
    """Placing a job's 8 shares one after another made a round of 300 such jobs
    4.6 times as long as one of 300 single-share jobs (all at once: 2.8)."""
    us = []
    for k in (1, 8):
        inst = _with_penalty_inputs(_jobs_of_several_gpus(300, k, k))
        model = workloads.iac_model(inst, gpus=[2048])
        for f in ("sensitivity", "pressure", "tau_base"):
            setattr(model, f, torch.as_tensor(getattr(model, f), device="cuda"))
        s = esp.Solver(inst)
        lam = s.prices(inst.lam0)
        t = []
        for _ in range(21):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            s.schedule(model, lam, 1, 0)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1) * 1e3)
        us.append(sorted(t)[10])
        s.close()
    _say(f"a round of 300 jobs of 1 and 8 shares: {us[0]:.0f} and {us[1]:.0f} us")
    assert us[1] < 3.6 * us[0]


# More clusters than compute units, two workgroups of the packing on one: clusters of
# one and several groups of GPUs, next to each other in LDS.
@pytest.mark.parametrize("clusters,n_jobs,gpus", [(300, 40, 700), (300, 90, 256), (300, 25, 1100)])
def test_packing_more_clusters_than_compute_units(clusters, n_jobs, gpus):
    _say(f"packing {clusters} clusters of {n_jobs} jobs on up to {gpus} GPUs")
    inst = workloads.make("batched", n_jobs=n_jobs, n_clusters=clusters)
    sizes = [gpus - (7 * b) % gpus for b in range(clusters)]
    _compare(inst, workloads.iac_model(inst, gpus=sizes), 2, 1, clusters=[0, 1, 37, 255, 256, 257, 298, 299])


def test_packing_of_clusters_sharing_a_compute_unit():
    """A round of 300 clusters on 512 GPUs each takes hardly longer than one of 256
    (with one workgroup on a compute unit 1.6 times as long)."""
    us = []
    for clusters in (300, 256):
        inst = _with_penalty_inputs(workloads.make("batched", n_jobs=400, n_clusters=clusters))
        model = workloads.iac_model(inst, gpus=[512] * clusters)
        for f in ("sensitivity", "pressure", "tau_base"):
            setattr(model, f, torch.as_tensor(getattr(model, f), device="cuda"))
        s = esp.Solver(inst)
        lam = s.prices(inst.lam0)
        t = []
        for _ in range(15):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            s.schedule(model, lam, 1, 0)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1) * 1e3)
        us.append(sorted(t)[7])
        s.close()
    _say(f"a round of 300 and of 256 clusters: {us[0]:.0f} and {us[1]:.0f} us")
    assert us[0] < 1.4 * us[1]
