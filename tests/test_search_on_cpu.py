"""The split search, run on the CPU from its own source (cpu_lanes): against the
oracle, and what it does where the GPU could not be asked without a fault."""
import ctypes as C
from concurrent.futures import ProcessPoolExecutor
from multiprocessing import get_context

import numpy as np
import pytest

import cpu_lanes as CL
from gpu_common import creeping_instance, large_profile, slow_outside_lds
from oracle import oracle as O
from workloads.gen import Workload, make_workload, random_instance

CO, F32 = O.F_COMPUTE_ONLY, O.F_FP32


def guarded(*args, **kw):
    """cpu_lanes.split in a process of its own: an access outside of the buffers
    ends that process and fails the test"""
    CL.lib()
    with ProcessPoolExecutor(1, mp_context=get_context("fork")) as ex:
        return ex.submit(CL.split, *args, **kw).result()


def repeated(w, n):
    """a batch of n templates in a fixed order out of a smaller one"""
    order = np.random.default_rng(5).permutation(np.arange(n) % w.n)
    return Workload(name=w.name, profile=w.profile, n_stages=np.ascontiguousarray(w.n_stages[order]),
                    stages=np.ascontiguousarray(w.stages[order]), m=w.m, s_max=w.s_max)


@pytest.fixture(scope="module")
def slow_links():
    """the 70B-like cluster with links 40 times slower: many templates are left to the split kernel"""
    w = make_workload("c3_70b_dense", 700)
    w.profile.link_bw_MBps = np.maximum(w.profile.link_bw_MBps // 40, 1)
    return w


@pytest.mark.parametrize("cus,n", [(1, 700), (20, 4300), (20, 9000)])
def test_sample_decides(cus, n):
    """the search runs from so many templates with windows in the window pass's
    sample (64 workgroups, spread over the batch), and leaves the batch alone
    below; grids of fewer workgroups, of 67 and of 70 (every tile taken once)"""
    w = repeated(make_workload("c1_tiny_dense", 500), n)
    assert CL.split(w, cus=cus)["ran"] == 1                    # need 0: not asked
    g = CL.split(w, cus=cus, need=1)
    CL.assert_split(w, g, 0)
    has = (g["status"][:, 0] == 0) | np.isin(np.arange(n), g["left"])
    V = g["counted"]
    assert g["ran"] == 1 and 0 < has.sum() < n
    assert abs(V - has.sum() * min(1, 64 * 64 / n if cus > 1 else 1)) <= (0 if cus == 1 else 0.05 * n)
    assert 2 < g["counted_stages"] / V < 4
    assert CL.split(w, cus=cus, need=V)["ran"] == 1
    idle = CL.split(w, cus=cus, need=V + 1)
    assert idle["ran"] == 0 and idle["left_count"] == 0 and ((idle["status"][:, 0] == 0xA5) == has).all()


def test_slow_links_need_more(slow_links):
    """transfers that outweigh the layers raise the need, fast ones do not"""
    fast = make_workload("c3_70b_dense", 700)
    assert CL.split(fast, need=100, need_slow=10**6)["ran"] == 1
    V = CL.split(slow_links, need=1)["counted"]
    assert CL.split(slow_links, need=100, need_slow=V - 101)["ran"] == 1
    assert CL.split(slow_links, need=100, need_slow=V - 99)["ran"] == 0


def test_left_list_holds_what_it_should(slow_links):
    g = guarded(slow_links)
    assert CL.assert_split(slow_links, g, 0) == g["left_count"] > 20
    assert len(set(g["left"].tolist())) == g["left_count"]
    assert (g["status"][g["left"]] == 8).all()                 # no split until the split kernel finds one


@pytest.mark.parametrize("flags", [0, CO, F32, F32 | CO])
@pytest.mark.parametrize("scale", [1, 10**9])
def test_templates_left(scale, flags):
    """templates are left to the split kernel where their cuts creep, and at any
    point of a search when few sweeps are allowed: in a first probe, between
    in-flight classes, in the last probe of fp32 costs. The others are whole."""
    w = creeping_instance(scale)
    assert CL.assert_split(w, CL.split(w, flags), flags, "creeping") >= 4
    few = make_workload("c2_7b_dense", 120)
    few.profile.layer_ns = np.ascontiguousarray(few.profile.layer_ns * (1 if scale == 1 else 1000))
    few.m = np.array([3, 9, 64], np.int32)
    at = [CL.assert_split(few, CL.split(few, flags, sweeps=s), flags, f"{s} sweeps") for s in (1, 3, 5, 8, 40)]
    assert at[0] > at[1] > at[2] > at[3] > at[4] == 0


def test_left_list_is_bounded(slow_links):
    """a call that overlaps on the same scratch may write any value where the
    list's length is kept (536,418,584: an iteration time of this profile, once
    found there): nothing is stored beyond the list"""
    n = slow_links.n
    for preset in (536_418_584, n - 1, n, 2**32 - 3):
        g = guarded(slow_links, preset=preset)
        assert g["rc"] == 0 and g["broken"] is None
        assert (g["left_count"] - preset) % 2**32 > 20


def test_left_list_reads_are_bounded():
    """the split kernel's side: a length or an entry beyond the batch ends the walk"""
    L = CL.lib()
    entry = lambda count, first, i, n: L.lanes_left_template(
        np.array([count] + [0] * (CL.LEFT_HEAD - 1) + [first] + [7] * 8, np.uint32).ctypes.data_as(C.c_void_p), i, n)
    assert entry(3, 5, 0, 9) == 5 and entry(3, 5, 2, 9) == 7
    assert entry(3, 5, 3, 9) == 9                              # past the length
    assert entry(536_418_584, 5, 9, 9) == 9                    # past the list
    assert entry(1, 9, 0, 9) == 9 and entry(1, 2**32 - 1, 0, 9) == 9


@pytest.mark.parametrize("flags", [0, CO, F32])
@pytest.mark.parametrize("in_lds", [True, False])
def test_windows_of_another_call(in_lds, flags):
    """a call of another batch or flags that overlaps on the same scratch leaves
    any status, in-flight class and window there, and calls templates valid that
    are not: the search ends and stays inside its tables and buffers"""
    for seed in range(1, 9):
        w = random_instance(40 + seed, L=[9, 30, 200][seed % 3], n_types=3 if in_lds else 200, s_max=[5, 12, 16][seed % 3], n=300,
                            max_cost=3000, moe=True, invalid_frac=0.6)
        if seed % 2:
            w.profile.layer_ns = np.ascontiguousarray(w.profile.layer_ns * 10**9)
        w.n_stages[::7] = 255
        g = guarded(w, flags, other=seed)
        assert g["rc"] == 0 and g["broken"] is None, (seed, g["broken"])


@pytest.mark.parametrize("flags", [0, F32])
@pytest.mark.parametrize("max_lds", [CL.LDS, 4096])
def test_evaluate_stays_inside_its_rows(flags, max_lds):
    """Evaluate, with its tables in LDS and through the caches, 4 stages at a time
    and one by one: the oracle's values on the oracle's splits, and no read past a
    row where another call left any layer counts"""
    for s_max in (16, 13):
        w = random_instance(60 + s_max, L=40, n_types=3, s_max=s_max, n=300, max_cost=3000, moe=True, cap_scale=30.0)
        o = O.price_plans(O.OracleProfile(w.profile), w.n_stages, w.stages, w.m, flags)
        it, pk, st, broken = CL.evaluate(w, flags, o["bottleneck"], o["layers"], o["status"], max_lds)
        ok = o["status"] == 0
        assert broken is None and ok.any()
        assert np.array_equal(st, o["status"]) and np.array_equal(pk, o["peak_mem"]) and np.array_equal(it, o["iter"])
        layers = np.random.default_rng(s_max).integers(0, 256, o["layers"].shape).astype(np.uint8)
        assert CL.evaluate(w, flags, o["bottleneck"], layers, o["status"], max_lds)[3] is None


@pytest.mark.parametrize("flags", [F32, F32 | CO])
def test_bounds_of_running_probes(slow_links, flags):
    """fp32 costs: lanes that take new templates while others are inside the probe
    of the rounded bound, p2p times above the layers' times: no bound falls below
    the least a stage can take, so no lookup leaves its row"""
    for w in [slow_links] + [random_instance(900 + seed, s_max=[6, 5, 4, 13, 16, 3][seed % 6], L=None if seed % 2 else 20 + seed,
                                             n=60, max_cost=6 if seed % 3 else 4000, cap_scale=[None, 0.5, 2.0][seed % 3])
                             for seed in (0, 4, 5, 7)]:
        w = repeated(w, 1000)
        g = CL.split(w, flags)
        CL.assert_split(w, g, flags, f"{w.name} flags {flags}")
    w = slow_outside_lds()
    g = CL.split(w, flags)
    CL.assert_split(w, g, flags, f"tables outside LDS, flags {flags}")
    assert not g["tables_in_lds"]


@pytest.mark.parametrize("flags", [0, CO, F32, F32 | CO])
def test_random_instances(flags):
    seen = set()
    for seed in range(12):
        w = repeated(random_instance(900 + seed, s_max=[6, 5, 4, 13, 16, 3][seed % 6], L=None if seed % 2 else 20 + seed,
                                     n=60, max_cost=6 if seed % 3 else 4000, cap_scale=[None, 0.5, 2.0][seed % 3]), 300)
        g = CL.split(w, flags)
        CL.assert_split(w, g, flags, f"seed {seed} flags {flags}")
        seen |= set(np.unique(g["status"]).tolist())
    assert 0 in seen and len(seen) > 4


@pytest.mark.parametrize("flags", [0, F32])
@pytest.mark.parametrize("n_types,L,s_max,scale,limits", [
    (61, 32, 8, 10**9, False), (22, 200, 4, 10**9, False), (51, 120, 3, 1, False), (26, 96, 7, 10**9, True),
    (20, 60, 12, 1, True), (85, 10, 5, 1, True)])
def test_tables_and_limits_near_the_size_of_lds(n_types, L, s_max, scale, limits, flags):
    """tables of 70 to 130 KB, memory limits that fit LDS alone but not beside
    them: the search runs with at least four wavefronts on a CU"""
    w = large_profile(n_types, L, s_max, scale, 100)
    g = CL.split(w, flags)
    CL.assert_split(w, g, flags, f"{n_types} types, L {L}")
    assert g["tables_in_lds"] and g["limits_in_lds"] == limits and g["per_cu"] >= 4


def test_search_without_room():
    """LDS too small for one wavefront's columns: not placed, nothing enqueued"""
    w = random_instance(3, L=100, s_max=64, n=4)
    g = CL.split(w, 0, max_lds=16 * 1024)
    assert g["rc"] == -4 and (g["left_count"], g["per_cu"]) == (0xA5A5A5A5, 0)
