"""The split search against the oracle: small batches whose every template the
oracle prices, repeated to a batch that takes the search whatever its templates
are (786,432 templates). Every copy has to equal the oracle's outputs bit for
bit."""
import numpy as np
import pytest

from gpu_common import CO, F32, assert_same, creeping_instance, gpu_price, large_profile, oracle_price, slow_outside_lds
from workloads.gen import Workload, make_workload, random_instance

pytestmark = pytest.mark.gpu
N = 786_432 + 77                                   # no multiple of a slice
N_ASKED = 196_608 + 77                             # the window pass's sample decides


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "no GPU"
    from paper_2609_34244_amd import heddle
    heddle.lib()
    return heddle


def check(H, w, flags, ctx, n=N):
    o = oracle_price(w, flags)
    reps = -(-n // w.n)
    order = np.random.default_rng(5).permutation(np.tile(np.arange(w.n), reps)[:n])
    big = Workload(name=w.name, profile=w.profile, n_stages=np.ascontiguousarray(w.n_stages[order]),
                   stages=np.ascontiguousarray(w.stages[order]), m=w.m, s_max=w.s_max)
    g = gpu_price(H, H.heddle_load_profile(w.profile), big, flags)
    assert_same(g, {k: v[order] for k, v in o.items()}, flags, ctx)
    return o


@pytest.mark.parametrize("flags", [0, CO, F32, F32 | CO])
def test_random_instances(H, flags):
    """ties, every status, stages that no layer fits, memory that binds, odd
    stage slots, several in-flight classes"""
    seen = set()
    for seed in range(12):
        w = random_instance(900 + seed, s_max=[6, 5, 4, 13, 16, 3][seed % 6], L=None if seed % 2 else 20 + seed, n=60,
                            max_cost=6 if seed % 3 else 4000, cap_scale=[None, 0.5, 2.0][seed % 3])
        seen |= set(np.unique(check(H, w, flags, f"seed {seed} flags {flags}")["status"]).tolist())
    assert 0 in seen and 8 in seen


@pytest.mark.parametrize("name,n", [("c2_7b_dense", 500), ("c3_70b_dense", 200), ("c4_moe", 300), ("c5_stress", 60)])
@pytest.mark.parametrize("flags", [0, F32])
def test_configs(H, name, n, flags):
    for n_batch in (N, N_ASKED):
        check(H, make_workload(name, n), flags, f"{name} flags {flags}", n_batch)


@pytest.mark.parametrize("flags", [0, CO, F32])
def test_wide_costs(H, flags):
    """stage times beyond 2^32: 64-bit rows, bucketed by their high bits"""
    for seed, scale in ((3, 10**9), (4, 10**12 + 7)):
        w = random_instance(seed, L=30, s_max=9, n=60, max_cost=3000)
        w.profile.layer_ns = np.ascontiguousarray(w.profile.layer_ns * scale)
        w.m = np.array([1, 7], np.int32)
        check(H, w, flags, f"scale {scale} flags {flags}")


@pytest.mark.parametrize("flags", [0, CO, F32])
def test_tables_outside_lds(H, flags):
    """more stage kinds than a byte holds, and tables too large for LDS: read
    through the caches"""
    rng = np.random.default_rng(11)
    w = random_instance(21, L=200, n_types=200, s_max=12, n=80, moe=True, invalid_frac=0.1)
    assert w.profile.n_types * len(w.profile.tp_degrees) * len(w.profile.ep_degrees) > 256
    w.profile.mem_cap_bytes[:] = rng.integers(60, 2000, size=200)
    check(H, w, flags, f"flags {flags}")


@pytest.mark.parametrize("n_types,L,s_max,scale", [(61, 32, 8, 10**9), (22, 200, 4, 10**9), (51, 120, 3, 1), (20, 60, 12, 1)])
def test_tables_near_the_size_of_lds(H, n_types, L, s_max, scale):
    """memory limits that would fit LDS alone, but not beside the tables (the
    last one: both fit)"""
    w = large_profile(n_types, L, s_max, scale, 60)
    for flags in (0, F32):
        check(H, w, flags, f"{n_types} types, L {L}, flags {flags}")


@pytest.mark.parametrize("flags", [0, CO, F32])
def test_few_templates_with_windows(H, flags):
    """large batches that the recurrence takes after all: mostly invalid
    templates, and links so slow that many searches would not settle"""
    w = make_workload("c3_70b_dense", 200)
    w.n_stages[np.random.default_rng(3).random(w.n) < 0.9] = 0
    check(H, w, flags, f"mostly invalid, flags {flags}", N_ASKED)
    for config in ("c3_70b_dense", "c1_tiny_dense"):
        w = make_workload(config, 200)
        w.profile.link_bw_MBps = np.maximum(w.profile.link_bw_MBps // 40, 1)
        check(H, w, flags, f"{config} with slow links, flags {flags}", N_ASKED)


@pytest.mark.parametrize("flags", [F32, F32 | CO])
def test_slow_links_outside_lds(H, flags):
    """transfers above the layers' times, tables read through the caches"""
    check(H, slow_outside_lds(), flags, f"flags {flags}")


@pytest.mark.parametrize("flags", [0, CO, F32])
@pytest.mark.parametrize("scale", [1, 10**9])
def test_left_to_the_split_kernel(H, scale, flags):
    """templates whose cuts move up one layer at a time, so that the search
    gives them up (test_search_on_cpu.py counts them)"""
    check(H, creeping_instance(scale), flags, f"heavy layers, scale {scale}, flags {flags}")


@pytest.mark.parametrize("flags", [0, F32, 4])
@pytest.mark.parametrize("n", [1200, N])
def test_addresses_off_16_bytes(H, n, flags):
    """records at 4 and layer counts at 1, 4 and 8 bytes past a multiple of 16: the
    paths that read and write 16 bytes are not taken"""
    import torch
    w = make_workload("c3_70b_dense", 200)
    o = oracle_price(w, flags)
    order = np.random.default_rng(5).permutation(np.arange(n) % w.n)
    prof = H.heddle_load_profile(w.profile)
    ns, st = H.to_device(w.n_stages[order], w.stages[order])
    for at, byte in ((0, 1), (1, 4), (1, 0), (2, 8)):
        rec = torch.empty(st.numel() + 4, dtype=st.dtype, device="cuda")[at:at + st.numel()].view(st.shape).copy_(st)
        out = H.alloc_outputs(n, 1, w.s_max, flags)
        size = out["layers"].numel()
        out["layers"] = torch.full((size + 16,), 0xAB, dtype=torch.uint8, device="cuda")[byte:byte + size].view(out["layers"].shape)
        assert rec.data_ptr() % 16 == 4 * at and out["layers"].data_ptr() % 16 == byte
        H.heddle_price_plans(prof, ns, rec, [64], flags, out)
        torch.cuda.synchronize()
        assert_same({k: v.cpu().numpy() for k, v in out.items()}, {k: v[order] for k, v in o.items()}, flags, f"records {at}, layers {byte}")


@pytest.mark.parametrize("chunk", [1, 15, 16, 17, 100, 0])
def test_count_of_fitting_plans(H, chunk):
    """the OK count of an enumerated space over chunks whose plan counts are and
    are not multiples of 16"""
    w = make_workload("c3_70b_dense", 1)
    prof = H.heddle_load_profile(w.profile)
    spec = H.EnumSpec(2, [0, 5], [0, 1, 2], [1, 2])
    ns, st = H.heddle_enum_templates(spec, 0, H.heddle_enum_count(spec))
    m = [8, 64, 65]
    out = H.heddle_price_plans(prof, ns, st, m, 0, H.alloc_outputs(len(ns), 3, 2, 0))
    assert H.heddle_best_enumerated(prof, spec, m, 0, chunk)[3] == int((out["status"] == 0).sum())
