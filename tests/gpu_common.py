"""Shared helpers of the GPU tests: run the HIP library through its C ABI
binding, run the CPU oracle on the same seeded inputs, compare."""
from __future__ import annotations

import numpy as np

from oracle import oracle as O
from workloads.gen import Workload, pack_stage, random_instance

F32 = 1
CO = 2
POISON = 0xAB


def sub_workload(w, idx):
    idx = np.asarray(idx)
    return Workload(name=w.name, profile=w.profile, n_stages=np.ascontiguousarray(w.n_stages[idx]),
                    stages=np.ascontiguousarray(w.stages[idx]), m=w.m, s_max=w.s_max, meta=w.meta)


def gpu_price(H, prof, w, flags, poison=True):
    """Price on the GPU; outputs pre-filled with a poison byte so that any
    slot the kernels do not write shows up."""
    import torch
    ns, st = H.to_device(w.n_stages, w.stages)
    out = H.alloc_outputs(w.n, len(w.m), w.s_max, flags)
    if poison:
        for v in out.values():
            v.view(torch.uint8).fill_(POISON)
    H.heddle_price_plans(prof, ns, st, [int(x) for x in w.m], flags, out)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def oracle_price(w, flags):
    return O.price_plans(O.OracleProfile(w.profile), w.n_stages, w.stages, w.m, flags)


def assert_same(g, o, flags, ctx=""):
    """Bit-exact comparison of every output."""
    for k in ("status", "layers", "peak_mem", "iter", "bottleneck"):
        a, b = g[k], o[k]
        if k in ("iter", "bottleneck") and flags & F32:
            a, b = a.view(np.uint32), b.view(np.uint32)
        if not np.array_equal(a, b):
            bad = np.argwhere(a != b)
            i = tuple(bad[0])
            t = i[0]
            raise AssertionError(
                f"{ctx}: {k} differs at {len(bad)} places, first {i}: gpu={a[i]} oracle={b[i]}; "
                f"template {t}: status gpu={g['status'][t]} oracle={o['status'][t]}, "
                f"layers gpu={g['layers'][t].tolist()} oracle={o['layers'][t].tolist()}, "
                f"iter gpu={g['iter'][t]} oracle={o['iter'][t]}")


def key_lt(it_a, m_a, it_b, m_b):
    """iter_a / m_a < iter_b / m_b, exactly"""
    from fractions import Fraction
    fa = Fraction(float(it_a)) if isinstance(it_a, (float, np.floating)) else int(it_a)
    fb = Fraction(float(it_b)) if isinstance(it_b, (float, np.floating)) else int(it_b)
    return fa * int(m_b) < fb * int(m_a)


def large_profile(n_types, L, s_max, scale, n):
    """every (type, TP) row in use, so that the search's tables come near LDS's size"""
    seed = next(s for s in range(100) if len(random_instance(s, L=2, n_types=1, n=1).profile.tp_degrees) == 3)
    w = random_instance(seed, L=L, n_types=n_types, s_max=s_max, n=n, max_cost=3000, moe=False, invalid_frac=0.1)
    p = w.profile
    p.profiled[:] = 1
    p.node_size[:] = 8
    p.n_gpus[:] = 64
    p.layer_ns = np.ascontiguousarray(p.layer_ns * scale)
    p.mem_cap_bytes[:] = np.random.default_rng(11).integers(L, 6 * L, size=n_types)
    return w


def slow_outside_lds():
    """more stage kinds than a byte holds (tables read through the caches), and
    transfers above the layers' times"""
    w = random_instance(21, L=100, n_types=200, s_max=12, n=40, moe=True, invalid_frac=0.1)
    w.profile.boundary_bytes = 10**6
    w.profile.mem_cap_bytes[:] = np.random.default_rng(11).integers(60, 2000, size=200)
    return w


def creeping_instance(scale=1):
    """heavy layers that only the first stages' type can hold: cuts move up one
    layer at a time. Three in-flight classes."""
    w = random_instance(1, L=120, n_types=2, s_max=12, n=40, moe=False, invalid_frac=0.0, cap_scale=100.0)
    rng = np.random.default_rng(2)
    p = w.profile
    p.profiled[:] = 1
    p.layer_ns[0] = 10 * scale
    p.layer_ns[1] = scale * np.where(rng.random(120) < 0.5, 10, 1000 + np.arange(120))[None, :]
    p.mem_cap_bytes[:] = 1 << 40
    p.node_size[:] = 8
    p.n_gpus[:] = 4096
    p.link_bw_MBps[:] = 1000
    p.boundary_bytes = 0
    S = rng.integers(8, 13, size=40)
    g = rng.integers(0, 2, size=(40, 12))
    w.m = np.array([2, 6, 64], np.int32)
    w.n_stages = S.astype(np.uint8)
    w.stages = np.ascontiguousarray(np.where(np.arange(12)[None] < S[:, None], pack_stage(g, 0, 0, 1), 0).astype(np.uint32))
    return w
