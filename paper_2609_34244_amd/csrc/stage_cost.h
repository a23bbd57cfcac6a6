// Cost of one pipeline stage holding layers [i, j) under the profile-based
// cost model (Heddle, arXiv 2609.34244, section 5.2): stage time (layer
// costs with the all-to-all of MoE layers, plus the outbound p2p), per-GPU
// memory with min(S - s, M_p) micro-batches of activations in flight, and
// gradient synchronisation (ring all-reduce of dense gradients over the D
// replicas and of expert gradients over D / EP). Shared by every kernel that
// evaluates a split, so they price identically.
#pragma once

#include "device_common.h"

namespace heddle {

struct StageCost {
    uint64_t T;        // stage time: ns, or fixed point (2^fx_exp) for fp32, not rounded
    int64_t mem;       // per-GPU bytes
    int64_t g;         // gradient synchronisation, ns
    bool fits;         // mem <= the GPU's memory
};

// Where a stage's cost is read from: the profile's tables through the caches.
template <bool F32> struct GlobalCost {
    const DevProfile &P;
    __device__ __forceinline__ void load(unsigned char *) {}
    struct At {                      // the places of one stage's kind
        int64_t cap, bw, p2p;
        const uint64_t *row;
        const longlong2 *sx, *ag;
    };
    __device__ __forceinline__ At at(uint32_t rec, int g_next, bool last, int D) const
    {
        const int R = P.L + 1, N = P.n_types;
        const int g = rec & 0xFF, l2tp = (rec >> 8) & 15, l2ep = (rec >> 12) & 15;
        const int tp = 1 << l2tp, ep = 1 << l2ep;
        const int ki = nibble(P.tp_index, l2tp), ei = nibble(P.ep_index, l2ep);
        const int node = P.node_size[g];
        At a;
        a.row = P.rows64[F32 ? 1 : 0] + ((size_t)(g * P.n_tp + ki) * 3 + a2a_variant(ep, tp, node)) * R;
        a.sx = P.pair_sx + (ki * P.n_ep + ei) * R;
        a.ag = P.pair_ag + ki * R;
        a.cap = P.mem_cap[g];
        a.bw = (int64_t)tp * D <= node ? P.intra_bw[g] : P.link_bw[g * N + g];
        a.p2p = 0;
        if (!last) a.p2p = F32 ? P.p2p_fx[g * N + g_next] : P.p2p_ns[g * N + g_next];
        return a;
    }
    __device__ __forceinline__ double inv_total(uint32_t rec) const
    {
        const int g = rec & 0xFF, l2tp = (rec >> 8) & 15, l2ep = (rec >> 12) & 15;
        const int ki = nibble(P.tp_index, l2tp);
        const size_t row = (size_t)(g * P.n_tp + ki) * 3 + a2a_variant(1 << l2ep, 1 << l2tp, P.node_size[g]);
        return 1.0 / (double)P.rows64[0][row * (P.L + 1) + P.L];
    }
};

// The same from a copy of the profile's cost block in LDS (V: entry type of its
// time rows). A stage's nine divergent reads go to LDS instead of taking the
// vector address unit one lane at a time.
template <bool F32, class V> struct LdsCost {
    const DevProfile &P;
    const unsigned char *block;
    __device__ __forceinline__ void load(unsigned char *lds)     // by the whole workgroup; the caller synchronises
    {
        const uint4 *src = (const uint4 *)P.cost_block[F32 ? 1 : 0];
        for (int i = threadIdx.x; i < P.cost_bytes[F32 ? 1 : 0] / 16; i += blockDim.x) ((uint4 *)lds)[i] = src[i];
        block = lds;
    }
    struct At {
        int64_t cap, bw, p2p;
        const V *row;
        const longlong2 *sx, *ag;
    };
    __device__ __forceinline__ const CostKind &kind(uint32_t rec) const
    {
        const uint32_t l2tp = (rec >> 8) & 15, l2ep = (rec >> 12) & 15;
        return ((const CostKind *)block)[((rec & 0xFF) * (uint32_t)P.n_tp + (uint32_t)nibble(P.tp_index, l2tp)) * (uint32_t)P.n_ep +
                                         (uint32_t)nibble(P.ep_index, l2ep)];
    }
    __device__ __forceinline__ At at(uint32_t rec, int g_next, bool last, int D) const
    {
        const CostKind &k = kind(rec);
        At a;
        a.row = (const V *)(block + P.cost_rows) + k.row;
        a.sx = (const longlong2 *)(block + P.cost_sx) + k.sx;
        a.ag = (const longlong2 *)(block + P.cost_ag) + k.ag;
        a.cap = k.cap;
        a.bw = ((int64_t)D << ((rec >> 8) & 15)) <= k.node ? k.intra : k.link;
        const int64_t p2p = ((const int64_t *)(block + P.cost_p2p))[last ? 0 : (rec & 0xFF) * (uint32_t)P.n_types + (uint32_t)g_next];
        a.p2p = last ? 0 : p2p;
        return a;
    }
    __device__ __forceinline__ double inv_total(uint32_t rec) const { return kind(rec).inv_total; }
};

// rec: the stage's packed record; g_next: the next stage's GPU type (ignored
// for the last stage). The record must have passed validation.
template <bool F32, class C>
__device__ __forceinline__ StageCost stage_cost(const C &tab, uint32_t rec, int g_next, int s, int S, int i, int j, int D,
                                                int64_t Mp)
{
    const auto a = tab.at(rec, g_next, s + 1 >= S, D);
    const longlong2 sx_i = a.sx[i], sx_j = a.sx[j];            // {state, expert grad}
    const longlong2 ag_i = a.ag[i], ag_j = a.ag[j];            // {activations, dense grad}
    StageCost c;
    c.T = (uint64_t)a.row[j] - (uint64_t)a.row[i] + (uint64_t)a.p2p;
    const int64_t f = (int64_t)(S - s) < Mp ? (int64_t)(S - s) : Mp;
    c.mem = (sx_j.x - sx_i.x) + f * (ag_j.x - ag_i.x);
    c.fits = c.mem <= a.cap;
    c.g = allreduce_ns(ag_j.y - ag_i.y, D, a.bw) +
          allreduce_ns(sx_j.y - sx_i.y, (int64_t)((uint32_t)D >> ((rec >> 12) & 15)), a.bw);
    return c;
}

// bytes of the cost block for a launch that reads it from LDS, 0 where three
// workgroups of it would not share a CU: Evaluate on c5 (85 KB, one workgroup of
// 512 per CU) took 0.395 ms from LDS against 0.300 ms through the caches
inline size_t cost_lds(const DevProfile &d, bool f32, int lds_cu)
{
    const size_t bytes = (size_t)d.cost_bytes[f32 ? 1 : 0];
    return 3 * (bytes + 2048) <= (size_t)lds_cu ? bytes : 0;
}

// 1F1B iteration time (section 5.3) from the bottleneck B, the sum of stage
// times and the largest synchronisation; fp32: B and every stage time are
// already rounded (exact integers with 24 significant bits), the largest
// synchronisation is rounded here and the total once more by the caller.
template <bool F32>
__device__ __forceinline__ uint64_t iteration_time(const DevProfile &P, int64_t Mp, uint64_t B, uint64_t sumT,
                                                   int64_t maxg)
{
    const uint64_t maxg_v = F32 ? rne24((uint64_t)maxg) << (-P.fx_exp) : (uint64_t)maxg;
    return (uint64_t)(Mp - 1) * B + sumT + maxg_v;
}

}  // namespace heddle
