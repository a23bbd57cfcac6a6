// Split search on gfx950: the exact min-max layer split (PartitionLayers of
// the planners' nested-loop backbone, Heddle, arXiv 2609.34244, section 3.1,
// aware of per-stage GPU speed and of memory) of many templates at once, one
// lane per template. It finds the same bottleneck and the same canonical split
// as the recurrence of the split kernel (price.hip), by search instead of by
// relaxing every (row, end) pair.
//
// For a bound B, a split c_0 = 0 < c_1 < ... < c_S = L keeps to B when every
// stage's time T(s, c_s, c_{s+1}) <= B and every stage fits memory. For a
// fixed end both conditions hold from some first row on, so they read
// c_s >= low_s(c_{s+1}), with low_s non-decreasing in the end; with
// c_{s+1} >= c_s + 1 these are the only constraints. Splits that keep to B
// are therefore closed under the componentwise minimum: there is a least one,
// it is the lexicographically smallest, and raising values from any lower
// bound until every constraint holds finds it or shows that there is none.
// A probe of B does that in sweeps from the last stage down, c_s = max(its
// lower bound, low_s(c_{s+1})). Where that leaves stage s no layer, c_{s+1}
// is raised to the next end whose last layer alone keeps to B, and one more
// sweep follows from the values reached.
//   - A feasible probe bounds B* from above by its largest stage time, and its
//     split is a lower bound of the split of every smaller B.
//   - An infeasible probe bounds B* from below by the smallest stage time that
//     any of its tests refused: under every B below that the probe would take
//     the same course.
// The two bounds meet exactly at B*, and the split of the last feasible probe
// is the canonical one. (fp32 pricing compares rounded times: one more probe
// at the largest value that rounds to B*'s rounding gives its split.)
//
// Mapping. A wavefront takes a slice of the batch, lists its templates that
// have windows by stage count, most first, and hands them to its lanes; all
// lanes sweep together, one stage per step counted from the last, and a lane
// whose search has ended takes the next of the list. The profile's
// time-prefix rows, with a table that turns a time into a first guess of a
// row's index (its bucket's first index), and the memory limits when they fit
// are copied into LDS once per workgroup; a lane's template is a column of one
// word per stage in its wavefront's LDS region, so those accesses are free of
// conflicts.
//
// What bounds it: the slices that take longest, and within them vector issue and the
// chain of three dependent LDS reads of a step (time at the end, bucket, rows around
// it). On c3 (1,000,000 templates, 16 wavefronts on a CU, a slice each) the vector units
// are busy 54% of the launch with 37.8 of 64 lanes on, 2.8 of a SIMD's 4 wavefronts are
// alive on average, and LDS is busy 32%, 44% of that with bank conflicts of the random
// reads (c5, 11 wavefronts: 42%, 30.4 lanes, 2.35 of 2.75, 23%, 50%). A template that
// fits takes 5.3 sweeps of one step per stage, where the recurrence takes about 960
// vector instructions of a whole wavefront: 0.23 ms against 1.05 ms (c5, 300,000
// templates x 6 micro-batch counts: 2.0 ms against 7.3 ms).
#include <cstring>

#include "dp_common.h"

namespace heddle {

template <class V> struct SearchTables;
template <> struct SearchTables<uint32_t> {
    static __device__ __forceinline__ const uint32_t *get(const DevProfile &P, bool f32) { return P.search32[f32 ? 1 : 0]; }
};
template <> struct SearchTables<uint64_t> {
    static __device__ __forceinline__ const uint64_t *get(const DevProfile &P, bool f32) { return P.search64[f32 ? 1 : 0]; }
};

// largest integer whose fp32 rounding is that of x
__device__ __forceinline__ uint64_t rne24_top(uint64_t x)
{
    const uint64_t v = rne24(x);
    if (v < (1ull << 24)) return v;
    const int sh = 40 - __clzll(v);                            // spacing above v is 2^sh
    return v + (1ull << (sh - 1)) - (((v >> sh) & 1) ? 1 : 0); // a tie goes to an even v
}

// LT: the tables are in LDS and a stage's kind (type, TP, EP) is a byte; else
// the tables are read through the caches and the kind has a column of its own
// LIM: the memory limits are 0 ignored, 1 in LDS, 2 read through the caches
template <class V, bool LT, int LIM>
__global__ void __launch_bounds__(1024) search_kernel(DevProfile P, PriceArgs A, SearchArgs X)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const V INF = DPInf<V>::value;
    enum { kEmpty, kRun, kDone };                              // lane states
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    // the same answer in every wavefront; the split kernel reads it
    bool runs = true;
    if (A.need > 0.f) runs = search_runs(A, (float)wave_sum(A.left[2 + lane]), (float)wave_sum(A.left[2 + kSamples + lane]));
    if (blockIdx.x == 0 && threadIdx.x == 0) A.left[1] = runs ? 1u : 0u;
    if (!runs) return;
    const int L = P.L, RS = P.search_stride[sizeof(V) == 8], N = P.n_types, ls = P.lim_stride, F = P.n_f;
    const bool f32 = (A.flags & HEDDLE_F_FP32) != 0;
    constexpr bool mem_aware = LIM != 0;
    const int shift = sizeof(V) == 4 ? 0 : P.search_shift[f32 ? 1 : 0];
    const V b_max = (V)(INF >> 1);                             // above every stage time
    const V *gtab = SearchTables<V>::get(P, f32);
    const V *tab;                                              // [rows][RS]: a word (read before P[0], not used), P[0 .. L], buckets
    if constexpr (LT) {
        uint4 *dst = (uint4 *)smem;
        const uint4 *src = (const uint4 *)gtab;
        for (int i = threadIdx.x; i < X.copy_bytes / 16; i += blockDim.x) dst[i] = src[i];
        tab = (const V *)smem;
    } else {
        tab = gtab;
    }
    const V *pm = tab + (size_t)P.search_rows * RS;            // [N * N + 1] p2p by type pair, 0 last
    // by kind: row | GPU type << 24, bucket scale (fp32 bits), least layer time
    const uint4 *gkinds = P.search_kind[(f32 ? 1 : 0) + (sizeof(V) == 8 ? 2 : 0)];
    const uint4 *kinds = LT ? (const uint4 *)(smem + X.kind_off) : gkinds;
    uint8_t *degree = smem + X.tab_bytes - 256;                // [256] by log2 TP | log2 EP << 4: index of (TP, EP)
    for (int i = threadIdx.x; i < 256; i += blockDim.x)
        degree[i] = (uint8_t)min(nibble(P.tp_index, i & 15) * P.n_ep + nibble(P.ep_index, i >> 4), X.degrees - 1);
    if constexpr (LT) {
        for (int i = threadIdx.x; i < X.n_kinds; i += blockDim.x) ((uint4 *)(smem + X.kind_off))[i] = gkinds[i];
    }
    // inverse memory-limit rows in LDS, [n_types][n_tp][n_ep][lim_f] of lim_words words
    uint32_t *limw = (uint32_t *)(smem + X.tab_bytes);
    const uint8_t *limb = (const uint8_t *)limw;
    if constexpr (LIM == 1) {
        const int used = (L + 4) >> 2, rows = X.lim_rows * used;   // words that hold entries 0 .. L
        for (int i = threadIdx.x; i < rows; i += blockDim.x) {
            const uint32_t r = (uint32_t)i / (uint32_t)used, q = (uint32_t)i - r * (uint32_t)used;
            const uint32_t kind = r / (uint32_t)X.lim_f, f = r - kind * (uint32_t)X.lim_f;
            limw[r * (uint32_t)X.lim_words + q] =
                ((const uint32_t *)(P.mem_lim + (size_t)(((kind * (uint32_t)F + f) * 2 + 1)) * ls))[q];
        }
    }
    __syncthreads();
    unsigned char *mine = smem + X.tab_bytes + X.lim_bytes + (size_t)wave * X.wave_bytes;
    uint16_t *list = (uint16_t *)mine;                         // [kSearchSlice] templates of the slice, most stages first
    // columns by position u = S - 1 - s, the stage counted from the last:
    // [s_cap + 2][64] c, c, last row, kind (LT); the first two bytes hold the
    // start of the stage in the last feasible probe's split (byte par, the lower
    // bound) and in the running probe (byte 1 - par)
    uint32_t *colW = (uint32_t *)(mine + 2 * kSearchSlice) + lane;
    uint32_t *colK = colW + (X.s_cap + 2) * 64;                // !LT: kind

    // What is read from the window pass's scratch (which templates have windows, their
    // in-flight classes and windows) may be another call's where calls overlap on one
    // buffer: it is read once or bounded on use, so that whatever it holds, every
    // access stays inside the batch and the tables, and every search ends.
    int state = kEmpty, S = 0, key = 0, k0 = 0, left = 0;
    int f_top = 0;                                             // micro-batches in flight, less one, at most
    int64_t t = 0;
    bool last_probe = false;                                   // fp32: the probe that gives the split
    bool warm = false;                                         // a bound of an earlier class is being tested
    V B = 0, lo = 0, hi = INF, nb = INF;
    int par = 0, shc = 0;                                      // shc: bit offset of the byte that bounds a sweep's starts

    // (columns past a template's stages hold anything: kept inside the kind table)
    auto kind_of = [&](int u, uint32_t w) -> uint32_t { return LT ? w >> 24 : min(colK[u * 64], (uint32_t)(X.n_kinds - 1)); };
    // entry x of the inverse memory-limit row of position u: the first row from which
    // layers up to x fit with min(u + 1, key) micro-batches in flight
    auto lim_at = [&](uint32_t kind, int f, int x) -> int {
        if constexpr (LIM == 1) return limb[(__umul24(kind, (uint32_t)X.lim_f) + (uint32_t)f) * (uint32_t)(4 * X.lim_words) + (uint32_t)x];
        return P.mem_lim[(size_t)(kind * (uint32_t)F + (uint32_t)f) * (uint32_t)(2 * ls) + (uint32_t)(ls + x)];
    };
    // four records of a template and the windows of its stages q0 .. q0 + 3 (q0 < S). By
    // 16 bytes where the rows are aligned: a wavefront's lanes read as many rows, and
    // the address unit takes them one by one
    auto fetch = [&](const uint32_t *rec, const uint16_t *win, int n, int q0, uint4 &r, uint2 &w) {
        if (X.vec_rec) {
            r = *(const uint4 *)(rec + q0);
        } else {
            r.x = rec[q0];
            r.y = rec[min(q0 + 1, n - 1)];
            r.z = rec[min(q0 + 2, n - 1)];
            r.w = rec[min(q0 + 3, n - 1)];
        }
        w = *(const uint2 *)(win + q0);
    };
    // columns of four stages, and their part of the template's bounds; r4: the record
    // after them (any after the last stage)
    float sw = 0.f, sp = 0.f;
    V least = 0;
    auto place = [&](int q0, uint4 r, uint32_t r4, uint2 w2) {
        const uint32_t rr[5] = {r.x, r.y, r.z, r.w, r4}, n_top = (uint32_t)N - 1;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int u = S - 1 - q0 - q;                      // below 0: past the last stage, into a spare row
            const bool in = u >= 0;
            const uint32_t g = min(rr[q] & 255u, n_top);
            const uint32_t k = in ? g * (uint32_t)X.degrees + degree[(rr[q] >> 8) & 255u] : 0u;
            const uint4 kd = kinds[k];
            const V p2p = pm[u > 0 ? g * N + min(rr[q + 1] & 255u, n_top) : (uint32_t)(N * N)];
            const uint32_t w = ((q & 2) ? w2.y : w2.x) >> ((q & 1) * 16);
            const uint32_t a = min(w & 255, (uint32_t)L), b = min((w >> 8) & 255, (uint32_t)L);
            const float fs = in ? __uint_as_float(kd.y) : 0.f;
            sw += fs;
            sp += fs * (float)p2p;
            least = in ? vmax<V>(least, (V)(p2p + (V)((uint64_t)kd.w << 32 | kd.z))) : least;
            const int row = in ? u : X.s_cap + 1;
            colW[row * 64] = a | a << 8 | b << 16 | (LT ? k << 24 : 0u);
            if constexpr (!LT) colK[row * 64] = k;
        }
    };

    const int64_t n_slices = (A.n + X.slice - 1) / X.slice;
    for (int64_t sl = (int64_t)blockIdx.x * waves + wave; sl < n_slices; sl += (int64_t)gridDim.x * waves) {
        // ---------------- the slice's templates that have windows, by stage count
        const int64_t base_t = sl * X.slice;
        const int nt = A.n - base_t < X.slice ? (int)(A.n - base_t) : X.slice;
        int n_list;
        {
            uint32_t *bins = colW - lane;                      // [64], free between slices
            auto usable = [&](int q) -> int {                  // stage count of a template with windows, else 0
                if (q >= nt) return 0;
                bool ok = false;
                for (int k = 0; k < A.n_m; k++) ok |= (A.wst[(base_t + q) * A.n_m + k] & 255u) == HEDDLE_S_OK;
                const int st = A.n_stages[base_t + q];
                return ok && st <= X.s_cap ? st : 0;
            };
            uint32_t has = 0;                                  // bit i: the template i * 64 + lane of the slice
            static_assert(kSearchSlice <= 32 * 64, "a bit per 64 templates of a slice");
            bins[lane] = 0;
            wave_sync();
            for (int q0 = 0; q0 < nt; q0 += 64) {
                const int st = usable(q0 + lane);
                has |= (st ? 1u : 0u) << (q0 >> 6);
                if (st) atomicAdd(&bins[64 - st], 1u);
            }
            wave_sync();
            const int c = (int)bins[lane], incl = wave_inclusive_sum(c);
            wave_sync();
            bins[lane] = (uint32_t)(incl - c);
            n_list = rl32(incl, 63);
            wave_sync();
            for (int q0 = 0; q0 < nt; q0 += 64) {
                if (!((has >> (q0 >> 6)) & 1u)) continue;
                const int st = A.n_stages[base_t + q0 + lane];
                list[atomicAdd(&bins[64 - st], 1u)] = (uint16_t)(q0 + lane | (st - 1) << 10);
                if (A.n_m == 1) continue;
                for (int k = 0; k < A.n_m; k++) {              // plans without windows beside ones with
                    const int64_t o = (base_t + q0 + lane) * A.n_m + k;
                    const uint32_t code = A.wst[o] & 255u;
                    if (code == HEDDLE_S_OK) continue;
                    A.status[o] = (uint8_t)code;
                    if (f32) ((float *)A.bottleneck)[o] = __builtin_inff();
                    else ((int64_t *)A.bottleneck)[o] = INT64_MAX;
                    for (int q = 0; q < A.s_max; q++) A.layers[o * A.s_max + q] = 0;
                }
            }
            wave_sync();
        }
        int head = 0, u_max = 0;
        for (;;) {
            // ---------------- lanes without a search: outputs of the ended ones, new templates
            const int n_idle = __popcll(ballot(state == kDone || (state == kEmpty && head < n_list)));
            if (n_idle >= X.refill || !ballot(state == kRun)) {
                // which lanes write outputs, and what each searches next: the split at a
                // rounded bound (fp32), the template's next class, a template of the list
                const bool found = hi != INF, ended = state == kDone;
                const bool again = ended && f32 && found && !last_probe, out = ended && !again;
                const int64_t obase = t * A.n_m;
                const int S_out = S, par_out = par, key_out = key;
                const V hi_out = hi;
                bool load = again;
                if (out && A.n_m > 1) {
                    int next_key = -1;
                    for (int k = 0; k < A.n_m; k++) {
                        const uint32_t wv = A.wst[obase + k];
                        const int kk = (int)((wv >> 8) & 255);
                        if ((wv & 255) == HEDDLE_S_OK && kk < key_out && kk > next_key) {
                            next_key = kk;
                            k0 = k;
                        }
                    }
                    load = next_key >= 0;
                    key = load ? next_key : key;
                }
                // (a lane whose probe is under way keeps what it is)
                last_probe = state == kRun ? last_probe : again;
                warm = state == kRun ? warm : load && !again && found && !f32;
                state = ended && !load ? kEmpty : state;
                const uint64_t empty = ballot(state == kEmpty);
                const int at = head + lanes_below(empty);
                if (state == kEmpty && at < n_list) {
                    const int en = list[at];
                    t = base_t + (en & 1023);
                    S = (en >> 10) + 1;
                    key = -1;
                    for (int k = 0; k < A.n_m; k++) {          // the class of the largest key first
                        const uint32_t wv = A.wst[t * A.n_m + k];
                        const int kk = (int)((wv >> 8) & 255);
                        if ((wv & 255) == HEDDLE_S_OK && kk > key) {
                            key = kk;
                            k0 = k;
                        }
                    }
                    load = true;
                }
                head += __popcll(empty);
                head = head < n_list ? head : n_list;
                // the new templates' records and windows are on their way before the
                // outputs are stored: a wait for a load also waits for the stores before it
                const uint32_t *rec = A.stages + t * A.s_max;
                const uint16_t *win = A.wwin + (t * A.n_m + k0) * win_stride(A.s_max);
                uint4 r0 = {}, r1 = {}, r2 = {}, r3 = {};
                uint2 w0 = {}, w1 = {}, w2 = {}, w3 = {};
                if (load) {
                    fetch(rec, win, S, 0, r0, w0);
                    if (S > 4) fetch(rec, win, S, 4, r1, w1);
                    if (S > 8) fetch(rec, win, S, 8, r2, w2);
                    if (S > 12) fetch(rec, win, S, 12, r3, w3);
                }
                if (out) {
                    for (int k = 0; k < A.n_m; k++) {
                        if (A.n_m > 1) {
                            const uint32_t wv = A.wst[obase + k];
                            if ((wv & 255) != HEDDLE_S_OK || (int)((wv >> 8) & 255) != key_out) continue;
                        }
                        const int64_t o = obase + k;
                        A.status[o] = (uint8_t)(found ? HEDDLE_S_OK : HEDDLE_S_OOM);
                        if (f32) ((float *)A.bottleneck)[o] = found ? exact_float(rne24((uint64_t)hi_out), P.fx_exp) : __builtin_inff();
                        else ((int64_t *)A.bottleneck)[o] = found ? (int64_t)hi_out : INT64_MAX;
                        uint8_t *lay = A.layers + o * A.s_max;
                        uint32_t c = 0;                        // c_q
                        auto word_at = [&](int q0) -> uint32_t {
                            uint32_t word = 0;
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                const int u1 = S_out - 2 - q0 - q;   // position of stage q0 + q + 1; -1: the end
                                const uint32_t x = (colW[max(u1, 0) * 64] >> (8 * par_out)) & 255u;
                                const uint32_t c1 = found && u1 >= -1 ? (u1 >= 0 ? x : (uint32_t)L) : c;
                                word |= (c1 - c) << (8 * q);
                                c = c1;
                            }
                            return word;
                        };
                        if (X.vec_lay) {
                            for (int q0 = 0; q0 < A.s_max; q0 += 16) {
                                uint4 v;
                                v.x = word_at(q0);
                                v.y = word_at(q0 + 4);
                                v.z = word_at(q0 + 8);
                                v.w = word_at(q0 + 12);
                                *(uint4 *)(lay + q0) = v;
                            }
                        } else {
                            for (int q0 = 0; q0 < A.s_max; q0 += 4) {
                                const uint32_t word = word_at(q0);
                                if (X.words) {
                                    *(uint32_t *)(lay + q0) = word;
                                } else {
                                    for (int q = 0; q < 4 && q0 + q < A.s_max; q++) lay[q0 + q] = (uint8_t)(word >> (8 * q));
                                }
                            }
                        }
                    }
                }
                if (load) {
                    f_top = max(key, 1) - 1;
                    sw = sp = 0.f;
                    least = 0;
                    place(0, r0, r1.x, w0);
                    if (S > 4) place(4, r1, r2.x, w1);
                    if (S > 8) place(8, r2, r3.x, w2);
                    if (S > 12) place(12, r3, S > 16 ? rec[16] : 0u, w3);
                    for (int q0 = 16; q0 < S; q0 += 4) {
                        uint4 r;
                        uint2 w;
                        fetch(rec, win, S, q0, r, w);
                        place(q0, r, q0 + 4 < S ? rec[q0 + 4] : 0u, w);
                    }
                    par = shc = 0;
                    nb = INF;
                    left = S <= 16 ? X.sweeps_short : X.sweeps;
                    state = kRun;
                    // the first probe: the bound that an even division of the work would reach, or
                    // an earlier class's bound (this class fits wherever that one does)
                    const float est = (sp + ldexpf((float)(P.search_buckets - 1), shift)) / sw;
                    V bf = est < (float)b_max ? (V)est : b_max;
                    bf = vmin<V>(vmax<V>(bf, least), b_max);
                    bf = warm ? hi_out : bf;
                    B = last_probe ? (V)vmin<uint64_t>(rne24_top((uint64_t)hi_out), (uint64_t)b_max) : bf;
                    lo = least;
                    hi = last_probe ? hi_out : INF;
                }
                wave_sync();
                if (!ballot(state != kEmpty)) break;           // the slice is done
                u_max = uni(wave_max(state == kRun ? S : 0));
            }
            // ---------------- a sweep: one step per stage, the last first
            // no bound is below a stage's p2p and least layer time, so its row holds an index
            // with P[row] >= B's remainder at or before its end: the lookup stays in the row
            HEDDLE_INVARIANT(state != kRun || B >= least);
            int e = L, upe = L, lu = state == kRun ? S : 0;    // lu: steps of this lane
            bool fail = false, redo = false;
            V mx = 0;
            uint32_t ws = colW[0], wn = colW[64];              // the words of position u and u + 1
            uint2 ks = *(const uint2 *)&kinds[kind_of(0, ws)];                  // (a lane without a template: any)
            uint32_t gn = (uint32_t)N;                         // GPU type of the stage after; N: none
#pragma unroll 1
            for (int u = 0; u < u_max; u++) {
                const bool on = u < lu;
                if (!ballot(on)) break;
                const uint32_t w = ws, kind = kind_of(u, w);
                const uint2 kd = ks;
                ws = wn;
                wn = colW[(u + 2) * 64];
                ks = *(const uint2 *)&kinds[kind_of(u + 1, ws)];
                const uint32_t g = kd.x >> 24;
                const V *pp = pm + (gn == (uint32_t)N ? (uint32_t)(N * N) : g * (uint32_t)N + gn);
                gn = g;
                if (on) {
                    const uint32_t row = (kd.x & 0xFFFFFFu) + 1;
                    int il = 0;
                    const int f = min(u, f_top);
                    if (mem_aware) il = lim_at(kind, f, e);
                    const V p2p = *pp;
                    const V pe = tab[row + (uint32_t)e] + p2p;
                    const float fs = __uint_as_float(kd.y);
                    const V tt = pe > B ? (V)(pe - B) : (V)0;  // low_s: the first row with P[row] >= tt
                    const uint32_t bu = (uint32_t)((float)(uint32_t)(tt >> shift) * fs);
                    HEDDLE_INVARIANT(tt <= tab[row + (uint32_t)e] && bu <= (uint32_t)P.search_buckets);
                    const int qi = ((const uint8_t *)&tab[row + (uint32_t)(L + 1)])[bu];
                    const int base = max((int)((w >> shc) & 255u), il);
                    int i = max(base, qi);
                    const V *pr = tab + row + (uint32_t)i;
                    V p1 = pr[-1], p0 = pr[0];
                    const V pn = pr[1];                        // (past P[L]: a bucket word, not used)
                    const bool one = p0 < tt;                  // a bucket rarely holds two rows below tt
                    i += one;
                    p1 = one ? p0 : p1;
                    p0 = one ? pn : p0;
                    if (p0 < tt) {
                        pr += 1;
                        do {
                            i++;
                            p1 = p0;
                            p0 = *++pr;
                        } while (p0 < tt);
                    }
                    nb = i > base ? vmin<V>(nb, (V)(pe - p1)) : nb;   // time, not memory or the bound, set the row
                    mx = vmax<V>(mx, (V)(pe - p0));
                    const int up = (int)((w >> 16) & 255u);
                    ((uint8_t *)&colW[u * 64])[1 - par] = (uint8_t)i;
                    fail = i > up;
                    if (i >= e) {
                        // no layer for the stage: raise its end (the start of the position before)
                        // past row i, over ends whose last layer alone does not keep to B or fit
                        redo = true;
                        int e2 = i + 1;
                        V pv = p0;
                        for (int tries = X.walk; tries > 0 && e2 <= upe; tries--) {
                            const V pw = tab[row + (uint32_t)e2], T = pw - pv + p2p;
                            if (T > B) nb = vmin<V>(nb, T);
                            else if (!mem_aware || lim_at(kind, f, e2) < e2) break;
                            pv = pw;
                            e2++;
                        }
                        fail |= e2 > upe;
                        if (!fail) ((uint8_t *)&colW[(u - 1) * 64])[1 - par] = (uint8_t)e2;   // u > 0: upe = L at u = 0
                    }
                    lu = fail ? 0 : lu;
                    e = i;
                    upe = up;
                }
            }
            // ---------------- what the sweep showed, and the next bound
            bool hard = false;
            if (state == kRun) {
                const bool pass = !fail && !redo;
                left--;
                const V lo_f = B == b_max ? INF : vmax<V>(nb, (V)(B + 1));   // every stage time is below b_max
                V lo_n = fail ? lo_f : lo, hi_n = pass && !last_probe ? mx : hi;
                const bool go_on = redo && !fail;                    // another sweep, from the values reached
                par = pass ? 1 - par : par;
                lo_n = pass && last_probe ? hi : lo_n;
                shc = 8 * (go_on ? 1 - par : par);
                const bool done = lo_n >= hi_n && !go_on;
                // the next bound: up by an eighth while no split is known, then halfway (just
                // below the first split's time when an earlier class's bound was tested)
                const V up = vmin<V>(vmax<V>(lo_n, (V)(B + (B >> 3))), b_max);
                const V mid = warm ? (V)(hi_n - 1) : (V)(lo_n + ((hi_n - lo_n) >> 1));
                const V bn = hi_n == INF ? up : mid;
                B = go_on ? B : bn;
                nb = go_on ? nb : INF;
                warm = warm && go_on;
                lo = lo_n;
                hi = hi_n;
                state = done ? kDone : kRun;
                hard = left < 0 && state == kRun;
                if (hard) {
                    state = kEmpty;
                    last_probe = false;
                }
            }
            const uint64_t hm = ballot(hard);
            if (hm) {
                // a search that takes its cuts up layer by layer: left to the split kernel,
                // without a split until then (Evaluate reads no layers of such a plan,
                // also when an overlapping call on this scratch loses the entry)
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(A.left, (uint32_t)__popcll(hm));
                at = (uint32_t)uni((int)at) + (uint32_t)lanes_below(hm);
                if (hard) {
                    if ((int64_t)at < A.n) A.left[kLeftHead + (size_t)at] = (uint32_t)t;
                    for (int k = 0; k < A.n_m; k++) A.status[t * A.n_m + k] = (uint8_t)HEDDLE_S_OOM;
                }
            }
        }
    }
}

// the LDS of a wavefront: the list of its slice and the stage columns
static size_t search_wave_bytes(int s_cap, bool lt)
{
    return (size_t)2 * kSearchSlice + (size_t)(lt ? 1 : 2) * (s_cap + 2) * 256;
}

template <class V, bool LT, int LIM>
static int launch_search_t(const heddle_profile *p, const PriceArgs &a, SearchArgs x, int waves, int blocks, size_t lds,
                           hipStream_t stream)
{
    if (lds > 65536)
        HEDDLE_HIP(hipFuncSetAttribute((const void *)search_kernel<V, LT, LIM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((search_kernel<V, LT, LIM>), dim3(blocks), dim3(64 * waves), lds, stream, p->dev, a, x);
    HEDDLE_HIP(hipGetLastError());
    return HEDDLE_OK;
}

template <class V>
static int launch_search_v(const heddle_profile *p, const PriceArgs &a, SearchArgs x, bool lt, int waves, int blocks, size_t lds,
                           hipStream_t stream)
{
    const int lim = (a.flags & HEDDLE_F_COMPUTE_ONLY) ? 0 : x.lim_words > 0 ? 1 : 2;
    if (!lt) return lim == 0 ? launch_search_t<V, false, 0>(p, a, x, waves, blocks, lds, stream)
                             : launch_search_t<V, false, 2>(p, a, x, waves, blocks, lds, stream);
    return lim == 0 ? launch_search_t<V, true, 0>(p, a, x, waves, blocks, lds, stream)
         : lim == 1 ? launch_search_t<V, true, 1>(p, a, x, waves, blocks, lds, stream)
                    : launch_search_t<V, true, 2>(p, a, x, waves, blocks, lds, stream);
}

bool place_search(const DevProfile &d, const PriceArgs &a, bool narrow, int max_lds, int lds_cu, int cus, SearchPlan &pl)
{
    std::memset(&pl, 0, sizeof(pl));
    SearchArgs &x = pl.x;
    x.s_cap = a.s_max < d.L ? a.s_max : d.L;
    const size_t tab = narrow ? (size_t)d.search_bytes32 : (size_t)d.search_bytes64;
    x.words = (a.s_max & 3) == 0 && ((uintptr_t)a.layers & 3) == 0;
    // tables in LDS while they leave room for wavefronts; kinds are bytes there
    constexpr size_t kRoom = 4;
    x.n_kinds = d.n_types * d.n_tp * d.n_ep;
    const size_t kind_bytes = (size_t)x.n_kinds * 16;
    const bool lt = x.n_kinds <= 256 && 256 + tab + kind_bytes + kRoom * search_wave_bytes(x.s_cap, true) <= (size_t)max_lds;
    pl.lt = lt;
    x.kind_off = lt ? (int32_t)tab : 0;
    x.copy_bytes = lt ? (int32_t)tab : 0;
    x.tab_bytes = 256 + (lt ? (int32_t)(tab + kind_bytes) : 0);
    x.degrees = d.n_tp * d.n_ep;
    x.vec_rec = (a.s_max & 3) == 0 && ((uintptr_t)a.stages & 15) == 0;
    x.vec_lay = (a.s_max & 15) == 0 && ((uintptr_t)a.layers & 15) == 0;
    x.wave_bytes = (int32_t)search_wave_bytes(x.s_cap, lt);
    // the memory limits too, when they fit a third of it and leave the same room
    // beside the tables
    x.lim_f = d.n_f < x.s_cap || !lt ? d.n_f : x.s_cap;
    x.lim_rows = x.n_kinds * x.lim_f;
    const int lim_words = ((d.L + 4) >> 2) | 1;                // odd: rows spread over the banks
    const size_t lim = ((size_t)x.lim_rows * lim_words * 4 + 15) & ~size_t(15);
    if (lt && !(a.flags & HEDDLE_F_COMPUTE_ONLY) && lim <= 56 * 1024 &&
        (size_t)x.tab_bytes + lim + kRoom * x.wave_bytes <= (size_t)max_lds) {
        x.lim_words = lim_words;
        x.lim_bytes = (int32_t)lim;
    } else {
        x.lim_f = d.n_f;
    }
    // wavefronts per workgroup (the registers allow 16 per CU at the most): the count that puts most wavefronts on a CU
    int waves = 1, wgs = 0;
    const int cap = 16;
    for (int w = 1; w <= 16; w++) {
        const size_t lds = (size_t)x.tab_bytes + x.lim_bytes + (size_t)w * x.wave_bytes;
        if (lds > (size_t)max_lds) break;
        int fit = (int)((size_t)lds_cu / ((lds + 511) & ~size_t(511)));
        fit = fit < cap / w ? fit : cap / w;
        if (fit * w > wgs * waves || wgs == 0) {
            wgs = fit;
            waves = w;
        }
    }
    if (wgs == 0 || cus < 1) return false;
    const int per_cu = wgs * waves;
    // every wavefront one slice, or as few equal ones as fit its list
    const int64_t slots = (int64_t)cus * per_cu;
    const int64_t rounds = (a.n + slots * kSearchSlice - 1) / (slots * kSearchSlice);
    x.slice = (int32_t)((a.n + slots * rounds - 1) / (slots * rounds));
    // new templates once 24 lanes are idle (16 and 32 are level within 2%); a template is left
    // to the split kernel after so many sweeps, where the lanes that wait for it cost more
    // than its recurrence: c3 (16 stages) 470 us a call at 12, 490 at 18, 560 at 30, c5 (32
    // stages, 300,000 templates) 3.4 ms at 12, 3.0 at 18, 3.3 at 24. By the template's own
    // stages: c2 in 64 stage slots 161 us at 12, 183 at 18 (131,072 templates; 138 with the
    // recurrence); but 18 for all templates of up to 32 stages with 64-bit costs, whose
    // recurrence is dearer (c5's at a micro-batch of 8: 897 us, 922 by their own)
    x.refill = 24;
    x.walk = 4;
    x.sweeps = 18;
    x.sweeps_short = narrow || x.s_cap <= 16 ? 12 : 18;
    const int64_t n_slices = (a.n + x.slice - 1) / x.slice;
    int64_t blocks = (n_slices + waves - 1) / waves;
    const int64_t most = (int64_t)cus * wgs;
    if (blocks > most) blocks = most;
    // a CU's share of LDS each, so that no CU takes more workgroups than another: they are
    // resident all at once, and the one that takes longest ends the launch
    size_t lds = ((size_t)lds_cu / wgs) & ~size_t(511);
    pl.lds = lds < (size_t)max_lds ? lds : (size_t)max_lds;
    pl.waves = waves;
    pl.per_cu = per_cu;
    pl.blocks = (int)blocks;
    return true;
}

int launch_search(const heddle_profile *p, const PriceArgs &a, const SearchPlan &pl, bool narrow, hipStream_t stream)
{
    return narrow ? launch_search_v<uint32_t>(p, a, pl.x, pl.lt, pl.waves, pl.blocks, pl.lds, stream)
                  : launch_search_v<uint64_t>(p, a, pl.x, pl.lt, pl.waves, pl.blocks, pl.lds, stream);
}

}  // namespace heddle
