// Runs the window pass and the split search on the CPU: the fibers behind
// hip/hip_runtime.h, and the calls that the tests make (cpu_lanes.py).
#include <sys/mman.h>
#include <ucontext.h>

#include <map>
#include <string>
#include <vector>

#include "profile.cpp"
#include "windows.hip"
#include "search.hip"
#include "evaluate.hip"

namespace heddle {
constexpr size_t kLds = 160 * 1024, kLdsTail = 16 * 1024;
alignas(16) unsigned char smem[kLds + kLdsTail];               // dynamic LDS of the workgroup that runs
bool tile_narrow(const heddle_profile *) { return false; }     // of the tile kernel, which is not compiled here
}  // namespace heddle

namespace lanes {

dim3 thread_idx, block_idx, block_dim, grid_dim;
int cus = 1, max_lds = heddle::kLds;
static std::string first_broken;
static int n_broken;

void broken(const char *what, const char *file, int line)
{
    if (n_broken++ == 0) first_broken = std::string(what) + " (" + file + ":" + std::to_string(line) + ")";
}

static std::map<void *, std::pair<void *, size_t>> blocks;

void *device_alloc(size_t bytes)
{
    const size_t page = 4096, body = (bytes + page - 1) / page * page;
    char *m = (char *)mmap(nullptr, body + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (m == MAP_FAILED) abort();
    mprotect(m, page, PROT_NONE);
    mprotect(m + page + body, page, PROT_NONE);
    char *p = m + page + (body - bytes) / 256 * 256;           // the end near the second page
    memset(m + page, 0xA5, body);
    blocks[p] = {m, body + 2 * page};
    return p;
}

void device_free(void *p)
{
    auto it = blocks.find(p);
    if (it == blocks.end()) return;
    munmap(it->second.first, it->second.second);
    blocks.erase(it);
}

struct Wave {
    uint64_t buf[2][64], there[2];
    uint64_t epoch;
    int arrived, alive;
};
struct Fiber {
    ucontext_t ctx;
    bool done;
};
constexpr size_t kStack = 128 * 1024;
static std::vector<Fiber> fibers;
static std::vector<Wave> waves;
static char *stacks;
static ucontext_t main_ctx;
static int cur, block_alive, block_arrived;
static uint64_t block_epoch, progress;
static const std::function<void()> *body;
static std::function<void()> meanwhile;                        // work of another call, now and then

static void yield()
{
    const int me = cur;
    swapcontext(&fibers[me].ctx, &main_ctx);
}

const uint64_t *exchange(uint64_t v, uint64_t *present)
{
    const int l = lane();
    Wave &w = waves[cur >> 6];
    const uint64_t e = w.epoch;
    const int par = e & 1;
    if (meanwhile && progress % 997 == 0) meanwhile();
    w.buf[par][l] = v;
    w.there[par] |= uint64_t(1) << l;
    progress++;
    if (++w.arrived == w.alive) {
        w.arrived = 0;
        w.there[par ^ 1] = 0;
        w.epoch++;
    } else {
        while (w.epoch == e) yield();
    }
    *present = w.there[par];
    return w.buf[par];
}

void sync_block()
{
    const uint64_t e = block_epoch;
    progress++;
    if (++block_arrived == block_alive) {
        block_arrived = 0;
        block_epoch++;
    } else {
        while (block_epoch == e) yield();
    }
}

static void fiber_main()
{
    (*body)();
    Wave &w = waves[cur >> 6];
    fibers[cur].done = true;
    progress++;
    if (--w.alive && w.arrived == w.alive) {
        w.arrived = 0;
        w.there[(w.epoch & 1) ^ 1] = 0;
        w.epoch++;
    }
    if (--block_alive && block_arrived == block_alive) {
        block_arrived = 0;
        block_epoch++;
    }
    setcontext(&main_ctx);
}

void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()> &kernel)
{
    if (lds > (size_t)max_lds || block.x > 1024 || block.x % 64) abort();
    const int nt = (int)block.x;
    if (!stacks) stacks = (char *)mmap(nullptr, 1024 * kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    body = &kernel;
    grid_dim = grid;
    block_dim = block;
    for (unsigned b = 0; b < grid.x; b++) {
        block_idx = dim3(b);
        memset(heddle::smem, 0xA5, sizeof(heddle::smem));
        fibers.assign(nt, Fiber());
        waves.assign(nt / 64, Wave());
        for (auto &w : waves) w.alive = 64;
        block_alive = nt;
        block_arrived = 0;
        block_epoch = 0;
        for (int i = 0; i < nt; i++) {
            getcontext(&fibers[i].ctx);
            fibers[i].ctx.uc_stack.ss_sp = stacks + (size_t)i * kStack;
            fibers[i].ctx.uc_stack.ss_size = kStack;
            fibers[i].ctx.uc_link = nullptr;
            makecontext(&fibers[i].ctx, fiber_main, 0);
        }
        while (block_alive) {
            const uint64_t before = progress;
            for (int i = 0; i < nt; i++) {
                if (fibers[i].done) continue;
                cur = i;
                thread_idx = dim3(i);
                swapcontext(&main_ctx, &fibers[i].ctx);
            }
            if (progress == before) {
                fprintf(stderr, "lanes wait for one another for ever\n");
                abort();
            }
        }
        for (size_t i = lds; i < sizeof(heddle::smem); i++)
            if (heddle::smem[i] != 0xA5) { broken("LDS written past the launch's size", __FILE__, __LINE__); break; }
    }
}

}  // namespace lanes

using namespace heddle;

struct SplitRun {
    int32_t cus, max_lds;            // in: the device
    int32_t preset_on;               // in: another call writes `preset` where the list's length is kept,
    uint32_t preset;                 //     after the window pass
    float need, need_slow;           // in: counted templates from which the search runs
    int32_t sweeps;                  // in: not 0: sweeps after which a template is left
    int32_t other;                   // in: not 0: the seed of another call's window pass over the same scratch
    int32_t placed, lt, lim, per_cu; // out: the search fits; tables, memory limits in LDS; wavefronts on a CU
    int32_t n_broken;
    char broken[256];
};

// window pass and split search; outputs of the templates that the search left
// are what it leaves there. left: their number, then their indices
extern "C" int lanes_split(const heddle_profile *p, int64_t n, int32_t s_max, const uint8_t *n_stages, const uint32_t *stages,
                           const int32_t *m, int32_t n_m, uint32_t flags, void *bottleneck, uint8_t *layers, uint8_t *status,
                           uint32_t *left, SplitRun *r)
{
    lanes::cus = r->cus;
    lanes::max_lds = r->max_lds;
    lanes::n_broken = 0;
    std::vector<void *> mem;
    auto dev = [&](size_t bytes, const void *from = nullptr) {
        void *q = lanes::device_alloc(bytes);
        if (from) memcpy(q, from, bytes);
        mem.push_back(q);
        return q;
    };
    const bool f32 = flags & HEDDLE_F_FP32, narrow = f32 ? p->narrow_f32 : p->narrow_i64;
    const size_t plans = (size_t)n * n_m, t = f32 ? 4 : 8;
    PriceArgs a;
    memset(&a, 0, sizeof(a));
    a.n = n;
    a.s_max = s_max;
    a.n_m = n_m;
    a.flags = (int32_t)flags;
    for (int k = 0; k < n_m; k++) a.m[k] = m[k];
    a.n_stages = (const uint8_t *)dev(n, n_stages);
    a.stages = (const uint32_t *)dev((size_t)n * s_max * 4, stages);
    a.iter = dev(plans * t);
    a.bottleneck = dev(plans * t);
    a.peak_mem = (int64_t *)dev(plans * 8);
    a.layers = (uint8_t *)dev(plans * s_max);
    a.status = (uint8_t *)dev(plans);
    a.wst = (uint32_t *)dev(plans * 4);
    a.wwin = (uint16_t *)dev(plans * win_stride(s_max) * 2);
    a.left = (uint32_t *)dev(left_bytes(n));
    a.need = r->need;
    a.need_slow = r->need_slow;
    a.p2p_share = p->p2p_share;
    SearchPlan pl;
    const auto limit = [&](int s) { return r->sweeps ? r->sweeps : s; };
    r->placed = place_search(p->dev, a, narrow, lanes::max_lds, lanes::max_lds, lanes::cus, pl);
    pl.x.sweeps = limit(pl.x.sweeps);
    pl.x.sweeps_short = limit(pl.x.sweeps_short);
    r->lt = pl.lt;
    r->lim = pl.x.lim_words > 0;
    r->per_cu = pl.per_cu;
    size_t lds = 0;
    int rc = r->placed ? 0 : HEDDLE_E_RANGE;
    if (!rc) rc = prepare_windows(p, a, lanes::max_lds, &lds);
    if (!rc) rc = launch_windows(p, a, lds, nullptr);
    if (!rc && r->preset_on) a.left[0] = r->preset;
    if (!rc && r->other) {
        auto draw = [x = (uint64_t)(uint32_t)r->other]() mutable { return (uint32_t)((x = x * 6364136223846793005ull + 1442695040888963407ull) >> 33); };
        lanes::meanwhile = [=]() mutable {
            for (size_t o = 0; o < plans; o++) a.wst[o] = (draw() % 10 < 7 ? 0u : draw() % 9) | draw() << 8;
            for (size_t o = 0; o < plans * win_stride(s_max); o++) a.wwin[o] = (uint16_t)draw();
        };
        lanes::meanwhile();
    }
    if (!rc) rc = launch_search(p, a, pl, narrow, nullptr);
    lanes::meanwhile = nullptr;
    memcpy(bottleneck, a.bottleneck, plans * t);
    memcpy(layers, a.layers, plans * s_max);
    memcpy(status, a.status, plans);
    memcpy(left, a.left, left_bytes(n));
    r->n_broken = lanes::n_broken;
    snprintf(r->broken, sizeof(r->broken), "%s", lanes::n_broken ? lanes::first_broken.c_str() : "");
    for (void *q : mem) lanes::device_free(q);
    return rc;
}

// Evaluate over given splits: iter, peak memory and status
extern "C" int lanes_evaluate(const heddle_profile *p, int64_t n, int32_t s_max, const uint8_t *n_stages, const uint32_t *stages,
                              const int32_t *m, int32_t n_m, uint32_t flags, const void *bottleneck, const uint8_t *layers,
                              uint8_t *status, void *iter, int64_t *peak_mem, SplitRun *r)
{
    lanes::cus = r->cus;
    lanes::max_lds = r->max_lds;
    lanes::n_broken = 0;
    PriceArgs a;
    memset(&a, 0, sizeof(a));
    a.n = n;
    a.s_max = s_max;
    a.n_m = n_m;
    a.flags = (int32_t)flags;
    for (int k = 0; k < n_m; k++) a.m[k] = m[k];
    a.n_stages = n_stages;
    a.stages = stages;
    a.bottleneck = (void *)bottleneck;
    a.layers = (uint8_t *)layers;
    a.status = status;
    a.iter = iter;
    a.peak_mem = peak_mem;
    const int rc = launch_evaluate(p, a, nullptr);
    r->n_broken = lanes::n_broken;
    snprintf(r->broken, sizeof(r->broken), "%s", lanes::n_broken ? lanes::first_broken.c_str() : "");
    return rc;
}

// the template of the split kernel's turn i over the list, or n
extern "C" int64_t lanes_left_template(const uint32_t *left, int64_t i, int64_t n) { return left_template(left, i, n); }
