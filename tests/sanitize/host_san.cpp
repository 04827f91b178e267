// Host logic of the library (pool bookkeeping, scheduler, buffer recycling, argument checks)
// under AddressSanitizer / UndefinedBehaviorSanitizer, on the CPU only.
//
// pool.cpp and plan.cpp are compiled unchanged.  This file supplies (1) a stand-in for the few
// HIP runtime calls they make - "device" memory is host heap, copies are memcpy, events are
// always complete - and (2) stand-ins for the kernel launchers that do not compute anything
// but CHECK what the kernels assume about their work lists and touch every byte of scratch the
// kernels would touch, so that a list entry out of range or an undersized buffer is reported by
// the sanitizer or by an explicit check.  Then a seeded random sequence of API calls runs, or, named
// on the command line, one of the directed cases.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <utility>
#include <vector>

#include "slora_internal.hpp"

#define REQUIRE(c)                                                          \
    do {                                                                    \
        if (!(c)) {                                                         \
            std::fprintf(stderr, "host_san: %s failed at line %d\n", #c, __LINE__); \
            std::abort();                                                   \
        }                                                                   \
    } while (0)

// ---------------------------------------------------------------------------------------------
// stand-in HIP runtime
// ---------------------------------------------------------------------------------------------
static long g_device_mallocs = 0;  // hipMalloc calls so far
static bool g_fail_malloc = false; // hipMalloc is out of memory
static size_t g_free_bytes = SIZE_MAX; // ... for a request of more than this
static long g_clears = 0;          // launches that clear memory so far
static bool g_captures = false;    // a HIP graph captures every stream but the default one

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipMalloc(void **p, size_t n)
{
    g_device_mallocs++;
    *p = g_fail_malloc || n > g_free_bytes ? nullptr : std::malloc(n ? n : 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n ? n : 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free((void *)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = g_captures ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeHost;
    a->devicePointer = const_cast<void *>(p);
    a->hostPointer = const_cast<void *>(p);
    return hipSuccess;
}
}

// ---------------------------------------------------------------------------------------------
// stand-in launchers: check the lists, touch the scratch
// ---------------------------------------------------------------------------------------------
namespace slora {

static std::vector<unsigned char> g_static_scratch; // exactly the size the library believes it has

int32_t static_scratch_address(int, void **out)
{
    if (g_static_scratch.empty()) g_static_scratch.resize(SLORA_STATIC_SCRATCH_BYTES);
    *out = g_static_scratch.data();
    return SLORA_OK;
}

int32_t launch_write_pages(slora_pool *pool, const int32_t *d_idx, int64_t n, const void *d_src, void *, int32_t)
{
    for (int64_t i = 0; i < n; ++i) {
        REQUIRE(d_idx[i] >= 0 && d_idx[i] < pool->n_pages);
        std::memcpy(static_cast<uint16_t *>(pool->dev_base) + (int64_t)d_idx[i] * pool->H,
                    static_cast<const uint16_t *>(d_src) + i * pool->H, (size_t)pool->H * 2);
    }
    return SLORA_OK;
}

int32_t launch_copy(void *dst, const void *src, size_t bytes, void *)
{
    REQUIRE(bytes > 0 && bytes % 16 == 0);
    std::memcpy(dst, src, bytes);
    return SLORA_OK;
}

int32_t launch_gather(slora_pool *pool, int64_t entry, int32_t rank, void *out, void *)
{
    for (int32_t j = 0; j < rank; ++j) {
        const int32_t p = pool->d_arena[entry + j];
        REQUIRE(p >= 0 && p < pool->n_pages);
        std::memcpy(static_cast<uint16_t *>(out) + (int64_t)j * pool->H,
                    static_cast<uint16_t *>(pool->dev_base) + (int64_t)p * pool->H, (size_t)pool->H * 2);
    }
    return SLORA_OK;
}

static int64_t g_seen; // consecutive items of an adapter: its list is checked once per launch

// every page number an item can reach through the device image of the arena
static void check_pages(const slora_plan *plan, int32_t arena_off, int32_t rank, int32_t slot)
{
    const slora_pool *pool = plan->pool;
    const int64_t key = (int64_t)arena_off * 64 + slot;
    if (key == g_seen) return;
    g_seen = key;
    REQUIRE(arena_off >= 0 && rank > 0);
    const int64_t first = arena_off + (int64_t)slot * 2 * rank;
    REQUIRE(first + 2 * rank <= pool->d_arena_cap);
    for (int32_t j = 0; j < 2 * rank; ++j) {
        const int32_t p = pool->d_arena[first + j];
        REQUIRE(p >= 0 && p < pool->n_pages);
        REQUIRE(pool->state[(size_t)p] == kAdapter);
    }
}

static void check_tokens(const slora_plan *plan, int32_t pos0, int32_t ntok)
{
    REQUIRE(pos0 >= 0 && ntok > 0 && pos0 + ntok <= plan->T_act);
    for (int32_t t = 0; t < ntok; ++t) {
        const int32_t tok = plan->d_tok_idx[pos0 + t];
        REQUIRE(tok >= 0 && tok < plan->T);
    }
}

// the v of all slots, in the layout of the route, lies inside the plan's buffer or the static scratch
static void check_scratch(const slora_plan *plan, int32_t n, const MultiArgs &a, const Route &route)
{
    const size_t floats = (size_t)plan->v_total_floats(n, plan->pool->dtype, plan->mfma_on(route));
    if (a.v[0] == plan->set->v)
        REQUIRE(floats <= plan->set->v_cap);
    else if (a.v[0] == (float *)g_static_scratch.data())
        REQUIRE(floats * sizeof(float) <= SLORA_STATIC_SCRATCH_BYTES);
    for (int32_t k = 1; k < n; ++k) REQUIRE(a.v[k] - a.v[0] == k * plan->v_slot_floats(plan->pool->dtype, plan->mfma_on(route)));
}

// Items of a vector kernel: of every position (token of an adapter) in them each of `units` ranks or columns once
struct Cover {
    const size_t row;
    std::vector<uint8_t> done;
    std::vector<int32_t> units, count; // of a position: how many there are (0: not in an item yet), how many are done
    Cover(int32_t positions, size_t most) : row(most), done((size_t)positions * most), units((size_t)positions), count((size_t)positions) {}
    void add(const Item &it, int32_t of, int32_t lo, int32_t hi)
    {
        for (int32_t p = it.pos0; p < it.pos0 + it.ntok; ++p) {
            REQUIRE(units[(size_t)p] == 0 || units[(size_t)p] == of);
            units[(size_t)p] = of;
            for (int32_t u = lo; u < hi; ++u) REQUIRE(!done[(size_t)p * row + (size_t)u]++);
            count[(size_t)p] += hi - lo;
        }
    }
    // every position is in the vector items, whole, or served elsewhere
    void check(const std::vector<uint8_t> &elsewhere) const
    {
        for (size_t p = 0; p < units.size(); ++p) {
            REQUIRE((units[p] != 0) != (elsewhere[p] != 0));
            REQUIRE(count[p] == units[p]);
        }
    }
};

// positions that the MFMA kernels or the one-launch decode kernel serve
static std::vector<uint8_t> served_elsewhere(const slora_plan *plan, const Route &route)
{
    std::vector<uint8_t> out((size_t)plan->T_act);
    for (size_t i = 0; plan->mfma_on(route) && i < plan->ms_items.size(); ++i)
        for (int32_t t = 0; t < plan->ms_items[i].ntok; ++t) out[(size_t)(plan->ms_items[i].pos0 + t)] = 1;
    for (size_t i = 0; route.fused && i < plan->vf_items.size(); ++i)
        for (int32_t t = 0; t < plan->vf_items[i].ntok; ++t) out[(size_t)(plan->vf_items[i].pos0 + t)] = 1;
    return out;
}

// what the latest apply, shrink or expand launched
struct Log {
    bool small = false, chain = false; // both vector stages in one launch: every workgroup computes v for itself; v is handed over
    bool fused = false, mfma_shrink = false, mfma_expand = false;
    bool wide = false, gang = false, gang_expand = false; // the larger items of the vector kernels
    size_t vec_shrink = 0, vec_expand = 0; // items
    size_t mfma_shrink_wgs = 0, mfma_expand_wgs = 0; // workgroups with work
};
static Log g_log;
static std::map<const slora_plan *, bool> g_wide; // whether the latest shrink of a plan left v in the MFMA layout of a dual plan
static volatile float g_sink; // reads of the stand-in kernels end here

// Items of the vector shrink of a call; words: of a launch that hands v over, how often each was left
static void vec_shrink(const slora_plan *plan, const MultiArgs &a, int32_t k, const Route &route, std::vector<uint8_t> *words)
{
    const slora_pool *pool = plan->pool;
    const size_t n_vs = plan->n_vs(route);
    const bool gang = n_vs > 0 && route.gang; // the larger items, then the small ones of the groups that are not in them
    REQUIRE(0 <= plan->n_gs_plain && (size_t)plan->n_gs_plain <= plan->gs_items.size());
    const size_t n_gs = gang ? plan->n_gs(route) : 0, n_vec = gang ? n_gs + plan->gv_items.size() : n_vs;
    REQUIRE(n_vec == plan->shrink_wgs(route));
    const std::vector<uint8_t> elsewhere = served_elsewhere(plan, route);
    float *v = a.v[k];
    Cover cover(plan->T_act, (size_t)plan->v_stride);
    for (size_t i = 0; i < n_vec; ++i) {
        const bool large = i < n_gs;
        const Item &it = large ? plan->d_gs[i] : gang ? plan->d_gv[i - n_gs] : plan->d_vs[i];
        REQUIRE(std::memcmp(&it, large ? &plan->gs_items[i] : gang ? &plan->gv_items[i - n_gs] : &plan->vs_items[i], sizeof it) == 0);
        check_pages(plan, it.arena_off, it.rank, a.slot[k]);
        check_tokens(plan, it.pos0, it.ntok);
        REQUIRE(it.a >= 0 && it.b > 0 && it.a + it.b <= it.rank);
        if (large) {
            REQUIRE(it.ntok <= kGangTok && it.b <= kGangPages && pool->shrink_pages == 0);
        } else { // its rows of x fit the LDS of the launch
            REQUIRE(it.ntok <= kShrinkTok && it.ntok <= (gang ? plan->max_gv_tok : plan->max_shrink_tok) && it.b <= (pool->shrink_pages > 0 ? pool->shrink_pages : kShrinkPages));
            REQUIRE(it.ntok == 1 || it.ntok * pool->H * 2 <= 65536);
            REQUIRE(!words || it.ntok <= plan->chain_of(route).tok);
        }
        cover.add(it, it.rank, it.a, it.a + it.b);
        for (int32_t t = 0; t < it.ntok; ++t)
            for (int32_t j = it.a; j < it.a + it.b; ++j) {
                v[(int64_t)(it.pos0 + t) * plan->v_stride + j] = 0.f;
                if (words) { // every word is left once
                    const int64_t w = it.run + (int64_t)t * it.rank + j;
                    REQUIRE(w >= 0 && w < plan->chain_of(route).words && !(*words)[(size_t)w]++);
                }
            }
    }
    cover.check(elsewhere);
}

// ... of the vector expand
static void vec_expand(const slora_plan *plan, const MultiArgs &a, int32_t k, const Route &route, const std::vector<uint8_t> *words)
{
    const slora_pool *pool = plan->pool;
    const size_t n_ve = plan->n_ve(route);
    const bool gang = n_ve > 0 && route.gang_expand;
    REQUIRE(!gang || plan->expand_split);
    REQUIRE(0 <= plan->n_ge_plain && (size_t)plan->n_ge_plain <= plan->ge_items.size());
    const size_t n_vec = gang ? plan->n_ge(route) : n_ve;
    REQUIRE(n_vec == plan->expand_wgs(route));
    const std::vector<uint8_t> elsewhere = served_elsewhere(plan, route);
    Cover cover(plan->T_act, (size_t)pool->H / 8);
    std::map<std::pair<int32_t, int32_t>, int> readers; // of the B rows of an adapter in a column range
    for (size_t i = 0; i < n_vec; ++i) readers[{(gang ? plan->d_ge : plan->d_ve)[i].arena_off, (gang ? plan->d_ge : plan->d_ve)[i].a}]++;
    for (size_t i = 0; i < n_vec; ++i) {
        const Item &it = gang ? plan->d_ge[i] : plan->d_ve[i];
        REQUIRE(std::memcmp(&it, gang ? &plan->ge_items[i] : &plan->ve_items[i], sizeof it) == 0);
        check_pages(plan, it.arena_off, it.rank, a.slot[k]);
        check_tokens(plan, it.pos0, it.ntok);
        REQUIRE(it.ntok <= (!gang ? kExpandTok : it.rank <= kOwnRanks ? kGangOwnTok : kGangExpandTok));
        for (int y16 = 0; gang && y16 < 2; ++y16) REQUIRE(plan->fours[y16] || !fours_pay(pool->dtype, y16, it.rank, it.ntok)); // the kernel instance has the code for it
        REQUIRE(it.a >= 0 && it.b > 0 && it.a % 8 == 0 && it.b % 8 == 0 && it.a + it.b <= pool->H);
        REQUIRE(it.b <= (plan->expand_split ? 512 : plan->expand_threads * 8));
        const int read_by = readers[std::make_pair(it.arena_off, it.a)];
        REQUIRE(it.tile == 0 || (it.tile == 1 && read_by == 1)); // streamed: read by this item only
        REQUIRE(it.tile == 1 || it.ntok > 2 || read_by > 1);
        cover.add(it, pool->H / 8, it.a / 8, (it.a + it.b) / 8);
        for (int32_t t = 0; t < it.ntok; ++t)
            for (int32_t j = 0; j < it.rank; j += words ? 1 : 16) {
                if (words) { // a word that is waited for is left
                    const int64_t w = it.run + (int64_t)t * it.rank + j;
                    REQUIRE(w >= 0 && w < plan->chain_of(route).words && (*words)[(size_t)w] == 1);
                } else {
                    g_sink = a.v[k][(int64_t)(it.pos0 + t) * plan->v_stride + j];
                }
            }
    }
    cover.check(elsewhere);
}

int32_t launch_clear(void *dst, size_t bytes, void *)
{
    REQUIRE(bytes > 0 && bytes % 16 == 0);
    g_clears++;
    std::memset(dst, 0, bytes);
    return SLORA_OK;
}

// both vector stages in one launch: the small items of both lists, v through the words of the plan's buffer set
int32_t launch_chain(slora_plan *plan, int32_t n, const MultiArgs &a, void *, bool y16, const Route &route)
{
    REQUIRE(a.n == n && route.chain && !route.small && !route.gang && !route.gang_expand && plan->expand_split);
    REQUIRE(plan->pool->H <= kChainMaxH && plan->pool->fuse_decode != 0 && plan->chain_wgs(route) <= 65535);
    const int64_t words_per_slot = plan->chain_of(route).words;
    REQUIRE(plan->set->launch > 0 && (size_t)(words_per_slot * n) <= plan->set->hand_cap);
    REQUIRE(plan->set->hand == (uint64_t *)(plan->set->v + plan->set->v_cap)); // behind every v
    for (size_t w = 0; w < plan->set->hand_cap; ++w) REQUIRE((uint32_t)(plan->set->hand[w] >> 32) != plan->set->launch); // a number of its own
    for (int32_t k = 0; k < n; ++k) {
        REQUIRE(a.x[k] && a.y[k] && a.v[k]);
        g_seen = -1;
        std::vector<uint8_t> words((size_t)words_per_slot);
        vec_shrink(plan, a, k, route, &words);
        g_seen = -1;
        vec_expand(plan, a, k, route, &words);
        for (size_t w = 0; w < words.size(); ++w)
            plan->set->hand[(size_t)(k * words_per_slot) + w] = (uint64_t)plan->set->launch << 32;
        for (uint8_t w : words) REQUIRE(w == 1); // no room for more
    }
    g_log.chain = true;
    g_log.vec_shrink = plan->n_vs(route);
    g_log.vec_expand = plan->n_ve(route);
    g_wide[plan] = route.wide;
    return SLORA_OK;
}

int32_t launch_shrink(slora_plan *plan, int32_t n, const MultiArgs &a, void *, const Route &route)
{
    const slora_pool *pool = plan->pool;
    const int32_t np = plan->pieces(pool->dtype);
    const int n_gran = (pool->H + kMsGranule - 1) / kMsGranule;
    const int n_kk = plan->v_stride / 16;
    REQUIRE(a.n == n && plan->v_stride % kRankPad == 0);
    REQUIRE(0 <= plan->n_vs_plain && plan->n_vs_plain <= plan->n_vs_head && (size_t)plan->n_vs_head <= plan->vs_items.size());
    g_seen = -1;
    check_scratch(plan, n, a, route);
    if (!route.chain) g_log.vec_shrink = plan->n_vs(route);
    g_log.wide = route.wide;
    g_log.gang = !route.chain && plan->n_vs(route) > 0 && route.gang;
    g_wide[plan] = route.wide;
    g_log.mfma_shrink = plan->mfma_on(route) && !plan->ms_items.empty();
    for (int32_t k = 0; k < n; ++k) {
        REQUIRE(a.x[k] && a.v[k]);
        float *v = a.v[k];
        if (!route.chain) vec_shrink(plan, a, k, route, nullptr);
        uint16_t *frag = reinterpret_cast<uint16_t *>(v + a.vfrag_off);
        int8_t *vexp = reinterpret_cast<int8_t *>(v + a.vexp_off);
        float *part = v + a.part_off;
        for (size_t i = 0; plan->mfma_on(route) && i < plan->ms_items.size(); ++i) {
            const MsItem &it = plan->d_ms[i];
            REQUIRE(std::memcmp(&it, &plan->ms_items[i], sizeof it) == 0);
            check_pages(plan, it.arena_off, it.rank, a.slot[k]);
            check_tokens(plan, it.pos0, it.ntok);
            REQUIRE(it.ntok <= kMsTok && it.nj > 0 && it.nj <= kMsRanks && it.j0 % kMsRanks == 0 && it.j0 + it.nj <= it.rank);
            REQUIRE(it.c0 >= 0 && it.c0 < it.c1 && it.c1 <= n_gran && it.part >= 0 && it.part < it.n_parts);
            const int mb = (it.ntok + 31) / 32, nb = (it.nj + 31) / 32;
            const int sub_tok = kMsTok >> route.sub;
            for (int p = 0; p < it.ntok; p += sub_tok) { // one workgroup each: its ring must fit
                const int rows = std::min(sub_tok, it.ntok - p);
                g_log.mfma_shrink_wgs++;
                REQUIRE(ms_lds_bytes((rows <= 32 ? 1 : rows <= 64 ? 2 : 4) + nb) <= plan->ms_lds[route.sub] && plan->ms_lds[route.sub] <= 80 * 1024);
            }
            REQUIRE(it.tile >= 0 && it.tile + mb <= plan->n_mfma_tiles);
            REQUIRE((it.sync >= 0) == (it.n_parts > 1 || plan->dual));
            if (it.sync >= 0) {
                REQUIRE(it.sync >= 0 && it.sync < plan->n_sync);
                REQUIRE(it.part_off >= 0 && it.part_off + (int64_t)it.n_parts * mb * nb * 1024 <= plan->part_floats);
                std::memset(part + it.part_off + (int64_t)it.part * mb * nb * 1024, 0, (size_t)mb * nb * 1024 * sizeof(float));
            }
            if (it.n_parts == 1 || it.part == it.n_parts - 1) { // the finished tile: fragments and exponents
                for (int w = 0; w < mb; ++w) {
                    for (int b = 0; b < nb; ++b)
                        for (int i2 = 0; i2 < 2; ++i2) {
                            const int kk = it.j0 / 16 + 2 * b + i2;
                            if (kk < n_kk)
                                std::memset(frag + (((int64_t)(it.tile + w) * n_kk + kk) * np) * 512, 0, (size_t)np * 1024);
                        }
                    std::memset(vexp + ((int64_t)(it.tile + w) * plan->n_rank_blocks + it.j0 / kMsRanks) * 32, 0, 32);
                }
            }
        }
        for (size_t i = 0; i < plan->mj_items.size(); ++i)
            REQUIRE(std::memcmp(&plan->d_mj[i], &plan->mj_items[i], sizeof(MsItem)) == 0);
    }
    return SLORA_OK;
}

int32_t launch_expand(slora_plan *plan, int32_t n, const MultiArgs &a, void *, bool, const Route &route)
{
    const slora_pool *pool = plan->pool;
    REQUIRE(a.n == n);
    REQUIRE(0 <= plan->n_ve_plain && plan->n_ve_plain <= plan->n_ve_head && (size_t)plan->n_ve_head <= plan->ve_items.size());
    g_seen = -1;
    check_scratch(plan, n, a, route);
    if (!route.chain) g_log.vec_expand = plan->n_ve(route);
    g_log.gang_expand = !route.chain && plan->n_ve(route) > 0 && route.gang_expand;
    REQUIRE(g_wide.count(plan) && g_wide[plan] == route.wide);
    g_log.mfma_expand = plan->mfma_on(route) && !plan->me_items.empty();
    const int n_kk = plan->v_stride / 16, np = plan->pieces(pool->dtype);
    for (int32_t k = 0; k < n; ++k) {
        REQUIRE(a.y[k] && a.v[k]);
        if (!route.chain) vec_expand(plan, a, k, route, nullptr);
        std::set<std::pair<int, int>> done; // every tile and column range is in one run
        for (size_t i = 0; plan->mfma_on(route) && i < plan->me_items.size(); ++i) {
            const Item &it = plan->d_me[i];
            REQUIRE(std::memcmp(&it, &plan->me_items[i], sizeof it) == 0);
            check_pages(plan, it.arena_off, it.rank, a.slot[k]);
            REQUIRE(it.a >= 0 && it.b > 0 && it.b <= kMfmaExpandCols && it.a % kMfmaExpandCols == 0 && it.a + it.b <= pool->H);
            const int tiles = it.run & 0xff, last = it.run >> 8; // a run: whole tiles, then one of `last` tokens
            g_log.mfma_expand_wgs += (size_t)std::min(tiles, route.parts);
            REQUIRE(tiles >= 1 && tiles <= plan->me_run && tiles <= kMfmaRunMax && last >= 1 && last <= kMfmaTok && it.ntok == (tiles == 1 ? last : kMfmaTok));
            check_tokens(plan, it.pos0, (tiles - 1) * kMfmaTok + last);
            REQUIRE(it.tile >= 0 && it.tile + tiles <= plan->n_mfma_tiles);
            const unsigned char *frag = reinterpret_cast<const unsigned char *>(a.v[k] + a.vfrag_off);
            const int8_t *vexp = reinterpret_cast<const int8_t *>(a.v[k] + a.vexp_off);
            for (int t = it.tile; t < it.tile + tiles; ++t) {
                REQUIRE(done.insert({t, it.a}).second);
                for (int kk = 0; kk < (it.rank + 31) / 32 * 2; ++kk)
                    for (int b = 0; b < np * 1024; b += 64) g_sink = frag[((int64_t)t * n_kk + kk) * np * 1024 + b];
                for (int b = 0; b < 32 * plan->n_rank_blocks; ++b) g_sink = vexp[(int64_t)t * plan->n_rank_blocks * 32 + b];
            }
        }
        int stages = 0; // an LDS buffer of V is as large as its widest user needs, see expand_mfma_kernel
        for (const Item &it : plan->me_items)
            if (it.rank <= kMsRanks || (it.rank <= 2 * kMsRanks && !(np == 3 && pool->dtype == SLORA_F16)))
                stages = std::max(stages, (std::min(it.rank, kMsRanks) + 31) / 32);
        REQUIRE(plan->me_stages == stages);
        REQUIRE(!g_log.mfma_expand || (int64_t)done.size() == (int64_t)plan->n_mfma_tiles * ((pool->H + kMfmaExpandCols - 1) / kMfmaExpandCols));
    }
    return SLORA_OK;
}

int32_t launch_fused(slora_plan *plan, int32_t n, const MultiArgs &a, void *, bool, const Route &route)
{
    const slora_pool *pool = plan->pool;
    REQUIRE(a.n == n && pool->H <= 8192);
    if (route.small) { // the whole batch, from the items of the rank-split expand
        g_log.small = true;
        g_wide[plan] = false;
        REQUIRE(plan->small && plan->ms_items.empty() && plan->vf_items.empty() && plan->expand_split && pool->H <= 4096);
        for (const Item &it : plan->ve_items)
            REQUIRE(it.rank <= kSmallRanks && it.ntok <= kExpandTok && it.ntok <= plan->max_expand_tok);
        return SLORA_OK;
    }
    g_log.fused = true;
    g_seen = -1;
    // every fused group is a whole group of at most kExpandTok tokens, and the tails of the two
    // vector lists are exactly these groups' two-stage items
    std::set<int32_t> fused_pos;
    for (size_t i = 0; i < plan->vf_items.size(); ++i) {
        const Item &it = plan->d_vf[i];
        REQUIRE(std::memcmp(&it, &plan->vf_items[i], sizeof it) == 0);
        REQUIRE(it.ntok >= 1 && it.ntok <= kExpandTok && it.rank <= plan->v_stride);
        check_tokens(plan, it.pos0, it.ntok);
        for (int32_t k = 0; k < n; ++k) {
            REQUIRE(a.x[k] && a.y[k]);
            check_pages(plan, it.arena_off, it.rank, a.slot[k]);
        }
        fused_pos.insert(it.pos0);
    }
    for (size_t i = 0; i < plan->vs_items.size(); ++i)
        REQUIRE((fused_pos.count(plan->vs_items[i].pos0) != 0) == (i >= (size_t)plan->n_vs_head));
    for (size_t i = 0; i < plan->ve_items.size(); ++i)
        REQUIRE((fused_pos.count(plan->ve_items[i].pos0) != 0) == (i >= (size_t)plan->n_ve_head));
    return SLORA_OK;
}

} // namespace slora

// ---------------------------------------------------------------------------------------------
// directed cases
// ---------------------------------------------------------------------------------------------
using namespace slora;

// A pool of one adapter per (rank, tokens) pair, its batch, and one x and y per slot.
struct Bench {
    int32_t H, n_slots, T = 0;
    std::vector<uint16_t> mem;
    slora_pool *pool = nullptr;
    slora_plan *plan = nullptr;
    std::vector<std::vector<uint16_t>> x;
    std::vector<std::vector<float>> y;
    std::vector<int32_t> ids;
    std::vector<const void *> xs;
    std::vector<float *> ys;
    int32_t slots[SLORA_MAX_MULTI] = {0, 1, 2, 3, 4, 5, 6, 7};

    Bench(int32_t H_, int32_t n_slots_, int32_t dtype, const std::vector<std::pair<int, int>> &groups,
          const std::vector<std::pair<const char *, int64_t>> &options = {})
        : H(H_), n_slots(n_slots_)
    {
        int64_t pages = 0;
        int32_t max_rank = 1;
        for (auto &g : groups) {
            pages += 2 * (int64_t)n_slots * g.first;
            max_rank = std::max(max_rank, g.first);
        }
        mem.assign((size_t)pages * H, 0);
        REQUIRE(slora_pool_init(&pool, H, pages, dtype, mem.data(), n_slots, max_rank) == SLORA_OK);
        for (auto &o : options) REQUIRE(slora_set_option(pool, o.first, o.second) == SLORA_OK);
        for (size_t a = 0; a < groups.size(); ++a) {
            REQUIRE(slora_adapter_alloc(pool, (int32_t)a, groups[a].first, nullptr) == SLORA_OK);
            ids.insert(ids.end(), (size_t)groups[a].second, (int32_t)a);
        }
        T = (int32_t)ids.size();
        for (int k = 0; k < n_slots; ++k) {
            x.emplace_back((size_t)T * H);
            y.emplace_back((size_t)T * H);
            xs.push_back(x.back().data());
            ys.push_back(y.back().data());
        }
        REQUIRE(slora_batch_plan(pool, &plan, ids.data(), T, nullptr, 0) == SLORA_OK);
    }
    ~Bench()
    {
        REQUIRE(slora_plan_destroy(plan) == SLORA_OK);
        REQUIRE(slora_pool_destroy(pool) == SLORA_OK);
    }
    int32_t apply(int32_t n) { g_log = {}; return slora_lora_apply_multi(plan, n, slots, xs.data(), ys.data(), nullptr); }
    int32_t apply_static(int32_t n) { g_log = {}; return slora_lora_apply_multi_static(plan, n, slots, xs.data(), ys.data(), nullptr); }
    int32_t apply_captured(int32_t n, bool y16)
    {
        g_log = {};
        g_captures = true;
        void *const stream = &n_slots; // a stream that is not the default one
        const int32_t rc = y16 ? slora_lora_apply_multi_y16(plan, n, slots, xs.data(), (void *const *)ys.data(), stream) : slora_lora_apply_multi(plan, n, slots, xs.data(), ys.data(), stream);
        g_captures = false;
        return rc;
    }
    int32_t apply16(int32_t n) { g_log = {}; return slora_lora_apply_multi_y16(plan, n, slots, xs.data(), (void *const *)ys.data(), nullptr); }
    int32_t shrink(int32_t n) { g_log = {}; return slora_lora_shrink(plan, n, slots, xs.data(), nullptr); }
    int32_t expand(int32_t n) { g_log = {}; return slora_lora_expand(plan, n, slots, ys.data(), nullptr); }
};

// An apply that fails leaves v as the shrink before it did: the expand that follows reads THAT layout.
static void failed_apply()
{
    for (int32_t n : {1, 2, 3, 4}) { // slots of the shrink; the apply of all eight needs a larger scratch
        Bench b(4096, 8, SLORA_F16, {{64, 512}});
        REQUIRE(b.shrink(n) == SLORA_OK && !g_log.mfma_shrink);
        g_fail_malloc = true;
        REQUIRE(b.apply(8) == SLORA_EHIP);
        g_fail_malloc = false;
        REQUIRE(b.expand(n) == SLORA_OK && !g_log.mfma_expand && g_log.vec_expand > 0);
        REQUIRE(b.apply(n) == SLORA_OK && g_log.mfma_expand);
    }
}

// The apply that allocates nothing takes the kernels of the one that does, also where the MFMA form is larger
// than the static scratch (512 tokens of rank 1024 on 8 slots: 80 MiB).
static void static_route()
{
    for (int32_t n : {1, 4, 8}) {
        Bench b(1024, 8, SLORA_F16, {{1024, 512}});
        REQUIRE(b.apply(n) == SLORA_OK);
        const Log multi = g_log;
        REQUIRE(b.apply_static(n) == SLORA_OK);
        REQUIRE(g_log.mfma_shrink == multi.mfma_shrink && g_log.mfma_expand == multi.mfma_expand);
        REQUIRE(g_log.vec_shrink == multi.vec_shrink && g_log.vec_expand == multi.vec_expand);
        REQUIRE(multi.mfma_expand == (n < 8) && (multi.vec_expand > 0) == (n == 8));
    }
}

// Once a plan has been applied (or shrunk) with n slots, whatever the type of y, further calls with at most n
// slots allocate nothing.
static void scratch_is_sized_once()
{
    for (int32_t H : {1024, 4096})
        for (int first = 0; first < 3; ++first) {
            Bench b(H, 8, SLORA_F16, {{H == 1024 ? 1024 : 64, 512}}); // H = 1024: 8 slots are too large for the MFMA form
            REQUIRE((first == 0 ? b.apply(8) : first == 1 ? b.apply16(8) : b.shrink(8)) == SLORA_OK);
            const long before = g_device_mallocs;
            for (int32_t n : {7, 1})
                REQUIRE(b.apply(n) == SLORA_OK && b.apply16(n) == SLORA_OK && b.shrink(n) == SLORA_OK && b.expand(n) == SLORA_OK);
            REQUIRE(g_device_mallocs == before);
        }
}

// "fuse_decode" 0: never one launch for both stages.  Otherwise a small batch takes the one that hands v over or, with the static scratch and
// under capture, the one in which every workgroup computes v for itself.
static void fuse_decode_never()
{
    for (int64_t mode : {0, 1, 2}) {
        Bench b(4096, 2, SLORA_BF16, {{8, 1}, {16, 2}}, {{"fuse_decode", mode}});
        for (bool y16 : {false, true}) {
            REQUIRE((y16 ? b.apply16(2) : b.apply(2)) == SLORA_OK);
            REQUIRE(g_log.chain == (mode == 1) && g_log.fused == (mode == 2) && !g_log.small);
            REQUIRE((g_log.vec_expand > 0) == (mode != 2));
            REQUIRE((y16 ? b.apply_captured(2, true) : b.apply_static(2)) == SLORA_OK);
            REQUIRE(g_log.small == (mode == 1) && g_log.fused == (mode == 2) && !g_log.chain);
            REQUIRE((g_log.vec_expand > 0) == (mode == 0));
        }
    }
}

// A workgroup of a kernel for both stages writes y while others still read x: calls in which a y overlaps an x take the two kernels.
static void y_in_the_buffer_of_x()
{
    Bench b(4096, 2, SLORA_BF16, {{8, 1}, {16, 2}});
    const size_t row = (size_t)b.H * 2; // bytes of a row of x, and of a 16-bit y
    std::vector<unsigned char> room(12 * row);
    b.xs = {room.data() + 3 * row, b.xs[1]};
    const auto one_launch = [&](int64_t y_off, bool y16) { // y of slot 1 at this offset from x of slot 0
        b.ys[1] = (float *)(room.data() + 3 * row + y_off);
        REQUIRE((y16 ? b.apply16(2) : b.apply(2)) == SLORA_OK);
        const bool one = g_log.chain;
        REQUIRE(g_log.vec_expand > 0 && !g_log.small);
        REQUIRE((y16 ? b.apply_captured(2, true) : b.apply_static(2)) == SLORA_OK);
        REQUIRE(g_log.small == one && (g_log.vec_expand == 0) == one && !g_log.chain);
        return one;
    };
    REQUIRE(!one_launch(0, true) && !one_launch((int64_t)(2 * row), true) && !one_launch(-(int64_t)(2 * row), true));
    REQUIRE(one_launch((int64_t)(3 * row), true) && one_launch(-(int64_t)(3 * row), true));
    REQUIRE(!one_launch(-(int64_t)(3 * row), false) && one_launch((int64_t)(3 * row), false)); // fp32: rows twice as long
}

// The MFMA expand list holds what its workgroups read: one record per run of tiles and column range, in runs that
// leave the launch at least 1024 workgroups.
static void expand_runs()
{
    std::vector<std::pair<int, int>> groups;
    for (int g = 0; g < 16; ++g) groups.push_back({32, 283}); // 16 x 9 tiles
    Bench b(4096, 4, SLORA_F16, groups);
    REQUIRE(b.plan->n_mfma_tiles == 144 && b.apply(4) == SLORA_OK && g_log.mfma_expand);
    REQUIRE(b.plan->me_items.size() == 16 * 16); // runs of 9 tiles: 144 x 16 x 4 / 1024
    int64_t info[SLORA_PLAN_INFO_N];
    REQUIRE(slora_plan_info(b.plan, info, SLORA_PLAN_INFO_N) == SLORA_OK && info[7] == 144 * 16);
}

// What a call takes depends on its own slots, not on the pool's: tokens per workgroup of the MFMA shrink, tiles per
// workgroup of the MFMA expand, and which kernels serve a batch of few tiles.
static void slots_of_the_call()
{
    const std::vector<std::pair<int, int>> prompts(8, {32, 283}); // 8 x 9 tiles, not dual
    for (int32_t n : {1, 3, 4, 8}) {
        Bench one(4096, n, SLORA_F16, prompts), all(4096, 8, SLORA_F16, prompts);
        REQUIRE(one.apply(n) == SLORA_OK && one.plan->mfma_on({}));
        const Log want = g_log;
        REQUIRE(all.apply(n) == SLORA_OK);
        REQUIRE(g_log.mfma_expand_wgs >= (size_t)std::min(1024, 72 * 16 * n));
        REQUIRE(g_log.mfma_expand_wgs <= 2 * want.mfma_expand_wgs);
        REQUIRE(g_log.mfma_shrink_wgs >= (size_t)std::min(160, 72 * n)); // 72: the items in quarters
    }
    Bench few(4096, 8, SLORA_F16, {{64, 32}}); // 8.4 MB of pages read again per slot: 30 MB from four slots on
    for (int32_t n = 1; n <= 8; ++n) REQUIRE(few.apply(n) == SLORA_OK && g_log.mfma_expand == (n >= 4));
    few.ids.assign(32, 0);
    g_log = {};
    REQUIRE(slora_lora_shrink_expand(few.pool, 0, few.xs[0], few.ids.data(), nullptr, 0, 32, few.ys[0], nullptr) == SLORA_OK);
    REQUIRE(!g_log.mfma_expand && g_log.vec_expand > 0);
}

// The larger items of the vector kernels: every call of a crowded plan covers each token's ranks and columns once,
// also where the plan's groups of many tokens are on the MFMA kernels (fp32 y) or not (16-bit y, two-stage calls).
static void larger_items()
{
    std::vector<std::pair<int, int>> groups;
    for (int g = 0; g < 60; ++g) groups.push_back({g % 3 == 0 ? 40 : 32, 7 + g % 9}); // 7 .. 15 tokens
    for (int g = 0; g < 8; ++g) groups.push_back({32, 1 + g % 4});
    Bench plain(1024, 8, SLORA_BF16, groups);
    groups.push_back({32, 800}); // too few tiles for a plan of MFMA groups: in both families' lists
    Bench dual(1024, 8, SLORA_F16, groups);
    for (Bench *b : {&plain, &dual}) {
        REQUIRE(b->plan->dual == (b == &dual));
        REQUIRE(b->apply(8) == SLORA_OK && g_log.gang && g_log.gang_expand && g_log.wide == (b == &dual));
        REQUIRE(b->apply16(8) == SLORA_OK && g_log.gang && g_log.gang_expand && !g_log.wide);
        REQUIRE(b->shrink(8) == SLORA_OK && g_log.gang && b->expand(8) == SLORA_OK && g_log.gang_expand);
    }
}

// They are taken, and their lists held, where they leave at most half the workgroups: beside many small groups a few
// larger ones would slow the small items down.
static void larger_items_pay()
{
    const auto with = [](int n_small, int n_large, int toks, bool taken) {
        std::vector<std::pair<int, int>> groups(n_small, {16, 1});
        groups.insert(groups.end(), n_large, {16, toks});
        Bench b(1024, 8, SLORA_F16, groups);
        REQUIRE(b.apply(8) == SLORA_OK && g_log.vec_shrink * 8 >= 1400 && g_log.gang == taken && b.plan->gs_items.empty() == !taken);
        REQUIRE(b.apply16(8) == SLORA_OK && g_log.gang == taken);
    };
    with(55, 5, 8, false);  // 260 small items / 225 larger and small
    with(60, 1, 5, false);
    with(40, 20, 8, false); // 320 / 180
    with(36, 24, 8, true);  // 336 / 168
    with(0, 60, 5, true);
}

// A plan holds no lists that calls of its pool's slots do not take.
static void larger_items_of_no_call()
{
    const std::vector<std::pair<int, int>> low(60, {16, 8}), high(60, {40, 8}); // 8 and 20 shrink items a group, 4 expand items
    for (int32_t n : {1, 2, 8}) {
        Bench b(1024, n, SLORA_F16, low), h(1024, n, SLORA_F16, high);
        REQUIRE(b.plan->gs_items.empty() == (480 * n < 1400) && b.plan->ge_items.empty() == (240 * n < 2000));
        REQUIRE(h.plan->gs_items.empty() == (1200 * n < 1400) && h.plan->ge_items.empty()); // its expand has no larger items
        REQUIRE(b.apply(n) == SLORA_OK && h.apply(n) == SLORA_OK);
    }
}

// Their tokens go through the matrix instruction, four at a time, where that pays: items of more than 32 ranks, those of 9 to 32 ranks that
// leave a wavefront three tokens (bf16) or four, and with a y in 16 bits those of up to 8 ranks that leave it three.
static void larger_items_in_fours()
{
    const auto with = [](int32_t dtype, int rank, int tok, bool fours, bool fours16) {
        Bench b(4096, 8, dtype, std::vector<std::pair<int, int>>(tok <= 16 ? 24 : 12, {rank, tok}));
        REQUIRE(b.apply16(8) == SLORA_OK && g_log.gang_expand && b.plan->fours[0] == fours && b.plan->fours[1] == fours16);
    };
    for (int32_t dtype : {SLORA_F16, SLORA_BF16}) {
        const bool bf16 = dtype == SLORA_BF16;
        for (int rank : {1, 8}) for (int tok : {5, 8, 9, 16, 33}) with(dtype, rank, tok, false, tok > 8);
        for (int rank : {9, 32})
            for (int tok : {5, 8, 9, 12, 13, 16, 24, 33}) with(dtype, rank, tok, tok > (bf16 ? 8 : 12), tok > (bf16 ? 8 : 12));
        for (int tok : {7, 8, 9, 33}) with(dtype, 33, tok, true, true);
        for (int tok : {5, 6}) with(dtype, 33, tok, false, false); // four, and one or two of their own
    }
}

// LDS of the MFMA expand: adapters of 129 to 256 ranks use its buffers but where v is in scaled pieces
static void expand_lds()
{
    for (int32_t dtype : {SLORA_F16, SLORA_BF16})
        for (int32_t rank : {32, 128, 129, 200, 256, 257}) {
            Bench b(1024, 8, dtype, {{rank, 512}});
            const bool scaled = dtype == SLORA_F16;
            REQUIRE(b.plan->dual && b.apply(8) == SLORA_OK && g_log.mfma_expand);
            REQUIRE(b.plan->me_stages == (rank == 32 ? 1 : rank == 128 ? 4 : rank > 256 || scaled ? 0 : 4));
        }
}

// "shrink_pages" as the caller sets it, be it the default, holds for every item
static void shrink_pages_of_the_caller()
{
    const std::vector<std::pair<int, int>> crowd(60, {32, 9});
    for (int64_t pages : {0, 1, 4, 12}) {
        std::vector<std::pair<const char *, int64_t>> options;
        if (pages > 0) options.push_back({"shrink_pages", pages});
        Bench b(1024, 8, SLORA_F16, crowd, options);
        REQUIRE(b.apply(8) == SLORA_OK && g_log.gang == (pages == 0) && g_log.gang_expand);
        REQUIRE(g_log.vec_shrink == (size_t)(60 * 3 * (pages == 1 ? 32 : pages == 12 ? 3 : 8)));
    }
}

// Both vector stages in one launch that hands v over: calls of up to a few thousand workgroups, beside MFMA groups too, never with the static
// scratch, the two-stage calls, "fuse_decode" 0, a y that overlaps an x or no memory for the words; a later expand finds v.
static void hand_over()
{
    std::vector<std::pair<int, int>> groups;
    for (int g = 0; g < 24; ++g) groups.push_back({8 + 24 * (g % 4), 1 + g % 5});
    const std::vector<std::pair<const char *, int64_t>> never{{"fuse_decode", 0}};
    for (int32_t H : {520, 4096, 8192, 8200}) {
        Bench b(H, 4, SLORA_BF16, groups), off(H, 4, SLORA_BF16, groups, never);
        for (int32_t n = 1; n <= 4; ++n) {
            const int64_t wgs = (b.plan->chain_wgs(Route{})) * n;
            const bool pays = H <= 8192 && wgs <= (std::min(b.plan->max_shrink_tok, 4) * H * 2 <= 40960 ? 4096 : 2048); // (more than 64 ranks times tokens an expand item)
            REQUIRE(b.apply(n) == SLORA_OK && g_log.chain == pays && g_log.vec_expand > 0);
            REQUIRE(b.expand(n) == SLORA_OK && !g_log.chain);
            REQUIRE(b.apply16(n) == SLORA_OK && g_log.chain == pays);
            REQUIRE(b.apply_static(n) == SLORA_OK && !g_log.chain);
            REQUIRE(b.shrink(n) == SLORA_OK && !g_log.chain && b.expand(n) == SLORA_OK && !g_log.chain);
            REQUIRE(off.apply(n) == SLORA_OK && !g_log.chain);
        }
    }
    Bench b(1024, 2, SLORA_F16, groups);
    const auto hand_overs = [&] {
        int64_t stats[SLORA_POOL_STATS_N];
        REQUIRE(slora_pool_stats(b.pool, stats, SLORA_POOL_STATS_N) == SLORA_OK);
        return stats[3];
    };
    REQUIRE(b.apply(1) == SLORA_OK && hand_overs() == 1 && b.apply_static(1) == SLORA_OK && b.apply_captured(1, false) == SLORA_OK && hand_overs() == 1);
    const void *const x1 = b.xs[1];
    b.xs[1] = b.ys[0]; // slot 0 writes what slot 1 reads
    REQUIRE(b.apply16(2) == SLORA_OK && !g_log.chain);
    b.xs[1] = x1;
    REQUIRE(b.apply(2) == SLORA_OK && g_log.chain && b.plan->set->launch == 1 && hand_overs() == 2); // (larger words than those of one slot)
    b.plan->set->launch = UINT32_MAX - 1; // numbers run out, and start again with none of theirs in the words
    for (int i = 0; i < 3; ++i) REQUIRE(b.apply(2) == SLORA_OK && g_log.chain);
    REQUIRE(b.plan->set->launch == 2);
    std::vector<std::pair<int, int>> mixed(20, {32, 64}); // 40 tiles
    mixed.push_back({16, 3});
    Bench m(2048, 3, SLORA_F16, mixed);
    REQUIRE(m.apply(3) == SLORA_OK && g_log.chain && g_log.mfma_expand && g_log.vec_expand > 0);
}

// Which calls take it, on both sides of every line.
static void hand_over_pays()
{
    const auto calls = [](int32_t H, int groups, int tok, int rank, std::initializer_list<std::pair<int32_t, bool>> slots) {
        Bench b(H, 8, SLORA_F16, std::vector<std::pair<int, int>>(groups, {rank, tok}));
        for (auto &s : slots) REQUIRE(b.apply16(s.first) == SLORA_OK && g_log.chain == s.second && !g_log.gang && !g_log.gang_expand);
    };
    calls(4096, 60, 4, 32, {{4, true}, {5, false}});           // 3840 and 4800 workgroups
    calls(3072, 71, 1, 1, {{5, true}, {6, false}});            // 2485, 2982: an expand item is one product a column
    calls(3072, 63, 1, 8, {{7, true}, {8, false}});            // 3528, 4032: eight
    calls(2560, 70, 4, 1, {{8, true}});                        // 3360: four
    calls(8192, 20, 4, 32, {{4, true}, {5, false}});           // 1920, 2400: 64 KiB of x
    calls(8192, 20, 4, 4, {{4, true}, {5, false}});            // 1360, 1700: and sixteen products
    calls(1024, 20, 1, 128, {{1, true}, {2, false}});          // 640 and 1280 shrink items, sixteen times as many as expand items
    calls(8192, 25, 2, 4, {{6, true}, {7, false}});            // 2550, 2975: eight products, three workgroups a compute unit
    calls(7168, 20, 4, 4, {{5, true}, {6, false}});            // 1500, 1800: sixteen, and 64 KiB of x
    calls(3072, 20, 2, 128, {{1, true}, {2, false}, {3, false}}); // 760, 1520, 2280: pairs, 5.3 times
    calls(3072, 8, 2, 128, {{3, true}, {4, false}, {6, true}, {7, false}}); // 912, 1216, 1824, 2128
    calls(3072, 8, 2, 96, {{4, true}, {5, true}, {8, true}}); // 960, 1200, 1920: of fewer ranks
    calls(3072, 20, 3, 128, {{3, true}});
    calls(2560, 5, 1, 100, {{6, true}, {8, false}});           // 900, 1200: single tokens, five times
    calls(2560, 13, 1, 100, {{2, true}, {3, false}, {4, true}}); // 780, 1170, 1560
    calls(1120, 40, 1, 64, {{1, true}, {2, true}, {3, false}}); // 760, 1520, 2280: short rows
    calls(4096, 42, 4, 128, {{1, true}, {2, false}});          // 1680, 3360: fours, four times
    // a call whose groups of many tokens are on the MFMA kernels keeps rows for the tokens of the others only
    std::vector<std::pair<int, int>> mixed{{64, 1}, {64, 3}, {64, 2}, {32, 400}};
    Bench b(8192, 4, SLORA_F16, mixed);
    REQUIRE(b.plan->dual && b.plan->max_shrink_tok == 4 && b.plan->chain[0].tok == 3 && b.plan->chain[1].tok == 4);
    REQUIRE(b.apply(4) == SLORA_OK && g_log.wide && g_log.chain && b.plan->chain[0].words == 64 * 6);
}

// Room for the words lies behind v, in one allocation; the first launch that uses it clears it, so calls that never hand v over launch
// nothing for it.  Without memory for it calls take the two kernels, and ask once per hand-out of the buffers.
static void words_of_the_calls_that_use_them()
{
    const std::vector<std::pair<int, int>> prompt{{64, 256}}, two{{64, 400}, {64, 200}}, crowd(40, {32, 8});
    for (auto *groups : {&prompt, &two, &crowd}) {
        Bench b(4096, 4, SLORA_BF16, *groups);
        const long mallocs = g_device_mallocs, clears = g_clears;
        REQUIRE(b.apply(4) == SLORA_OK && !g_log.chain && (g_log.mfma_expand || g_log.gang_expand));
        REQUIRE(g_device_mallocs == mallocs + 1 && g_clears == clears);
    }
    const std::vector<std::pair<int, int>> some(20, {16, 2});
    {
        Bench b(1024, 4, SLORA_F16, some);
        const long mallocs = g_device_mallocs, clears = g_clears;
        for (int i = 0; i < 3; ++i)
            for (int32_t n : {4, 1, 3}) REQUIRE(b.apply(n) == SLORA_OK && g_log.chain && b.shrink(n) == SLORA_OK && b.apply16(n) == SLORA_OK && g_log.chain);
        REQUIRE(g_device_mallocs == mallocs + 1 && g_clears == clears + 1);
        REQUIRE(b.plan->chain_of(Route{}).words == 20 * 2 * 16);
    }
    int place = 0;
    void *const stream = &place;
    Bench few(1024, 1, SLORA_F16, std::vector<std::pair<int, int>>(60, {40, 4})); // 15360 floats and 9600 words: 64 and 128 KiB
    g_free_bytes = (size_t)1 << 16;
    long mallocs = g_device_mallocs;
    REQUIRE(few.apply(1) == SLORA_OK && !g_log.chain && g_log.vec_expand > 0 && g_device_mallocs == mallocs + 2);
    for (int i = 0; i < 3; ++i) REQUIRE(few.apply(1) == SLORA_OK && !g_log.chain && g_device_mallocs == mallocs + 2); // not asked for again
    g_free_bytes = SIZE_MAX;
    REQUIRE(few.apply(1) == SLORA_OK && !g_log.chain);
    REQUIRE(slora_plan_destroy(few.plan) == SLORA_OK && slora_batch_plan(few.pool, &few.plan, few.ids.data(), few.T, nullptr, 0) == SLORA_OK);
    mallocs = g_device_mallocs;
    g_captures = true; // nothing is allocated, and nothing cleared, under capture
    REQUIRE(slora_lora_apply_multi(few.plan, 1, few.slots, few.xs.data(), few.ys.data(), stream) == SLORA_OK && g_device_mallocs == mallocs);
    g_captures = false;
    REQUIRE(few.apply(1) == SLORA_OK && g_log.chain && g_device_mallocs == mallocs + 1);
    g_captures = true;
    g_log = {};
    REQUIRE(slora_lora_apply_multi(few.plan, 1, few.slots, few.xs.data(), few.ys.data(), stream) == SLORA_OK && !g_log.chain && g_log.vec_expand > 0);
    g_captures = false;
}

static const struct { const char *name; void (*run)(); } kCases[] = {
    {"hand_over", hand_over},
    {"hand_over_pays", hand_over_pays},
    {"words_of_the_calls_that_use_them", words_of_the_calls_that_use_them},
    {"shrink_pages_of_the_caller", shrink_pages_of_the_caller},
    {"expand_lds", expand_lds},
    {"larger_items_of_no_call", larger_items_of_no_call},
    {"larger_items_pay", larger_items_pay},
    {"larger_items", larger_items},
    {"larger_items_in_fours", larger_items_in_fours},
    {"failed_apply", failed_apply},
    {"static_route", static_route},
    {"scratch_is_sized_once", scratch_is_sized_once},
    {"fuse_decode_never", fuse_decode_never},
    {"y_in_the_buffer_of_x", y_in_the_buffer_of_x},
    {"expand_runs", expand_runs},
    {"slots_of_the_call", slots_of_the_call},
};

// ---------------------------------------------------------------------------------------------
// driver
// ---------------------------------------------------------------------------------------------
int main(int argc, char **argv)
{
    for (auto &c : kCases)
        if (argc > 1 && !std::strcmp(argv[1], c.name)) {
            c.run();
            std::printf("host_san OK: %s\n", c.name);
            return 0;
        }
    const unsigned seed = argc > 1 ? (unsigned)std::atoi(argv[1]) : 1u;
    std::mt19937 rng(seed);
    auto rnd = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    long calls = 0, plans_made = 0, both_families = 0, larger = 0, chains = 0;
    for (int round = 0; round < 12; ++round) {
        const int32_t H = 8 * rnd(8, 160);
        const int64_t n_pages = rnd(200, 3000);
        const int32_t n_slots = rnd(1, 5), max_rank = rnd(1, 300);
        const int32_t dtype = rnd(0, 1);
        std::vector<uint16_t> mem((size_t)n_pages * H, 0x3c00);
        slora_pool *pool = nullptr;
        REQUIRE(slora_pool_init(&pool, H, n_pages, dtype, mem.data(), n_slots, max_rank) == SLORA_OK);
        REQUIRE(slora_set_option(pool, "mfma_min_tokens", rnd(1, 40)) == SLORA_OK);
        REQUIRE(slora_set_option(pool, "mfma_min_tiles", rnd(0, 2) ? rnd(1, 4) : 1000) == SLORA_OK); // 1000: plans of both families
        REQUIRE(slora_set_option(pool, "mfma_split_bytes", 4096 << rnd(0, 6)) == SLORA_OK);
        REQUIRE(slora_set_option(pool, "mfma_split_min_h", 128 << rnd(0, 3)) == SLORA_OK);
        REQUIRE(slora_set_option(pool, "xcd_group", rnd(0, 3)) == SLORA_OK);
        const int pages = rnd(1, 12); // the half of the pools that does not set it may take the larger items
        if (pages % 2) REQUIRE(slora_set_option(pool, "shrink_pages", pages) == SLORA_OK);
        REQUIRE(slora_set_option(pool, "fuse_decode", rnd(0, 2)) == SLORA_OK);
        std::vector<int32_t> loaded;
        std::vector<slora_plan *> plans;
        std::vector<uint16_t> x((size_t)4096 * H, 0x3800), w;
        std::vector<float> y((size_t)SLORA_MAX_MULTI * 4096 * H, 0.f);
        // one to four calls on a plan, any entry point, now and then without device memory to be had
        auto use = [&](slora_plan *plan, int32_t most) {
            int32_t slots[SLORA_MAX_MULTI];
            const void *xs[SLORA_MAX_MULTI];
            float *ys[SLORA_MAX_MULTI];
            for (int k = 0; k < most; ++k) {
                slots[k] = rnd(0, n_slots - 1);
                xs[k] = x.data();
                ys[k] = y.data() + (size_t)k * 4096 * H;
            }
            for (int c = rnd(1, 4); c > 0; --c) {
                const int32_t n = rnd(0, 1) ? most : (most + 1) / 2;
                const bool no_memory = g_fail_malloc = rnd(0, 7) == 0;
                g_log = {};
                int32_t rc = SLORA_OK;
                const int entry = rnd(0, 6);
                switch (entry) {
                case 0: rc = slora_lora_apply_multi_static(plan, n, slots, xs, ys, nullptr); break;
                case 1: rc = slora_lora_apply_multi_y16(plan, n, slots, xs, (void *const *)ys, nullptr); break;
                case 2: rc = slora_lora_shrink(plan, n, slots, xs, nullptr); break;
                case 3: rc = slora_lora_expand(plan, n, slots, ys, nullptr); break;
                case 4: rc = slora_lora_expand_y16(plan, n, slots, (void *const *)ys, nullptr); break;
                default: rc = slora_lora_apply_multi(plan, n, slots, xs, ys, nullptr);
                }
                g_fail_malloc = false;
                both_families += plan->dual && g_log.mfma_expand;
                larger += g_log.gang || g_log.gang_expand;
                chains += g_log.chain;
                REQUIRE(rc == SLORA_OK || rc == SLORA_EBUSY || (rc == SLORA_ERANGE && entry == 0) ||
                        (rc == SLORA_EINVAL && (entry == 3 || entry == 4)) || (rc == SLORA_EHIP && no_memory));
            }
        };
        for (int step = 0; step < 120; ++step, ++calls) {
            const int what = rnd(0, 9);
            if (what <= 2) { // make an adapter resident on pages of the library's choice, then fill them
                const int32_t id = rnd(0, 60), rank = rnd(0, max_rank + 2);
                std::vector<int32_t> pages((size_t)n_slots * 2 * std::max(rank, 1));
                const int32_t rc = slora_adapter_alloc(pool, id, rank, pages.data());
                if (rc == SLORA_OK) {
                    loaded.push_back(id);
                    w.assign((size_t)n_slots * 2 * rank * H + 8, 0x2e66);
                    REQUIRE(slora_adapter_upload(pool, id, w.data(), nullptr) == SLORA_OK);
                } else {
                    REQUIRE(rc == SLORA_EBUSY || rc == SLORA_ENOMEM || rc == SLORA_ERANGE);
                }
            } else if (what == 3 && !loaded.empty()) { // evict
                const size_t k = rng() % loaded.size();
                REQUIRE(slora_adapter_unload(pool, loaded[k]) == SLORA_OK);
                loaded.erase(loaded.begin() + (long)k);
            } else if (what == 4) { // KV pages come and go
                const int64_t n = rnd(0, 40);
                std::vector<int32_t> kv((size_t)std::max<int64_t>(n, 1));
                if (slora_pool_alloc_kv(pool, n, kv.data()) == SLORA_OK) {
                    std::vector<uint16_t> src((size_t)n * H, 0x7e00);
                    REQUIRE(slora_pool_write_pages(pool, kv.data(), n, src.data(), 0, nullptr) == SLORA_OK);
                    if (rnd(0, 1)) REQUIRE(slora_pool_mark_kv(pool, kv.data(), n, 0) == SLORA_OK);
                }
            } else if (what <= 7) { // a batch: prefill segments and decode tokens
                std::vector<int32_t> ids, seg{0};
                const int n_seg = rnd(0, 12);
                for (int s = 0; s < n_seg; ++s) {
                    const int32_t id = (loaded.empty() || rnd(0, 9) == 0) ? -1 : loaded[rng() % loaded.size()];
                    const int len = rnd(0, 3) ? rnd(1, 6) : rnd(20, 300);
                    if ((int)ids.size() + len > 4096) break;
                    ids.insert(ids.end(), (size_t)len, id);
                    seg.push_back((int32_t)ids.size());
                }
                slora_plan *plan = nullptr;
                const bool decode = rnd(0, 3) == 0;
                REQUIRE(slora_batch_plan(pool, &plan, ids.data(), (int32_t)ids.size(), decode ? nullptr : seg.data(),
                                         (int32_t)seg.size() - 1) == SLORA_OK);
                plans_made++;
                use(plan, rnd(1, SLORA_MAX_MULTI));
                int64_t info[SLORA_PLAN_INFO_N];
                REQUIRE(slora_plan_info(plan, info, SLORA_PLAN_INFO_N) == SLORA_OK);
                if (rnd(0, 2))
                    REQUIRE(slora_plan_destroy(plan) == SLORA_OK);
                else
                    plans.push_back(plan);
            } else if (what == 8 && !plans.empty()) { // an older plan again: stale after an eviction, else fine
                slora_plan *plan = plans[rng() % plans.size()];
                use(plan, rnd(1, 2));
            } else if (!loaded.empty()) { // gather a matrix back
                const int32_t id = loaded[rng() % loaded.size()];
                std::vector<uint16_t> out((size_t)(max_rank + 2) * H + 8);
                REQUIRE(slora_adapter_gather(pool, id, rnd(0, n_slots - 1), rnd(0, 1), out.data(), nullptr) == SLORA_OK);
            }
        }
        REQUIRE(slora_pool_destroy(pool) == SLORA_EBUSY || plans.empty());
        for (slora_plan *p : plans) REQUIRE(slora_plan_destroy(p) == SLORA_OK);
        int64_t stats[SLORA_POOL_STATS_N];
        REQUIRE(slora_pool_stats(pool, stats, SLORA_POOL_STATS_N) == SLORA_OK);
        REQUIRE(slora_pool_destroy(pool) == SLORA_OK);
    }
    REQUIRE(both_families > 0); // MFMA calls on plans that hold both kernel families' lists
    REQUIRE(chains > 0);        // calls that hand v over inside a launch
    REQUIRE(larger > 0);        // calls that take the vector kernels' larger items
    std::printf("host_san OK: seed %u, %ld calls, %ld plans, %ld on both families, %ld of larger items\n", seed, calls, plans_made, both_families, larger);
    return 0;
}
