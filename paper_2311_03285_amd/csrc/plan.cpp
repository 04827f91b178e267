// Batch scheduler: turns (adapter id per token, request segments) into device work lists.
//
// The paper batches requests of different adapters and ranks in one iteration (Sec. 4.1) and
// runs the LoRA term with kernels that take no padding (Sec. 5.3); how the work is ordered is
// left open there.  Here tokens are grouped by adapter so that each adapter's pages are
// streamed once per group, groups are ordered by rank (longest work first, so the tail of a
// launch is made of short items), and each group goes either to the wavefront-reduction
// matrix-vector kernels (few tokens: decode) or to the MFMA kernels (many tokens: prefill).
// A plan depends only on the ids, so one plan serves every projection of every layer.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>

#include "slora_internal.hpp"

using namespace slora;

namespace {

struct Group {
    int32_t id;
    int32_t rank;
    int64_t arena_off;
    int32_t first_tok;
    std::vector<int32_t> toks;
};

int32_t hip_fail(hipError_t e, const char *what) { return fail(SLORA_EHIP, "%s: %s", what, hipGetErrorString(e)); }

} // namespace

int32_t slora::build_plan(slora_pool *pool, slora_plan *plan, const int32_t *ids, int32_t T,
                          const int32_t *seg_offsets, int32_t n_seg, int32_t call_slots)
{
    // ---- validate ----------------------------------------------------------------------
    if (T < 0) return fail(SLORA_EINVAL, "T=%d must be >= 0", T);
    if (T > 0 && !ids) return fail(SLORA_EINVAL, "token_adapter_ids is NULL");
    if (seg_offsets) {
        if (n_seg < 0) return fail(SLORA_ESEG, "n_seg=%d must be >= 0", n_seg);
        if (seg_offsets[0] != 0) return fail(SLORA_ESEG, "seg_offsets[0]=%d must be 0", seg_offsets[0]);
        if (seg_offsets[n_seg] != T)
            return fail(SLORA_ESEG, "seg_offsets[n_seg]=%d must equal T=%d", seg_offsets[n_seg], T);
        for (int32_t s = 0; s < n_seg; ++s) {
            if (seg_offsets[s + 1] <= seg_offsets[s] || seg_offsets[s + 1] > T)
                return fail(SLORA_ESEG, "seg_offsets must be strictly increasing and end at T (segment %d)", s);
            const int32_t id0 = ids[seg_offsets[s]];
            for (int32_t t = seg_offsets[s] + 1; t < seg_offsets[s + 1]; ++t)
                if (ids[t] != id0)
                    return fail(SLORA_ESEG, "token %d has id %d but its segment %d starts with id %d", t, ids[t], s, id0);
        }
    }
    std::unordered_map<int32_t, int32_t> group_of;
    std::vector<Group> groups;
    try {
        for (int32_t t = 0; t < T; ++t) {
            const int32_t id = ids[t];
            if (id == -1) continue;
            auto g = group_of.find(id);
            if (g == group_of.end()) {
                auto a = pool->adapters.find(id);
                if (id < 0 || a == pool->adapters.end())
                    return fail(SLORA_ENOENT, "token %d names adapter %d, which is not loaded", t, id);
                group_of.emplace(id, (int32_t)groups.size());
                groups.push_back(Group{id, a->second.rank, a->second.arena_off, t, {}});
                g = group_of.find(id);
            }
            groups[(size_t)g->second].toks.push_back(t);
        }

        // ---- order: rank bucket (descending), then more tokens first, then first appearance --
        std::vector<int32_t> order;
        for (int32_t g = 0; g < (int32_t)groups.size(); ++g)
            if (groups[(size_t)g].rank > 0) order.push_back(g);
        std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
            const Group &x = groups[(size_t)a], &y = groups[(size_t)b];
            if (x.rank != y.rank) return x.rank > y.rank;
            if (x.toks.size() != y.toks.size()) return x.toks.size() > y.toks.size();
            return x.first_tok < y.first_tok;
        });

        plan->T = T;
        plan->tok_idx.clear();
        plan->vs_items.clear();
        plan->ve_items.clear();
        plan->ms_items.clear();
        plan->mj_items.clear();
        plan->me_items.clear();
        plan->sum_rank = 0;
        plan->n_groups = (int32_t)order.size();
        plan->n_groups_vec = plan->n_groups_mfma = 0;
        plan->n_mfma_tiles = 0;
        plan->n_sync = 0;
        plan->part_floats = 0;
        plan->max_shrink_tok = 0;
        const int32_t n_chunks = (pool->H + kMsGranule - 1) / kMsGranule;
        int32_t max_rank = 0;
        const int32_t H = pool->H;
        // The MFMA kernels pay off when adapters have many tokens AND there are enough 32-token
        // tiles to fill the GPU: a handful of tiles is a few long, latency-bound workgroups, and
        // such groups are faster on the vector path (their pages are re-read from L2).
        int64_t mfma_tiles = 0;
        for (int32_t gi : order) {
            const int64_t n = (int64_t)groups[(size_t)gi].toks.size();
            if (n >= pool->mfma_min_tokens) mfma_tiles += (n + kMfmaTok - 1) / kMfmaTok;
        }
        const int64_t min_tokens = mfma_tiles >= pool->mfma_min_tiles ? pool->mfma_min_tokens : INT64_MAX;
        const int64_t launch_slots = std::min<int64_t>(pool->n_slots, SLORA_MAX_MULTI);
        const int64_t most_slots = call_slots > 0 ? call_slots : launch_slots; // ... of a call
        // One launch for both stages of decode groups (at most kExpandTok tokens): a workgroup per
        // group streams the whole adapter.  That pays when the batch has enough groups to fill
        // the GPU about three times over with whole-group workgroups AND the groups are large
        // (a workgroup's waits for its work item, page lists and first pages are then short beside
        // its streaming): measured per step inside one process, 2.41 -> 2.38 ms on the mixed
        // configuration (H = 8192, 2.3 MB of pages per group); on the large-pool decode one (0.6 MB
        // per group) 109.0 -> 112.3 us in one process and 111.7 -> 110.8 us in the next.
        // x rows are staged in LDS (64 KiB: H <= 8192).
        int64_t n_small = 0, small_bytes = 0;
        for (int32_t gi : order) {
            const int64_t n = (int64_t)groups[(size_t)gi].toks.size();
            if (n < min_tokens && n <= kExpandTok) {
                n_small++;
                small_bytes += (int64_t)groups[(size_t)gi].rank * H * 4; // A and B pages
            }
        }
        const bool fuse = pool->fuse_decode != 0 && H <= 8192 &&
                          (pool->fuse_decode > 1 ||
                           (n_small * launch_slots >= 3 * 256 && small_bytes >= n_small * (int64_t(1) << 20)));
        // ... these groups run in that launch whatever else the plan holds
        auto fused_group = [&](int64_t n) { return fuse && n < min_tokens && n <= kExpandTok; };
        // Fewer tiles than that: applies to fp32 y take the MFMA kernels all the same where the vector kernels
        // would read very much again - every four tokens of a group read all of its pages, while an MFMA
        // tile of a small batch is spread over many workgroups (shares of H, quarters of its tokens).
        // Measured, vector / MFMA, us per call, for pages read (all slots): 30 MB 18.0 / 16.2, 67 MB 43 / 27,
        // 134 MB 35 / 18, 268 MB 60 / 22, 537 MB (512 tokens of rank 64, 4 slots) 110 / 32.  Groups that stay
        // on the vector kernels put the three MFMA launches behind theirs: 59 MB 26 / 34, 214 MB 85 / 67,
        // 236 MB 116 / 103.  A plan does not know the type of y nor the slots of its calls: it holds both forms
        // (dual) if a call of as many slots as it may have reads that much, route() decides call by call, and
        // 16-bit y and the two-stage calls keep the vector kernels, whose sums 16-bit results are rounded from.
        int64_t sums = 0; // floats of one set of partial sums
        plan->reread = 0;
        bool few_tokens = false;
        for (int32_t gi : order) {
            const int64_t n = (int64_t)groups[(size_t)gi].toks.size();
            if (n >= pool->mfma_min_tokens && !fused_group(n)) {
                plan->reread += (n + kExpandTok - 1) / kExpandTok * groups[(size_t)gi].rank * (int64_t)H * 4;
                sums += (n + kMfmaTok - 1) / kMfmaTok * kMfmaTok * ((groups[(size_t)gi].rank + kRankPad - 1) / kRankPad * kRankPad);
            } else {
                few_tokens = true;
            }
        }
        // (a form whose partial sums of one slot exceed the static scratch is never taken: see route)
        plan->reread_min = few_tokens ? 128000000 : 30000000;
        plan->dual = min_tokens == INT64_MAX && plan->reread * most_slots >= plan->reread_min &&
                     sums * (int64_t)sizeof(float) <= (int64_t)SLORA_STATIC_SCRATCH_BYTES;
        const int64_t mfma_tokens = plan->dual ? pool->mfma_min_tokens : min_tokens;
        auto mfma_group = [&](int64_t n) { return n >= mfma_tokens && !fused_group(n); }; // has MFMA items
        // Size of a share of an MFMA shrink tile (see below): mfma_split_bytes, or more when the
        // batch is so large that shares of that size would be far more than the GPU can hold at a
        // time (every share of a split tile costs a set of partial sums) - about three workgroups
        // per compute unit for a launch of up to eight slots.
        int64_t ms_bytes = 0;
        for (int32_t gi : order) {
            const Group &g = groups[(size_t)gi];
            const int64_t n = (int64_t)g.toks.size();
            if (!mfma_group(n)) continue;
            const int64_t n_tok_tiles = (n + kMsTok - 1) / kMsTok, n_rank_blocks = (g.rank + kMsRanks - 1) / kMsRanks;
            ms_bytes += (n * n_rank_blocks + (int64_t)g.rank * n_tok_tiles) * H * 2;
        }
        // A dual batch is small: there the shares are as short as pays, 256 elements of H (512 tokens of rank 64,
        // H = 4096, 4 slots: 24 us for the stage with shares of 1 MiB, 18 at 512 KiB, 15 from 256 KiB on).  Short
        // chains also keep the error where the vector kernels have it: 1.08e-7 against 1.09e-7 for these
        // tokens in binary16 (2.9e-7 unsplit), 1.25e-7 against 1.41e-7 for rank 128 and H = 8192.
        const int64_t split_bytes = plan->dual ? std::min<int64_t>(pool->mfma_split_bytes, 32 << 10) : pool->mfma_split_bytes;
        const int64_t split_min_h = plan->dual ? std::min<int64_t>(pool->mfma_split_min_h, 256) : pool->mfma_split_min_h;
        const int64_t share_bytes = std::max<int64_t>(split_bytes, ms_bytes * launch_slots / (3 * 256));
        // MFMA expand: a workgroup keeps the B operands of its columns and walks a run of tiles.  Long runs
        // pay for them once, but the launch still needs several workgroups per compute unit.  The list's runs are
        // for calls of the most slots; calls of fewer share a run out over several workgroups (see route).
        int64_t me_tiles = 0;
        for (int32_t gi : order) {
            const int64_t n = (int64_t)groups[(size_t)gi].toks.size();
            if (mfma_group(n)) me_tiles += (n + kMfmaTok - 1) / kMfmaTok;
        }
        const int64_t me_pairs = me_tiles * ((H + kMfmaExpandCols - 1) / kMfmaExpandCols) * most_slots;
        const int32_t me_run = (int32_t)std::min<int64_t>(kMfmaRunMax, std::max<int64_t>(1, me_pairs / 1024));
        plan->me_run = me_run;
        plan->me_stages = 0;
        int32_t n_vec_groups = 0, most_vec_tokens = 0;
        for (int32_t gi : order) {
            const int64_t n = (int64_t)groups[(size_t)gi].toks.size();
            if (n >= min_tokens) continue;
            n_vec_groups++;
            most_vec_tokens = std::max(most_vec_tokens, (int32_t)n);
        }
        // vector-expand items: long runs of columns, halved while a launch would have fewer
        // workgroups than the GPU has CUs
        int32_t chunks = (H + kExpandColsMax - 1) / kExpandColsMax;
        auto cols_of = [&](int32_t c) { return ((H + c - 1) / c + 511) / 512 * 512; };
        while ((int64_t)n_vec_groups * chunks < 256 && cols_of(chunks) > 512) chunks *= 2;
        int32_t ecols = cols_of(chunks);
        // still short of workgroups at the smallest items: split the ranks over the wavefronts
        plan->expand_split = ecols == 512 && (int64_t)n_vec_groups * chunks < 512;
        // the vector shrink stages its tokens' x rows in LDS: at most 64 KiB of them per item
        const int32_t shrink_tok = std::max(1, std::min(kShrinkTok, 65536 / (H * 2)));
        const int32_t shrink_pages = pool->shrink_pages > 0 ? (int32_t)pool->shrink_pages : kShrinkPages;
        plan->expand_threads = ecols / 8;
        std::vector<Item> vs_tail, ve_tail, vs_dual, ve_dual;
        plan->vf_items.clear();
        plan->chain[0] = plan->chain[1] = {}; // of the plain items, and of the dual ones until they are behind those
        auto word = [](int64_t w) { return (int32_t)std::min<int64_t>(w, INT32_MAX); }; // (plans of so many hand nothing over)
        for (int32_t gi : order) {
            const Group &g = groups[(size_t)gi];
            const int32_t n = (int32_t)g.toks.size();
            const int32_t pos_base = (int32_t)plan->tok_idx.size();
            plan->tok_idx.insert(plan->tok_idx.end(), g.toks.begin(), g.toks.end());
            plan->sum_rank += g.rank;
            max_rank = std::max(max_rank, g.rank);
            const int32_t off = (int32_t)g.arena_off;
            if (mfma_group(n)) {
                // v tiles of 32 tokens, numbered in order; an expand item covers one tile, a shrink
                // item up to four consecutive ones (its pages are then read once for them all)
                const int32_t tile0 = plan->n_mfma_tiles;

                const int32_t n_tiles = (n + kMfmaTok - 1) / kMfmaTok;
                plan->n_mfma_tiles += n_tiles;
                for (int32_t p = 0; p < n; p += kMsTok) {
                    const int32_t nt = std::min(kMsTok, n - p);
                    for (int32_t j = 0; j < g.rank; j += kMsRanks) {
                        const int32_t nj = std::min(kMsRanks, g.rank - j);
                        // Shares of H: a workgroup streams its rows at a rate set by what it keeps in
                        // flight, so a tile of (nt + nj) rows x H is cut into shares of about
                        // share_bytes each - the launch then consists of many workgroups of
                        // similar, small size and every compute unit is busy to the end.  A share is
                        // never shorter than mfma_split_min_h elements: the partial sums a share
                        // leaves behind (and the last one reads back) must stay small beside its rows.
                        const int64_t cost = (int64_t)(nt + nj) * H * 2;
                        int64_t parts = (cost + share_bytes / 2) / share_bytes;
                        parts = std::min<int64_t>(parts, H / std::max<int64_t>(split_min_h, kMsGranule));
                        parts = std::min<int64_t>(parts, std::min<int64_t>(n_chunks, 64));
                        const int64_t mb = (nt + 31) / 32, nb = (nj + 31) / 32;
                        if (parts < 2 || plan->part_floats + parts * mb * nb * 1024 > (int64_t(1) << 30))
                            parts = 1;
                        MsItem it{};
                        it.arena_off = off;
                        it.rank = g.rank;
                        it.j0 = j;
                        it.nj = nj;
                        it.pos0 = pos_base + p;
                        it.ntok = nt;
                        it.tile = tile0 + p / kMfmaTok;
                        it.n_parts = (int32_t)parts;
                        it.sync = -1;
                        if (parts > 1 || plan->dual) {
                            it.sync = plan->n_sync++;
                            it.part_off = (int32_t)plan->part_floats;
                            plan->part_floats += parts * mb * nb * 1024;
                            plan->mj_items.push_back(it);
                        }
                        for (int32_t q = 0; q < (int32_t)parts; ++q) {
                            it.part = q;
                            it.c0 = (int32_t)((int64_t)n_chunks * q / parts);
                            it.c1 = (int32_t)((int64_t)n_chunks * (q + 1) / parts);
                            plan->ms_items.push_back(it);
                        }
                    }
                }
                // expand: the tiles in runs of equal length; a run of one column range is one workgroup
                // V of at most kMsRanks ranks at a time passes through LDS; that of an adapter of more ranks than twice as many, or than
                // kMsRanks if its pieces are scaled (see expand_mfma_kernel), does not
                if (g.rank <= (plan->dual && pool->dtype == SLORA_F16 ? kMsRanks : 2 * kMsRanks))
                    plan->me_stages = std::max(plan->me_stages, (std::min(g.rank, kMsRanks) + 31) / 32);
                const int32_t n_runs = (n_tiles + me_run - 1) / me_run;
                for (int32_t k = 0; k < n_runs; ++k) {
                    const int32_t t0 = n_tiles * k / n_runs, t1 = n_tiles * (k + 1) / n_runs;
                    const int32_t last = std::min(kMfmaTok, n - (t1 - 1) * kMfmaTok);
                    for (int32_t c = 0; c < H; c += kMfmaExpandCols) {
                        plan->me_items.push_back(Item{off, g.rank, c, std::min(kMfmaExpandCols, H - c), pos_base + t0 * kMfmaTok,
                                                      std::min(kMfmaTok, n - t0 * kMfmaTok), tile0 + t0, (t1 - t0) + 256 * last});
                    }
                }
            }
            if ((int64_t)n >= min_tokens) {
                plan->n_groups_mfma++;
            } else {
                plan->n_groups_vec++;
                // a group the one-launch decode kernel can take goes to the end of the two lists
                // (the two-stage calls run the whole lists, a fused apply only their heads)
                const bool fused = fused_group(n);
                const bool both = mfma_group(n); // in the MFMA lists as well
                std::vector<Item> &vs = fused ? vs_tail : both ? vs_dual : plan->vs_items;
                std::vector<Item> &ve = fused ? ve_tail : both ? ve_dual : plan->ve_items;
                slora_plan::Chain none, &chain = fused ? none : plan->chain[both]; // (a call that hands v over runs the others in launch_fused)
                const int64_t hand = chain.words;
                chain.words += (int64_t)n * g.rank;
                chain.work += (int64_t)n * g.rank * ((H + ecols - 1) / ecols);
                chain.tok = std::max(chain.tok, std::min(n, shrink_tok));
                chain.shared = chain.shared || n > kExpandTok;
                if (fused) plan->vf_items.push_back(Item{off, g.rank, 0, H, pos_base, n, 0, 0});
                for (int32_t p = 0; p < n; p += shrink_tok) {
                    const int32_t nt = std::min(shrink_tok, n - p), run = word(hand + (int64_t)p * g.rank);
                    plan->max_shrink_tok = std::max(plan->max_shrink_tok, nt);
                    for (int32_t j = 0; j < g.rank; j += shrink_pages)
                        vs.push_back(Item{off, g.rank, j, std::min(shrink_pages, g.rank - j), pos_base + p, nt, 0, run});
                }
                for (int32_t p = 0; p < n; p += kExpandTok) {
                    const int32_t nt = std::min(kExpandTok, n - p), run = word(hand + (int64_t)p * g.rank);
                    for (int32_t c = 0; c < H; c += ecols)
                        ve.push_back(Item{off, g.rank, c, std::min(ecols, H - c), pos_base + p, nt, n <= kExpandTok, run});
                }
            }
        }
        // Groups of many tokens on the vector kernels: every item of the lists above reads its pages, and its x again for
        // every few pages, for four tokens.
        plan->gs_items.clear();
        plan->gv_items.clear();
        plan->ge_items.clear();
        plan->n_gs_plain = plan->n_ge_plain = plan->max_gv_tok = 0;
        plan->fours[0] = plan->fours[1] = false;
        // (only if a call of most_slots may take them, see route: they make a plan dearer, 40 groups of eight tokens of rank 64, H = 4096,
        // 22 -> 27 us on the host.  A call that names a slot twice may have more; it takes the small items.)
        const bool crowds = plan->expand_split && plan->vf_items.empty() && most_vec_tokens > kExpandTok;
        const int64_t n_vs = (int64_t)plan->vs_items.size(), n_vs_all = n_vs + (int64_t)vs_dual.size();
        bool gang = crowds && pool->shrink_pages == 0 && n_vs_all * most_slots >= kGangFrom;
        const bool gang_expand = crowds && (int64_t)(plan->ve_items.size() + ve_dual.size()) * most_slots >= kGangExpandFrom;
        if (gang) {
            int64_t few = 0, few_dual = 0; // shrink items of a call that takes the larger ones
            for (int32_t gi : order) {
                const Group &g = groups[(size_t)gi];
                const int32_t n = (int32_t)g.toks.size(), tok = n > kExpandTok ? kGangTok : shrink_tok, pages = n > kExpandTok ? kGangPages : shrink_pages;
                if ((int64_t)n < min_tokens) (mfma_group(n) ? few_dual : few) += (int64_t)((n + tok - 1) / tok) * ((g.rank + pages - 1) / pages);
            }
            gang = gang_pays(n_vs, few) || gang_pays(n_vs_all, few + few_dual);
        }
        if (gang || gang_expand) {
            std::vector<Item> gs_dual, ge_dual;
            int32_t pos = 0;
            for (int32_t gi : order) {
                const Group &g = groups[(size_t)gi];
                const int32_t n = (int32_t)g.toks.size(), off = (int32_t)g.arena_off, pos0 = pos;
                pos += n;
                if ((int64_t)n >= min_tokens) continue;
                std::vector<Item> &gs = mfma_group(n) ? gs_dual : plan->gs_items;
                std::vector<Item> &ge = mfma_group(n) ? ge_dual : plan->ge_items;
                if (!gang) {
                } else if (n <= kExpandTok) {
                    plan->max_gv_tok = std::max(plan->max_gv_tok, std::min(n, shrink_tok));
                    for (int32_t p = 0; p < n; p += shrink_tok)
                        for (int32_t j = 0; j < g.rank; j += shrink_pages)
                            plan->gv_items.push_back(Item{off, g.rank, j, std::min(shrink_pages, g.rank - j), pos0 + p, std::min(shrink_tok, n - p), 0, 0});
                } else {
                    const int32_t runs = (g.rank + kGangPages - 1) / kGangPages; // of about equal length
                    for (int32_t p = 0; p < n; p += kGangTok)
                        for (int32_t k = 0; k < runs; ++k) {
                            const int32_t j0 = (int32_t)((int64_t)g.rank * k / runs), j1 = (int32_t)((int64_t)g.rank * (k + 1) / runs);
                            gs.push_back(Item{off, g.rank, j0, j1 - j0, pos0 + p, std::min(kGangTok, n - p), 0, 0});
                        }
                }
                // (one or two tokens left over from the fours have blocks of 16 ranks: an item of their own, unless a wavefront forms whole sums)
                const int32_t fours = g.rank > kOwnRanks && n % kExpandTok <= 2 ? n - n % kExpandTok : n;
                for (int32_t p = 0, nt; gang_expand && p < n; p += nt) {
                    nt = p < fours ? std::min(g.rank <= kOwnRanks ? kGangOwnTok : kGangExpandTok, fours - p) : n - p;
                    for (int y16 = 0; y16 < 2; ++y16) plan->fours[y16] = plan->fours[y16] || fours_pay(pool->dtype, y16, g.rank, nt);
                    for (int32_t c = 0; c < H; c += ecols)
                        ge.push_back(Item{off, g.rank, c, std::min(ecols, H - c), pos0 + p, nt, n <= kExpandTok, 0});
                }
            }
            plan->n_gs_plain = (int32_t)plan->gs_items.size();
            plan->n_ge_plain = (int32_t)plan->ge_items.size();
            plan->gs_items.insert(plan->gs_items.end(), gs_dual.begin(), gs_dual.end());
            plan->ge_items.insert(plan->ge_items.end(), ge_dual.begin(), ge_dual.end());
        }
        plan->n_vs_plain = (int32_t)plan->vs_items.size();
        plan->n_ve_plain = (int32_t)plan->ve_items.size();
        if (plan->chain[0].words > 0)
            for (std::vector<Item> *items : {&vs_dual, &ve_dual}) // their words follow those of the plain items
                for (Item &i : *items) i.run = word(i.run + plan->chain[0].words);
        plan->chain[1].words += plan->chain[0].words;
        plan->chain[1].work += plan->chain[0].work;
        plan->chain[1].tok = std::max(plan->chain[1].tok, plan->chain[0].tok);
        plan->chain[1].shared = plan->chain[1].shared || plan->chain[0].shared;
        plan->vs_items.insert(plan->vs_items.end(), vs_dual.begin(), vs_dual.end());
        plan->ve_items.insert(plan->ve_items.end(), ve_dual.begin(), ve_dual.end());
        plan->n_vs_head = (int32_t)plan->vs_items.size();
        plan->n_ve_head = (int32_t)plan->ve_items.size();
        plan->vs_items.insert(plan->vs_items.end(), vs_tail.begin(), vs_tail.end());
        plan->ve_items.insert(plan->ve_items.end(), ve_tail.begin(), ve_tail.end());
        for (int32_t sub = 0; sub < kMsSubs; ++sub) {
            plan->ms_wgs[sub] = 0;
            plan->ms_lds[sub] = 0;
            for (const MsItem &i : plan->ms_items)
                for (int32_t p = 0; p < i.ntok; p += kMsTok >> sub) {
                    const int32_t rows = std::min(kMsTok >> sub, i.ntok - p);
                    plan->ms_wgs[sub]++;
                    plan->ms_lds[sub] = std::max(plan->ms_lds[sub], ms_lds_bytes((rows <= 32 ? 1 : rows <= 64 ? 2 : 4) + (i.nj + 31) / 32));
                }
        }
        // longest first: the hardware hands a workgroup to a compute unit as one becomes free, so
        // with the big shares at the head of the list and the small ones at its end the launch
        // ends on every unit at about the same time
        std::stable_sort(plan->ms_items.begin(), plan->ms_items.end(), [](const MsItem &a, const MsItem &b) {
            return (int64_t)(a.ntok + a.nj) * (a.c1 - a.c0) > (int64_t)(b.ntok + b.nj) * (b.c1 - b.c0);
        });
        plan->T_act = (int32_t)plan->tok_idx.size();
        // Small batches in one launch, every workgroup computing v for itself: while that is a page or two per
        // wavefront and token.  Measured, us per call, two kernels / one: rank x H x tokens of the largest item
        // 32 Ki and 64 Ki 9.6 / 6.6 (one token of 4 slots), 128 Ki 11.8 / 10.0 (19 groups of rank 8), 10.5 / 10.0 (H = 2048),
        // 9.8 / 9.3 (7 groups of rank 16); 256 Ki 11.3 / 12.6; H = 8192 (two blocks of loads per page) 9.1 / 10.1.
        // Only calls of at most 256 workgroups: a larger launch streams the A pages eight times.
        plan->max_expand_tok = 0;
        bool few_pages = true;
        for (const Item &i : plan->ve_items) {
            plan->max_expand_tok = std::max(plan->max_expand_tok, i.ntok);
            few_pages = few_pages && i.rank <= kSmallRanks && (int64_t)i.rank * H * i.ntok <= 128 * 1024;
        }
        plan->small = pool->fuse_decode != 0 && plan->expand_split && plan->ms_items.empty() && plan->vf_items.empty() && few_pages && H <= 4096;
        plan->v_stride = std::max(kRankPad, (max_rank + kRankPad - 1) / kRankPad * kRankPad);
        plan->n_rank_blocks = (plan->v_stride + kMsRanks - 1) / kMsRanks;
    } catch (const std::bad_alloc &) {
        return fail(SLORA_ENOMEM, "out of host memory while planning");
    }
    return SLORA_OK;
}

int32_t slora_plan::upload(bool once, void *stream)
{
    if (!pool->dev_base) return SLORA_OK; // host-only pool: the plan stays on the host
    const size_t n_tok = tok_idx.size();
    if (n_tok == 0) return SLORA_OK;
    const size_t tok_bytes = (n_tok * sizeof(int32_t) + 63) / 64 * 64;
    const size_t bytes = tok_bytes + (ms_items.size() + mj_items.size()) * sizeof(MsItem) +
                         (vs_items.size() + ve_items.size() + me_items.size() + vf_items.size() + gs_items.size() + gv_items.size() + ge_items.size()) * sizeof(Item);
    // The image is assembled in the pinned half of a recycled buffer set and copied to the
    // device half on the pool's own upload stream: the copy runs beside whatever the caller's
    // streams are doing, and the first launch of the plan waits for it through an event.
    int32_t rc = pool->take_set(&set, bytes, bytes);
    if (rc != SLORA_OK) return rc;
    unsigned char *img = static_cast<unsigned char *>(set->h);
    std::memcpy(img, tok_idx.data(), n_tok * sizeof(int32_t));
    unsigned char *at = img + tok_bytes;
    auto put = [&](const auto &v) {
        const size_t n_bytes = v.size() * sizeof(v[0]);
        if (!v.empty()) std::memcpy(at, v.data(), n_bytes);
        at += n_bytes;
    };
    put(ms_items); // 64-byte records first: everything stays aligned to its size
    put(mj_items);
    put(vs_items);
    put(ve_items);
    put(me_items);
    put(vf_items);
    put(gs_items);
    put(gv_items);
    put(ge_items);
    d_tok_idx = (int32_t *)set->d;
    d_ms = (MsItem *)((unsigned char *)set->d + tok_bytes);
    d_mj = d_ms + ms_items.size();
    d_vs = (Item *)(d_mj + mj_items.size());
    d_ve = d_vs + vs_items.size();
    d_me = d_ve + ve_items.size();
    d_vf = d_me + me_items.size();
    d_gs = d_vf + vf_items.size();
    d_gv = d_gs + gs_items.size();
    d_ge = d_gv + gv_items.size();
    if (once) {
        // A plan of one call: its lists travel on that call's own stream, by a kernel that reads the pinned image, so
        // there is no copy engine to start and no event between two streams, both of which cost the host more than the
        // launch.  236 decode and prompt tokens, H = 4096: 51.3 -> 27.0 us per call back to back.
        rc = pool->arena_ready(stream);
        if (rc == SLORA_OK) rc = launch_copy(set->d, set->h, bytes, stream);
        last_stream = stream;
        return rc;
    }
    void *up_v = nullptr;
    rc = pool->uploads(&up_v);
    if (rc != SLORA_OK) {
        pool->give_set(set, nullptr);
        set = nullptr;
        return rc;
    }
    hipStream_t up = (hipStream_t)up_v;
    hipError_t e = hipMemcpyAsync(set->d, set->h, bytes, hipMemcpyHostToDevice, up);
    if (e == hipSuccess) e = hipEventRecord((hipEvent_t)set->order, up);
    if (e != hipSuccess) {
        rc = hip_fail(e, "uploading the work lists");
        pool->give_set(set, pool->upload_stream);
        set = nullptr;
        return rc;
    }
    last_stream = pool->upload_stream;
    order_recorded = true;
    return SLORA_OK;
}

Route slora_plan::route(int32_t n, bool apply, bool y16) const
{
    Route r;
    r.wide = dual && apply && !y16 && reread * n >= reread_min &&
             v_total_floats(n, pool->dtype, true) * (int64_t)sizeof(float) <= (int64_t)SLORA_STATIC_SCRATCH_BYTES;
    r.fused = apply && !vf_items.empty();
    r.small = apply && small && (int64_t)ve_items.size() * n <= 256;
    // Larger vector items, where the small ones are more workgroups than the GPU holds at a time.  us per kernel, small / large:
    // shrink, 2066 / 294 workgroups 22.1 / 13.7, 2604 / 333 12.4 / 9.6, 1446 / 363 15.2 / 13.1, but 1520 / 208 7.6 / 8.1,
    // 792 / 748 9.2 / 12.5, 752 / 376 8.4 / 10.6, 744 / 96 9.6 / 13.1; expand, 6016 / 1536 22.6 / 15.8, 4338 / 1098 16.0 / 11.1,
    // 912 / 792 7.8 / 7.5, but 600 / 288 8.3 / 11.2, 414 / 333 10.4 / 12.8.
    // The small items beside the larger ones pay for them (fewer of the gang kernel's workgroups fit a compute unit), so the larger ones
    // must leave half the workgroups at most.  Workgroups small / large, us per call: 4992 / 2016 60 / 53, 4920 / 2085 53.6 / 49.0, 4480 / 2240
    // 59 / 56, 2880 / 1200 40.9 / 39.1, but 2560 / 1440 44.8 / 46.6, 5056 / 3392 38.8 / 40.8, 10068 / 6993 49 / 52, 2080 / 1800 33.0 / 35.7, 7680 / 6560
    // 37.5 / 43.5; 2304 / 1408 32.4 / 32.3, 2880 / 1760 39.4 / 39.4, and one composition found the other way round, 3072 / 2064 39.4 / 37.3.
    const int64_t small_wgs = (int64_t)n_vs(r), large_wgs = (int64_t)(n_gs(r) + gv_items.size());
    r.gang = n_gs(r) > 0 && small_wgs * n >= kGangFrom && large_wgs * n >= 256 && gang_pays(small_wgs, large_wgs);
    r.gang_expand = !ge_items.empty() && (int64_t)n_ve(r) * n >= kGangExpandFrom && (int64_t)n_ge(r) * n >= 512;
    // Tokens of an item per workgroup of the MFMA shrink.  The items of a call of modest size are too
    // few for the GPU; halves or quarters of their tokens read the pages two or four times as often,
    // which pays only while compute units stand idle: 111 items 62 us in as many workgroups, 48 in 153,
    // 35 in 222, but 236 items 47 -> 52 and 252 items 55 -> 58 us (launches of three or four slots).
    // Between: 177 items of three slots 39 us whole, 44 in halves; 189 halves against 345 quarters 15 us less.
    // Quarters pay a little less long than halves: 126 halves 31.6, 252 quarters 29.0 us; 132 / 264 38.4 / 36.2, but 148 / 296
    // 33.4 / 41.0, 184 / 368 34.0 / 43.6 us; 148 whole / 296 halves 63.8 / 51.2.
    while (r.sub + 1 < kMsSubs && ms_wgs[r.sub] * n < (r.sub == 0 ? 160 : 140)) r.sub++;
    // Calls of fewer slots than the list's runs are made for share a run out until there are 1024 workgroups.  Sixteen
    // prompts in a pool of 64 slots, us per call of one slot in 256 / 768 / 1024 / 1536 / 2048 workgroups 84 / 63 /
    // 63 / 63 / 67 (16-bit y 81 / 54 / 54 / 55 / 59), of two in 512 / 1024 / 1536 / 2048 101 / 91 / 90 / 93 (87 / 74 / 71 /
    // 76), of three in 768 / 1536 / 2304 129 / 124 / 127 (96 / 95 / 99).
    if (!me_items.empty()) {
        const int64_t wgs = (int64_t)me_items.size() * n;
        r.parts = (int32_t)std::min<int64_t>(me_run, (1024 + wgs - 1) / wgs);
    }
    return r;
}

// Both stages in one launch, us two kernels / one launch.  Large calls are bound by HBM, and the two kernels hold more wavefronts: 4096 workgroups, four (three from H = 6152 on)
// of which a compute unit holds at a time.  128 tokens of rank 32, H = 4096, 1 / 2 / 4 slots, 2048 / 4096 / 8192: 18.5 / 15.5, 29.8 / 26.4, 52.8 / 56.6; 60 groups of four of
// rank 32, 4 slots, 3840: 39.4 / 36.9; 100 of rank 64, H = 2048, 4 slots, 8000: 41.0 / 42.3, fours of them 52.3 / 60.4; 20 groups of eight tokens of rank 64, 3 slots, 2880: 29.8 / 23.0.
// Fewer where
//  - an expand item is little work (ranks x tokens below 16, below 4): its workgroups wait in their places all the same.  71 tokens of rank 1, H = 3072, 8 slots, 3976: 13.2 / 14.6, 252
//    pairs, H = 1024, 4 slots, 3024: 10.6 / 11.2, but 200 of rank 4, 2400: 10.6 / 9.8; 63 of rank 8, H = 3072, 8 slots, 4032: 15.9 / 16.6, but 70 groups of four of rank 1, 3360: 18.8 / 17.8.  Three quarters of
//    that from H = 6152 on, where three of its workgroups fit a compute unit: pairs of ranks 1-8, H = 8192, 25 groups, 8 slots, 3448: 16.5 / 18.4, H = 7168, 33 groups, 6 slots, 3042: 15.8 / 17.7, 47 calls of up to 2560 1.05 times as fast.
//  - rows of x leave a compute unit three or two workgroups (more than 40 or 56 KiB): 60 groups of four tokens of rank 64, H = 8192, 2 slots, 3840: 67.8 / 75.9, but 20 of rank 32, 4 slots,
//    1920: 30.0 / 26.1; with little work in an expand item 30 groups of eight of rank 4, H = 8192, 2 slots, 2040: 18.7 / 20.6, ten of sixteen of rank 8, 1440: 16.4 / 17.3, but of rank 4, 1360: 16.0 / 15.8;
//    fours of ranks 1-8, H = 7168 (64 KiB as well: whole chunks of 512 elements, 16 from H = 6152 on), 30 groups, 4 slots, 1920: 16.0 / 18.5, 33, 6 slots, 1824: 15.9 / 17.9, but 36 calls of 1408 to 1664 1.05 times as fast.
// Calls that are mostly shrink (many ranks of short rows) have little in flight in its wavefronts; five or more workgroups fit a compute unit in a kernel of its own; and rows
// of a second 64 ranks are requested after the wait.
//  - Six times as many shrink items as expand items: 640 of them.  60 tokens of rank 128, H = 2048, 2160: 16.8 / 18.9, 100 pairs in 3600 25.5 / 30.4, but 20 of rank 128, H = 1024, 680: 10.4 / 7.9.
//  - Four times, pairs of tokens (whose B rows are not streamed here): 2048.  20 of rank 128, H = 3072, 4 slots, 3040: 29.0 / 34.0; 14 of rank 128, H = 4096, 4 slots, 2240: 26.4 / 28.6; 9, 6 slots, 2160: 26.9 / 28.7, but
//    7 of them, 7 slots, 1960: 26.5 / 25.7; nor, of 112 ranks or more each, between one round of the GPU's 1024 places (a few expand items may wait) and one and a half: ten of rank 128, H = 3072, 3 slots,
//    1140: 13.2 / 15.7, 16 of rank 128, H = 3584, 2 slots, 1248: 14.6 / 15.9, 40, H = 2888, 1520: 15.7 / 18.1, 95 such calls 0.94 times as fast, but 10 of rank 128, H = 4096, 1600 and H = 3584, 1.07.  Threes and fours: 3072.  42 fours of rank 128, H = 4096, 2 slots, 3360: 42.8 / 45.6, but 17 of rank 100, H = 3072, 5 slots, 2635: 30.5 / 28.3.
//  - Four and a half times, single tokens: H < 2048 2048.  18 of ranks 30-130, H = 1920, 8 slots, 3744: 21.9 / 23.9; 15 of rank 64, H = 1072, 8 slots, 2280: 12.7 / 13.0; but 59 of rank 64, H = 1536, 3 slots, 3363: 19.5 / 18.1.
//    H >= 2048 not between one round of the GPU's 1024 places and one and a half.  Ten of rank 100, H = 2560, 4 slots, 1200: 13.3 / 14.5, five, 8 slots 12.9 / 14.6, but 6 slots, 900: 12.0 / 11.0;
//    13, 8 slots, 3120: 25.2 / 23.7; 30 of rank 128, H = 2048, 1080: 12.3 / 13.2; but 32 of ranks 5-130, H = 1120, 2 slots, 1292: 13.0 / 12.0.
bool slora_plan::chain_pays(int32_t n, const Route &r) const
{
    const Chain &c = chain_of(r);
    const int64_t shrinks = (int64_t)n_vs(r) * n, expands = (int64_t)n_ve(r) * n, wgs = shrinks + expands;
    if (!expand_split || pool->fuse_decode == 0 || shrinks == 0 || r.gang || r.gang_expand || pool->H > kChainMaxH || wgs > 65535 || c.words * n > INT32_MAX) return false;
    if (shrinks > 6 * expands && shrinks > 640) return false;
    if (shrinks >= 4 * expands && c.tok >= 2 && wgs > (c.tok == 2 ? 2048 : 3072)) return false;
    if (shrinks >= 4 * expands && c.tok == 2 && shrinks * ((pool->H + 511) / 512) >= 28 * expands && wgs > 1088 && wgs <= 1536) return false;
    if (2 * shrinks > 9 * expands && c.tok == 1 && (pool->H < 2048 ? wgs > 2048 : wgs > 1024 && wgs <= 1536)) return false;
    const int64_t work = c.work * n / expands, rows = (int64_t)c.tok * pool->H * 2;
    if (rows > 40960) return wgs <= (c.tok < 4 || pool->H <= 6144 || work >= 64 ? 2048 : pool->H <= 7168 ? 1664 : 1408);
    return wgs <= (work < 4 ? 2560 : work < 16 ? (pool->H > 6144 ? 2688 : 3584) : 4096);
}

size_t slora_plan::most_chain_words(int32_t n) const
{
    int64_t most = 0;
    for (int32_t m = 1; m <= n; ++m)
        for (int y16 = 0; y16 <= (dual ? 1 : 0); ++y16) {
            const Route r = route(m, true, y16 != 0);
            if (chain_pays(m, r)) most = std::max(most, chain_of(r).words * m);
        }
    return (size_t)most;
}

int64_t slora_plan::v_most_floats(int32_t n, int32_t dtype) const
{
    int64_t most = v_total_floats(n, dtype, !dual);
    for (int32_t m = 1; dual && m <= n; ++m) // more slots may need less: not every call of a dual plan takes the MFMA form
        if (route(m, true, false).wide) most = std::max(most, v_total_floats(m, dtype, true));
    return most;
}

void slora_plan::fill_args(MultiArgs &a, int32_t n, float *v, const Route &r) const
{
    const int64_t per_slot = v_slot_floats(pool->dtype, mfma_on(r));
    for (int32_t k = 0; k < n; ++k) a.v[k] = v + (int64_t)k * per_slot;
    a.vfrag_off = (int64_t)T_act * v_stride;
    a.vexp_off = a.vfrag_off + vfrag_floats(pool->dtype);
    a.part_off = a.vexp_off + vexp_floats();
}

int32_t slora_plan::enter(void *stream)
{
    if (!set || stream == last_stream) return SLORA_OK;
    hipError_t e = hipSuccess;
    if (!order_recorded) e = hipEventRecord((hipEvent_t)set->order, (hipStream_t)last_stream);
    if (e == hipSuccess) e = hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)set->order, 0);
    if (e != hipSuccess) return hip_fail(e, "ordering the plan's work between two streams");
    last_stream = stream;
    order_recorded = false;
    return SLORA_OK;
}

namespace {

int32_t check_plan(slora_plan *plan, int32_t n, const int32_t *slots)
{
    if (!plan) return fail(SLORA_EINVAL, "plan is NULL");
    if (n < 1 || n > SLORA_MAX_MULTI) return fail(SLORA_EINVAL, "n=%d must be in [1, %d]", n, SLORA_MAX_MULTI);
    if (!slots) return fail(SLORA_EINVAL, "slots is NULL");
    for (int32_t k = 0; k < n; ++k)
        if (slots[k] < 0 || slots[k] >= plan->pool->n_slots)
            return fail(SLORA_ERANGE, "slot=%d outside [0, %d)", slots[k], plan->pool->n_slots);
    if (plan->generation != plan->pool->unload_generation)
        return fail(SLORA_EBUSY, "plan is stale: an adapter was unloaded after it was built");
    if (!plan->pool->dev_base) return fail(SLORA_EHIP, "pool is host-only (dev_base == NULL)");
    return SLORA_OK;
}

// whether a y of the call shares memory with an x
bool y_overlaps_x(const slora_plan *plan, int32_t n, const void *const *x, void *const *y, bool y16)
{
    const uintptr_t x_bytes = (uintptr_t)plan->T * (uintptr_t)plan->pool->H * 2, y_bytes = y16 ? x_bytes : 2 * x_bytes;
    for (int32_t k = 0; k < n; ++k)
        for (int32_t m = 0; m < n; ++m) {
            const uintptr_t xa = reinterpret_cast<uintptr_t>(x[k]), ya = reinterpret_cast<uintptr_t>(y[m]);
            if (xa < ya + y_bytes && ya < xa + x_bytes) return true;
        }
    return false;
}

// scratch: where v goes; NULL = the plan's own buffer (grown on demand)
// y != NULL: part of an apply - decode groups the plan marked for it run both stages in one
// launch here, and the two-stage launches (here and in do_expand) cover the other groups only.
int32_t do_shrink(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x, void *stream,
                  float *scratch = nullptr, void *const *y = nullptr, bool y16 = false)
{
    if (!x) return fail(SLORA_EINVAL, "x is NULL");
    if (plan->T_act == 0) return SLORA_OK;
    MultiArgs a{};
    a.n = n;
    for (int32_t k = 0; k < n; ++k) {
        if (!x[k]) return fail(SLORA_EINVAL, "x[%d] is NULL", k);
        if (reinterpret_cast<uintptr_t>(x[k]) & 15) return fail(SLORA_EINVAL, "x[%d] must be 16-byte aligned", k);
        a.x[k] = x[k];
        a.slot[k] = slots[k];
    }
    DeviceScope dev(plan->pool->device);
    if (dev.status() != SLORA_OK) return dev.status();
    Route route = plan->route(n, y != nullptr, y16);
    // the two kernels have read all of x before y is written; in the one-launch kernels other workgroups
    // still read it
    const bool overlaps = y && y_overlaps_x(plan, n, x, y, y16);
    if (overlaps) route.small = false;
    // the page lists of every adapter the plan names went to the device when it was built
    float *v = scratch;
    int32_t rc = SLORA_OK;
    if (!v) {
        // (room for the words is made whatever the call, so that a plan's buffers are sized once)
        if (plan->most_slots < n) {
            plan->most_words = plan->most_chain_words(n);
            plan->most_slots = n;
        }
        rc = plan->pool->grow_v(plan->set, (size_t)plan->v_most_floats(n, plan->pool->dtype), plan->most_words, stream);
        v = plan->set->v;
    }
    if (rc == SLORA_OK) rc = plan->enter(stream);
    if (rc == SLORA_OK && !scratch && y && !overlaps && plan->chain_pays(n, route) && (size_t)(plan->chain_of(route).words * n) <= plan->set->hand_cap &&
        !stream_captures(stream) && plan->pool->next_launch(plan->set, stream)) {
        route.chain = true;
        route.small = false;
    }
    if (rc != SLORA_OK) return rc;
    plan->fill_args(a, n, v, route);
    if (route.fused || route.small || route.chain)
        for (int32_t k = 0; k < n; ++k) a.y[k] = y[k];
    if (route.fused || route.small) rc = launch_fused(plan, n, a, stream, y16, route);
    if (rc == SLORA_OK && route.chain) {
        rc = launch_chain(plan, n, a, stream, y16, route);
        plan->pool->hand_overs += rc == SLORA_OK;
    }
    if (rc == SLORA_OK && !route.small) rc = launch_shrink(plan, n, a, stream, route);
    if (rc == SLORA_OK) {
        plan->v_slots = n;
        plan->v_used = v;
        plan->v_route = route;
    }
    return rc;
}

int32_t check_y(int32_t n, void *const *y)
{
    if (!y) return fail(SLORA_EINVAL, "y is NULL");
    for (int32_t k = 0; k < n; ++k) {
        if (!y[k]) return fail(SLORA_EINVAL, "y[%d] is NULL", k);
        if (reinterpret_cast<uintptr_t>(y[k]) & 15) return fail(SLORA_EINVAL, "y[%d] must be 16-byte aligned", k);
        for (int32_t m = 0; m < k; ++m)
            if (y[m] == y[k]) return fail(SLORA_EINVAL, "y[%d] and y[%d] are the same buffer", m, k);
    }
    return SLORA_OK;
}

int32_t do_expand(slora_plan *plan, int32_t n, const int32_t *slots, void *const *y, void *stream, bool y16,
                  bool after_apply = false)
{
    int32_t rc = check_y(n, y);
    if (rc != SLORA_OK) return rc;
    if (plan->T_act == 0) return SLORA_OK;
    MultiArgs a{};
    a.n = n;
    for (int32_t k = 0; k < n; ++k) {
        a.y[k] = y[k];
        a.slot[k] = slots[k];
    }
    Route route = plan->v_route;
    if (!after_apply) route.chain = false; // v is in memory as well
    if (plan->v_slots != n || !plan->v_used || (!after_apply && route.fused))
        return fail(SLORA_EINVAL, "expand of %d slot(s) needs a preceding slora_lora_shrink of %d slot(s)", n, n);
    if (after_apply && route.small) return SLORA_OK; // both stages ran in one launch
    DeviceScope dev(plan->pool->device);
    if (dev.status() != SLORA_OK) return dev.status();
    rc = plan->enter(stream);
    if (rc != SLORA_OK) return rc;
    plan->fill_args(a, n, plan->v_used, route);
    return launch_expand(plan, n, a, stream, y16, route);
}

} // namespace

namespace {
int32_t make_plan(slora_pool *pool, slora_plan **out, const int32_t *token_adapter_ids, int32_t T,
                  const int32_t *seg_offsets, int32_t n_seg, int32_t call_slots, void *stream = nullptr)
{
    clear_error();
    if (!pool || !out) return fail(SLORA_EINVAL, "NULL argument");
    *out = nullptr;
    slora_plan *p = new (std::nothrow) slora_plan;
    if (!p) return fail(SLORA_ENOMEM, "out of host memory");
    p->pool = pool;
    p->generation = pool->unload_generation;
    int32_t rc = build_plan(pool, p, token_adapter_ids, T, seg_offsets, n_seg, call_slots);
    if (rc == SLORA_OK && pool->dev_base) {
        DeviceScope dev(pool->device);
        rc = dev.status();
        // page lists of adapters loaded since the last plan, then this plan's work lists
        if (rc == SLORA_OK) rc = pool->sync_device();
        // (a capturing stream takes no copy that reads an image which is recycled: such a call is refused when it waits)
        bool once = call_slots > 0 && rc == SLORA_OK;
        if (once) {
            hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
            once = hipStreamIsCapturing((hipStream_t)stream, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone;
            if (!once) (void)hipGetLastError();
        }
        if (rc == SLORA_OK) rc = p->upload(once, stream);
    }
    if (rc != SLORA_OK) {
        if (p->set) pool->give_set(p->set, p->last_stream);
        delete p;
        return rc;
    }
    pool->live_plans++;
    *out = p;
    return SLORA_OK;
}
} // namespace

extern "C" {

int32_t slora_batch_plan(slora_pool *pool, slora_plan **out, const int32_t *token_adapter_ids, int32_t T,
                         const int32_t *seg_offsets, int32_t n_seg)
{
    return make_plan(pool, out, token_adapter_ids, T, seg_offsets, n_seg, 0);
}

int32_t slora_plan_destroy(slora_plan *plan)
{
    clear_error();
    if (!plan) return SLORA_OK;
    if (plan->set) {
        // Nothing is freed and nothing is waited for: the buffers go back to the pool with an
        // event recorded behind the plan's last launch and are handed out again after it.
        DeviceScope dev(plan->pool->device);
        plan->pool->give_set(plan->set, plan->last_stream);
        plan->set = nullptr;
    }
    plan->pool->live_plans--;
    delete plan;
    return SLORA_OK;
}

int32_t slora_plan_info(const slora_plan *plan, int64_t *out, int32_t n)
{
    clear_error();
    if (!plan || !out || n < 0 || n > SLORA_PLAN_INFO_N) return fail(SLORA_EINVAL, "bad arguments");
    const int64_t v[SLORA_PLAN_INFO_N] = {plan->T_act,
                                          plan->n_groups,
                                          plan->n_groups_vec,
                                          plan->n_groups_mfma,
                                          (int64_t)plan->vs_items.size(),
                                          (int64_t)plan->ve_items.size(),
                                          (int64_t)plan->ms_items.size(),
                                          plan->me_wgs(),
                                          plan->v_stride,
                                          plan->sum_rank,
                                          plan->n_sync,
                                          plan->v_slot_floats(plan->pool->dtype, true) * (int64_t)sizeof(float),
                                          (int64_t)plan->vf_items.size()};
    for (int32_t k = 0; k < n; ++k) out[k] = v[k];
    return SLORA_OK;
}

int32_t slora_lora_shrink(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x, void *stream)
{
    clear_error();
    int32_t rc = check_plan(plan, n, slots);
    return rc != SLORA_OK ? rc : do_shrink(plan, n, slots, x, stream);
}

int32_t slora_lora_expand(slora_plan *plan, int32_t n, const int32_t *slots, float *const *y, void *stream)
{
    clear_error();
    int32_t rc = check_plan(plan, n, slots);
    return rc != SLORA_OK ? rc : do_expand(plan, n, slots, reinterpret_cast<void *const *>(y), stream, false);
}

int32_t slora_lora_expand_y16(slora_plan *plan, int32_t n, const int32_t *slots, void *const *y, void *stream)
{
    clear_error();
    int32_t rc = check_plan(plan, n, slots);
    return rc != SLORA_OK ? rc : do_expand(plan, n, slots, y, stream, true);
}

namespace {
int32_t apply_multi(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x, void *const *y,
                    void *stream, bool y16, bool static_scratch = false)
{
    clear_error();
    int32_t rc = check_plan(plan, n, slots);
    if (rc != SLORA_OK) return rc;
    rc = check_y(n, y); // validate the y side before the shrink is enqueued
    if (rc != SLORA_OK) return rc;
    float *scratch = nullptr;
    if (static_scratch) {
        const bool mfma = plan->mfma_on(plan->route(n, true, y16));
        const int64_t need = plan->v_total_floats(n, plan->pool->dtype, mfma) * (int64_t)sizeof(float);
        if (need > (int64_t)SLORA_STATIC_SCRATCH_BYTES)
            return fail(SLORA_ERANGE,
                        "this batch needs %lld bytes of scratch for %d slot(s), the static scratch holds %lld: use "
                        "fewer slots per call or slora_lora_apply_multi",
                        (long long)need, n, (long long)SLORA_STATIC_SCRATCH_BYTES);
        scratch = static_cast<float *>(plan->pool->static_scratch);
        if (!scratch) return fail(SLORA_EHIP, "the static scratch was not resolved for this pool's device");
    }
    rc = do_shrink(plan, n, slots, x, stream, scratch, y, y16);
    if (rc != SLORA_OK) return rc;
    return do_expand(plan, n, slots, y, stream, y16, true);
}
} // namespace

int32_t slora_lora_apply_multi_static(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x,
                                      float *const *y, void *stream)
{
    return apply_multi(plan, n, slots, x, reinterpret_cast<void *const *>(y), stream, false, true);
}

int32_t slora_lora_apply_multi(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x,
                               float *const *y, void *stream)
{
    return apply_multi(plan, n, slots, x, reinterpret_cast<void *const *>(y), stream, false);
}

int32_t slora_lora_apply_multi_y16(slora_plan *plan, int32_t n, const int32_t *slots, const void *const *x,
                                   void *const *y, void *stream)
{
    return apply_multi(plan, n, slots, x, y, stream, true);
}

int32_t slora_lora_apply(slora_plan *plan, int32_t slot, const void *x, float *y, void *stream)
{
    const void *xs[1] = {x};
    float *ys[1] = {y};
    return slora_lora_apply_multi(plan, 1, &slot, xs, ys, stream);
}

int32_t slora_lora_shrink_expand(slora_pool *pool, int32_t slot, const void *x, const int32_t *token_adapter_ids,
                                 const int32_t *seg_offsets, int32_t n_seg, int32_t T, float *y, void *stream)
{
    slora_plan *plan = nullptr;
    int32_t rc = make_plan(pool, &plan, token_adapter_ids, T, seg_offsets, n_seg, 1, stream);
    if (rc != SLORA_OK) return rc;
    rc = slora_lora_apply(plan, slot, x, y, stream);
    std::string keep = last_error_cstr();
    (void)slora_plan_destroy(plan); // the plan's buffers are recycled after the launches have run
    if (rc != SLORA_OK) fail(rc, "%s", keep.c_str());
    return rc;
}

} // extern "C"
