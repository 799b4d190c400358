// Host side of the SP-KV C ABI: configuration checks, arena carving, the host's
// conservative capacity bound (the "safe budget" idea of the paper's appendix "Inference
// Kernels": capacity is checked on the host without reading the device until a worst-case
// bound trips), and kernel launches.  See include/spkv.h for the contract.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "spkv_internal.h"

namespace {

constexpr size_t kAlign = 256;
constexpr int kFallbackItems = 2944;   // 11.5 one-wave workgroups per CU on 256 CUs (MI355X, 12 fit)
constexpr int kMaxTimedLaunches = 8192;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Carve {
    size_t ring, ring_logit, t_pair, kept_len, gate_on, pool_next, free_top, free_pages, err_flag,
        page_table, pool,
        pos_pool, logit_pool, seg_count, seg_on, bulk_info, part_acc, part_ml, pair_items,
        pair_ticket, pos_scratch, total;
    int n_pairs, G, n_ring_pages, pt_cap, n_pages, n_seg_cap, max_items;
};

bool config_ok(const spkv_config_t* c) {
    if (c == nullptr) return false;
    if (c->batch < 1 || c->batch > SPKV_MAX_BATCH) return false;
    if (c->n_kv_heads < 1 || c->n_q_heads < 1 || c->n_q_heads % c->n_kv_heads != 0) return false;
    if (c->n_q_heads / c->n_kv_heads > 16) return false;
    if ((int64_t)c->batch * c->n_kv_heads > 16384) return false;
    if (c->head_dim != 64 && c->head_dim != 128) return false;
    if (c->window < 1 || c->window > (1 << 20)) return false;
    if (c->page_tokens != 0 && c->page_tokens != SPKV_PAGE_TOKENS) return false;
    if (std::isnan(c->tau)) return false;
    if (c->max_context < 1 || c->max_context > (1 << 30)) return false;
    if (c->max_total_kept_tokens < 0 || c->max_total_kept_tokens > ((int64_t)1 << 40)) return false;
    return true;
}

bool carve(const spkv_config_t* c, Carve* out) {
    if (!config_ok(c)) return false;
    Carve k{};
    k.n_pairs = c->batch * c->n_kv_heads;
    k.G = c->n_q_heads / c->n_kv_heads;
    k.n_ring_pages = (c->window + kPageTokens - 1) / kPageTokens;
    const int64_t max_evicted = c->max_context > c->window ? c->max_context - c->window : 0;
    k.pt_cap = (int)((max_evicted + kPageTokens - 1) / kPageTokens) + 1;
    const int64_t n_pages = (c->max_total_kept_tokens + kPageTokens - 1) / kPageTokens + k.n_pairs;
    if (n_pages > ((int64_t)1 << 30)) return false;
    k.n_pages = (int)n_pages;
    k.n_seg_cap = (int)(((int64_t)c->max_context + kSegTokens - 1) / kSegTokens) + 1;
    // Work-item slots: 128 per pair leaves room for a pair 40 times longer than the mean at
    // the default item count; at least enough for the largest item target on one pair.
    // The multi-token kernels store 16, 32 or 64 columns per slot instead of G: two slots of
    // 64 columns per pair must fit whatever the shape (only caches of thousands of pairs
    // with small groups reach this term).
    k.max_items = std::max(kMaxItemTarget + k.n_pairs, std::min(k.n_pairs * 128, 1 << 17));
    k.max_items = std::max(k.max_items, (k.n_pairs * 128 + k.G - 1) / k.G);
    const size_t page_bytes = (size_t)spkv_page_elems(c->head_dim) * 2;
    size_t off = 0;
    auto take = [&off](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes);
        return at;
    };
    k.ring = take((size_t)k.n_pairs * k.n_ring_pages * page_bytes);
    k.ring_logit = take((size_t)k.n_pairs * c->window * 4);
    k.t_pair = take((size_t)k.n_pairs * 4);
    k.kept_len = take((size_t)k.n_pairs * 4);
    k.gate_on = take((size_t)k.n_pairs * 4);
    k.pool_next = take(4);
    k.free_top = take(4);
    k.free_pages = take((size_t)k.n_pages * 4);
    k.err_flag = take(4);
    k.page_table = take((size_t)k.n_pairs * k.pt_cap * 4);
    k.pool = take((size_t)k.n_pages * page_bytes);
    k.pos_pool = take((size_t)k.n_pages * kPageTokens * 4);
    k.logit_pool = take((size_t)k.n_pages * kPageTokens * 4);
    k.seg_count = take((size_t)k.n_pairs * k.n_seg_cap * 4);
    k.seg_on = take((size_t)k.n_pairs * k.n_seg_cap * 4);
    k.bulk_info = take((size_t)k.n_pairs * 32);
    k.part_acc = take((size_t)k.max_items * k.G * c->head_dim * 4);
    k.part_ml = take((size_t)k.max_items * k.G * 2 * 4);
    k.pair_items = take((size_t)k.n_pairs * 4);
    k.pair_ticket = take((size_t)k.n_pairs * 4);
    k.pos_scratch = take((size_t)k.pt_cap * kPageTokens * 4);
    k.total = off;
    *out = k;
    return true;
}

float logit_threshold(float tau) {
    const double t = (double)tau;
    if (t <= 0.0) return -INFINITY;
    if (t >= 1.0) return INFINITY;
    return (float)std::log(t / (1.0 - t));
}

int64_t pages_for(int64_t len) { return (len + kPageTokens - 1) / kPageTokens; }

}  // namespace

// Scratch for spkv_decode_attention_static: the split-K partials of callers that cannot
// allocate.  One copy per GPU the library runs on, held until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress; kernels get the address
// that call returns for the current device.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

// Device address of the current device's copy of `scratch` (looked up once per device);
// null if the runtime cannot tell.
void* static_scratch_of_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

struct spkv_cache {
    spkv_config_t cfg;
    Carve carve;
    SpkvView view;
    char* arena;
    size_t arena_bytes;
    std::vector<int32_t> T;       // tokens per sequence (exact: the host sees every append)
    std::vector<int32_t> L_ub;    // per (seq, head): upper bound of the long-term length
    int64_t pages_ub;             // sum of pages_for(L_ub): upper bound of pool pages in use
    bool bound_is_loose;          // a bulk append grew L_ub by far more than the truth
    // Single-token steps add one to L_ub per pair and step although only the keep rate's share
    // is kept, so the bound drifts away from the lengths and the work partition derived from
    // it would come out too coarse.  `slack` counts what was added since the bound was last
    // exact; past 1/16 of the bound the lengths are copied to pinned host memory behind the
    // step just issued (no wait) and adopted by the first later call that finds the copy done.
    int64_t slack;
    int32_t* snap_host;           // pinned, twice [n_pairs] and a ticket; null if the allocation failed
    int32_t snap_ticket;          // the ticket that comes with the copy enqueued last
    bool snap_pending;
    std::vector<int32_t> snap_ev; // per sequence: pairs pushed out of the window since the copy
    // Lengths that a prompt append sent by itself (second half of the buffer): current while no call
    // has changed any since.
    int32_t sent_ticket;
    bool sent;
    // What is known of the lengths themselves: L_ub less what `since_exact` (per sequence) added to
    // it is the length when the bound was last exact -- from which the lists have grown by single
    // tokens and short chunks only (lists_known), or by a prompt as well.
    std::vector<int32_t> since_exact;
    bool lists_known, snap_covers;    // snap_covers: no prompt since the copy was enqueued
    bool chunk_since_prompt;          // a copy costs a call some 8 us: not for a single short chunk
    int item_target;
    int merge_waves;              // SPKV_OPT_MERGE_WAVES (0 = per call)
    int step_launches;            // SPKV_OPT_STEP_LAUNCHES (0 = per call)
    int n_sink;                   // always-kept first positions (SPKV_OPT_SINK_TOKENS)
    int one_round_items;          // items the chip runs in one resident round, with a margin
    int compact_items;            // item target under the gapless numbering
    int chunk_round_items;        // as one_round_items, for the chunk kernel
    SpkvSplit split;              // partition used by the last decode call
    mutable std::vector<uint64_t> seen;   // scratch of sequences_alike: room for every sequence
    bool timing;
    bool split_only;
    std::vector<hipEvent_t> events;   // pairs (before, after)
    int n_timed;
};

namespace {

// Point the device-side view at the regions of the cache's arena.
void bind_view(spkv_cache* c) {
    const spkv_config_t* cfg = &c->cfg;
    const Carve& k = c->carve;
    SpkvView& v = c->view;
    v.B = cfg->batch;
    v.Hq = cfg->n_q_heads;
    v.Hkv = cfg->n_kv_heads;
    v.G = k.G;
    v.D = cfg->head_dim;
    v.w = cfg->window;
    v.n_pairs = k.n_pairs;
    v.n_ring_pages = k.n_ring_pages;
    v.pt_cap = k.pt_cap;
    v.n_pages = k.n_pages;
    v.n_seg_cap = k.n_seg_cap;
    v.max_items = k.max_items;
    v.theta = logit_threshold(cfg->tau);
    v.n_sink = c->n_sink;
    char* a = c->arena;
    v.ring = reinterpret_cast<uint16_t*>(a + k.ring);
    v.ring_logit = reinterpret_cast<float*>(a + k.ring_logit);
    v.t_pair = reinterpret_cast<int32_t*>(a + k.t_pair);
    v.kept_len = reinterpret_cast<int32_t*>(a + k.kept_len);
    v.gate_on = reinterpret_cast<int32_t*>(a + k.gate_on);
    v.pool_next = reinterpret_cast<int32_t*>(a + k.pool_next);
    v.free_top = reinterpret_cast<int32_t*>(a + k.free_top);
    v.free_pages = reinterpret_cast<int32_t*>(a + k.free_pages);
    v.err_flag = reinterpret_cast<int32_t*>(a + k.err_flag);
    v.page_table = reinterpret_cast<int32_t*>(a + k.page_table);
    v.pool = reinterpret_cast<uint16_t*>(a + k.pool);
    v.pos_pool = reinterpret_cast<int32_t*>(a + k.pos_pool);
    v.logit_pool = reinterpret_cast<float*>(a + k.logit_pool);
    v.seg_count = reinterpret_cast<int32_t*>(a + k.seg_count);
    v.seg_on = reinterpret_cast<int32_t*>(a + k.seg_on);
    v.bulk_info = reinterpret_cast<int32_t*>(a + k.bulk_info);
    v.part_acc = reinterpret_cast<float*>(a + k.part_acc);
    v.part_ml = reinterpret_cast<float*>(a + k.part_ml);
    v.pair_items = reinterpret_cast<int32_t*>(a + k.pair_items);
    v.pair_ticket = reinterpret_cast<int32_t*>(a + k.pair_ticket);
    v.pos_scratch = reinterpret_cast<int32_t*>(a + k.pos_scratch);
}

// What an empty cache needs cleared: everything up to the pool (ring, counters, tables) and the
// counters behind it.  Pages keep what they hold: whoever begins a half-page clears the values behind
// the list's end (clear_list_end).  Nothing else is read before it is written.
hipError_t clear_arena(char* arena, const Carve& k, hipStream_t s) {
    return spkv_launch_reset(arena, k.pool, k.pair_items, k.pos_scratch - k.pair_items, s);
}

// The host's bound from the exact lengths.
void adopt_lengths(spkv_cache* c, const int32_t* len) {
    int64_t pages = 0;
    for (int p = 0; p < c->carve.n_pairs; ++p) {
        c->L_ub[p] = len[p];
        pages += pages_for(len[p]);
    }
    c->pages_ub = pages;
    c->bound_is_loose = false;
    c->slack = 0;
    std::fill(c->since_exact.begin(), c->since_exact.end(), 0);
    c->lists_known = true;
    c->snap_pending = c->sent = false;
}

// Read the exact long-term lengths back and tighten the host's bound.  Synchronises.
int refresh_bound(spkv_cache* c, hipStream_t s, int32_t* kept_len_out) {
    std::vector<int32_t> len(c->carve.n_pairs);
    if (hipStreamSynchronize(s) != hipSuccess) return SPKV_E_HIP;
    if (hipMemcpy(len.data(), c->view.kept_len, len.size() * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return SPKV_E_HIP;
    adopt_lengths(c, len.data());      // a copy still on its way is older than what was just read
    if (kept_len_out != nullptr) std::memcpy(kept_len_out, len.data(), len.size() * 4);
    return SPKV_OK;
}

bool being_captured(hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) == hipSuccess) return cap != hipStreamCaptureStatusNone;
    (void)hipGetLastError();          // no answer: not an error of the next launch
    return true;
}

// A prompt append sends the lengths it leaves to the host by itself (spkv_bulk_scatter).  Not under
// capture: a replay would send them again, with an old ticket.
SpkvLengthCopy prompt_length_copy(spkv_cache* c, int n_max, hipStream_t s) {
    if (c->snap_host == nullptr || !spkv_append_copies_lengths(c->view, n_max) || being_captured(s))
        return SpkvLengthCopy{nullptr, 0};
    return SpkvLengthCopy{c->snap_host + c->carve.n_pairs + 1, ++c->sent_ticket};
}
// ... once it has been launched and its tokens are counted.  (No event behind it: the launch after an
// event starts 5 to 6 us late, 45 of the 556 us of a prompt of 16 sequences in 8 pieces.)
void prompt_copy_enqueued(spkv_cache* c, const SpkvLengthCopy& to) { c->sent = to.host != nullptr; }

// The exact lengths, where a call cannot go on without them: those that the last call sent, as soon as
// they are there -- the stream goes on meanwhile -- else read back.  (A prompt of 16 sequences in 8
// pieces of 4096 tokens: five read-backs, each of which drained the stream, were 84 us of 642.)
// The wait is bounded: past it the stream is waited for.
constexpr auto kLengthsPatience = std::chrono::milliseconds(20);
int exact_lengths(spkv_cache* c, hipStream_t s) {
    // Under capture never from the copy: whether a call can be captured would depend on whether the prompt
    // before it has run yet.  Refused as ever by the read-back.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (c->sent && hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    if (!c->sent || cap == hipStreamCaptureStatusActive) return refresh_bound(c, s, nullptr);
    const int n_pairs = c->carve.n_pairs;
    const int32_t* len = c->snap_host + n_pairs + 1;
    const auto until = std::chrono::steady_clock::now() + kLengthsPatience;
    while (__atomic_load_n(len + n_pairs, __ATOMIC_ACQUIRE) != c->sent_ticket)
        if (std::chrono::steady_clock::now() > until) return refresh_bound(c, s, nullptr);
    adopt_lengths(c, len);
    return SPKV_OK;
}

// Until no copy of the lengths can be writing the buffer any more: both halves hold the ticket of the
// copy enqueued last, or -- one of them was never launched, or is far behind -- the device has run dry.
void await_copies(const spkv_cache* c) {
    const int n_pairs = c->carve.n_pairs;
    const int32_t* behind = c->snap_host + n_pairs;
    auto arrived = [&]() {
        return __atomic_load_n(behind, __ATOMIC_ACQUIRE) == c->snap_ticket &&
               __atomic_load_n(behind + n_pairs + 1, __ATOMIC_ACQUIRE) == c->sent_ticket;
    };
    const auto until = std::chrono::steady_clock::now() + kLengthsPatience;
    while (!arrived() && std::chrono::steady_clock::now() < until) {}
    if (!arrived()) (void)hipDeviceSynchronize();
}

// Keeps the host's bound of the lengths close to the truth during long runs of single-token
// steps without ever waiting: adopts a finished copy of the device lengths (plus whatever has
// left the windows since it was enqueued: still an upper bound), and enqueues a new copy when
// the slack has grown past 1/share of the bound.  Never while the stream is being captured (the
// copy would become a graph node and the host would read it at the wrong time).
void tighten_bound(spkv_cache* c, hipStream_t s, int share = 16) {
    if (c->snap_host == nullptr) return;
    const int n_pairs = c->carve.n_pairs, Hkv = c->cfg.n_kv_heads;
    if (c->snap_pending) {
        if (__atomic_load_n(c->snap_host + n_pairs, __ATOMIC_ACQUIRE) == c->snap_ticket) {
            int64_t pages = 0, slack = 0;
            for (int p = 0; p < n_pairs; ++p) {
                const int64_t L = (int64_t)c->snap_host[p] + c->snap_ev[p / Hkv];
                if (L < c->L_ub[p]) c->L_ub[p] = (int32_t)L;
                pages += pages_for(c->L_ub[p]);
                slack += c->snap_ev[p / Hkv];
            }
            c->pages_ub = pages;
            c->slack = slack;
            c->since_exact = c->snap_ev;
            if (c->snap_covers) c->lists_known = true;
            c->snap_pending = false;
        } else {
            return;
        }
    }
    int64_t sum = 0;
    for (int p = 0; p < n_pairs; ++p) sum += c->L_ub[p] + std::min(c->T[p / Hkv], c->cfg.window);
    if (c->slack * share <= sum) return;
    if (being_captured(s)) return;
    c->snap_ticket += 1;
    if (spkv_launch_copy_lengths(c->view, SpkvLengthCopy{c->snap_host, c->snap_ticket}, s) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    std::fill(c->snap_ev.begin(), c->snap_ev.end(), 0);
    c->snap_pending = true;
    c->snap_covers = true;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Work partition for one decode call from the host's upper bound of the lengths: items of
// about (all half-pages / item_target) half-pages, and enough slots per pair for the
// longest pair.  The kernels apply it to the exact device-side lengths, which never
// exceed the bound, so every pair fits its slots.
// mw: work items per workgroup and partial slot; the target counts items either way.
SpkvSplit choose_split_mw(const spkv_cache* c, int one_round_items, int64_t slots_total_cap, int mw,
                          int64_t* n_items = nullptr) {
    const int n_pairs = c->carve.n_pairs, Hkv = c->cfg.n_kv_heads;
    std::vector<int64_t> hp(n_pairs);
    int64_t sum_hp = 0, max_hp = 1;
    for (int p = 0; p < n_pairs; ++p) {
        const int Tw = std::min(c->T[p / Hkv], c->cfg.window);
        hp[p] = (c->L_ub[p] + kHalfTokens - 1) / kHalfTokens + (Tw + kHalfTokens - 1) / kHalfTokens;
        sum_hp += hp[p];
        max_hp = std::max(max_hp, hp[p]);
    }
    // Item count: the caller's target, else one resident round, whatever the cache size and
    // however the pairs differ in length -- every pair is cut evenly, so no item is longer
    // than the others.  (Measured: more, shorter items cost 6 % on a batch of 64 sequences
    // of 1k-64k tokens with keep rates from 0 to 1, 2.9 GB kept, and 11 % on 2.1 GB in 128
    // equal lists: every item pays its own start-up round trips.)
    int64_t target = c->item_target;
    if (target <= 0) target = one_round_items;
    target = std::max<int64_t>(1, std::min<int64_t>(target, slots_total_cap - n_pairs));
    const int64_t groups_target = std::max<int64_t>(1, target / mw);
    int64_t per = std::max<int64_t>(1, (sum_hp + groups_target * mw - 1) / (groups_target * mw));
    // Every pair rounds its workgroup count up; keep the total within the target, because one
    // more than the chip holds at once costs a whole second round of the longest items.
    for (int guard = 0; guard < 64; ++guard) {
        int64_t groups = 0;
        for (int p = 0; p < n_pairs; ++p) groups += (hp[p] + per * mw - 1) / (per * mw);
        if (groups <= groups_target || groups <= n_pairs) break;
        per += std::max<int64_t>(1, per / 16);
    }
    const int64_t slots_cap = std::max<int64_t>(1, slots_total_cap / n_pairs - 1);
    if ((max_hp + per * mw - 1) / (per * mw) > slots_cap) per = (max_hp + slots_cap * mw - 1) / (slots_cap * mw);
    SpkvSplit sp;
    sp.hp_per_item = (int32_t)per;
    sp.slots = (int32_t)((max_hp + per * mw - 1) / (per * mw)) | 1;   // odd: see spkv_decode_split
    sp.mw = mw;
    sp.compact = sp.runs = sp.most = 0;
    if (n_items != nullptr) {
        *n_items = 0;
        for (int p = 0; p < n_pairs; ++p)
            *n_items += std::min<int64_t>((hp[p] + per * mw - 1) / (per * mw) * mw, hp[p]);
    }
    return sp;
}

// Single-token decode: workgroups of 4 or 2 items when the cache has few pairs and the
// whole-workgroup rounding per pair neither lengthens the items nor leaves fewer of them than
// one item per workgroup would.  Measured (step time, 32 query / 8 KV heads of 128, keep rates
// drawn per pair): one sequence of 128k tokens 26 -> 22 us, 4 of 128k 39 -> 38, 3 of 64k
// 47 -> 44, equal lists of 1 to 4 sequences 1 to 2.5 us less, two of twelve shapes 1.5 us
// more; but 16 sequences of 32k (128 pairs of about 23 items) 78 -> 92 at the same item
// length, and 64 sequences of 1k-64k 459 -> 540: workgroup ids go round-robin to the 8 XCDs,
// pair p's run starts at id p * slots, and when the lengths repeat from sequence to sequence
// (keep rates that depend on the head) every sequence adds the same uneven pattern -- in
// units of whole workgroups -- until some XCD is handed more waves than it holds and runs
// the surplus in a second round.  Hence the limit of kMergePairs pairs.
// Large caches are cut into equal shares before any of this is asked (share_split, below).
// Caches of more pairs take one item per workgroup, and where their lists are uneven
// (worth_gapless) the gapless numbering (spkv_decode_split_compact) with seven items per
// compute unit, as far as its prefix sum reaches; an explicit item target, merge width or the
// one-launch step keep the plain numbering.
constexpr int kMergePairs = 32, kCompactItemsPerCu = 7, kCompactChunkItemsPerCu = 4,
              kCompactChunkPairs = 384;
// Where the gapless numbering is worth its search and its longer items: at least three slots to
// an item.  Step, plain -> gapless, us: a quarter of the heads keep all, a quarter nothing but
// the window, the rest 0.10-0.33 (four to five slots an item), 64 sequences of 1k-64k 604 -> 500
// (0.05-0.30: 536 -> 471), 40 of 2k-20k 131 -> 110, 24 of 1k-30k 116 -> 96, 16 of 4k-8k
// 36 -> 33, with the predictor inside 641 -> 512, 128 -> 114, 103 -> 98, 37 -> 34.  Sparse heads
// alone (one to 2.7 slots an item) gain or lose a few percent in no order that slots, lengths or the share per XCD would
// tell apart, and stay plain: 16 of 32k 82.6 -> 81.3 (all kept 322 -> 313), 40 of 16k
// 104.7 -> 104.5, 24 of 20k 77.8 -> 77.1, but 32 of 16k 61.1 -> 63.3, 64 of 1k-30k 158 -> 163,
// 128 of 0.5k-16k 195 -> 207.
// The search costs more with more lengths per lane: above 384 pairs the lists must be worth it
// (64 sequences x 8 heads mixed, 300-3000 tokens, 400 keys a pair: 45 -> 51; 100 x 8 of 1k-12k,
// 2300 keys: 201 -> 181).
constexpr int kGapRatio = 3, kGapFewPairs = 384, kGapMeanKeys = 1024;
bool worth_gapless(const spkv_cache* c, const SpkvSplit& plain, int64_t items) {
    const int n = c->carve.n_pairs;
    if (n > kCompactPairs || (int64_t)n * plain.slots < kGapRatio * items) return false;
    if (n <= kGapFewPairs) return true;
    int64_t keys = 0;
    for (int p = 0; p < n; ++p) keys += c->L_ub[p];
    return keys >= (int64_t)n * kGapMeanKeys;
}
// The same for a multi-token step of one column group, whose gapless items are fewer (four per
// compute unit) and longer, which short lists have no use for: not where the longest is below 40
// half-pages; and from there on for few pairs (up to 64, 32 with head_dim 64: the plain
// numbering's many partial results cost more to merge), for items of at least five half-pages, or
// for uneven lists (the longest half as long again as the mean, twice with head_dim 64).  Plain /
// gapless, us: 64 x 3 heads of 64, 1k-2k tokens, 2 drafts 24.6 / 27.7; 48 x 8 of 500-1000 34 / 37;
// 48 x 3 of 2k-4k 26 / 28; but 8 heads of 40k 26 / 23, 3 heads of 64, 100k 30 / 24, 24 x 8 of
// 4k-16k 73 / 69, 10 x 8 of 4k-12k 26.5 / 24.8, 16 x 8 of 1k-4k with dense and local-only heads
// 38 / 35, 32 x 8 of 8k-32k so 275 / 189.  Over 9900 caches of up to 384 pairs, of all kinds,
// drawn at random: always plain 5.1 % slower on average than the faster of the two, always
// gapless 1.2 %, by this rule 0.8 %; what is left is even lists, up to 10 % either way (20 % with
// head_dim 64) by how the plain numbering happens to fall on the compute units.
constexpr int kGapFewChunkPairs = 64, kGapChunkLongestHps = 40, kGapChunkItemHps = 5;
bool worth_gapless_chunk(const spkv_cache* c, int items) {
    const int n = c->carve.n_pairs, Hkv = c->cfg.n_kv_heads;
    if (n > kCompactChunkPairs) return false;
    int64_t sum = 0, longest = 0;                          // half-pages
    for (int p = 0; p < n; ++p) {
        const int Tw = std::min(c->T[p / Hkv], c->cfg.window);
        const int64_t hp = (c->L_ub[p] + kHalfTokens - 1) / kHalfTokens + (Tw + kHalfTokens - 1) / kHalfTokens;
        sum += hp;
        longest = std::max(longest, hp);
    }
    if (longest < kGapChunkLongestHps) return false;
    return n * 128 <= kGapFewChunkPairs * c->cfg.head_dim || sum >= (int64_t)items * kGapChunkItemHps ||
           2 * longest * n >= sum * (c->cfg.head_dim == 128 ? 3 : 4);
}
// Large caches in equal shares (spkv_decode_shares): two runs per compute unit.  From which size on, by what a wave
// with two half-pages in registers costs at its start, and few pairs with many partial results each, against
// what equal shares save; D = 64 has half the bytes to a half-page and the same arithmetic.  Step replayed from a graph
// over enough caches that every one comes cold, 4 query heads to a KV head, items / shares, us: 32 pairs of 18 MB
// 11.4 / 11.4, 26 MB 13.2 / 12.4, 64 MB 19.4 / 18.3, 240 MB 48.7 / 44.1; 128 pairs of 18 MB 11.8 / 12.1, 26 MB 13.9 / 13.4, 100 MB
// 26.6 / 25.0; 256 of 26 MB 15.0 / 15.1, 40 MB 17.9 / 17.2; 512 of 60 MB 23.9 / 23.5, 1 GB 200 / 167 (one dense head in
// eight 174 / 170).  Around the line 12 to 20 pairs have the most to merge: 26 MB, 1 / 2 / 4 / 8 query heads to a KV head, 12
// pairs 13.1 13.2 13.7 14.4 / 13.5 13.6 13.7 14.0, 16 pairs 12.8 13.2 13.4 14.0 / 13.0 13.3 13.5 13.9, even at 29 MB; the step
// with the predictor, 256 hidden units, is ahead everywhere: 14.9 15.6 15.9 16.6 / 12.9 13.8 13.8 14.1, 14.2 14.4 15.0 15.5 /
// 13.1 13.6 13.8 14.2.  Up to 8 the line lies where the shares were ahead with every merge in four waves; in sixteen they
// would be from 26 MB on (8 pairs 14.5 / 13.6, one pair of 40 MB 22.3 / 20.2).  head_dim 64: 32 pairs of 110 MB
// 26.9 / 26.8, 170 MB 37.5 / 35.3; 128 of 110 MB 26.6 / 27.4, 170 MB
// 36.8 / 35.9; 8 of 170 MB 37.0 / 36.0.  The multi-token step, whose partial results are four times as long, gains
// earlier and with any number of pairs: 4 drafts, 1 pair of 40 MB 35.8 / 25.6, 8 pairs of 26 MB 21.2 / 17.9, 32 pairs of
// 18 MB 17.0 / 16.3, 64 MB 28.2 / 23.4, 256 of 40 MB 24.5 / 22.4; head_dim 64, 128 pairs of 110 MB 35.6 / 32.6.  (Lists
// very unlike, a few long ones among many short: steps 1.0 to 2.0 times as fast as items, drafts 0.97 to 2.9.)
// (Repeated on one cache, which stays in the last-level cache, all take 1 to 2 us less.)
// Not where two sequences have the same lengths throughout: an item's place in its pair depends on the pair's
// length and the call, a run's on the pairs before it as well, and copies of a sequence are given the same bits.  The host
// knows lengths alone, so two unlike sequences whose contexts and kept lengths coincide (equal dense batches,
// many sequences of one KV head) keep the items too, at the items' speed.  Copies fed by the same calls have the same bound;
// a captured launch is not asked again when it is replayed.
constexpr int kShareFewPairs = 8;
constexpr int64_t kShareBytes = (int64_t)24 << 20, kShareBytesFewPairs = (int64_t)144 << 20, kShareBytes64 = (int64_t)160 << 20;
constexpr int64_t kShareBytesChunk = (int64_t)20 << 20, kShareBytesChunk64 = (int64_t)100 << 20;
// Do two sequences have the same lengths in every head?  (Copies of a sequence do.)  Those of one half-page
// a head do not count: it is never cut.
bool sequences_alike(const spkv_cache* c) {
    const int B = c->cfg.batch, Hkv = c->cfg.n_kv_heads;
    std::vector<uint64_t>& seen = c->seen;
    seen.clear();
    for (int b = 0; b < B; ++b) {
        uint64_t x = (uint64_t)c->T[b] * 0x9e3779b97f4a7c15ull;
        bool any = std::min(c->T[b], c->cfg.window) > kHalfTokens;
        for (int h = 0; h < Hkv; ++h) {
            const int32_t L = c->L_ub[b * Hkv + h];
            x = (x ^ (uint32_t)L) * 0xff51afd7ed558ccdull;
            x ^= x >> 32;
            any = any || L > 0;
        }
        if (any) seen.push_back(x);
    }
    std::sort(seen.begin(), seen.end());
    return std::adjacent_find(seen.begin(), seen.end()) != seen.end();
}
// The equal shares of a call; runs = 0 where they are not taken.
SpkvSplit share_split(const spkv_cache* c, int64_t slots_total_cap, bool chunk) {
    const int n = c->carve.n_pairs, D = c->cfg.head_dim, runs = 2 * (c->compact_items / kCompactItemsPerCu);
    if (n > kSharePairs || runs + n > slots_total_cap) return SpkvSplit{};
    int64_t hps = 0, longest = 0;
    for (int p = 0; p < n; ++p) {
        const int Tw = std::min(c->T[p / c->cfg.n_kv_heads], c->cfg.window);
        const int64_t hp = (c->L_ub[p] + kHalfTokens - 1) / kHalfTokens + (Tw + kHalfTokens - 1) / kHalfTokens;
        hps += hp;
        longest = std::max(longest, hp);
    }
    const int64_t least = D == 64 ? (chunk ? kShareBytesChunk64 : kShareBytes64)
                                  : chunk ? kShareBytesChunk : n <= kShareFewPairs ? kShareBytesFewPairs : kShareBytes;
    if (hps * (kHalfTokens * 4 * D) < least || sequences_alike(c)) return SpkvSplit{};
    return SpkvSplit{1, runs + n, 1, 0, runs, (int32_t)(longest * runs / std::max<int64_t>(1, hps) + 1)};
}
SpkvSplit choose_split(const spkv_cache* c, int one_round_items, int64_t slots_total_cap) {
    if (c->merge_waves > 0) return choose_split_mw(c, one_round_items, slots_total_cap, c->merge_waves);
    if (c->item_target <= 0 && c->step_launches != 1) {
        const SpkvSplit sp = share_split(c, slots_total_cap, false);
        if (sp.runs > 0) return sp;
    }
    int64_t items_one = 0;
    const SpkvSplit one = choose_split_mw(c, one_round_items, slots_total_cap, 1, &items_one);
    if (c->carve.n_pairs <= kMergePairs) {
        for (int mw = 4; mw > 1; mw >>= 1) {
            int64_t items = 0;
            const SpkvSplit sp = choose_split_mw(c, one_round_items, slots_total_cap, mw, &items);
            if (sp.hp_per_item <= one.hp_per_item && items >= items_one) return sp;
        }
        return one;
    }
    if (c->item_target > 0 || c->step_launches == 1 || !worth_gapless(c, one, items_one))
        return one;
    SpkvSplit sp = choose_split_mw(c, c->compact_items, slots_total_cap, 1, &items_one);
    sp.compact = (int32_t)std::max<int64_t>(1, items_one);
    return sp;
}

// Slots of partial results that a launch may write.
int64_t partial_slots(const spkv_cache* c, const SpkvSplit& sp) {
    return sp.runs > 0 ? sp.slots : (int64_t)c->carve.n_pairs * sp.slots;
}

// A captured launch is replayed while the lists grow: until every pair has gained a whole item,
// one workgroup more per pair has a place for every item.  Without them a replay gives some
// workgroups a second item and waits for those.  Eager launches take none: the host's bound is never
// short.
void room_to_grow(spkv_cache* c, hipStream_t s) {
    if (c->split.compact > 0 && being_captured(s)) c->split.compact += c->carve.n_pairs;
}

SpkvSplit choose_split(const spkv_cache* c) {
    return choose_split(c, c->one_round_items, c->carve.max_items);
}

// One launch (merge and append by the last workgroup of every pair) or two (a merge launch)
// for the single-token decode calls.
// Measured on MI355X (16 sequences, 32 query / 8 KV heads of 128, step time in us against kept
// K/V bytes): one launch 22.3 / 36.8 / 54.6 / 87.3 at 51 / 115 / 222 / 436 MB, two launches
// 17.6 / 28.0 / 45.0 / 78.5 -- the tickets (an atomic per workgroup on one address per pair,
// served one after the other) and the merge's dependent round trips inside the launch cost
// more than a second launch does.  At the smallest sizes the kernels say the same (one sequence
// of 2k, 0.25 MB, replayed from a graph: 8.1 one launch, 6.9 two), but a step issued by itself is
// as long as the host takes to issue it (10.7 one, 14.1 two).  Two launches unless the caller asks.
bool one_launch(const spkv_cache* c, hipStream_t) {
    return c->step_launches == 1;
}

// Short lists: one workgroup per pair does the whole call (spkv_decode_short) in place of a split and
// a merge launch.  What limits it is one compute unit's share of a pair: 16 half-pages with
// head_dim 128 (two rounds of eight waves; 8 for groups of more than eight heads, whose merge is
// longer), 24 with 64.  Longer lists only where there are pairs for most compute units and the lists are
// alike, so that no unit works on alone.  Step replayed from a graph, two launches / this, us:
// 2 pairs of 64, 4 half-pages 6.6 / 4.9, 24 6.8 / 6.2, 48 7.0 / 8.0; 8 pairs of 128, 4 half-pages
// 8.6 / 5.4, 16 8.3 / 7.2, 32 8.4 / 9.0; 4 pairs of 16 heads, 8 half-pages 9.3 / 9.0, 16 9.4 / 10.2;
// 128 pairs of 128, 16 half-pages 15.3 / 10.7; 256 pairs, 16 22 / 15, 64 52 / 44; 512 pairs, 4 23 / 15, 64
// 94 / 88; but 300 pairs, 64 the longest and 16 the mean, 1.3 times as long.  (Issued call by call,
// short steps take what the host takes: 13 / 10.)  Over 500 caches of up to 512 pairs drawn at random
// this takes 0.80 of the time on those it is chosen for, 1.01 at most.
// A captured launch is replayed on lists of any length: it is one only of lists so short that the split
// kernel, frozen with as few workgroups, is never the faster one.  us a replay, split / this, captured at
// 4 half-pages: 2 pairs of 64 at 4 5.8 / 3.3, at 64 14.0 / 7.7, at 1024 273 / 150; 8 of 128 at 64 20 / 15, at 1024
// 547 / 283; 128 at 64 40 / 28, at 1024 504 / 364.  Captured at 5 already, 8 of 128 at 64 13 / 17, at 1024 189 / 285;
// 2 of 64 captured at 24, at 48 6.3 / 6.5, at 384 18 / 54.
constexpr int kShortHps = 16, kShortHpsWideGroup = 8, kShortHps64 = 24, kShortEvenPairs = 192, kShortEvenHps = 64;
constexpr int kShortHpsCaptured = 4;
bool short_lists(const spkv_cache* c, hipStream_t s) {
    if (c->item_target > 0 || c->merge_waves > 0 || c->step_launches > 0) return false;
    const int n = c->carve.n_pairs, Hkv = c->cfg.n_kv_heads;
    int64_t longest = 0, sum = 0;                          // half-pages
    for (int p = 0; p < n; ++p) {
        const int Tw = std::min(c->T[p / Hkv], c->cfg.window);
        const int64_t hp = (c->L_ub[p] + kHalfTokens - 1) / kHalfTokens + (Tw + kHalfTokens - 1) / kHalfTokens;
        longest = std::max(longest, hp);
        sum += hp;
    }
    if (longest <= kShortHpsCaptured) return true;
    const bool few = longest <= (c->cfg.head_dim == 64 ? kShortHps64 : c->carve.G > 8 ? kShortHpsWideGroup : kShortHps);
    const bool even = n >= kShortEvenPairs && longest <= kShortEvenHps && 2 * longest * n <= 3 * sum;
    return (few || even) && !being_captured(s);
}
// spkv_decode_attention: what times or measures the split kernel alone is given that kernel.
bool short_attention(const spkv_cache* c, hipStream_t s) { return !c->timing && !c->split_only && short_lists(c, s); }
// The partition reported for such a call: one workgroup per pair.
SpkvSplit short_split(const spkv_cache* c) {
    return SpkvSplit{1 << 16, 1, spkv_short_waves(c->cfg.head_dim), 0, 0, 0};
}

// Tokens sequence b receives in a call: from cu_seqlens, or one each (cu == nullptr).
int tokens_for(const int32_t* cu, int b) { return cu == nullptr ? 1 : cu[b + 1] - cu[b]; }

// Capacity check before any launch.  Worst case for the pool: every pair pushed out of
// the window by this call is kept.  If that does not fit, the true lengths are read back
// once (synchronises) and the check repeated; SPKV_E_CAPACITY if it still does not fit.
int reserve_capacity(spkv_cache* c, const int32_t* cu, hipStream_t s) {
    const int B = c->cfg.batch, Hkv = c->cfg.n_kv_heads, w = c->cfg.window;
    for (int b = 0; b < B; ++b)
        if ((int64_t)c->T[b] + tokens_for(cu, b) > c->cfg.max_context) return SPKV_E_CAPACITY;
    for (int attempt = 0;; ++attempt) {
        int64_t pages = c->pages_ub;
        for (int b = 0; b < B; ++b) {
            const int n = tokens_for(cu, b);
            const int64_t ev = std::max<int64_t>(0, (int64_t)c->T[b] + n - w) -
                               std::max<int64_t>(0, (int64_t)c->T[b] - w);
            if (ev == 0) continue;
            for (int h = 0; h < Hkv; ++h) {
                const int64_t L = c->L_ub[b * Hkv + h];
                pages += pages_for(L + ev) - pages_for(L);
            }
        }
        if (pages <= c->carve.n_pages) return SPKV_OK;
        if (attempt == 1) return SPKV_E_CAPACITY;
        const int rc = exact_lengths(c, s);
        if (rc != SPKV_OK) return rc;
    }
}

// After an append whose keep rate says more about the lengths than the bound does.
void prompt_appended(spkv_cache* c) {
    c->bound_is_loose = true;
    c->lists_known = c->snap_covers = c->chunk_since_prompt = false;
}

// Host bookkeeping after the launch: exact token counts, upper bounds of the lengths.
void commit_lengths(spkv_cache* c, const int32_t* cu) {
    const int B = c->cfg.batch, Hkv = c->cfg.n_kv_heads, w = c->cfg.window;
    c->sent = false;
    for (int b = 0; b < B; ++b) {
        const int n = tokens_for(cu, b);
        const int64_t ev = std::max<int64_t>(0, (int64_t)c->T[b] + n - w) -
                           std::max<int64_t>(0, (int64_t)c->T[b] - w);
        c->T[b] += n;
        if (ev == 0) continue;
        for (int h = 0; h < Hkv; ++h) {
            int32_t& L = c->L_ub[b * Hkv + h];
            c->pages_ub += pages_for(L + ev) - pages_for(L);
            L += (int32_t)ev;
        }
        c->slack += ev * Hkv;
        c->snap_ev[b] += (int32_t)ev;
        c->since_exact[b] += (int32_t)ev;
    }
}

}  // namespace

extern "C" {

size_t spkv_cache_required_bytes(const spkv_config_t* cfg) {
    Carve k;
    return carve(cfg, &k) ? k.total : 0;
}

int spkv_cache_create(const spkv_config_t* cfg, void* dev_arena, size_t arena_bytes, void* stream,
                      spkv_cache_t** out) {
    if (out == nullptr) return SPKV_E_INVAL;
    *out = nullptr;
    Carve k;
    if (!carve(cfg, &k)) return SPKV_E_INVAL;
    if (dev_arena == nullptr || (reinterpret_cast<uintptr_t>(dev_arena) % kAlign) != 0 ||
        arena_bytes < k.total)
        return SPKV_E_INVAL;
    spkv_cache* c = new (std::nothrow) spkv_cache();
    if (c == nullptr) return SPKV_E_NOMEM;
    c->cfg = *cfg;
    c->cfg.page_tokens = SPKV_PAGE_TOKENS;
    c->carve = k;
    c->arena = static_cast<char*>(dev_arena);
    c->arena_bytes = k.total;
    c->T.assign(cfg->batch, 0);
    c->L_ub.assign(k.n_pairs, 0);
    c->pages_ub = 0;
    c->bound_is_loose = false;
    c->slack = 0;
    c->snap_host = nullptr;
    c->snap_ticket = 0;
    c->snap_pending = false;
    c->sent_ticket = 0;
    c->sent = false;
    c->snap_ev.assign(cfg->batch, 0);
    c->since_exact.assign(cfg->batch, 0);
    c->seen.reserve(cfg->batch);
    c->lists_known = true;
    c->snap_covers = false;
    c->chunk_since_prompt = false;
    c->item_target = 0;
    c->merge_waves = 0;
    c->step_launches = 0;
    c->n_sink = 0;
    {
        // Measured on MI355X: up to 94 % of the resident slots run in one round; at 99 % some
        // compute units already queue a second item and the launch takes 15-20 % longer.
        const int resident = spkv_split_resident_items(cfg->head_dim);
        c->one_round_items = resident > 0 ? resident - resident / 24 : kFallbackItems;
        const int cus = spkv_compute_units();
        c->compact_items = kCompactItemsPerCu * (cus > 0 ? cus : 256);
        c->chunk_round_items = 0;
    }
    c->split = SpkvSplit{1, 1, 1, 0, 0, 0};
    c->timing = false;
    c->split_only = false;
    c->n_timed = 0;
    bind_view(c);
    if (clear_arena(c->arena, k, static_cast<hipStream_t>(stream)) != hipSuccess) {
        delete c;
        return SPKV_E_HIP;
    }
    (void)static_scratch_of_current_device();     // set-up for spkv_decode_attention_static
    // pinned host buffer for the length snapshots (see tighten_bound); the cache works
    // without it, with a coarser partition on very long generations
    void* pinned = nullptr;
    if (hipHostMalloc(&pinned, (size_t)(k.n_pairs + 1) * 8, hipHostMallocCoherent) == hipSuccess) {
        c->snap_host = static_cast<int32_t*>(pinned);
        c->snap_host[k.n_pairs] = c->snap_host[2 * k.n_pairs + 1] = 0;
    } else {
        (void)hipGetLastError();
    }
    *out = c;
    return SPKV_OK;
}

int spkv_cache_grow(spkv_cache_t* c, const spkv_config_t* cfg, void* dev_arena, size_t arena_bytes,
                    void* stream) {
    if (c == nullptr || cfg == nullptr) return SPKV_E_INVAL;
    const spkv_config_t& o = c->cfg;
    if (cfg->batch != o.batch || cfg->n_q_heads != o.n_q_heads || cfg->n_kv_heads != o.n_kv_heads ||
        cfg->head_dim != o.head_dim || cfg->window != o.window)
        return SPKV_E_INVAL;
    if (cfg->max_context < o.max_context || cfg->max_total_kept_tokens < o.max_total_kept_tokens)
        return SPKV_E_INVAL;
    Carve k;
    if (!carve(cfg, &k)) return SPKV_E_INVAL;
    char* na = static_cast<char*>(dev_arena);
    if (na == nullptr || (reinterpret_cast<uintptr_t>(na) % kAlign) != 0 || arena_bytes < k.total)
        return SPKV_E_INVAL;
    // the two arenas must not overlap
    if (na < c->arena + c->arena_bytes && c->arena < na + k.total) return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Carve& q = c->carve;
    const size_t page_bytes = (size_t)spkv_page_elems(o.head_dim) * 2;
    if (clear_arena(na, k, s) != hipSuccess) return SPKV_E_HIP;
    struct Region { size_t to, from, bytes; };
    const Region regions[] = {
        {k.ring, q.ring, (size_t)q.n_pairs * q.n_ring_pages * page_bytes},
        {k.ring_logit, q.ring_logit, (size_t)q.n_pairs * o.window * 4},
        {k.t_pair, q.t_pair, (size_t)q.n_pairs * 4},
        {k.kept_len, q.kept_len, (size_t)q.n_pairs * 4},
        {k.gate_on, q.gate_on, (size_t)q.n_pairs * 4},
        {k.pool_next, q.pool_next, 4},
        {k.free_top, q.free_top, 4},
        {k.free_pages, q.free_pages, (size_t)q.n_pages * 4},
        {k.err_flag, q.err_flag, 4},
        {k.pool, q.pool, (size_t)q.n_pages * page_bytes},
        {k.pos_pool, q.pos_pool, (size_t)q.n_pages * kPageTokens * 4},
        {k.logit_pool, q.logit_pool, (size_t)q.n_pages * kPageTokens * 4},
    };
    // every region starts on a 256-byte boundary and is padded to one, and no region
    // shrinks, so copying the padded size stays inside the new region
    for (const Region& r : regions)
        if (spkv_launch_copy(na + r.to, c->arena + r.from, align_up(r.bytes), s) != hipSuccess)
            return SPKV_E_HIP;
    if (spkv_launch_copy_rows(reinterpret_cast<int32_t*>(na + k.page_table),
                              reinterpret_cast<const int32_t*>(c->arena + q.page_table), q.n_pairs,
                              q.pt_cap, k.pt_cap, s) != hipSuccess)
        return SPKV_E_HIP;
    const float tau = c->cfg.tau;
    c->cfg = *cfg;
    c->cfg.page_tokens = SPKV_PAGE_TOKENS;
    c->cfg.tau = tau;                    // the live threshold stays (see spkv_cache_set_tau)
    c->carve = k;
    c->arena = na;
    c->arena_bytes = k.total;
    bind_view(c);
    return SPKV_OK;
}

int spkv_cache_destroy(spkv_cache_t* c) {
    if (c == nullptr) return SPKV_E_INVAL;
    for (hipEvent_t e : c->events) (void)hipEventDestroy(e);
    if (c->snap_host != nullptr) {
        await_copies(c);
        (void)hipHostFree(c->snap_host);
    }
    delete c;
    return SPKV_OK;
}

int spkv_cache_reset(spkv_cache_t* c, void* stream) {
    if (c == nullptr) return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (clear_arena(c->arena, c->carve, s) != hipSuccess) return SPKV_E_HIP;
    std::fill(c->T.begin(), c->T.end(), 0);
    std::fill(c->L_ub.begin(), c->L_ub.end(), 0);
    c->pages_ub = 0;
    c->bound_is_loose = false;
    c->slack = 0;
    std::fill(c->since_exact.begin(), c->since_exact.end(), 0);
    c->lists_known = true;
    c->snap_pending = c->sent = false;
    return SPKV_OK;
}

int spkv_append(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                const int32_t* cu_seqlens, void* stream) {
    if (c == nullptr || cu_seqlens == nullptr) return SPKV_E_INVAL;
    const int B = c->cfg.batch;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (cu_seqlens[0] != 0) return SPKV_E_INVAL;
    int n_max = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = (int64_t)cu_seqlens[b + 1] - cu_seqlens[b];
        if (n < 0) return SPKV_E_INVAL;
        if (n > n_max) n_max = (int)std::min<int64_t>(n, INT32_MAX);
    }
    if (n_max == 0) return SPKV_OK;
    if (k == nullptr || v == nullptr || util_logits == nullptr) return SPKV_E_INVAL;
    if (!aligned16(k) || !aligned16(v) || !aligned16(util_logits)) return SPKV_E_INVAL;
    const int rc = reserve_capacity(c, cu_seqlens, s);
    if (rc != SPKV_OK) return rc;

    SpkvCu cu;
    std::memcpy(cu.v, cu_seqlens, (size_t)(B + 1) * 4);
    const uint16_t* kk = static_cast<const uint16_t*>(k);
    const uint16_t* vv = static_cast<const uint16_t*>(v);
    const SpkvLengthCopy to = prompt_length_copy(c, n_max, s);
    hipError_t e = (n_max == 1)
                       ? spkv_launch_append_step(c->view, kk, vv, util_logits, cu, s)
                       : spkv_launch_append_bulk(c->view, kk, vv, util_logits, cu, n_max, nullptr, SpanCut{0, 1}, SpkvStage{}, to, s);
    if (e != hipSuccess) return SPKV_E_HIP;
    commit_lengths(c, cu_seqlens);
    if (n_max > SPKV_MAX_CHUNK_TOKENS) prompt_appended(c);         // short chunks: see tighten_bound
    prompt_copy_enqueued(c, to);
    return SPKV_OK;
}

int spkv_decode_step(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                     const void* q, void* out, float* lse, float sm_scale, void* stream) {
    if (c == nullptr || k == nullptr || v == nullptr || util_logits == nullptr || q == nullptr ||
        out == nullptr)
        return SPKV_E_INVAL;
    if (!aligned16(k) || !aligned16(v) || !aligned16(util_logits) || !aligned16(q) ||
        !aligned16(out) || (lse != nullptr && !aligned16(lse)))
        return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)c->cfg.head_dim);
    if (c->bound_is_loose) {
        const int rc = exact_lengths(c, s);
        if (rc != SPKV_OK) return rc;
    }
    tighten_bound(c, s);
    const int rc = reserve_capacity(c, nullptr, s);
    if (rc != SPKV_OK) return rc;
    if (short_lists(c, s)) {
        const SpkvStepIO io = {static_cast<uint16_t*>(out), lse, static_cast<const uint16_t*>(k),
                               static_cast<const uint16_t*>(v), util_logits};
        c->split = short_split(c);
        if (spkv_launch_decode_short(c->view, static_cast<const uint16_t*>(q), sm_scale, io, s) != hipSuccess)
            return SPKV_E_HIP;
        commit_lengths(c, nullptr);
        return SPKV_OK;
    }
    c->split = choose_split(c);          // partition of the state BEFORE the append
    room_to_grow(c, s);
    if (spkv_launch_decode_step(c->view, static_cast<const uint16_t*>(k),
                                static_cast<const uint16_t*>(v), util_logits,
                                static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out), lse,
                                sm_scale, c->split, one_launch(c, s), s) != hipSuccess)
        return SPKV_E_HIP;
    commit_lengths(c, nullptr);
    return SPKV_OK;
}

size_t spkv_decode_step_predict_workspace_bytes(int32_t batch, int32_t d_hidden) {
    if (batch <= 0 || d_hidden <= 0) return 0;
    return (size_t)kPredictSplit * batch * d_hidden * sizeof(float);
}

int spkv_decode_step_predict(spkv_cache_t* c, const void* hidden, const void* w1, const float* b1,
                             const void* w2, const float* b2, int32_t d_model, int32_t d_hidden,
                             const void* k, const void* v, const void* q, void* out, float* lse,
                             float* util_logits, void* workspace, size_t workspace_bytes,
                             float sm_scale, void* stream) {
    if (c == nullptr || hidden == nullptr || w1 == nullptr || w2 == nullptr || k == nullptr ||
        v == nullptr || q == nullptr || out == nullptr || util_logits == nullptr || workspace == nullptr)
        return SPKV_E_INVAL;
    if (d_model <= 0 || d_model % 128 != 0 || d_hidden <= 0 || d_hidden % 16 != 0) return SPKV_E_INVAL;
    if (!aligned16(hidden) || !aligned16(w1) || !aligned16(w2) || !aligned16(k) || !aligned16(v) ||
        !aligned16(q) || !aligned16(out) || !aligned16(util_logits) || !aligned16(workspace) ||
        (b1 != nullptr && !aligned16(b1)) || (b2 != nullptr && !aligned16(b2)) ||
        (lse != nullptr && !aligned16(lse)))
        return SPKV_E_INVAL;
    if (workspace_bytes < spkv_decode_step_predict_workspace_bytes(c->cfg.batch, d_hidden))
        return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)c->cfg.head_dim);
    if (c->bound_is_loose) {
        const int rc = exact_lengths(c, s);
        if (rc != SPKV_OK) return rc;
    }
    tighten_bound(c, s);
    const int rc = reserve_capacity(c, nullptr, s);
    if (rc != SPKV_OK) return rc;
    // the predictor's workgroups share the launch: leave them room in the resident round
    const int n_pred = spkv_predict_blocks(c->cfg.batch, d_hidden);
    c->split = choose_split(c, std::max(c->carve.n_pairs, c->one_round_items - n_pred),
                            c->carve.max_items);
    room_to_grow(c, s);
    SpkvPredict pr = {};
    pr.x = static_cast<const uint16_t*>(hidden);
    pr.w1 = static_cast<const uint16_t*>(w1);
    pr.b1 = b1;
    pr.w2 = static_cast<const uint16_t*>(w2);
    pr.b2 = b2;
    pr.part = static_cast<float*>(workspace);
    pr.logits = util_logits;
    pr.d_model = d_model;
    pr.d_hidden = d_hidden;
    if (spkv_launch_decode_step_predict(c->view, static_cast<const uint16_t*>(k),
                                        static_cast<const uint16_t*>(v),
                                        static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out),
                                        lse, sm_scale, c->split, pr, s) != hipSuccess)
        return SPKV_E_HIP;
    commit_lengths(c, nullptr);
    return SPKV_OK;
}

int spkv_decode_attention(spkv_cache_t* c, const void* q, void* out, float* lse, float sm_scale,
                          void* stream) {
    if (c == nullptr || q == nullptr || out == nullptr) return SPKV_E_INVAL;
    if (!aligned16(q) || !aligned16(out) || (lse != nullptr && !aligned16(lse))) return SPKV_E_INVAL;
    for (int b = 0; b < c->cfg.batch; ++b)
        if (c->T[b] == 0) return SPKV_E_STATE;
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)c->cfg.head_dim);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (c->bound_is_loose) {   // first decode after a bulk append: one read-back of the lengths
        const int rc = exact_lengths(c, s);
        if (rc != SPKV_OK) return rc;
    }
    tighten_bound(c, s);
    if (short_attention(c, s)) {
        const SpkvStepIO io = {static_cast<uint16_t*>(out), lse, nullptr, nullptr, nullptr};
        c->split = short_split(c);
        return spkv_launch_decode_short(c->view, static_cast<const uint16_t*>(q), sm_scale, io, s) == hipSuccess
                   ? SPKV_OK
                   : SPKV_E_HIP;
    }
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (c->timing && c->n_timed < kMaxTimedLaunches) {
        if ((size_t)(2 * c->n_timed + 2) > c->events.size()) {
            hipEvent_t a, b2;
            if (hipEventCreate(&a) != hipSuccess) return SPKV_E_HIP;
            if (hipEventCreate(&b2) != hipSuccess) {
                (void)hipEventDestroy(a);
                return SPKV_E_HIP;
            }
            c->events.push_back(a);
            c->events.push_back(b2);
        }
        ev0 = c->events[2 * c->n_timed];
        ev1 = c->events[2 * c->n_timed + 1];
        c->n_timed += 1;
    }
    c->split = choose_split(c);
    room_to_grow(c, s);
    if (spkv_launch_decode(c->view, static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out),
                           lse, sm_scale, c->split, c->split_only, one_launch(c, s), ev0, ev1, s) != hipSuccess)
        return SPKV_E_HIP;
    return SPKV_OK;
}

int spkv_decode_attention_static(spkv_cache_t* c, const void* q, void* out, float* lse,
                                 float sm_scale, void* stream) {
    if (c == nullptr || q == nullptr || out == nullptr) return SPKV_E_INVAL;
    if (!aligned16(q) || !aligned16(out) || (lse != nullptr && !aligned16(lse))) return SPKV_E_INVAL;
    // partial slots the scratch holds for this shape: [cap][G][D] sums, then [cap][G][2]
    const int G = c->carve.G, D = c->cfg.head_dim;
    const int64_t cap = (int64_t)((kStaticScratchBytes - kAlign) / ((size_t)G * (D + 2) * sizeof(float)));
    if (cap < 2 * (int64_t)c->carve.n_pairs) return SPKV_E_CAPACITY;
    for (int b = 0; b < c->cfg.batch; ++b)
        if (c->T[b] == 0) return SPKV_E_STATE;
    if (c->bound_is_loose) return SPKV_E_STATE;      // would have to wait for the device
    char* base = static_cast<char*>(static_scratch_of_current_device());
    if (base == nullptr) return SPKV_E_HIP;
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)D);
    SpkvView v = c->view;
    v.part_acc = reinterpret_cast<float*>(base);
    v.part_ml = reinterpret_cast<float*>(base + align_up((size_t)cap * G * D * sizeof(float)));
    v.max_items = (int32_t)std::min<int64_t>(cap, INT32_MAX);
    if (short_lists(c, static_cast<hipStream_t>(stream))) {      // no partial results at all
        const SpkvStepIO io = {static_cast<uint16_t*>(out), lse, nullptr, nullptr, nullptr};
        c->split = short_split(c);
        return spkv_launch_decode_short(c->view, static_cast<const uint16_t*>(q), sm_scale, io,
                                        static_cast<hipStream_t>(stream)) == hipSuccess
                   ? SPKV_OK
                   : SPKV_E_HIP;
    }
    c->split = choose_split(c, c->one_round_items, cap);
    room_to_grow(c, static_cast<hipStream_t>(stream));
    if (partial_slots(c, c->split) > cap) return SPKV_E_CAPACITY;
    if (spkv_launch_decode(v, static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out), lse,
                           sm_scale, c->split, false, false, nullptr, nullptr,
                           static_cast<hipStream_t>(stream)) != hipSuccess)
        return SPKV_E_HIP;
    return SPKV_OK;
}

namespace {
int chunk_call(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
               const void* q, const int32_t* cu_seqlens, void* out, float* lse, float sm_scale,
               void* stream, bool append);
int prefill_core(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                 const void* q, const int32_t* cu_seqlens, int n_max, void* out, float* lse,
                 float sm_scale, uint16_t* stage, int32_t* prefix, int shp, float* part,
                 size_t part_bytes, bool exact_fit, hipStream_t s);
}

int spkv_decode_chunk(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                      const void* q, const int32_t* cu_seqlens, void* out, float* lse,
                      float sm_scale, void* stream) {
    return chunk_call(c, k, v, util_logits, q, cu_seqlens, out, lse, sm_scale, stream, true);
}

int spkv_score_chunk(spkv_cache_t* c, const void* k, const void* v, const void* q,
                     const int32_t* cu_seqlens, void* out, float* lse, float sm_scale, void* stream) {
    return chunk_call(c, k, v, nullptr, q, cu_seqlens, out, lse, sm_scale, stream, false);
}

namespace {
int chunk_call(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
               const void* q, const int32_t* cu_seqlens, void* out, float* lse, float sm_scale,
               void* stream, bool append) {
    if (c == nullptr || cu_seqlens == nullptr) return SPKV_E_INVAL;
    const int B = c->cfg.batch, G = c->carve.G;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (cu_seqlens[0] != 0) return SPKV_E_INVAL;
    int n_max = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = (int64_t)cu_seqlens[b + 1] - cu_seqlens[b];
        if (n < 0 || n > SPKV_MAX_CHUNK_TOKENS || n > c->cfg.window || n * G > 64) return SPKV_E_INVAL;
        n_max = std::max(n_max, (int)n);
    }
    if (n_max == 0) return SPKV_OK;
    if (k == nullptr || v == nullptr || (append && util_logits == nullptr) || q == nullptr ||
        out == nullptr)
        return SPKV_E_INVAL;
    if (!aligned16(k) || !aligned16(v) || (append && !aligned16(util_logits)) || !aligned16(q) ||
        !aligned16(out) || (lse != nullptr && !aligned16(lse)))
        return SPKV_E_INVAL;
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)c->cfg.head_dim);
    if (n_max * G > 16) {
        if (!append && c->bound_is_loose) {
            const int rc = exact_lengths(c, s);
            if (rc != SPKV_OK) return rc;
        }
        // More than one group of 16 query columns: the prefill kernels (each tile serves all
        // columns of a workgroup); their split-K partials live in the cache's partial buffers.
        return prefill_core(c, k, v, util_logits, q, cu_seqlens, n_max, out, lse, sm_scale, nullptr, nullptr, 0,
                            c->view.part_acc, (size_t)c->carve.max_items * G * c->cfg.head_dim * sizeof(float), false, s);
    }
    if (c->bound_is_loose) {       // the split-K partition below wants the exact lengths
        const int rc = exact_lengths(c, s);
        if (rc != SPKV_OK) return rc;
    } else {
        tighten_bound(c, s);
    }
    if (append) {
        const int rc = reserve_capacity(c, cu_seqlens, s);
        if (rc != SPKV_OK) return rc;
    }

    if (c->chunk_round_items == 0) {
        const int resident = spkv_chunk_resident_items(c->cfg.head_dim);
        c->chunk_round_items = resident > 0 ? resident - resident / 24 : 960;
    }
    // every slot holds 16 columns of partials instead of G
    const int64_t slot_cap = (int64_t)c->carve.max_items * G / 16;
    c->split = c->item_target <= 0 ? share_split(c, slot_cap, true) : SpkvSplit{};
    if (c->split.runs == 0) {
        // May take the gapless numbering with few items (spkv_chunk_split<D, 1, true>).
        const int chunk_items = c->compact_items / kCompactItemsPerCu * kCompactChunkItemsPerCu;
        const bool compact = c->item_target <= 0 && worth_gapless_chunk(c, chunk_items);
        int64_t items = 0;
        c->split = choose_split_mw(c, compact ? chunk_items : c->chunk_round_items, slot_cap, 1, &items);
        if (compact) c->split.compact = (int32_t)std::max<int64_t>(1, items);
    }
    room_to_grow(c, s);

    // every slot the launch may write must lie inside the partial buffers (they are sized
    // for this at create; checked again here because an overrun would be a wild device write)
    if (partial_slots(c, c->split) * 16 > (int64_t)c->carve.max_items * G)
        return SPKV_E_CAPACITY;

    SpkvCu cu;
    std::memcpy(cu.v, cu_seqlens, (size_t)(B + 1) * 4);
    const uint16_t* kk = static_cast<const uint16_t*>(k);
    const uint16_t* vv = static_cast<const uint16_t*>(v);
    if (spkv_launch_decode_chunk(c->view, kk, vv, static_cast<const uint16_t*>(q),
                                 static_cast<uint16_t*>(out), lse, sm_scale, c->split, cu,
                                 append ? util_logits : nullptr, s) != hipSuccess)
        return SPKV_E_HIP;
    if (append) commit_lengths(c, cu_seqlens);
    return SPKV_OK;
}
}  // namespace

namespace {
// Few spans (short chunks, small batch) leave most of the chip idle while each workgroup
// walks a whole list: cut every span's tiles into ranges so that the launch has about as
// many workgroups as the chip holds at once -- one eight-wave workgroup per compute unit,
// two of four or two waves; more ranges than that only add partial results to write and merge.
constexpr int kPrefillResident = 512;
int prefill_split_cap(int spans, int nw) {
    const int resident = nw == 8 ? kPrefillResident8 : kPrefillResident;
    if (spans <= 0) return 1;
    return std::max(1, std::min(32, (resident + spans / 2) / spans));
}
// Short chunks, one span per pair: ranges of about equal length over all pairs (spkv_prefill_slots) in
// place of ks per pair?  In units of the time of a tile: ks per pair wait for the longest pair's
// range, twice where the ranges do not fit the chip at once, and merge ks partial results; the equal
// ranges cost every workgroup the search for its own (about five tiles) and are merged up to 64 per
// pair.  ks ranges / equal ones, us per call of 16 tokens: heads of unlike lists, 16 sequences of 32k
// 109 / 101, 4 of 128k 56 / 54, 40 of 2k-20k with dense and local-only heads 257 / 159; like or short
// ones, 64 of 4k-8k with 2 heads of 64 26 / 28, one of 10k 20 / 23, one of 100k 38 / 40, 48 of 2k-4k
// with 2 heads of 64 19 / 23, 16 of 250-500 24 / 28.  Before the lengths are known (after a prompt,
// until a copy of them has arrived) the bound says nothing about how unlike they are: equal
// ranges only where it is far above what the search costs.
bool ranges_over_all_pairs(int ks, int pairs, int slots, int64_t longest, int64_t all, bool known) {
    const int64_t each = (all + slots - 1) / slots;
    if (!known) return each >= 64;
    const int64_t rounds = ((int64_t)pairs * ks + kPrefillResident - 1) / kPrefillResident;
    const int64_t unit = std::max<int64_t>(8, each);
    return rounds * ((longest + ks - 1) / ks) + ks / 2 >
           unit + 5 + std::min<int64_t>(64, (longest + unit - 1) / unit) / 2;
}
}  // namespace

size_t spkv_prefill_workspace_bytes(const spkv_cache_t* c, int32_t max_tokens_per_sequence,
                                    int64_t max_total_tokens) {
    if (c == nullptr || max_tokens_per_sequence <= 0 || max_total_tokens <= 0) return 0;
    const size_t prefix = align_up((size_t)max_total_tokens * c->cfg.n_kv_heads * 4);
    const size_t shp = ((size_t)c->cfg.window + max_tokens_per_sequence + kHalfTokens - 1) / kHalfTokens;
    const size_t half_bytes = (size_t)2 * kHalfTokens * c->cfg.head_dim * 2;
    // Split-K partials.  A call cuts its spans into ks = round(resident / spans) ranges, which
    // is above one only while spans <= 2/3 resident, so it never holds more than 4/3 resident
    // workgroups of nw * 32 columns: 4/3 * 65536 columns (256 x 8 x 32 = 512 x 4 x 32),
    // whatever the chunk length.  Caches with more (sequence, head) pairs than that never split.
    const size_t partial = c->carve.n_pairs <= kPrefillResident * 2 / 3
                               ? align_up(((size_t)65536 * 4 / 3 + 64) * (c->cfg.head_dim + 2) * 4)
                               : 0;
    return prefix + align_up((size_t)c->carve.n_pairs * shp * half_bytes) + partial;
}

namespace {
// Prefill attention + append of a call whose arguments have been checked: staging rows,
// prefix counts (neither for spkv_prefill_direct chunks) and split-K partials in the buffers given
// (part_bytes: what `part` holds; the number of key ranges per span is cut down to what fits).
// exact_fit: fail instead.  util_logits = null: attention alone (spkv_prefill_direct chunks).
int prefill_core(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                 const void* q, const int32_t* cu_seqlens, int n_max, void* out, float* lse,
                 float sm_scale, uint16_t* stage, int32_t* prefix, int shp, float* part,
                 size_t part_bytes, bool exact_fit, hipStream_t s) {
    const int B = c->cfg.batch;
    // without staging rows, prefix counts or logits only what needs none of them
    if ((stage == nullptr || prefix == nullptr || util_logits == nullptr) && !spkv_prefill_direct(c->view, n_max))
        return SPKV_E_INVAL;
    if (util_logits != nullptr) {
        const int rc = reserve_capacity(c, cu_seqlens, s);
        if (rc != SPKV_OK) return rc;
    }
    SpkvCu cu;
    std::memcpy(cu.v, cu_seqlens, (size_t)(B + 1) * 4);
    // split-K over every span's tiles when the spans alone would not fill the chip; each
    // range keeps at least a few tiles (lengths from the host's upper bound)
    const SpkvPrefillShape sh = spkv_prefill_shape(c->carve.G, n_max);
    const bool short_chunk = sh.nw != 8;
    if (short_chunk && (c->lists_known || c->chunk_since_prompt)) tighten_bound(c, s, 4);
    c->chunk_since_prompt = short_chunk;
    const int64_t window_tiles = c->cfg.window / kHalfTokens + 1;
    int64_t longest = 0, known_longest = 0, all = 0;               // in tiles; known_longest and all:
    for (int p = 0; p < c->carve.n_pairs; ++p) {                   // of the lengths rather than the bound
        const int64_t bound = c->L_ub[p];
        const int64_t known = c->lists_known ? std::max<int64_t>(0, bound - c->since_exact[p / c->cfg.n_kv_heads]) : bound;
        longest = std::max(longest, bound / kHalfTokens);
        known_longest = std::max(known_longest, known / kHalfTokens + window_tiles);
        all += known / kHalfTokens + window_tiles;
    }
    const bool ordered = spkv_prefill_ordered(c->view, n_max, longest == 0);
    const int spans = spkv_prefill_spans(c->view, cu, n_max, ordered);
    const int64_t tiles = longest + (c->cfg.window + 64) / kHalfTokens;
    int ks = (int)std::max<int64_t>(1, std::min<int64_t>(prefill_split_cap(spans, sh.nw), tiles / 4));
    // Long chunks: not for less than it costs to merge (a tile takes about 1 us, writing and merging 250
    // partial results 14), and not into a second round of workgroups that are over soon.  us, two
    // sequences of 1.7k in pieces of 500, a last piece of 56 spans in 5 ranges 29, in 4 20; four of 700-3000,
    // last piece whole 35, in 2 ranges 28 and the merge 11.
    if (!short_chunk && spans * ks > kPrefillResident8 && tiles / ks < 24) ks = std::max(1, kPrefillResident8 / spans);
    if (!short_chunk && tiles * (ks - 1) < 40 * ks) ks = 1;
    // exactly what this call writes must fit (spans in order are no reason to refuse: counted without the
    // order, by n_max alone, they are too many to be cut into ranges)
    while (spkv_prefill_partial_bytes(spans, ks, sh, c->cfg.head_dim) > part_bytes) {
        if (exact_fit && !ordered) return SPKV_E_INVAL;
        ks -= 1;                    // ks = 1 writes no partials
    }
    int slots = 0;
    bool once = false;
    if (short_chunk) {
        slots = ks > 1 ? spkv_prefill_slots(c->carve.n_pairs, sh, c->cfg.head_dim, part_bytes) : 0;
        if (slots > 0 && !ranges_over_all_pairs(ks, spans, slots, known_longest, all, c->lists_known)) slots = 0;
        if (slots > 0) ks = 1;      // (ranges cut on the device, which also decides `once` then)
        once = c->lists_known && all * (int64_t)(kHalfTokens * 4 * c->cfg.head_dim) > kOnceBytes;
    }
    const SpkvLengthCopy to = prompt_length_copy(c, n_max, s);
    if (spkv_launch_prefill(c->view, static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v),
                            util_logits, static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out),
                            lse, sm_scale, cu, n_max, stage, prefix, shp, ordered, ks, slots, once, part, to, s) != hipSuccess)
        return SPKV_E_HIP;
    if (util_logits == nullptr) return SPKV_OK;
    commit_lengths(c, cu_seqlens);
    if (n_max > SPKV_MAX_CHUNK_TOKENS) {          // shorter ones: see tighten_bound
        if (short_chunk) c->bound_is_loose = true;
        else prompt_appended(c);
    }
    prompt_copy_enqueued(c, to);
    return SPKV_OK;
}
}  // namespace

int spkv_prefill_attention(spkv_cache_t* c, const void* k, const void* v, const float* util_logits,
                           const void* q, const int32_t* cu_seqlens, void* out, float* lse,
                           float sm_scale, void* workspace, size_t workspace_bytes, void* stream) {
    if (c == nullptr || cu_seqlens == nullptr) return SPKV_E_INVAL;
    const int B = c->cfg.batch;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (cu_seqlens[0] != 0) return SPKV_E_INVAL;
    int n_max = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t n = (int64_t)cu_seqlens[b + 1] - cu_seqlens[b];
        if (n < 0) return SPKV_E_INVAL;
        n_max = std::max<int64_t>(n_max, n);
    }
    if (n_max == 0) return SPKV_OK;
    bool one_each = true;
    for (int b = 0; b < B; ++b) one_each = one_each && cu_seqlens[b + 1] - cu_seqlens[b] == 1;
    if (one_each)       // a plain decode step
        return spkv_decode_step(c, k, v, util_logits, q, out, lse, sm_scale, stream);
    // The shortest chunks go to the multi-token step: with one group of 16 query columns its
    // one-wave items read the lists at the decode step's rate, and it needs fewer launches
    // (2 and 4 tokens, there / here, us a call: 16 sequences of 32k 89 / 92, 91 / 92, 4 of 128k 45 / 48, 47 / 49,
    // one of 8k 14 / 19, 15 / 18, 40 of 2k-20k with dense and local-only heads 124 / 151, 126 / 153).
    if (n_max <= SPKV_MAX_CHUNK_TOKENS && n_max <= c->cfg.window && n_max * c->carve.G <= 16)
        return spkv_decode_chunk(c, k, v, util_logits, q, cu_seqlens, out, lse, sm_scale, stream);
    if (k == nullptr || v == nullptr || util_logits == nullptr || q == nullptr || out == nullptr ||
        workspace == nullptr)
        return SPKV_E_INVAL;
    if (!aligned16(k) || !aligned16(v) || !aligned16(util_logits) || !aligned16(q) ||
        !aligned16(out) || (lse != nullptr && !aligned16(lse)) ||
        (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
        return SPKV_E_INVAL;
    if (cu_seqlens[B] <= 0) return SPKV_E_INVAL;
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)c->cfg.head_dim);
    char* ws = static_cast<char*>(workspace);
    const size_t prefix_bytes = align_up((size_t)cu_seqlens[B] * c->cfg.n_kv_heads * 4);
    const int shp = (c->cfg.window + n_max + kHalfTokens - 1) / kHalfTokens;
    const size_t stage_bytes =
        align_up((size_t)c->carve.n_pairs * shp * ((size_t)2 * kHalfTokens * c->cfg.head_dim * 2));
    if (prefix_bytes + stage_bytes > workspace_bytes) return SPKV_E_INVAL;
    return prefill_core(c, k, v, util_logits, q, cu_seqlens, n_max, out, lse, sm_scale,
                        reinterpret_cast<uint16_t*>(ws + prefix_bytes), reinterpret_cast<int32_t*>(ws), shp,
                        reinterpret_cast<float*>(ws + prefix_bytes + stage_bytes),
                        workspace_bytes - prefix_bytes - stage_bytes, true, s);
}

namespace {
// Workspace of spkv_soft_gated_attention: [zeros: n_pairs int32][bias][staging half-pages].
struct SoftCarve {
    size_t zeros, bias, stage, total;
    int shp, n_pairs;
};
bool soft_carve(int batch, int n_kv_heads, int head_dim, int window, int64_t n_max, SoftCarve* o) {
    if (batch < 1 || batch > SPKV_MAX_BATCH || n_kv_heads < 1 || (head_dim != 64 && head_dim != 128) ||
        window < 1 || window > (1 << 20) || n_max < 1 || n_max > (1 << 30) ||
        (int64_t)batch * n_kv_heads > 16384)
        return false;
    o->n_pairs = batch * n_kv_heads;
    o->shp = (int)((window + n_max + kHalfTokens - 1) / kHalfTokens);
    const size_t half_bytes = (size_t)2 * kHalfTokens * head_dim * 2;
    o->zeros = 0;
    o->bias = align_up((size_t)o->n_pairs * 4);
    o->stage = o->bias + align_up((size_t)o->n_pairs * o->shp * kHalfTokens * 4);
    o->total = o->stage + (size_t)o->n_pairs * o->shp * half_bytes;
    return true;
}
}  // namespace

size_t spkv_soft_gated_workspace_bytes(int32_t batch, int32_t n_kv_heads, int32_t head_dim,
                                       int32_t window, int32_t max_tokens_per_sequence) {
    SoftCarve k;
    return soft_carve(batch, n_kv_heads, head_dim, window, max_tokens_per_sequence, &k) ? k.total : 0;
}

int spkv_soft_gated_attention(const void* q, const void* k, const void* v, const float* util_logits,
                              const int32_t* cu_seqlens, int32_t batch, int32_t n_q_heads,
                              int32_t n_kv_heads, int32_t head_dim, int32_t window, void* out,
                              float* lse, float sm_scale, void* workspace, size_t workspace_bytes,
                              void* stream) {
    if (cu_seqlens == nullptr || batch < 1 || batch > SPKV_MAX_BATCH || n_kv_heads < 1 ||
        n_q_heads < 1 || n_q_heads % n_kv_heads != 0 || n_q_heads / n_kv_heads > 16)
        return SPKV_E_INVAL;
    if (cu_seqlens[0] != 0) return SPKV_E_INVAL;
    int64_t n_max = 0;
    for (int b = 0; b < batch; ++b) {
        const int64_t n = (int64_t)cu_seqlens[b + 1] - cu_seqlens[b];
        if (n < 0) return SPKV_E_INVAL;
        n_max = std::max(n_max, n);
    }
    if (n_max == 0) return SPKV_OK;
    SoftCarve sc;
    if (!soft_carve(batch, n_kv_heads, head_dim, window, n_max, &sc)) return SPKV_E_INVAL;
    if (q == nullptr || k == nullptr || v == nullptr || util_logits == nullptr || out == nullptr ||
        workspace == nullptr || workspace_bytes < sc.total)
        return SPKV_E_INVAL;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(util_logits) || !aligned16(out) ||
        (lse != nullptr && !aligned16(lse)) || (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
        return SPKV_E_INVAL;
    if (!(sm_scale > 0.f)) sm_scale = 1.0f / std::sqrt((float)head_dim);
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    if (spkv_launch_fill_zero(ws + sc.zeros, sc.bias, s) != hipSuccess) return SPKV_E_HIP;
    // A view that only carries the shape: no sequence holds a token (t_pair = kept_len = 0),
    // so the kernels take every key from the staging rows of this call.
    SpkvView vw{};
    vw.B = batch;
    vw.Hq = n_q_heads;
    vw.Hkv = n_kv_heads;
    vw.G = n_q_heads / n_kv_heads;
    vw.D = head_dim;
    vw.w = window;
    vw.n_pairs = sc.n_pairs;
    vw.n_ring_pages = (window + kPageTokens - 1) / kPageTokens;
    vw.pt_cap = 1;
    vw.n_pages = 1;
    vw.t_pair = reinterpret_cast<int32_t*>(ws + sc.zeros);
    vw.kept_len = vw.t_pair;
    vw.page_table = vw.t_pair;
    vw.pool = reinterpret_cast<uint16_t*>(ws + sc.stage);
    vw.ring = vw.pool;
    SpkvCu cu;
    std::memcpy(cu.v, cu_seqlens, (size_t)(batch + 1) * 4);
    if (spkv_launch_soft_gated(vw, static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v),
                               util_logits, static_cast<const uint16_t*>(q), static_cast<uint16_t*>(out),
                               lse, sm_scale, cu, (int)n_max, reinterpret_cast<uint16_t*>(ws + sc.stage),
                               reinterpret_cast<float*>(ws + sc.bias), sc.shp, s) != hipSuccess)
        return SPKV_E_HIP;
    return SPKV_OK;
}

namespace {
// Pool pages the host's bound would reach after `n` more single-token steps of every
// sequence with every pair that leaves a window kept.
int64_t pages_after_steps(const spkv_cache* c, int64_t n) {
    const int B = c->cfg.batch, Hkv = c->cfg.n_kv_heads, w = c->cfg.window;
    int64_t pages = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t ev = std::max<int64_t>(0, (int64_t)c->T[b] + n - w) -
                           std::max<int64_t>(0, (int64_t)c->T[b] - w);
        for (int h = 0; h < Hkv; ++h) pages += pages_for((int64_t)c->L_ub[b * Hkv + h] + ev);
    }
    return pages;
}
}  // namespace

int spkv_cache_safe_steps(spkv_cache_t* c, void* stream, int64_t* n_steps) {
    if (c == nullptr || n_steps == nullptr) return SPKV_E_INVAL;
    const int rc = refresh_bound(c, static_cast<hipStream_t>(stream), nullptr);
    if (rc != SPKV_OK) return rc;
    int64_t hi = INT64_MAX;
    for (int b = 0; b < c->cfg.batch; ++b)
        hi = std::min<int64_t>(hi, (int64_t)c->cfg.max_context - c->T[b]);
    hi = std::max<int64_t>(hi, 0);
    int64_t lo = 0;                      // largest n known to fit
    if (pages_after_steps(c, 0) > c->carve.n_pages) hi = 0;
    while (lo < hi) {                    // pages_after_steps is non-decreasing in n
        const int64_t mid = lo + (hi - lo + 1) / 2;
        if (pages_after_steps(c, mid) <= c->carve.n_pages) lo = mid;
        else hi = mid - 1;
    }
    *n_steps = lo;
    return SPKV_OK;
}

int spkv_cache_advance(spkv_cache_t* c, int64_t n_steps) {
    if (c == nullptr || n_steps < 0) return SPKV_E_INVAL;
    if (n_steps == 0) return SPKV_OK;
    for (int b = 0; b < c->cfg.batch; ++b)
        if ((int64_t)c->T[b] + n_steps > c->cfg.max_context) return SPKV_E_CAPACITY;
    if (pages_after_steps(c, n_steps) > c->carve.n_pages) return SPKV_E_CAPACITY;
    const int B = c->cfg.batch, Hkv = c->cfg.n_kv_heads, w = c->cfg.window;
    c->sent = false;
    for (int b = 0; b < B; ++b) {
        const int64_t ev = std::max<int64_t>(0, (int64_t)c->T[b] + n_steps - w) -
                           std::max<int64_t>(0, (int64_t)c->T[b] - w);
        c->T[b] += (int32_t)n_steps;
        for (int h = 0; h < Hkv; ++h) {
            int32_t& L = c->L_ub[b * Hkv + h];
            c->pages_ub += pages_for((int64_t)L + ev) - pages_for(L);
            L += (int32_t)ev;
        }
        c->slack += ev * Hkv;
        c->snap_ev[b] += (int32_t)ev;
        c->since_exact[b] += (int32_t)ev;
    }
    return SPKV_OK;
}

int spkv_cache_stats(spkv_cache_t* c, spkv_stats_t* st, int32_t* kept_len, void* stream) {
    if (c == nullptr || st == nullptr) return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n_pairs = c->carve.n_pairs, Hkv = c->cfg.n_kv_heads, w = c->cfg.window;
    std::vector<int32_t> len(n_pairs), gate(n_pairs);
    int rc = refresh_bound(c, s, len.data());
    if (rc != SPKV_OK) return rc;
    int32_t pool_next = 0, free_top = 0, err = 0;
    if (hipMemcpy(gate.data(), c->view.gate_on, (size_t)n_pairs * 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&pool_next, c->view.pool_next, 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&free_top, c->view.free_top, 4, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&err, c->view.err_flag, 4, hipMemcpyDeviceToHost) != hipSuccess)
        return SPKV_E_HIP;
    std::memset(st, 0, sizeof(*st));
    for (int b = 0; b < c->cfg.batch; ++b) {
        st->total_tokens += c->T[b];
        st->evicted_tokens += (int64_t)std::max(0, c->T[b] - w) * Hkv;
        st->window_tokens += (int64_t)std::min(c->T[b], w) * Hkv;
    }
    for (int p = 0; p < n_pairs; ++p) {
        st->kept_tokens += len[p];
        st->gate_on_tokens += gate[p];
    }
    st->density_evicted = st->evicted_tokens ? (double)st->kept_tokens / (double)st->evicted_tokens : 0.0;
    st->density_all = st->total_tokens ? (double)st->gate_on_tokens / ((double)st->total_tokens * Hkv) : 0.0;
    const int64_t row_bytes = (int64_t)2 * c->cfg.head_dim * 2;
    st->kept_kv_bytes = (st->kept_tokens + st->window_tokens) * row_bytes;
    st->dense_kv_bytes = st->total_tokens * Hkv * row_bytes;
    st->pool_pages_used = (int64_t)pool_next - free_top;
    st->pool_pages_total = c->carve.n_pages;
    st->arena_bytes = (int64_t)c->arena_bytes;
    st->device_error = err;
    auto work_items = [&](const SpkvSplit& sp) -> int32_t {
        int64_t n = 0;
        for (int p = 0; p < n_pairs; ++p) {
            const int Tw = std::min(c->T[p / Hkv], w);
            const int64_t hp = (len[p] + kHalfTokens - 1) / kHalfTokens + (Tw + kHalfTokens - 1) / kHalfTokens;
            const int64_t per = (int64_t)sp.hp_per_item * sp.mw;
            n += sp.runs > 0 ? hp : std::min<int64_t>(std::min<int64_t>((hp + per - 1) / per, sp.slots) * sp.mw, hp);
        }
        return (int32_t)(sp.runs > 0 ? std::min<int64_t>(n, sp.runs) : n);
    };
    st->n_work_items = work_items(short_attention(c, s) ? short_split(c) : choose_split(c));   // of the next spkv_decode_attention
    st->n_work_items_last_call = work_items(c->split);             // of the most recent decode call
    if (kept_len != nullptr) std::memcpy(kept_len, len.data(), (size_t)n_pairs * 4);
    return err ? SPKV_E_DEVICE : SPKV_OK;
}

int spkv_cache_release_sequence(spkv_cache_t* c, int32_t b, void* stream) {
    if (c == nullptr || b < 0 || b >= c->cfg.batch) return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Exact lengths first (synchronises): the host's page bound must drop by exactly what
    // the sequence gives back.
    const int rc = refresh_bound(c, s, nullptr);
    if (rc != SPKV_OK) return rc;
    if (spkv_launch_release_sequence(c->view, b, s) != hipSuccess) return SPKV_E_HIP;
    const int Hkv = c->cfg.n_kv_heads;
    for (int h = 0; h < Hkv; ++h) {
        int32_t& L = c->L_ub[b * Hkv + h];
        c->pages_ub -= pages_for(L);
        L = 0;
    }
    c->T[b] = 0;
    return SPKV_OK;
}

int spkv_cache_kept_positions(spkv_cache_t* c, int32_t b, int32_t h, int32_t* pos, int32_t cap,
                              int32_t* n, void* stream) {
    if (c == nullptr || n == nullptr || b < 0 || b >= c->cfg.batch || h < 0 ||
        h >= c->cfg.n_kv_heads || cap < 0)
        return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int pair = b * c->cfg.n_kv_heads + h;
    if (spkv_launch_gather_positions(c->view, pair, s) != hipSuccess) return SPKV_E_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SPKV_E_HIP;
    int32_t L = 0;
    if (hipMemcpy(&L, c->view.kept_len + pair, 4, hipMemcpyDeviceToHost) != hipSuccess) return SPKV_E_HIP;
    *n = L;
    if (L > cap || (L > 0 && pos == nullptr)) return SPKV_E_INVAL;
    if (L > 0 &&
        hipMemcpy(pos, c->view.pos_scratch, (size_t)L * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return SPKV_E_HIP;
    return SPKV_OK;
}

int spkv_cache_threshold_logit(const spkv_cache_t* c, float* theta) {
    if (c == nullptr || theta == nullptr) return SPKV_E_INVAL;
    *theta = c->view.theta;
    return SPKV_OK;
}

int spkv_cache_set_tau(spkv_cache_t* c, float tau) {
    if (c == nullptr || tau != tau) return SPKV_E_INVAL;
    c->cfg.tau = tau;
    c->view.theta = logit_threshold(tau);
    return SPKV_OK;
}

int spkv_cache_prune(spkv_cache_t* c, void* stream) {
    if (c == nullptr) return SPKV_E_INVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (spkv_launch_prune(c->view, s) != hipSuccess) return SPKV_E_HIP;
    return refresh_bound(c, s, nullptr);      // exact lengths and page count again (synchronises)
}

int spkv_cache_set_option(spkv_cache_t* c, int32_t option, int64_t value) {
    if (c == nullptr) return SPKV_E_INVAL;
    switch (option) {
        case SPKV_OPT_ITEM_TARGET:
            if (value < 0 || value > kMaxItemTarget) return SPKV_E_INVAL;
            c->item_target = (int)value;
            return SPKV_OK;
        case SPKV_OPT_SPLIT_ONLY:
            c->split_only = value != 0;
            return SPKV_OK;
        case SPKV_OPT_MERGE_WAVES:
            if (value != 0 && value != 1 && value != 2 && value != 4) return SPKV_E_INVAL;
            c->merge_waves = (int)value;
            return SPKV_OK;
        case SPKV_OPT_STEP_LAUNCHES:
            if (value != 0 && value != 1 && value != 2) return SPKV_E_INVAL;
            c->step_launches = (int)value;
            return SPKV_OK;
        case SPKV_OPT_SINK_TOKENS:
            if (value < 0 || value > c->cfg.max_context) return SPKV_E_INVAL;
            for (int32_t t : c->T)
                if (t != 0) return SPKV_E_STATE;
            c->n_sink = (int)value;
            c->view.n_sink = (int)value;
            return SPKV_OK;
        case SPKV_OPT_KERNEL_TIMING:
            c->timing = value != 0;
            c->n_timed = 0;
            return SPKV_OK;
        default:
            return SPKV_E_INVAL;
    }
}

int spkv_cache_read_kernel_timing(spkv_cache_t* c, float* ms, int32_t cap, int32_t* n) {
    if (c == nullptr || n == nullptr || cap < 0 || (cap > 0 && ms == nullptr)) return SPKV_E_INVAL;
    const int count = std::min<int>(c->n_timed, cap);
    for (int i = 0; i < count; ++i) {
        if (hipEventSynchronize(c->events[2 * i + 1]) != hipSuccess) return SPKV_E_HIP;
        if (hipEventElapsedTime(&ms[i], c->events[2 * i], c->events[2 * i + 1]) != hipSuccess)
            return SPKV_E_HIP;
    }
    *n = count;
    c->n_timed = 0;
    return SPKV_OK;
}

int64_t spkv_debug_layout_offset(int32_t head_dim, int32_t is_v, int32_t kidx, int32_t d) {
    if ((head_dim != 64 && head_dim != 128) || kidx < 0 || kidx >= kPageTokens || d < 0 ||
        d >= head_dim)
        return -1;
    return is_v ? spkv_v_off(head_dim, kidx, d) : spkv_k_off(head_dim, kidx, d);
}

int spkv_utility_logits(const void* hidden, const void* w1, const float* b1, const void* w2,
                        const float* b2, float* logits, float* workspace, int32_t n_tokens,
                        int32_t d_model, int32_t d_hidden, int32_t n_kv_heads, void* stream) {
    if (hidden == nullptr || w1 == nullptr || w2 == nullptr || logits == nullptr ||
        workspace == nullptr)
        return SPKV_E_INVAL;
    if (n_tokens < 0 || n_tokens > (1 << 24) || d_model < 128 || d_model % 128 != 0 ||
        d_hidden < 16 || d_hidden % 16 != 0 || d_hidden > (1 << 16) || n_kv_heads < 1 ||
        n_kv_heads > 1024)
        return SPKV_E_INVAL;
    if (!aligned16(hidden) || !aligned16(w1) || !aligned16(w2) || !aligned16(logits) ||
        !aligned16(workspace))
        return SPKV_E_INVAL;
    if (n_tokens == 0) return SPKV_OK;
    return spkv_launch_predictor(static_cast<const uint16_t*>(hidden),
                                 static_cast<const uint16_t*>(w1), b1,
                                 static_cast<const uint16_t*>(w2), b2, logits, workspace, n_tokens,
                                 d_model, d_hidden, n_kv_heads,
                                 static_cast<hipStream_t>(stream)) == hipSuccess
               ? SPKV_OK
               : SPKV_E_HIP;
}

int spkv_debug_copy(void* dst, const void* src, size_t bytes, void* stream) {
    if (dst == nullptr || src == nullptr || (bytes & 15u) != 0 || !aligned16(dst) || !aligned16(src))
        return SPKV_E_INVAL;
    return spkv_launch_copy(dst, src, bytes, static_cast<hipStream_t>(stream)) == hipSuccess
               ? SPKV_OK
               : SPKV_E_HIP;
}

int spkv_debug_read(const void* src, size_t region_bytes, int32_t run_bytes, int64_t first_run,
                    int64_t n_runs, int64_t stride, int32_t n_workgroups, void* sink, void* stream) {
    if (src == nullptr || sink == nullptr || !aligned16(src) || !aligned16(sink)) return SPKV_E_INVAL;
    if (run_bytes < 16384 || run_bytes % 16384 != 0) return SPKV_E_INVAL;
    const int64_t total_runs = (int64_t)(region_bytes / (size_t)run_bytes);
    if (total_runs < 1 || n_runs < 1 || n_runs > total_runs || first_run < 0 || stride < 1 ||
        stride > ((int64_t)1 << 31) || first_run > ((int64_t)1 << 31) || total_runs > ((int64_t)1 << 31))
        return SPKV_E_INVAL;               // (first_run + i) * stride stays below 2^64
    if (n_workgroups < 1 || n_workgroups > (1 << 20)) return SPKV_E_INVAL;
    return spkv_launch_read(src, total_runs, run_bytes / 16384, first_run, n_runs, stride, n_workgroups,
                            sink, static_cast<hipStream_t>(stream)) == hipSuccess
               ? SPKV_OK
               : SPKV_E_HIP;
}

const char* spkv_strerror(int code) {
    switch (code) {
        case SPKV_OK: return "ok";
        case SPKV_E_INVAL: return "invalid argument";
        case SPKV_E_STATE: return "decode on a sequence that holds no token";
        case SPKV_E_CAPACITY: return "cache capacity (pool pages, page table or max_context) exceeded";
        case SPKV_E_HIP: return "HIP runtime error";
        case SPKV_E_NOMEM: return "host allocation failed";
        case SPKV_E_DEVICE: return "kernel flagged an inconsistent cache state";
        default: return "unknown error";
    }
}

}  // extern "C"
