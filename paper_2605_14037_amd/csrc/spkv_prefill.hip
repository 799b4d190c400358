// Prefill attention (chunks of any length over the cache, then the append) and the
// soft-gated attention forward, on gfx950: keys staged in the page layout, tiles shared by a
// workgroup through LDS, MFMA tile loop with lazily raised softmax references.
#include "spkv_device.h"

// ------------------------------------------------- prefill attention (any chunk length)
// n new tokens per sequence attend causally with the availability rule of Eq. 3-4 and are
// appended, in four steps:
//   1. spkv_stage_ring (or spkv_prefill_stage) copies the window as it stands (ring, un-rotated into position
//      order) and the n new K/V rows into staging half-pages in the page layout: staging
//      row u holds position T_old - w + u, so query i (position T_old + i) has exactly the
//      rows i < u <= i + w in its window.
//   2. the bulk append runs, its first launch beside step 1, and records, per new token, how long a prefix of the long-term
//      list lies at least w behind it (see spkv_bulk_ring).
//   3. spkv_prefill_attend32 (long chunks) or spkv_prefill_attend: one wave per block of
//      tb = 32 / G consecutive tokens of one (sequence, KV head) -- 32 MFMA columns (token,
//      head), in the latter in two groups of 16 or, for the shortest chunks, one -- walks the
//      long-term prefix and then the staging rows of the block's windows, one online softmax per
//      column, and writes the normalised bf16 rows (or, when a span's keys are cut into ranges,
//      partial results that spkv_prefill_combine merges).
// Chunks of at most kFewTokens tokens skip the first two steps and are appended beside the merge
// (DIRECT below).
// Window keys and long-term entries are disjoint (positions > t - w against <= t - w), so
// every available key is counted once.

struct SpkvPrefill {
    uint16_t* stage;     // [n_pairs][shp] half-pages
    int32_t*  prefix;    // [total tokens][H_kv]
    float*    bias;      // soft gating only: [n_pairs][shp][32] log2 u of every staging row, in units of a score
    float     bias_unit; // soft gating only: 1 / (sm_scale log2 e)
    int32_t   shp;       // staging half-pages per pair
    int32_t   tb;        // tokens per wave (16 nq / G)
    int32_t   nblk;      // workgroups (spans of nw tb tokens) per pair in the grid
    int32_t   pin_xcd;   // 1: all blocks of a pair run on one XCD (shared L2)
    int32_t   nw;        // waves per workgroup (2, 4 or 8): a span is nw * tb tokens
    int32_t   nq;        // column groups of 16 per wave (1 or 2)
    int32_t   ks;        // workgroups per span, its tiles are cut into ks ranges (split-K)
    int32_t   slots;     // > 0 (fewer than eight waves): ranges of about equal length over all pairs
                         // instead, at most this many in all
    int32_t   once;      // fewer than eight waves, slots = 0: the lists pass the caches by (kOnceBytes)
    float*    part;      // partial (acc, m, l) of every (range, column); slots > 0: then [n_pairs] int2
                         // (first range, ranges) of every pair
    const int32_t* order;    // not null: the spans in the order that the append leaves here (SpanOrder)
    int32_t   groups;    // with `order`: groups of pairs, 8 / groups XCDs each (1, 2, 4 or 8; ks > 1: 1)
    int32_t   steps;     // with `order`: workgroups per XCD
    int32_t   spans;     // spans in all: n_pairs nblk; with `order` those that hold a token
};

// A workgroup per (staging half-page, pair), in a launch of its own: soft gating, and chunks whose append
// writes the ring in its first launch.
template <int D>
__global__ __launch_bounds__(256) void spkv_prefill_stage(SpkvView v, const uint16_t* __restrict__ k,
                                                          const uint16_t* __restrict__ vv,
                                                          const float* __restrict__ f, SpkvCu cu, SpkvStage st) {
    stage_half_page<D>(v, k, vv, f, cu, st, blockIdx.y, blockIdx.x);
}

// Bits e = 0..7 set for a <= e <= b (empty if the range misses 0..7); branch-free.
__device__ __forceinline__ unsigned bit_range8(int a, int b) {
    const int lo = min(max(a, 0), 8), hi = max(min(b, 7), -8);
    return (0xffu << lo) & (0xffu >> (7 - hi)) & 0xffu;
}

// One half-page from LDS for the NQ column groups of a wave, in pieces so that the
// accumulators are only ever touched by MFMA inside the tile loop:
//   tile_scores      S = K Q^T for the groups (2 NQ independent accumulator chains),
//                    masked keys to -inf
//   tile_weights     weights p = 2^(x - m) against the column references m as they stand,
//                    and their per-lane sums; reports (wave-uniform) whether a reference
//                    is too low -- some sum above 2^11, so a weight may exceed 2^8 -- or
//                    not set yet.  Weights up to 2^11 are harmless in bf16 / fp32, so in
//                    the steady state no maximum is taken and nothing is rescaled.
//   tile_accumulate  sums and P V with the weights accepted
//   rescale_columns  raises the references to the column maxima of the tile and rescales
//                    sums and accumulators; the tile loop leaves its inner loop for this
//                    (rare once a few tiles have been seen) and then redoes the tile
constexpr float kWeightSumLimit = 2048.0f;
// Shape of a workgroup: long chunks take eight waves of 32 columns (spkv_prefill_attend32: two
// waves per SIMD, one workgroup per compute unit, 256 query columns per tile fetch).  Chunks of
// fewer tokens than eight such waves hold would leave waves without a token, so they get
// four waves of two groups, and the shortest four or two waves of one group each (measured
// on 16-token chunks: as fast as two waves of two groups on 16 sequences at 32k, 10 % faster
// on 4 sequences at 128k; eight waves of one group for 32 tokens were 15 % slower than four
// of two -- twice the waves read every tile from LDS).
static SpkvPrefillShape prefill_shape(int group, int n_max) {
    SpkvPrefillShape sh;
    const int tb1 = 16 / group, tb2 = 32 / group;    // tokens of one, two column groups (group <= 16)
    if (n_max <= 4 * tb1) {
        sh.nq = 1;
        sh.nw = n_max <= 2 * tb1 ? 2 : 4;
    } else {
        sh.nq = 2;
        sh.nw = n_max <= 4 * tb2 ? 4 : 8;
    }
    sh.tb = 16 * sh.nq / group;
    return sh;
}

template <int D, int NQ>
__device__ __forceinline__ void tile_scores(const uint16_t* tile, int lane,
                                            const bf16x8 (&qb)[NQ][D / 32], const unsigned (&kill)[NQ],
                                            bool any_kill, float (&x)[NQ][8]) {
    constexpr int NS = D / 32;
    f32x4 s0[NQ], s1[NQ];
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        s0[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
        s1[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
        const bf16x8 k0 = *reinterpret_cast<const bf16x8*>(tile + sl * 512 + lane * 8);
        const bf16x8 k1 = *reinterpret_cast<const bf16x8*>(tile + (NS + sl) * 512 + lane * 8);
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            s0[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qb[c][sl], s0[c], 0, 0, 0);
            s1[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qb[c][sl], s1[c], 0, 0, 0);
        }
    }
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[c][i] = s0[c][i];
            x[c][4 + i] = s1[c][i];
        }
    }
    if (any_kill) {
#pragma unroll
        for (int c = 0; c < NQ; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((kill[c] >> e) & 1u) x[c][e] = SPKV_NEG_INF;
    }
}

template <int NQ>
__device__ __forceinline__ bool tile_weights(const float (&x)[NQ][8], float scale_log2e,
                                             const float (&m)[NQ], f32x8 (&p)[NQ], float (&psum)[NQ]) {
    bool low = false;
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        const bool unset = m[c] == SPKV_NEG_INF;
        const float neg_ref = unset ? 0.f : -m[c];
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            p[c][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[c][e], scale_log2e, neg_ref));
            sum += p[c][e];
        }
        psum[c] = sum;
        low = low || unset || !(sum <= kWeightSumLimit);
    }
    return __ballot(low) != 0ull;
}

template <int D, int NQ>
__device__ __forceinline__ void tile_accumulate(const uint16_t* tile, int lane, const f32x8 (&p)[NQ],
                                                const float (&psum)[NQ], f32x4 (&acc)[NQ][D / 16],
                                                float (&l)[NQ]) {
    constexpr int NS = D / 32, NB = D / 16;
    bf16x8 va[NB];
#pragma unroll
    for (int db = 0; db < NB; ++db)
        va[db] = *reinterpret_cast<const bf16x8*>(tile + (2 * NS + db) * 512 + lane * 8);
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        l[c] += psum[c];
        const bf16x8 pb = __builtin_convertvector(p[c], bf16x8);
#pragma unroll
        for (int db = 0; db < NB; ++db)
            acc[c][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[db], pb, acc[c][db], 0, 0, 0);
    }
}

// x: the masked scores of the tile that did not fit the references.  A column whose keys
// are all excluded so far keeps the reference -inf (its sums and accumulators are zero).
template <int D, int NQ>
__device__ __forceinline__ void rescale_columns(const float (&x)[NQ][8], float scale_log2e,
                                                f32x4 (&acc)[NQ][D / 16], float (&m)[NQ], float (&l)[NQ]) {
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        float cm = fmaxf(fmaxf(fmaxf(x[c][0], x[c][1]), fmaxf(x[c][2], x[c][3])),
                         fmaxf(fmaxf(x[c][4], x[c][5]), fmaxf(x[c][6], x[c][7]))) * scale_log2e;
        cm = fmaxf(cm, __shfl_xor(cm, 16));
        cm = fmaxf(cm, __shfl_xor(cm, 32));
        const float m_new = fmaxf(m[c], cm);
        const float m_ref = (m_new == SPKV_NEG_INF) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m[c] - m_ref);
        l[c] *= alpha;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) acc[c][db] *= alpha;
        m[c] = m_new;
    }
}

// Ranges of about equal length for the workgroups of a short chunk (host: ranges_over_all_pairs):
// pair p's tiles (at most, by its kept length) in units of `unit` tiles, rounded up, give its number
// of ranges.  The unit is the smallest of eight whose ranges fit `slots` (all tiles / unit from slots
// down to slots - pairs; the last one always fits), at least kRangeMinTiles.  Every wave works it out
// from the lengths: a handful of loads per lane, nine wave sums and a prefix sum, 3 to 4 us.  Equal
// pairs are cut alike.  512 slots are one round of two workgroups per compute unit (16 tokens, per
// call: 16 sequences of 32k 101 us, 40 of 2k-20k with dense and local-only heads 159); 640 take 124
// and 187.  Ranges below eight tiles cost more to merge than they hide.
constexpr int kRangePairsPerLane = 6, kRangeSlots = 512, kRangeMinTiles = 8, kRangeCap = 64;
// Range `id` of all pairs' ranges in order: its pair, the id of the pair's first range and the
// pair's number of ranges; false past the last one.  all: the tiles of all pairs.
// n_pairs <= 64 kRangePairsPerLane, < slots.
__device__ __forceinline__ bool locate_range(const SpkvView& v, const SpkvCu& cu, int slots, int id,
                                             int& pair, int& first, int& ranges, int& all) {
    constexpr int kTries = 8;
    const int lane = threadIdx.x & 63, per_lane = (v.n_pairs + 63) >> 6, p0 = lane * per_lane;
    int tiles[kRangePairsPerLane], sum = 0;
#pragma unroll
    for (int i = 0; i < kRangePairsPerLane; ++i) {
        const int p = min(p0 + i, v.n_pairs - 1), b = p / v.Hkv;
        const bool mine = i < per_lane && p0 + i < v.n_pairs && cu.v[b + 1] > cu.v[b];
        tiles[i] = mine ? ((v.kept_len[p] + kHalfTokens - 1) >> 5) + (v.w >> 5) + 1 : 0;
        sum += tiles[i];
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o);
    all = __builtin_amdgcn_readfirstlane(sum);
    // ceil(tiles / unit) in floats: the half keeps the truncation exact below 2^21 tiles
    auto ranges_of = [](int t, int unit, float inv) -> int {
        return min((int)(((float)(t + unit - 1) + 0.5f) * inv), kRangeCap);
    };
    int unit = 0;
    float inv = 0.f;
#pragma unroll
    for (int k = kTries - 1; k >= 0; --k) {
        const int target = slots - (v.n_pairs * k + kTries - 2) / (kTries - 1);
        const int u = max(kRangeMinTiles, (all + target - 1) / target);
        const float iu = 1.0f / (float)u;
        int n = 0;
#pragma unroll
        for (int i = 0; i < kRangePairsPerLane; ++i) n += ranges_of(tiles[i], u, iu);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o);
        if (k == kTries - 1 || __builtin_amdgcn_readfirstlane(n) <= slots) {
            unit = u;
            inv = iu;
        }
    }
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kRangePairsPerLane; ++i) mine += ranges_of(tiles[i], unit, inv);
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (id >= __builtin_amdgcn_readlane(incl, 63)) return false;
    int run = incl - mine, at = -1, at_first = 0, at_ranges = 0;
#pragma unroll
    for (int i = 0; i < kRangePairsPerLane; ++i) {
        const int r = ranges_of(tiles[i], unit, inv);
        if (id >= run && id < run + r) {
            at = p0 + i;
            at_first = run;
            at_ranges = r;
        }
        run += r;
    }
    const int src = __builtin_ctzll(__ballot(at >= 0));
    pair = __builtin_amdgcn_readlane(at, src);
    first = __builtin_amdgcn_readlane(at_first, src);
    ranges = __builtin_amdgcn_readlane(at_ranges, src);
    return true;
}

// Short chunks (long ones: spkv_prefill_attend32 below).  One workgroup of NW (4 or 2) waves per (sequence,
// KV head) and tile range, which holds the whole chunk: wave wv owns tokens i0 = wv tb .. + tb - 1 as
// its 16 NQ MFMA columns (tb = 16 NQ / G tokens times G heads; NQ = 2 groups of 16, one for the
// shortest chunks).  The waves walk the same half-pages, so each 16 KB tile is fetched from memory
// once per workgroup into a ring of LDS buffers (every wave copies its share of a tile straight from
// memory into LDS, two tiles ahead of the one all waves consume) and each wave reads its MFMA A
// operands from LDS with conflict-free 16-byte reads.
// DIRECT (at most kFewTokens tokens, no more than the window): attended BEFORE the append, without the
// staging rows and prefix counts of the longer chunks, two launches less.  The tiles are the whole list, the ring's
// half-pages as they lie -- a ring key counts for the tokens that still have it in their window, and
// for all if it passes the gate -- and, for the last range of a pair, the chunk's own rows, which its waves
// lay out in LDS themselves.  16 tokens, 16 sequences of 32k: stage 11, append 7.5, attention 95.6
// and merge 7.5 us as four launches; attention 93.6 and merge with the append beside it 9.1 as two
// (118 -> 101 us a call; one of 4 x 2k 31 -> 19.5).  The gates of the ring tiles are looked up once, before the
// loop: left to the tiles, each waited for its own (windows of 2048 / 4096, 104 / 145 us; 81 / 100 so).  What is left is the read at 5 TB/s: ranges up to a
// tenth longer than their mean (a pair has a whole number of them), about 4 us of search.  Tried and
// slower: tiles in registers, a wave per 32 columns and tile (115 us: two waves load a tile, half the
// bytes in flight); a ring of LDS per wave, all columns in one wave, no barrier (102 us, and 8 us more
// for short lists, where one wave's products are the longest chain).
template <int D, int NW, int NQ, bool DIRECT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_prefill_attend(SpkvView v, const uint16_t* __restrict__ q,
                                                           uint16_t* __restrict__ out,
                                                           float* __restrict__ lse, float scale_log2e,
                                                           SpkvPrefill pf, SpkvCu cu,
                                                           const uint16_t* __restrict__ k_new,
                                                           const uint16_t* __restrict__ v_new) {
    constexpr int NS = D / 32, NB = D / 16;
    constexpr int kHalfElems = 2 * kHalfTokens * D;
    constexpr int kRows = kHalfElems / 512;     // 1 KB rows of a tile
    constexpr int kRowsPerWave = kRows / NW;
    // Tiles in flight ahead of the one in use (three measured no faster than two, for long
    // chunks and for the two-wave workgroups of short ones alike).
    constexpr int kAhead = 2, kBufs = kAhead + 1;
    __shared__ __attribute__((aligned(16))) uint16_t s_tile[kBufs + (DIRECT ? 1 : 0)][kHalfElems];
    constexpr int kGateTiles = 256;
    __shared__ unsigned s_gate[DIRECT ? kGateTiles : 1];       // gates of the first ring tiles of this workgroup
    int pair, kr, ranges;
    bool once = pf.once != 0;
    if (pf.slots == 0) {
        pair = blockIdx.x / pf.ks;
        kr = (int)blockIdx.x - pair * pf.ks;
        ranges = pf.ks;
    } else {
        int first, all;
        if (!locate_range(v, cu, pf.slots, blockIdx.x, pair, first, ranges, all)) return;
        kr = (int)blockIdx.x - first;
        once = (int64_t)all * (2 * kHalfElems) > kOnceBytes;
        if (kr == 0 && threadIdx.x == 0)
            reinterpret_cast<int2*>(pf.part + (size_t)pf.slots * (NW * NQ * 16) * (D + 2))[pair] =
                make_int2(first, ranges);
    }
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row0 = cu.v[b], n_tok = cu.v[b + 1] - row0;
    if (n_tok <= 0) return;
    const int last_tok = n_tok - 1;
    const int tid = threadIdx.x, lane = tid & 63, kc = lane >> 4, n = lane & 15;
    // wave index as a scalar: everything derived from it (token range, loop bounds, the
    // branches on them) then stays in scalar registers and scalar branches
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = wv * pf.tb;
    const int tbv = max(0, min(pf.tb, n_tok - i0)), i_last = i0 + tbv - 1, cols = tbv * v.G;
    const bool active = tbv > 0;
    // the cache is in the state after the append (DIRECT: before it)
    const int T0 = v.t_pair[pair] - (DIRECT ? 0 : n_tok), L = v.kept_len[pair];
    const int u_min = max(0, v.w - T0);     // first staging row that holds a position

    auto prefix_of = [&](int i) -> int {   // long-term entries at least w behind token i
        if (DIRECT) return L;
        if (T0 + i - v.w < 0) return 0;
        return min(max(pf.prefix[((size_t)row0 + i) * v.Hkv + h], 0), L);
    };

    bf16x8 qb[NQ][NS];
    int tok[NQ], cnt[NQ];
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        const int col = c * 16 + n;
        const int i = i0 + col / v.G, g = col - (col / v.G) * v.G;
        const bool valid = col < cols;
        tok[c] = valid ? i : -1;
        cnt[c] = valid ? prefix_of(i) : 0;
        const uint16_t* qrow = q + ((size_t)(row0 + i) * v.Hq + (size_t)h * v.G + g) * D + kc * 8;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            uint4 raw = {0u, 0u, 0u, 0u};
            if (valid) raw = *reinterpret_cast<const uint4*>(qrow + sl * 32);
            qb[c][sl] = __builtin_bit_cast(bf16x8, raw);
        }
    }
    // long-term half-pages: the workgroup visits those some token of the chunk can see; this
    // wave computes on those below its own last count, unmasked below its first count
    const int nA = (prefix_of(last_tok) + kHalfTokens - 1) >> 5;
    const int nA_wave = active ? (prefix_of(i_last) + kHalfTokens - 1) >> 5 : 0;
    const int fullA = active ? prefix_of(i0) >> 5 : 0;
    // staging half-pages: rows [1, last_tok + w] that hold a position; this wave's windows
    // cover rows [lo_w, hi_w]
    // (DIRECT: ring half-pages that hold a key, and one tile more, which the loop does not reach)
    const int sB0 = DIRECT ? 0 : max(1, u_min) >> 5, held = min(T0, v.w);
    const int nB = DIRECT ? (held + kHalfTokens - 1) >> 5 : ((last_tok + v.w) >> 5) - sB0 + 1;
    const int lo_w = max(i0 + 1, u_min), hi_w = i_last + v.w;
    const int n_loop = nA + nB, n_hp = n_loop + (DIRECT ? 1 : 0), last = max(n_loop - 1, 0);
    // split-K: this workgroup takes tiles [x_begin, x_stop) of the span's n_hp
    const int x_begin = (int)(((long long)kr * n_hp) / ranges);
    const int x_stop = (int)(((long long)(kr + 1) * n_hp) / ranges), x_end = min(x_stop, n_loop);
    // DIRECT: age of a ring slot's key, 0 = the position w behind the first new token; does it pass the gate?
    const int slot0 = T0 >= v.w ? T0 % v.w : T0 - v.w;
    auto age_of = [&](int at) -> int { return at - slot0 + (at < slot0 ? v.w : 0); };
    auto ring_gate = [&](int at) -> bool {
        return gate_passes(v, v.ring_logit[(size_t)pair * v.w + at], T0 - v.w + age_of(at));
    };
    const int ring0 = max(x_begin - nA, 0);     // DIRECT: this workgroup's first ring tile
    if (DIRECT) {
        // two tiles' gates per wave and pass, the loads of four passes together
        const int tiles = min(x_end - nA - ring0, kGateTiles);
        for (int t0 = wv * 2; t0 < tiles; t0 += 4 * 2 * NW) {
            bool on[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                on[u] = ring_gate(min((ring0 + t0 + u * 2 * NW) * kHalfTokens + lane, held - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long gates = __ballot(on[u]);
                const int t = t0 + u * 2 * NW + lane;
                if (lane < 2 && t < tiles) s_gate[t] = (unsigned)(gates >> (32 * lane));
            }
        }
    }
    if (DIRECT && x_stop > n_loop) {        // the chunk's own rows as a tile: key j is token j, then zeros
        uint16_t* tile = s_tile[kBufs];
#pragma unroll 2
        for (int e = tid; e < kHalfElems / 16; e += 64 * NW) {          // 16-byte units of K, then of V
            const int mm = e & 15, chunk = (e >> 4) % (D / 8), t = (e >> 4) / (D / 8);
            const int key = 8 * (mm >> 2) + 4 * t + (mm & 3);
            uint4 kk = {0u, 0u, 0u, 0u};
            if (key < n_tok) kk = *reinterpret_cast<const uint4*>(k_new + ((size_t)(row0 + key) * v.Hkv + h) * D + chunk * 8);
            const int d = (e >> 6) * 16 + (e & 15), key0 = 8 * ((e >> 4) & 3);
            unsigned w[4] = {0u, 0u, 0u, 0u};
            if (key0 < n_tok) {
                unsigned x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = v_new[((size_t)(row0 + min(key0 + j, last_tok)) * v.Hkv + h) * D + d];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (key0 + j < n_tok) w[j >> 1] |= x[j] << (16 * (j & 1));
            }
            *reinterpret_cast<uint4*>(tile + (size_t)e * 8) = kk;
            *reinterpret_cast<uint4*>(tile + kHalfTokens * D + (size_t)e * 8) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }

    const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
    const uint16_t* stage = pf.stage + (size_t)pair * pf.shp * (size_t)kHalfElems;
    // Page ids are fetched 64 at a time, one per lane, and picked by readlane: the tile
    // loop then issues no memory load of its own whose wait would also wait for the tile
    // copies in flight (a fetch happens once per 128 tiles and is waited for on the spot).
    int page_lane0 = -64, my_page = 0;      // logical page held by lane 0; this lane's page id
    auto page_of = [&](int lp) -> int {     // lp wave-uniform, never decreasing
        if (lp >= page_lane0 + 64) {
            page_lane0 = lp;
            my_page = pt[min(lp + lane, v.pt_cap - 1)];
            __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
        }
        return __builtin_amdgcn_readlane(my_page, lp - page_lane0);
    };
    auto base_of = [&](int x) -> const uint16_t* {
        x = min(x, last);
        if (x < nA) {
            const int page = min(max(page_of(min(x >> 1, v.pt_cap - 1)), 0), v.n_pages - 1);
            return pool_page(v, page) + (x & 1) * kHalfElems;
        }
        if (DIRECT) return ring_page(v, pair, (x - nA) >> 1) + ((x - nA) & 1) * kHalfElems;
        return stage + (size_t)min(sB0 + x - nA, pf.shp - 1) * kHalfElems;
    };

    f32x4 acc[NQ][NB];
    float m[NQ], l[NQ];
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        m[c] = SPKV_NEG_INF;
        l[c] = 0.f;
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[c][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }

    // Tiles go from memory straight into LDS (no registers in between), two tiles ahead of
    // their use: the copy of tile x + 2 is issued when tile x is begun, into the buffer that
    // tile x - 1 vacated, and has a whole tile's time more than it needs before the barrier
    // that ends tile x + 1's wait.  Every wave copies its kRowsPerWave 1 KB rows of a tile;
    // a wave-wide 16-byte load lands at the row's LDS address plus 16 bytes per lane.
    const int my_off = (wv * kRowsPerWave * 64 + lane) * 8;     // this lane's part of a tile
    const unsigned lds_rows = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&s_tile[0][0] +
                              (unsigned)wv * (kRowsPerWave * 1024);
    auto stage_tile = [&](const uint16_t* base, int buf) {
        const uint16_t* p = base + my_off;
        const unsigned dst = lds_rows + (unsigned)buf * (kHalfElems * 2);
        if (once) {
#pragma unroll
            for (int r = 0; r < kRowsPerWave; ++r) load_row_to_lds_once(p + r * 512, dst + r * 1024);
        } else {
#pragma unroll
            for (int r = 0; r < kRowsPerWave; ++r) load_row_to_lds(p + r * 512, dst + r * 1024);
        }
    };
    // Everything loaded so far (queries, counts) is waited for here, once: left pending, the
    // first use inside the tile loop would carry a wait for all loads in flight -- on every
    // tile, tile copies included.
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    stage_tile(base_of(x_begin), 0);
#pragma unroll
    for (int a = 1; a < kAhead; ++a) stage_tile(base_of(x_begin + a), a);
    const uint16_t* p_next = base_of(x_begin + kAhead);
    wait_loads_but<(kAhead - 1) * kRowsPerWave>();        // tile x_begin has landed
    __syncthreads();

    // Tile loop.  The inner loop never touches the accumulators except by MFMA; when the
    // references do not fit a tile the wave leaves it before using the tile, rescales, and
    // resumes at the same tile (prefetch and barrier of a tile are issued exactly once, so
    // the waves stay in step whatever each one does).  After a rescale the references
    // are at least the tile's column maxima, so the second attempt is accepted; a column
    // with every key excluded so far keeps m = -inf and is accepted on the retry as well.
    int x = x_begin, buf = 0;            // buf: LDS buffer of tile x
    bool resume = false, pending = false;
    float xs[NQ][8];
    while (x < x_end) {
        if (pending) rescale_columns<D, NQ>(xs, scale_log2e, acc, m, l);
        for (; x < x_end; ++x) {
            if (!resume) {
                // the tile after next (past the last one: the last tile again, never used)
                stage_tile(p_next, buf >= 1 ? buf - 1 : kBufs - 1);
                p_next = base_of(x + kAhead + 1);
            }
            resume = false;
            const uint16_t* tile = s_tile[buf];
            bool mine;
            int u_tile = 0;
            if (x < nA) {
                mine = x < nA_wave;
            } else {
                u_tile = (sB0 + x - nA) * kHalfTokens;
                mine = active && (DIRECT || (u_tile <= hi_w && u_tile + kHalfTokens > lo_w));
            }
            if (mine) {
                // per column group: which of this lane's eight keys are excluded
                unsigned kill[NQ] = {};
                bool any = true;
                if (x < nA) {
                    any = x >= fullA;
                    if (any) {
                        const int k0 = x * kHalfTokens + kc * 8;   // list index of this lane's first key
#pragma unroll
                        for (int c = 0; c < NQ; ++c) kill[c] = bit_range8(0, cnt[c] - k0 - 1) ^ 0xffu;
                    }
                } else if (DIRECT) {
                    const int u0 = u_tile + kc * 8;
                    unsigned gate = 0u;
                    if (x - nA - ring0 < kGateTiles) {
                        gate = s_gate[x - nA - ring0] >> (kc * 8);
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (ring_gate(min(u0 + e, held - 1))) gate |= 1u << e;
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int at = u0 + e, age = age_of(at);
#pragma unroll
                        for (int c = 0; c < NQ; ++c)       // in token i's window iff its age is above i
                            if (at >= held || !(((gate >> e) & 1u) || age > tok[c])) kill[c] |= 1u << e;
                    }
                } else {
                    const int u0 = u_tile + kc * 8;
                    // window of token i: rows i < u <= i + w that hold a position
#pragma unroll
                    for (int c = 0; c < NQ; ++c)
                        kill[c] = (tok[c] >= 0 ? bit_range8(max(tok[c] + 1, u_min) - u0,
                                                            tok[c] + v.w - u0)
                                               : 0u) ^ 0xffu;
                }
                tile_scores<D, NQ>(tile, lane, qb, kill, any, xs);
                f32x8 pw[NQ];
                float psum[NQ];
                if (tile_weights<NQ>(xs, scale_log2e, m, pw, psum) && !pending) {
                    pending = true;
                    resume = true;
                    break;
                }
                pending = false;
                tile_accumulate<D, NQ>(tile, lane, pw, psum, acc, l);
            }
            wait_loads_but<(kAhead - 1) * kRowsPerWave>();    // all but the newest copies: tile x + 1 has landed
            __syncthreads();
            buf = buf == kBufs - 1 ? 0 : buf + 1;
        }
    }
    wait_loads_but<0>();
    if (DIRECT && x_stop > n_loop && active) {
        unsigned kill[NQ];
#pragma unroll
        for (int c = 0; c < NQ; ++c) kill[c] = bit_range8(0, tok[c] - kc * 8) ^ 0xffu;
        tile_scores<D, NQ>(s_tile[kBufs], lane, qb, kill, true, xs);
        f32x8 pw[NQ];
        float psum[NQ];
        if (tile_weights<NQ>(xs, scale_log2e, m, pw, psum)) {
            rescale_columns<D, NQ>(xs, scale_log2e, acc, m, l);
            (void)tile_weights<NQ>(xs, scale_log2e, m, pw, psum);
        }
        // these weights stay in 32 bits, as in spkv_chunk_combine: three bf16 parts hold all 24 of one
#pragma unroll
        for (int part = 0; part < 3; ++part) {
            tile_accumulate<D, NQ>(s_tile[kBufs], lane, pw, psum, acc, l);
#pragma unroll
            for (int c = 0; c < NQ; ++c) {
                psum[c] = 0.f;
                pw[c] -= __builtin_convertvector(__builtin_convertvector(pw[c], bf16x8), f32x8);
            }
        }
    }

#pragma unroll
    for (int c = 0; c < NQ; ++c) {
        float lc = l[c];
        lc += __shfl_xor(lc, 16);
        lc += __shfl_xor(lc, 32);
        if (tok[c] >= 0 && (pf.slots > 0 || pf.ks > 1)) {
            // partial of this tile range: un-normalised accumulators, reference, sum
            // layout: [all columns][D] accumulators, then [all columns][2] (m, l)
            const size_t n_cols = (size_t)(pf.slots > 0 ? pf.slots : v.n_pairs * pf.ks) * (NW * NQ * 16);
            const size_t pc = (size_t)blockIdx.x * (NW * NQ * 16) + wv * (NQ * 16) + c * 16 + n;
            float* pa = pf.part + pc * D + kc * 4;
#pragma unroll
            for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(pa + db * 16) = acc[c][db];
            if (kc == 0) {
                pf.part[n_cols * D + pc * 2] = m[c];
                pf.part[n_cols * D + pc * 2 + 1] = lc;
            }
        } else if (tok[c] >= 0) {
            const int col = c * 16 + n;
            const int g = col - (col / v.G) * v.G;
            const size_t o = (size_t)(row0 + tok[c]) * v.Hq + (size_t)h * v.G + g;
            const float inv = 1.0f / lc;
            uint16_t* po = out + o * D + kc * 4;
#pragma unroll
            for (int db = 0; db < NB; ++db) {
                const __bf16 r0 = (__bf16)(acc[c][db][0] * inv), r1 = (__bf16)(acc[c][db][1] * inv);
                const __bf16 r2 = (__bf16)(acc[c][db][2] * inv), r3 = (__bf16)(acc[c][db][3] * inv);
                uint2 pk;
                pk.x = (unsigned)__builtin_bit_cast(uint16_t, r0) | ((unsigned)__builtin_bit_cast(uint16_t, r1) << 16);
                pk.y = (unsigned)__builtin_bit_cast(uint16_t, r2) | ((unsigned)__builtin_bit_cast(uint16_t, r3) << 16);
                *reinterpret_cast<uint2*>(po + db * 16) = pk;
            }
            if (lse != nullptr && kc == 0) lse[o] = (m[c] + log2f(lc)) * 0.6931471805599453f;
        }
    }
}

// Span `id` of a group of pairs in the order that the append has left (SpanOrder): its pair, and its index
// among the pair's spans, counted from the last one.  Where the group has none: -1.  Past its last one: an
// index past the pair's spans.  e: the entry of this lane.
__device__ __forceinline__ SpanOrder span_entry(const int32_t* __restrict__ order, int n_pairs) {
    const int lane = threadIdx.x & 63;
    return *reinterpret_cast<const SpanOrder*>(order + (size_t)min(lane, n_pairs - 1) * kSpanOrderStride);
}
__device__ __forceinline__ void find_span(SpanOrder e, int n_pairs, int group, int id, int& pair, int& at) {
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(lane < n_pairs && e.pair_group >> 16 == group && e.before <= id);
    const int r = m != 0ull ? 63 - __builtin_clzll(m) : 0;
    pair = min(__builtin_amdgcn_readlane(e.pair_group, r) & 0xffff, n_pairs - 1);
    at = m != 0ull ? id - __builtin_amdgcn_readlane(e.before, r) : -1;
}

// Long chunks and the soft-gated forward: one workgroup of eight waves per span of 8 tb tokens,
// each wave with 32 columns (token, head) as ONE group of MFMA 32x32x16, so that 256 query columns
// share one tile fetch.  Half the matrix instructions of two groups of 16x16x32 for the same
// flops: what a matrix instruction holds back of a SIMD's vector issue counts half as often
// (probe: four 32x32x16 with eight fma each, two waves per SIMD, 154 ns; eight 16x16x32 with four
// each 204 ns; the products alone 115 ns either way).
// Software pipeline over half-pages x (32 keys): the products K Q^T of x + 1 stand beside the
// weights of x, then V P of x; LDS holds four steps of two half-pages, copied two steps ahead,
// and every operand read goes out half a unit or more before its use, also across the one
// barrier per step.  One code path for all half-pages: masks are a branch around the scores
// alone, and a wave that sees no key of a half-page skips the product with V.
// Soft gating: the bias log2 u of a key, in units of a score, is what its products start from.
// 4 sequences of 16 384 tokens, 32 query / 8 KV heads of 128 (8.8 TFLOP): 9.37 -> 7.87 ms =
// 1.12 PFLOP/s (two groups of 16 columns, reads and products of a tile one after the other,
// before; a large matrix product reaches 1.35 here); prompts of 3 to 19.5 thousand tokens, keep
// rates 0.1 to 0.33, 4 sequences: 2.26 -> 1.90 ms.  What is left, by counters: the matrix units are
// busy 56 % of the SIMD time, with 5.6 vector instructions beside each product; waves wait 27 %
// of their time (copies and the barrier) and 33 % for an issue slot; the clock falls as the
// load rises (1.85 GHz; 1.7 on the last chunks of a 32k prompt).
template <int D, bool SOFT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_prefill_attend32(
    SpkvView v, const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float* __restrict__ lse,
    float scale_log2e, SpkvPrefill pf, SpkvCu cu) {
    constexpr int NW = 8, NS = D / 16, NB = D / 32;
    constexpr int kHalfElems = 2 * kHalfTokens * D;
    constexpr int kStepElems = 2 * kHalfElems;              // a step: two half-pages, 64 keys
    constexpr int kRowsPerWave = kStepElems / 512 / NW;     // 1 KB rows of a step per wave
    constexpr int kBufs = 4;
    __shared__ __attribute__((aligned(16))) uint16_t s_tile[kBufs][kStepElems];
    __shared__ __attribute__((aligned(16))) float s_bias[SOFT ? kBufs : 1][SOFT ? NW : 1][SOFT ? 64 : 4];
    __shared__ __attribute__((aligned(16))) float s_zero[32];
    if (SOFT && threadIdx.x < 32) s_zero[threadIdx.x] = 0.f;      // (the barrier before the loop)
    int pair, qblk, kr, id = 0;      // (sequence, KV head), span, tile range of the span
    if (!SOFT && pf.order != nullptr) {
        // `share` XCDs for a group; two neighbours of a pair at a time on one (they share most of their windows)
        const int share = 8 / pf.groups, xcd = blockIdx.x & 7, group = xcd / share, at = blockIdx.x >> 3;
        const int j = ((at >> 1) * share + xcd - group * share) * 2 + (at & 1);
        id = j / pf.ks;
        kr = j - id * pf.ks;
        find_span(span_entry(pf.order, v.n_pairs), v.n_pairs, group, id, pair, qblk);
    } else if (pf.pin_xcd) {
        // workgroups go round-robin to the 8 XCDs: id % 8 picks the XCD, and every pair lives on one
        // XCD, so its list is fetched into one L2 and re-read there; rotated inside every full group
        // of 8 pairs by the group index: with 8 KV heads a plain pair % 8 would give each XCD one
        // head of every sequence, and heads differ several-fold in kept length
        const int local = blockIdx.x >> 3, lp = local / (pf.nblk * pf.ks);
        const int rem = local - lp * pf.nblk * pf.ks;
        qblk = rem / pf.ks;
        kr = rem - qblk * pf.ks;
        const int rot = (lp * 8 + 8 <= v.n_pairs) ? lp : 0;
        pair = lp * 8 + (((blockIdx.x & 7) + rot) & 7);
        if (pair >= v.n_pairs) return;
    } else if (SOFT) {                    // the last, longest spans of all pairs first
        qblk = (int)blockIdx.x / v.n_pairs;
        pair = (int)blockIdx.x - qblk * v.n_pairs;
        kr = 0;
    } else {
        pair = blockIdx.x / (pf.nblk * pf.ks);
        const int rem = blockIdx.x - pair * pf.nblk * pf.ks;
        qblk = rem / pf.ks;
        kr = rem - qblk * pf.ks;
    }
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row0 = cu.v[b], n_tok = cu.v[b + 1] - row0;
    // longest prefixes first
    qblk = (!SOFT && pf.order != nullptr ? (n_tok + NW * pf.tb - 1) / (NW * pf.tb) : pf.nblk) - 1 - qblk;
    const int span0 = qblk * NW * pf.tb;
    if (span0 < 0 || span0 >= n_tok) return;
    const int span_last = min(span0 + NW * pf.tb, n_tok) - 1;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = span0 + wv * pf.tb;
    const int tbv = max(0, min(pf.tb, n_tok - i0)), i_last = i0 + tbv - 1, cols = tbv * v.G;
    const bool active = tbv > 0;
    const bool valid = col < cols;
    const int tok = valid ? i0 + col / v.G : -1;
    // Counters, prefix counts and the first page ids are fetched together, before any of them is
    // looked at (prefix counts of tokens whose window starts at 0 are never written: any value).
    const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
    int page_lane0 = 0, my_page = 0;        // logical page held by lane 0; this lane's page id
    int T0 = 0, L = 0, p_span = 0, p_first = 0, p_last = 0, p_tok = 0;
    if (!SOFT) {
        const int32_t* pp = pf.prefix + (size_t)row0 * v.Hkv + h;
        my_page = pt[min(lane, v.pt_cap - 1)];
        T0 = v.t_pair[pair] - n_tok;
        L = v.kept_len[pair];
        p_span = pp[(size_t)span_last * v.Hkv];
        p_first = pp[(size_t)min(i0, n_tok - 1) * v.Hkv];
        p_last = pp[(size_t)min(max(i_last, i0), n_tok - 1) * v.Hkv];
        p_tok = pp[(size_t)(valid ? tok : span0) * v.Hkv];
    }
    const int u_min = max(0, v.w - T0);     // first staging row that holds a position
    // long-term entries at least w behind token i
    auto prefix_of = [&](int i, int p) -> int { return T0 + i - v.w < 0 ? 0 : min(max(p, 0), L); };
    const int cnt = valid ? prefix_of(tok, p_tok) : 0;
    bf16x8 qb[NS];
    {
        const uint16_t* qrow = q + ((size_t)(row0 + (valid ? tok : i0)) * v.Hq + (size_t)h * v.G + (col - (col / v.G) * v.G)) * D + half * 8;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            uint4 raw = {0u, 0u, 0u, 0u};
            if (valid) raw = *reinterpret_cast<const uint4*>(qrow + sl * 16);
            qb[sl] = __builtin_bit_cast(bf16x8, raw);
        }
    }
    const int nA = (prefix_of(span_last, p_span) + kHalfTokens - 1) >> 5;
    const int nA_wave = active ? (prefix_of(i_last, p_last) + kHalfTokens - 1) >> 5 : 0;
    const int fullA = active ? prefix_of(i0, p_first) >> 5 : 0;
    const int sB0 = (SOFT ? u_min : max(span0 + 1, u_min)) >> 5;
    const int nB = ((span_last + v.w) >> 5) - sB0 + 1;
    const int lo_w = SOFT ? u_min : max(i0 + 1, u_min), hi_w = i_last + v.w;
    const int n_hp = nA + nB, last = n_hp - 1;
    const int x_begin = (int)(((long long)kr * n_hp) / pf.ks);
    const int x_end = (int)(((long long)(kr + 1) * n_hp) / pf.ks);

    const uint16_t* stage = pf.stage + (size_t)pair * pf.shp * (size_t)kHalfElems;
    auto page_of = [&](int lp) -> int {
        if (lp >= page_lane0 + 64) {
            page_lane0 = lp;
            my_page = pt[min(lp + lane, v.pt_cap - 1)];
            __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
        }
        return __builtin_amdgcn_readlane(my_page, lp - page_lane0);
    };
    auto base_of = [&](int x) -> const uint16_t* {
        x = min(x, last);
        if (x < nA) {
            const int page = min(max(page_of(min(x >> 1, v.pt_cap - 1)), 0), v.n_pages - 1);
            return pool_page(v, page) + (x & 1) * kHalfElems;
        }
        return stage + (size_t)min(sB0 + x - nA, pf.shp - 1) * kHalfElems;
    };

    // Copies of a step: waves 0-3 the first half-page, 4-7 the second, a quarter each.  Rows land
    // in LDS in operand order, so that every operand read is 1 KB in lane order: K row sl holds,
    // for lane (half, r), 16 bytes (d = 16 sl + 8 half ..) of key 16 (r >> 4) + 8 ((r >> 2) & 1) +
    // 4 ((r >> 3) & 1) + (r & 3) -- the score of row r of an MFMA then comes out in the register
    // and lane in which the product with V wants the weight of that key; V row (g, db) holds
    // keys 16 g + 8 half .. + 7 of d = 32 db + r.
    const int quarter = wv & 3;
    const unsigned k_lane = ((((col >> 3) & 1) * (D / 8) + half) * 16 + 8 * (col >> 4) + 4 * ((col >> 2) & 1) + (col & 3)) * 16;
    const unsigned v_lane = (((col >> 4) * 4 + half) * 16 + (col & 15)) * 16;
    const unsigned my_off = quarter < 2 ? k_lane + quarter * kRowsPerWave * 512
                                        : v_lane + kHalfTokens * D * 2 + (quarter - 2) * 512;
    const int row_bytes = quarter < 2 ? 512 : 2048;
    const unsigned lds_rows = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)&s_tile[0][0] +
                              (unsigned)wv * (kRowsPerWave * 1024);
    const unsigned lds_bias = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)&s_bias[0][0][0] +
                              (unsigned)wv * 256;
    constexpr int kCopies = kRowsPerWave + (SOFT ? 1 : 0);
    auto stage_step = [&](int x, int buf) {                 // half-pages x, x + 1
        const char* p = reinterpret_cast<const char*>(base_of(x + (wv >> 2)));
#pragma unroll
        for (int r = 0; r < kRowsPerWave; ++r)
            load_row_to_lds(p + r * row_bytes, my_off, lds_rows + (unsigned)buf * (kStepElems * 2) + r * 1024);
        if (SOFT) {
            const int hp = min(sB0 + min(x + (lane >> 5), last) - nA, pf.shp - 1);
            load_word_to_lds(pf.bias + ((size_t)pair * pf.shp + hp) * kHalfTokens + (lane & 31),
                             lds_bias + (unsigned)buf * (NW * 256));
        }
    };

    f32x16 acc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    float m = valid ? SPKV_NEG_INF : 0.f, l = 0.f;

    // K operands and (soft gating) biases of the half-page after the current one
    bf16x8 kf[NS];
    f32x16 cb;
    auto load_k = [&](const uint16_t* hp, const float* bias) {
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) kf[sl] = *reinterpret_cast<const bf16x8*>(hp + sl * 512 + lane * 8);
        if (SOFT) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 t = *reinterpret_cast<const float4*>(bias + (g >> 1) * 16 + half * 8 + (g & 1) * 4);
                cb[4 * g] = t.x;
                cb[4 * g + 1] = t.y;
                cb[4 * g + 2] = t.z;
                cb[4 * g + 3] = t.w;
            }
        }
    };
    // Does any token of the wave see a key of the half-page?  The values of the others are not
    // touched at all (a weight of zero would still turn an infinity among them into a NaN).
    auto mine = [&](int x) -> bool {
        if (x >= x_end) return false;
        if (x < nA) return x < nA_wave;
        const int u = (sB0 + x - nA) * kHalfTokens;
        return active && u <= hi_w && u + kHalfTokens > lo_w;
    };
    // soft gating: every row of the half-page lies outside every window of the wave
    auto all_biased = [&](int x) -> bool { return (sB0 + x - nA) * kHalfTokens + kHalfTokens - 1 <= i0; };
    // scores of a half-page from kf; with soft gating started at the bias (in units of a score)
    auto scores = [&](f32x16& s) {
        if (SOFT) {
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qb[0], cb, 0, 0, 0);
        } else {
            f32x16 zero;
#pragma unroll
            for (int e = 0; e < 16; ++e) zero[e] = 0.f;
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qb[0], zero, 0, 0, 0);
        }
#pragma unroll
        for (int sl = 1; sl < NS; ++sl) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[sl], qb[sl], s, 0, 0, 0);
    };
    // Excluded keys to -inf: past the list prefix of the column's token, outside its window, past
    // this workgroup's range.  Soft gating: the bias of the rows that only some tokens have outside
    // their windows.
    auto mask = [&](f32x16& s, int x, const float* bias) {
        const int u = (sB0 + x - nA) * kHalfTokens;
        const bool some_biased = SOFT && !all_biased(x);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int k0 = 16 * g + 8 * half, u0 = u + k0;
            unsigned ok = 0u;
            if (x >= x_end) ok = 0u;
            else if (x < nA) ok = bit_range8(0, cnt - (x * kHalfTokens + k0) - 1);
            else if (tok >= 0) ok = bit_range8((SOFT ? u_min : max(tok + 1, u_min)) - u0, tok + v.w - u0);
            if (some_biased) {
#pragma unroll
                for (int e = 0; e < 8; ++e) s[8 * g + e] += u0 + e <= tok ? bias[k0 + e] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) s[8 * g + e] = ((ok >> e) & 1u) ? s[8 * g + e] : SPKV_NEG_INF;
        }
    };
    // weights against the column reference as it stands: bf16 operands of P V and their sum;
    // true (wave-uniform) if a reference is too low or not set yet
    bf16x8 pb[2];
    float psum, neg_ref = valid ? 0.f : -m, limit = valid ? -1.f : kWeightSumLimit;
    auto weights = [&](const f32x16& s) -> bool {
        f32x8 p[2];
#pragma unroll
        for (int e = 0; e < 16; ++e)
            p[e >> 3][e & 7] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2e, neg_ref));
        float s4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s4[e] = (p[0][e] + p[0][4 + e]) + (p[1][e] + p[1][4 + e]);
        psum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        pb[0] = __builtin_convertvector(p[0], bf16x8);
        pb[1] = __builtin_convertvector(p[1], bf16x8);
        return __builtin_amdgcn_ballot_w64(!(psum <= limit)) != 0ull;
    };
    auto rescale = [&](const f32x16& s) {
        float cm = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) cm = fmaxf(cm, s[e]);
        cm *= scale_log2e;
        cm = fmaxf(cm, __shfl_xor(cm, 32));
        const float m_new = fmaxf(m, cm);
        const bool unset = m_new == SPKV_NEG_INF;      // every key so far excluded
        const float m_ref = unset ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m - m_ref);
        l *= alpha;
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] *= alpha;
        m = m_new;
        neg_ref = -m_ref;
        limit = unset ? -1.f : kWeightSumLimit;
        (void)weights(s);
    };
    bf16x8 va[2][NB];
    auto load_v = [&](const uint16_t* hp, int g) {
#pragma unroll
        for (int db = 0; db < NB; ++db)
            va[g][db] = *reinterpret_cast<const bf16x8*>(hp + kHalfTokens * D + (g * NB + db) * 512 + lane * 8);
    };
    auto accumulate = [&](int g) {
#pragma unroll
        for (int db = 0; db < NB; ++db)
            acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[g][db], pb[g], acc[db], 0, 0, 0);
    };
    // half-pages fast_begin <= x < fast_end need no mask
    int fast_begin = 0, fast_end = min(x_end, fullA);
    if (SOFT) {
        fast_begin = (u_min + kHalfTokens - 1) / kHalfTokens - sB0;
        fast_end = active ? min(x_end, (i0 + 1) / kHalfTokens - sB0) : 0;
    }
    // One half-page x at hp: its scores are in sc and its first V operands in va[0]; the scores of
    // the next one (hp1) go to sn from the K operands in kf, which are then those of hp2.  Every
    // LDS read is issued half a unit or more before its use, also across the barrier of a step
    // (what is read was announced by the barrier before); `more` runs between the products.
    auto unit = [&](f32x16& sc, f32x16& sn, int x, const uint16_t* hp, const float* bias,
                    const uint16_t* hp1, const uint16_t* hp2, const float* bias2, auto&& more) {
        const bool edge = x < fast_begin || x >= fast_end, seen = !edge || mine(x);
        if (edge) mask(sc, x, bias);
        __builtin_amdgcn_sched_barrier(0);
        scores(sn);
        const bool low = weights(sc);
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(low && seen, 0)) rescale(sc);
        load_v(hp, 1);
        load_k(hp2, SOFT && !all_biased(x + 2) ? s_zero : bias2);
        __builtin_amdgcn_sched_barrier(0);
        if (seen) {
            l += psum;
            accumulate(0);
        }
        load_v(hp1, 0);
        more();
        __builtin_amdgcn_sched_barrier(0);
        if (seen) accumulate(1);
        __builtin_amdgcn_sched_barrier(0);
    };

    // Queries and counts, and the kernel arguments the loop uses (a scalar load still pending at
    // its head makes the first operand wait of every pass wait for all LDS reads).
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    asm volatile("" : : "s"(scale_log2e));
    // Soft gating: where the loop lies against the 32-byte lines that instructions are fetched in counts,
    // with the same instructions: 4 sequences of 16k at the eight places 8275 (this one) to 8351 us, head_dim 64
    // 1333 (this one) to 1352.  (Moved by anything between here and the loop.)
    if (SOFT && D == 128) asm volatile(".p2align 5\n\t.rept 5\n\ts_nop 0\n\t.endr");
    if (SOFT && D != 128) asm volatile(".p2align 5\n\t.rept 7\n\ts_nop 0\n\t.endr");
    stage_step(x_begin, 0);
    stage_step(x_begin + 2, 1);
    stage_step(x_begin + 4, 2);
    wait_loads_but<kCopies>();                   // the first two steps have landed
    __syncthreads();
    f32x16 s0, s1;
    const int wb = SOFT ? wv : 0, b32 = SOFT ? 32 : 0;
    load_k(s_tile[0], SOFT && !all_biased(x_begin) ? s_zero : &s_bias[0][wb][0]);
    scores(s0);
    load_k(s_tile[0] + kHalfElems, SOFT && !all_biased(x_begin + 1) ? s_zero : &s_bias[0][wb][b32]);
    load_v(s_tile[0], 0);
    int buf = 0;
    for (int x = x_begin; x < x_end; x += 2) {
        const int nb = (buf + 1) & 3;
        const uint16_t* t0 = s_tile[buf];
        const uint16_t* t1 = s_tile[nb];
        const float* b0 = &s_bias[SOFT ? buf : 0][wb][0];
        const float* b1 = &s_bias[SOFT ? nb : 0][wb][0];
        unit(s0, s1, x, t0, b0, t0 + kHalfElems, t1, b1, [&]() { stage_step(x + 6, (buf + 3) & 3); });
        if (x + 1 >= x_end) break;               // (an odd last half-page: nothing left to read or wait for)
        unit(s1, s0, x + 1, t0 + kHalfElems, b0 + b32, t1, t1 + kHalfElems, b1 + b32, [&]() {});
        wait_loads_but<kCopies>();               // all but the newest: the step after next has landed
        __syncthreads();
        buf = nb;
    }
    wait_loads_but<0>();

    l += __shfl_xor(l, 32);
    if (!valid) return;
    if (pf.ks > 1) {
        const size_t n_cols = (size_t)pf.spans * pf.ks * (NW * 32);
        const size_t range = !SOFT && pf.order != nullptr ? (size_t)id * pf.ks + kr : ((size_t)pair * pf.nblk + qblk) * pf.ks + kr;
        const size_t pc = range * (NW * 32) + wv * 32 + col;
        float* pa = pf.part + pc * D + half * 4;
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f32x4*>(pa + db * 32 + g * 8) =
                    (f32x4){acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]};
        if (half == 0) {
            pf.part[n_cols * D + pc * 2] = m;
            pf.part[n_cols * D + pc * 2 + 1] = l;
        }
        return;
    }
    const size_t o = (size_t)(row0 + tok) * v.Hq + (size_t)h * v.G + (col - (col / v.G) * v.G);
    const float inv = 1.0f / l;
    uint16_t* po = out + o * D + half * 4;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const __bf16 r0 = (__bf16)(acc[db][4 * g] * inv), r1 = (__bf16)(acc[db][4 * g + 1] * inv);
            const __bf16 r2 = (__bf16)(acc[db][4 * g + 2] * inv), r3 = (__bf16)(acc[db][4 * g + 3] * inv);
            uint2 pk;
            pk.x = (unsigned)__builtin_bit_cast(uint16_t, r0) | ((unsigned)__builtin_bit_cast(uint16_t, r1) << 16);
            pk.y = (unsigned)__builtin_bit_cast(uint16_t, r2) | ((unsigned)__builtin_bit_cast(uint16_t, r3) << 16);
            *reinterpret_cast<uint2*>(po + db * 32 + g * 8) = pk;
        }
    if (lse != nullptr && half == 0) lse[o] = (m + log2f(l)) * 0.6931471805599453f;
}

// Merge of the tile ranges of one (span, column): out = sum_r 2^(m_r - M) acc_r /
// sum_r 2^(m_r - M) l_r.  A workgroup of 256 threads takes 256 / (D / 4) consecutive columns
// of a span's workgroup; a thread owns four consecutive output elements of one column.
// With f set (chunks attended before their append) the first n_pairs workgroups append the chunk
// meanwhile: the merge reads nothing of the cache.
template <int D>
__global__ __launch_bounds__(256) void spkv_prefill_combine(SpkvView v, uint16_t* __restrict__ out,
                                                            float* __restrict__ lse, SpkvPrefill pf,
                                                            SpkvCu cu, const uint16_t* __restrict__ k,
                                                            const uint16_t* __restrict__ vv,
                                                            const float* __restrict__ f) {
    const int n_append = f != nullptr ? v.n_pairs : 0;
    if ((int)blockIdx.x < n_append) {
        append_few<D>(v, blockIdx.x, k, vv, f, cu);
        return;
    }
    constexpr int TPC = D / 4, CPB = 256 / TPC;          // threads per column, columns per block
    const int kCols = pf.nw * pf.nq * 16;               // a multiple of CPB (of 16)
    const int blocks_per_span = kCols / CPB;
    const int id = (int)blockIdx.x - n_append, span = id / blocks_per_span;
    const int cs = (id - span * blocks_per_span) * CPB + (int)threadIdx.x / TPC;
    const int d = ((int)threadIdx.x % TPC) * 4;
    int pair = span / pf.nblk, qblk = span - pair * pf.nblk;
    size_t o = 0;
    auto holds_token = [&]() -> bool {                         // o: its output row
        const int b = pair / v.Hkv, h = pair - b * v.Hkv;
        const int row0 = cu.v[b], n_tok = cu.v[b + 1] - row0;
        if (pf.order != nullptr) qblk = (n_tok + pf.nw * pf.tb - 1) / (pf.nw * pf.tb) - 1 - qblk;
        const int wv = cs / (pf.nq * 16), col = cs - wv * (pf.nq * 16);
        const int i0 = qblk * pf.nw * pf.tb + wv * pf.tb;
        const int tbv = max(0, min(pf.tb, n_tok - i0));
        const int i = i0 + col / v.G, g = col - (col / v.G) * v.G;
        o = (size_t)(row0 + i) * v.Hq + (size_t)h * v.G + g;
        return col < tbv * v.G;
    };
    // in order, the pair is looked up beside the merge: columns without a token merge what nobody wrote
    SpanOrder e = {0, 0};
    if (pf.order != nullptr) e = span_entry(pf.order, v.n_pairs);
    else if (!holds_token()) return;
    const size_t n_cols = (size_t)(pf.slots > 0 ? pf.slots : pf.spans * pf.ks) * kCols;
    int2 cut = make_int2(span * pf.ks, pf.ks);                 // first range, ranges
    if (pf.slots > 0) cut = reinterpret_cast<const int2*>(pf.part + n_cols * (D + 2))[pair];
    const size_t pc0 = (size_t)cut.x * kCols + cs;             // range r: pc0 + r * kCols
    const float* ml = pf.part + n_cols * D;
    // Ranges kFold at a time, all their loads in flight together; only the rescaling is chained.
    constexpr int kFold = 8;
    float M = SPKV_NEG_INF, den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < cut.y; r0 += kFold) {
        float2 x[kFold];
        f32x4 a[kFold];
#pragma unroll
        for (int u = 0; u < kFold; ++u) {
            const size_t pc = pc0 + (size_t)min(r0 + u, cut.y - 1) * kCols;      // past the end: re-read, ignored
            x[u] = *reinterpret_cast<const float2*>(ml + pc * 2);
            a[u] = *reinterpret_cast<const f32x4*>(pf.part + pc * D + d);
        }
        float m_new = M;
#pragma unroll
        for (int u = 0; u < kFold; ++u)
            if (r0 + u < cut.y) m_new = fmaxf(m_new, x[u].x);
        const float m_ref = m_new == SPKV_NEG_INF ? 0.f : m_new, so = __builtin_amdgcn_exp2f(M - m_ref);
        den *= so;
        num *= so;
#pragma unroll
        for (int u = 0; u < kFold; ++u)
            if (r0 + u < cut.y) {
                const float sc = __builtin_amdgcn_exp2f(x[u].x - m_ref);         // 0 for a range without keys
                num += a[u] * sc;
                den += x[u].y * sc;
            }
        M = m_new;
    }
    if (pf.order != nullptr) {
        find_span(e, v.n_pairs, 0, span, pair, qblk);
        if (!holds_token()) return;
    }
    const float inv = 1.0f / den;
    uint2 packed;
    packed.x = (unsigned)__builtin_bit_cast(uint16_t, (__bf16)(num[0] * inv)) |
               ((unsigned)__builtin_bit_cast(uint16_t, (__bf16)(num[1] * inv)) << 16);
    packed.y = (unsigned)__builtin_bit_cast(uint16_t, (__bf16)(num[2] * inv)) |
               ((unsigned)__builtin_bit_cast(uint16_t, (__bf16)(num[3] * inv)) << 16);
    *reinterpret_cast<uint2*>(out + o * D + d) = packed;
    if (lse != nullptr && d == 0) lse[o] = (M + log2f(den)) * 0.6931471805599453f;
}

static SpkvPrefill prefill_params(const SpkvView& v, int n_max, uint16_t* stage, int32_t* prefix,
                                  float* bias, int shp, int ks = 1, float* part = nullptr,
                                  int slots = 0, bool once = false) {
    SpkvPrefill pf;
    pf.once = once ? 1 : 0;
    pf.ks = ks;
    pf.slots = slots;
    pf.part = part;
    pf.stage = stage;
    pf.prefix = prefix;
    pf.bias = bias;
    pf.bias_unit = 0.f;
    pf.shp = shp;
    SpkvPrefillShape sh = prefill_shape(v.G, n_max);
    if (bias != nullptr) sh = SpkvPrefillShape{2, 8, 32 / v.G};       // soft gating: one shape
    pf.tb = sh.tb;
    pf.nw = sh.nw;
    pf.nq = sh.nq;
    pf.nblk = (n_max + pf.nw * pf.tb - 1) / (pf.nw * pf.tb);   // spans of one workgroup
    pf.spans = v.n_pairs * pf.nblk;
    pf.order = nullptr;
    pf.groups = 1;
    pf.steps = 0;
    pf.pin_xcd = (pf.nw == 8 && v.n_pairs >= 8 && pf.nblk * pf.ks >= 4) ? 1 : 0;
    return pf;
}

static unsigned prefill_grid(const SpkvView& v, const SpkvPrefill& pf) {
    if (pf.slots > 0) return (unsigned)pf.slots;
    if (pf.order != nullptr) return 8u * (unsigned)pf.steps;
    return pf.pin_xcd ? 8u * (unsigned)((v.n_pairs + 7) / 8) * (unsigned)(pf.nblk * pf.ks)
                      : (unsigned)v.n_pairs * (unsigned)(pf.nblk * pf.ks);
}

SpkvPrefillShape spkv_prefill_shape(int group, int n_max) { return prefill_shape(group, n_max); }

// Spans in order (SpanOrder) for few pairs.  With each pair on an XCD of its own, pairs in turn (below,
// as from 65 pairs on), the XCD with the densest heads finishes last, and sequences that have ended
// leave theirs idle.  us for prompts in pieces of 4096 tokens, keep rates 0.1 to 0.33, pairs in turn / in
// order: one sequence of 16k 832 / 698, two 1400 / 1214, four 2500 / 2295, eight 4478 / 4428, four of
// 3k-19k 1872 / 1630; three of
// 3k-19k with 3 KV heads of 64 1520 / 807; one of 128k 35.0 / 26.9 ms.  Pairs share the XCDs in groups, so that a list is
// fetched into few L2s and neighbours find their windows there: all pairs on all XCDs took 2409
// (four) and 4825 us (eight), 112 against 105 ms for four of 128k; neighbours on different XCDs
// 2332 (four), but one whole prompt of 16k 700 instead of 728.
// Not where the spans run in one round, which the order cannot even out, nor for pieces of up to 4096 tokens
// that begin prompts (no list yet), whose spans differ by their own place more than by their pair's list:
// us a call, one sequence of 2100 66 / 67, 4096 106 / 106; two of 1100 62 / 65, 2048 81 / 83, 4096 163 / 152; four of
// 600 61 / 63, 4096 288 / 279; eight of 300 57 / 61, 2048 232 / 240, 4096 537 / 536.  Longer ones gain as others
// do: one of 4500 123 / 108, 12 000 437 / 353, two of 5000 222 / 195, eight of 6000 870 / 873.
bool spkv_prefill_ordered(const SpkvView& v, int n_max, bool from_empty) {
    const SpkvPrefillShape sh = prefill_shape(v.G, n_max);
    const int spans = v.n_pairs * ((n_max + sh.nw * sh.tb - 1) / (sh.nw * sh.tb));
    return sh.nw == 8 && v.n_pairs <= kSpanOrderPairs && spans > kPrefillResident8 &&
           !(from_empty && n_max <= 4096 && v.n_pairs % 8 == 0) && spkv_append_copies_lengths(v, n_max);
}
static void order_params(const SpkvView& v, const SpkvCu& cu, int n_max, SpkvPrefill& pf) {
    pf.order = v.bulk_info + kSpanOrderAt;
    pf.spans = spkv_prefill_spans(v, cu, n_max, true);
    pf.pin_xcd = 0;
    const int64_t pairs = (int64_t)cu.v[v.B] * v.Hkv / n_max;       // as many as would bring n_max tokens each
    // at least eight such pairs to a group: their unlike lengths even out
    pf.groups = 1;
    while (pf.ks == 1 && pairs >= 16 * pf.groups && v.Hkv % (2 * pf.groups) == 0 && pf.groups < 8) pf.groups *= 2;
    const int each = pf.spans / pf.groups * pf.ks;                  // a group has as many heads of every sequence
    const int run = 2 * (8 / pf.groups);
    pf.steps = (each + run - 1) / run * 2;
}

int spkv_prefill_spans(const SpkvView& v, const SpkvCu& cu, int n_max, bool ordered) {
    const SpkvPrefillShape sh = prefill_shape(v.G, n_max);
    const int span = sh.nw * sh.tb;
    if (!ordered) return v.n_pairs * ((n_max + span - 1) / span);
    int n = 0;
    for (int b = 0; b < v.B; ++b) n += (cu.v[b + 1] - cu.v[b] + span - 1) / span;
    return n * v.Hkv;
}

int spkv_prefill_slots(int n_pairs, SpkvPrefillShape sh, int head_dim, size_t part_bytes) {
    const size_t table = (size_t)n_pairs * sizeof(int2);
    const size_t slot = (size_t)(sh.nw * sh.nq * 16) * (head_dim + 2) * 4;
    if (sh.nw == 8 || n_pairs > 64 * kRangePairsPerLane || part_bytes < table) return 0;
    const size_t fit = (part_bytes - table) / slot;
    const int slots = fit < (size_t)kRangeSlots ? (int)fit : kRangeSlots;
    return slots > n_pairs ? slots : 0;
}

size_t spkv_prefill_partial_bytes(int spans, int ks, SpkvPrefillShape sh, int head_dim) {
    return ks > 1 ? (size_t)spans * ks * (sh.nw * sh.nq * 16) * (head_dim + 2) * 4 : 0;
}

// The attention launch of the shape chosen for the call.
template <int D, bool DIRECT>
static void launch_attend(const SpkvView& v, const uint16_t* q, uint16_t* out, float* lse, float sl,
                          const SpkvPrefill& pf, const SpkvCu& cu, const uint16_t* k, const uint16_t* vv,
                          hipStream_t s) {
    const dim3 grid(prefill_grid(v, pf));
    if (pf.nw == 8)
        spkv_prefill_attend32<D, false><<<grid, dim3(512), 0, s>>>(v, q, out, lse, sl, pf, cu);
    else if (pf.nq == 2)
        spkv_prefill_attend<D, 4, 2, DIRECT><<<grid, dim3(256), 0, s>>>(v, q, out, lse, sl, pf, cu, k, vv);
    else if (pf.nw == 4)
        spkv_prefill_attend<D, 4, 1, DIRECT><<<grid, dim3(256), 0, s>>>(v, q, out, lse, sl, pf, cu, k, vv);
    else
        spkv_prefill_attend<D, 2, 1, DIRECT><<<grid, dim3(128), 0, s>>>(v, q, out, lse, sl, pf, cu, k, vv);
}

static_assert(SPKV_MAX_CHUNK_TOKENS <= kFewTokens, "spkv_decode_chunk and spkv_score_chunk have no staging rows");
bool spkv_prefill_direct(const SpkvView& v, int n_max) {
    return n_max <= kFewTokens && n_max <= v.w && prefill_shape(v.G, n_max).nw != 8;
}

template <int D>
static hipError_t launch_prefill(const SpkvView& v, const uint16_t* k, const uint16_t* vv, const float* f,
                                 const uint16_t* q, uint16_t* out, float* lse, float sl, const SpkvCu& cu, int n_max,
                                 const SpkvPrefill& pf, SpkvLengthCopy to, hipStream_t s) {
    const bool direct = spkv_prefill_direct(v, n_max), merge = pf.ks > 1 || pf.slots > 0;
    if (direct) {
        launch_attend<D, true>(v, q, out, lse, sl, pf, cu, k, vv, s);
    } else {
        const int stage_hps = (v.w + n_max + kHalfTokens - 1) / kHalfTokens;
        SpkvStage st = {pf.stage, pf.bias, pf.bias_unit, pf.shp, stage_hps};
        if (!spkv_append_stages(v, n_max)) {
            spkv_prefill_stage<D><<<dim3(stage_hps, v.n_pairs), dim3(256), 0, s>>>(v, k, vv, f, cu, st);
            st.stage = nullptr;
        }
        const SpanCut cut = {pf.order != nullptr ? pf.nw * pf.tb : 0, pf.groups};
        const hipError_t e = spkv_launch_append_bulk(v, k, vv, f, cu, n_max, pf.prefix, cut, st, to, s);
        if (e != hipSuccess) return e;
        launch_attend<D, false>(v, q, out, lse, sl, pf, cu, nullptr, nullptr, s);
    }
    if (merge) {
        const float* fa = direct ? f : nullptr;
        const int blocks = pf.spans * (pf.nw * pf.nq * 16 / (256 / (D / 4)));
        spkv_prefill_combine<D><<<dim3((fa != nullptr ? v.n_pairs : 0) + blocks), dim3(256), 0, s>>>(v, out, lse, pf, cu, k, vv, fa);
    } else if (direct && f != nullptr) {
        return spkv_launch_append_bulk(v, k, vv, f, cu, n_max, nullptr, SpanCut{0, 1}, SpkvStage{}, to, s);
    }
    return hipGetLastError();
}

hipError_t spkv_launch_prefill(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                               const float* f, const uint16_t* q, uint16_t* out, float* lse,
                               float sm_scale, const SpkvCu& cu, int n_max, uint16_t* stage,
                               int32_t* prefix, int shp, bool ordered, int ks, int slots, bool once,
                               float* part, SpkvLengthCopy to, hipStream_t s) {
    SpkvPrefill pf = prefill_params(v, n_max, stage, prefix, nullptr, shp, ks, part, slots, once);
    if (ordered) order_params(v, cu, n_max, pf);
    const float sl = sm_scale * 1.4426950408889634f;
    return v.D == 128 ? launch_prefill<128>(v, k, vv, f, q, out, lse, sl, cu, n_max, pf, to, s)
                      : launch_prefill<64>(v, k, vv, f, q, out, lse, sl, cu, n_max, pf, to, s);
}

// Soft-gated attention of whole sequences (no cache): the same staging and the same tile
// loop with every earlier row visible and the bias log2 u on the rows outside the window.
// v: a view that only describes the shape (B, heads, D, w, n_pairs) and whose t_pair points
// at n_pairs zeros.
hipError_t spkv_launch_soft_gated(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                  const float* f, const uint16_t* q, uint16_t* out, float* lse,
                                  float sm_scale, const SpkvCu& cu, int n_max, uint16_t* stage,
                                  float* bias, int shp, hipStream_t s) {
    SpkvPrefill pf = prefill_params(v, n_max, stage, nullptr, bias, shp);
    // A pair to an XCD leaves some XCDs more pairs than others where their number is no multiple of eight:
    // then all pairs on all XCDs, unless the spans run in one round, whose tiles come sooner from one L2.
    // us, pairs of an XCD / all: 9 pairs of 700 tokens (99 spans) 37.3 / 39.2, of 2000 91 / 75, of 8000
    // 913 / 611, with head_dim 64 and groups of 8 1303 / 770; 12 of those 1347 / 1009; 20 pairs of 8000 834 / 700,
    // 30 2053 / 1953, 36 2552 / 2330.
    if (v.n_pairs % 8 != 0 && pf.spans > kPrefillResident8) pf.pin_xcd = 0;
    // (below 1e-30 a score no longer shows beside the biases: keeps bias / scale finite)
    const float sl = std::max(sm_scale * 1.4426950408889634f, 1e-30f);
    pf.bias_unit = 1.0f / sl;
    const int stage_hps = (v.w + n_max + kHalfTokens - 1) / kHalfTokens;
    const unsigned grid = prefill_grid(v, pf);
    const SpkvStage st = {pf.stage, pf.bias, pf.bias_unit, pf.shp, stage_hps};
    if (v.D == 128) {
        spkv_prefill_stage<128><<<dim3(stage_hps, v.n_pairs), dim3(256), 0, s>>>(v, k, vv, f, cu, st);
        spkv_prefill_attend32<128, true><<<dim3(grid), dim3(512), 0, s>>>(v, q, out, lse, sl, pf, cu);
    } else {
        spkv_prefill_stage<64><<<dim3(stage_hps, v.n_pairs), dim3(256), 0, s>>>(v, k, vv, f, cu, st);
        spkv_prefill_attend32<64, true><<<dim3(grid), dim3(512), 0, s>>>(v, q, out, lse, sl, pf, cu);
    }
    return hipGetLastError();
}

