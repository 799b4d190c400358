// Read path of the SP-KV cache on gfx950 (MI355X, wave64, MFMA):
//   spkv_decode_split    split-K flash decoding, one wave per work item, K/V tiles consumed
//                        as MFMA operands straight from the page layout
//                        (.._split_compact: the same items, workgroups numbered without gaps;
//                        spkv_decode_shares: large caches in equal shares)
//   spkv_decode_combine  log-sum-exp merge of the partials
//   fused step           spkv_decode_split<.., true> + spkv_combine_append: append and decode
//                        of one token per sequence in two launches instead of three; with
//                        the utility predictor riding along: spkv_decode_split_predict
//   multi-token step     spkv_chunk_split + spkv_chunk_combine: up to 16 new tokens per sequence
#include "spkv_device.h"

// One wavefront per work item.  The G <= 16 query heads of the GQA group are the N = 16
// columns of every MFMA, so each K/V tile is read exactly once per group.  Every wave-wide
// load is 1 KB contiguous.
// MW = sp.mw consecutive items of a pair form a workgroup.  With MW > 1 the waves work
// independently and meet once, at the end, to merge their (max, sum, acc) triples in LDS, so
// that one partial per workgroup goes to memory (the partial stores sit in the tail of every
// wave; a quarter of them measured 1.5-2 us less per launch) and the merge launch has a
// quarter to fold.  The host picks MW > 1 only when packing the items of every pair into whole
// workgroups does not lengthen the items (few pairs with long lists).
// Block id = pair * slots + jj with an odd slot count: workgroups go round-robin to the 8
// XCDs, so the items of every pair -- long or short -- spread evenly over all of them
// (heads differ in kept length by several times; pinning a head to one XCD would leave
// the others idle), and the odd stride keeps the per-pair remainders from piling up on
// the low XCDs.
//
// FUSED = false: the cache already holds the newest token (spkv_append ran before).
// FUSED = true (spkv_decode_step): the cache is in the state before the append of the
// newest token.  The kernel then excludes the ring slot that token will overwrite unless
// the pair in it passes the gate (it is the pair leaving the window: kept -> it stays
// attended, as the next long-term entry; dropped -> it is gone), and publishes every
// pair's item count for spkv_combine_append, which adds the new token's own term.
//
// Modes of the split kernel:
//   kSplitPlain     partials only (spkv_decode_attention in two launches, split-only timing)
//   kSplitFusedTwo  first launch of the two-launch fused step (FUSED above)
//   kSplitMerge     one launch for spkv_decode_attention: every workgroup of a (sequence, KV
//                   head), with or without work, takes a ticket of the pair once its partial
//                   (stored through to device scope) has arrived; the one that draws the last
//                   ticket -- all partials of the pair are then visible to it after a
//                   device-scope acquire -- merges them and writes `out` / `lse`
//   kSplitStep      one launch for the whole fused step: kSplitMerge in the state before the
//                   append (FUSED masking), the merging workgroup adds the new token's own term
//                   and then performs the pair's append.  Workgroups without work take a
//                   ticket too because they have read the pair's counters: the append may only
//                   change them once nobody will read them again in this launch.
// No workgroup ever waits for another: tickets are a single fetch-and-add, so the launch
// drains whatever the order in which its workgroups run.
constexpr int kSplitPlain = 0, kSplitFusedTwo = 1, kSplitMerge = 2, kSplitStep = 3;
constexpr int kMergePad = 16;    // floats between the rows of the LDS copy: no bank conflicts for G = 4

static size_t split_lds_bytes(int mw, int group, int head_dim) {
    if (mw == 1) return 0;
    return ((size_t)mw * group * (head_dim + kMergePad) + 2 * mw * 16) * sizeof(float);
}

// The work of one workgroup that has some: MW items of pair `pair`, their partial to slot
// pair * slots + jj.
template <int D, bool FUSED, int MW, bool SHARED>
__device__ __forceinline__ void split_compute(const SpkvView& v, const uint16_t* __restrict__ q,
                                              float scale_log2e, SpkvSplit sp, const PairSplit& ps,
                                              int pair, int jj, float* s_mem) {
    constexpr int NS = D / 32;   // head-dim slabs of one K tile
    constexpr int NB = D / 16;   // 16-wide output blocks
    const int wave = MW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int j = jj * MW + wave;
    // a wave past the pair's last item takes an empty range and joins the merge with weight 0
    const bool has_item = j < ps.items;
    const int hbase = ps.nhp / ps.items, hrem = ps.nhp - hbase * ps.items;
    const int hp0 = has_item ? j * hbase + min(j, hrem) : 0;
    const int hp1 = has_item ? hp0 + hbase + (j < hrem ? 1 : 0) : 0;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int lane = threadIdx.x & 63, kc = lane >> 4, n = lane & 15;

    bf16x8 qb[NS];
    {
        const uint16_t* qrow = q + ((size_t)b * v.Hq + (size_t)h * v.G + n) * D + kc * 8;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            uint4 raw = {0u, 0u, 0u, 0u};
            if (n < v.G) raw = *reinterpret_cast<const uint4*>(qrow + sl * 32);
            qb[sl] = __builtin_bit_cast(bf16x8, raw);
        }
    }
    f32x4 acc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = SPKV_NEG_INF, l = 0.f;
    const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;

    // Fused step: which ring key (if any) must be left out.  Only items that reach into
    // the ring look (most do not), and only after their query loads are under way.
    int drop_hp = -1, drop_r = -1;
    if (FUSED && hp1 > ps.ghp && ps.T >= v.w) {
        const int slot = ps.T % v.w;
        if (!gate_passes(v, v.ring_logit[(size_t)pair * v.w + slot], ps.T - v.w)) {
            drop_hp = ps.ghp + (slot >> 5);
            drop_r = slot & 31;
        }
    }

    int hp = hp0;
    while (hp < hp1) {
        // Page ids of the next 64 logical pages, one per lane; read back with readlane so
        // that no half-page waits on a dependent table lookup.
        const int pbase = hp >> 1;
        const int my_page = pt[min(pbase + lane, v.pt_cap - 1)];
        const int hp_end = min(hp1, (pbase + 64) << 1);
        for (; hp < hp_end; ++hp) {
            const uint16_t* base;
            int nvalid;
            if (hp < ps.ghp) {
                const int page = __builtin_amdgcn_readlane(my_page, (hp >> 1) - pbase);
                base = pool_page(v, page) + (hp & 1) * (2 * kHalfTokens * D);
                nvalid = min(kHalfTokens, ps.L - hp * kHalfTokens);
            } else {
                const int r = hp - ps.ghp;
                base = ring_page(v, pair, r >> 1) + (r & 1) * (2 * kHalfTokens * D);
                nvalid = min(kHalfTokens, ps.Tw - r * kHalfTokens);
            }
            // keys past the valid length, and (fused step) the pair leaving the window
            const int masked_r = (FUSED && hp == drop_hp) ? drop_r : -1;
            const bool any_kill = nvalid < kHalfTokens || masked_r >= 0;
            unsigned kill = 0u;
            if (any_kill) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (kc * 8 + e >= nvalid || kc * 8 + e == masked_r) kill |= 1u << e;
            }
            const uint16_t* kp = base + lane * 8;
            const uint16_t* vp = base + kHalfTokens * D + lane * 8;
            bf16x8 ka[2][NS], va[NB];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int sl = 0; sl < NS; ++sl)
                    ka[t][sl] = load_stream_b128(kp + (t * (D / 8) + sl * 4) * 128);
#pragma unroll
            for (int db = 0; db < NB; ++db) va[db] = load_stream_b128(vp + db * 512);
            // (Forcing all 16 loads ahead of the first MFMA with a scheduling barrier was
            // measured 2 % slower than the compiler's interleaving of loads and MFMAs.)
            attend_half_page<D>(ka, va, qb, kill, any_kill, scale_log2e, acc, m, l);
        }
    }

    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const size_t slot = (size_t)pair * sp.slots + jj;
    // SHARED: the partial is read by another workgroup of this launch (see ticket_merge)
    if (MW == 1) {
        if (n < v.G) {
            float* pa = v.part_acc + (slot * v.G + n) * D + kc * 4;
#pragma unroll
            for (int db = 0; db < NB; ++db) {
                if (SHARED) store_device_b128(pa + db * 16, acc[db]);
                else *reinterpret_cast<f32x4*>(pa + db * 16) = acc[db];
            }
            if (kc == 0) {
                float* pm = v.part_ml + (slot * v.G + n) * 2;
                if (SHARED) {
                    store_device_b32(pm, m);
                    store_device_b32(pm + 1, l);
                } else {
                    pm[0] = m;
                    pm[1] = l;
                }
            }
        }
        return;
    }
    // the workgroup's waves meet: acc[wave][head][d] (rows kMergePad floats apart), m, l
    constexpr int kRow = D + kMergePad;
    float* s_acc = s_mem;
    float* s_m = s_mem + MW * v.G * kRow;
    float* s_l = s_m + MW * 16;
    if (n < v.G) {
        float* pa = s_acc + (wave * v.G + n) * kRow + kc * 4;
#pragma unroll
        for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(pa + db * 16) = acc[db];
        if (kc == 0) {
            s_m[wave * 16 + n] = m;
            s_l[wave * 16 + n] = l;
        }
    }
    __syncthreads();
    // one partial per workgroup: with M the largest reference of the waves,
    // acc = sum_w 2^(m_w - M) acc_w,  l = sum_w 2^(m_w - M) l_w
    for (int e = threadIdx.x; e < v.G * D; e += 64 * MW) {
        const int g = e / D, d = e - g * D;
        float mw[MW], M = SPKV_NEG_INF;
#pragma unroll
        for (int w = 0; w < MW; ++w) {
            mw[w] = s_m[w * 16 + g];
            M = fmaxf(M, mw[w]);
        }
        const float m_ref = (M == SPKV_NEG_INF) ? 0.f : M;      // no key at all: every weight 0
        float a = 0.f, lsum = 0.f;
#pragma unroll
        for (int w = 0; w < MW; ++w) {
            const float sc = __builtin_amdgcn_exp2f(mw[w] - m_ref);
            a += sc * s_acc[(w * v.G + g) * kRow + d];
            lsum += sc * s_l[w * 16 + g];
        }
        float* pa = v.part_acc + (slot * v.G + g) * D + d;
        float* pm = v.part_ml + (slot * v.G + g) * 2;
        if (SHARED) {
            store_device_b32(pa, a);
            if (d == 0) {
                store_device_b32(pm, M);
                store_device_b32(pm + 1, lsum);
            }
        } else {
            *pa = a;
            if (d == 0) {
                pm[0] = M;
                pm[1] = lsum;
            }
        }
    }
}

// Ticket and merge.  Every workgroup of the pair calls this once, after its partial (if it
// had work) has been stored.  In the merging workgroup a thread owns eight consecutive
// floats of the pair's G x D outputs (a "unit": two float4 of one head); the waves share the
// partials round-robin, their loads go out eight partials at a time and only the cheap
// rescaling is chained; with several waves the wave results meet in LDS.
template <int D, bool STEP, int MW>
__device__ __forceinline__ void ticket_merge(const SpkvView& v, const uint16_t* __restrict__ q,
                                             float scale_log2e, SpkvSplit sp, const PairSplit& ps,
                                             int pair, float* s_mem, int* s_page, const SpkvStepIO& io) {
    constexpr int NT = 64 * MW, UPH = D / 8, U = 8, kRow = D + kMergePad;
    const int tid = threadIdx.x;
    wait_all_vmem();          // this thread's partial stores (written through) have arrived
    int ticket = 0;
    if (MW == 1) {
        if (tid == 0) ticket = atomicAdd(v.pair_ticket + pair, 1);
        ticket = __builtin_amdgcn_readfirstlane(ticket);
    } else {
        int* s_t = reinterpret_cast<int*>(s_mem);
        __syncthreads();                                     // all threads released; LDS is free
        if (tid == 0) *s_t = atomicAdd(v.pair_ticket + pair, 1);
        __syncthreads();
        ticket = *s_t;
        __syncthreads();                                     // before LDS is written again
    }
    if (ticket != sp.slots - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");       // the others' partials
    if (tid == 0) v.pair_ticket[pair] = 0;                   // for the next launch

    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int lane = tid & 63, wave = MW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t kv_row = ((size_t)b * v.Hkv + h) * D;
    const int n_part = ps.groups, NU = v.G * UPH;            // units of the pair
    const size_t slot0 = (size_t)pair * sp.slots;
    float* s_acc = s_mem;                                    // [MW][G][kRow]   (MW > 1 only)
    float* s_m = s_mem + MW * v.G * kRow;                    // [MW][16]
    float* s_l = s_m + MW * 16;

    // The finish of one unit: the new token's own term (step), normalisation, bf16, store.
    auto finish = [&](int g, int d8, bool ok, float M, float den, const f32x4 (&acc)[2]) {
        const size_t o_row = (size_t)b * v.Hq + (size_t)h * v.G + g;
        float Mt = M, w_tok = 0.f;
        f32x4 vn[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        if (STEP) {
            // score q . k_new in fp32 (the UPH lanes of a head add up), weight sum 1, value v_new
            const uint4 qe = *reinterpret_cast<const uint4*>(q + o_row * D + d8 * 8);
            const uint4 ke = *reinterpret_cast<const uint4*>(io.k_new + kv_row + d8 * 8);
            const uint4 ve = *reinterpret_cast<const uint4*>(io.v_new + kv_row + d8 * 8);
            const unsigned qw[4] = {qe.x, qe.y, qe.z, qe.w}, kw[4] = {ke.x, ke.y, ke.z, ke.w};
            const unsigned vw[4] = {ve.x, ve.y, ve.z, ve.w};
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dot += __builtin_bit_cast(float, qw[e] << 16) * __builtin_bit_cast(float, kw[e] << 16);
                dot += __builtin_bit_cast(float, qw[e] & 0xffff0000u) * __builtin_bit_cast(float, kw[e] & 0xffff0000u);
                vn[e >> 1][(e & 1) * 2] = __builtin_bit_cast(float, vw[e] << 16);
                vn[e >> 1][(e & 1) * 2 + 1] = __builtin_bit_cast(float, vw[e] & 0xffff0000u);
            }
            if (!ok) dot = 0.f;
#pragma unroll
            for (int o = UPH / 2; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
            const float m_tok = dot * scale_log2e;
            Mt = fmaxf(M, m_tok);
            w_tok = __builtin_amdgcn_exp2f(m_tok - Mt);
        }
        const float m_ref = (Mt == SPKV_NEG_INF) ? 0.f : Mt;
        const float sc = __builtin_amdgcn_exp2f(M - m_ref);
        const float dsum = den * sc + w_tok;
        if (ok) {
            unsigned pk[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = (acc[e >> 1][(e & 1) * 2] * sc + vn[e >> 1][(e & 1) * 2] * w_tok) / dsum;
                const float x1 = (acc[e >> 1][(e & 1) * 2 + 1] * sc + vn[e >> 1][(e & 1) * 2 + 1] * w_tok) / dsum;
                const __bf16 r0 = (__bf16)x0, r1 = (__bf16)x1;
                pk[e] = (unsigned)__builtin_bit_cast(uint16_t, r0) | ((unsigned)__builtin_bit_cast(uint16_t, r1) << 16);
            }
            *reinterpret_cast<uint4*>(io.out + o_row * D + d8 * 8) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            if (io.lse != nullptr && d8 == 0) io.lse[o_row] = (Mt + log2f(dsum)) * 0.6931471805599453f;
        }
    };

    AppendRegs<D, NT> ar;
    if (STEP)      // the append's loads travel while the partials are merged
        ar = append_load<D, NT>(v, pair, h, b, ps.T, ps.L, io.k_new, io.v_new,
                                io.f_new[(size_t)b * v.Hkv + h], tid);

    for (int u0 = 0; u0 < NU; u0 += 64) {        // every wave: all units, its share of the partials
        const int unit = u0 + lane;
        const bool ok = unit < NU;
        const int g = ok ? unit / UPH : 0, d8 = ok ? unit - g * UPH : 0;
        float M = SPKV_NEG_INF, den = 0.f;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        for (int i0 = wave; i0 < n_part; i0 += U * MW) {
            f32x4 a[U][2];
            float2 ml[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t row = (slot0 + min(i0 + u * MW, n_part - 1)) * v.G + g;   // past the end: re-read, ignored
                const float* pa = v.part_acc + row * D + d8 * 8;
                a[u][0] = *reinterpret_cast<const f32x4*>(pa);
                a[u][1] = *reinterpret_cast<const f32x4*>(pa + 4);
                ml[u] = *reinterpret_cast<const float2*>(v.part_ml + row * 2);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * MW < n_part) {
                    const float m_new = fmaxf(M, ml[u].x);
                    const float m_ref = (m_new == SPKV_NEG_INF) ? 0.f : m_new;   // partials with no key: weight 0
                    const float so = __builtin_amdgcn_exp2f(M - m_ref);
                    const float si = __builtin_amdgcn_exp2f(ml[u].x - m_ref);
                    den = den * so + ml[u].y * si;
                    acc[0] = acc[0] * so + a[u][0] * si;
                    acc[1] = acc[1] * so + a[u][1] * si;
                    M = m_new;
                }
            }
        }
        if (MW == 1) {
            finish(g, d8, ok, M, den, acc);
        } else if (ok) {
            float* pa = s_acc + (wave * v.G + g) * kRow + d8 * 8;
            *reinterpret_cast<f32x4*>(pa) = acc[0];
            *reinterpret_cast<f32x4*>(pa + 4) = acc[1];
            if (d8 == 0) {
                s_m[wave * 16 + g] = M;
                s_l[wave * 16 + g] = den;
            }
        }
    }
    if (MW > 1) {
        __syncthreads();
        for (int u0 = 0; u0 < NU; u0 += NT) {
            const int unit = u0 + tid;
            const bool ok = unit < NU;
            const int g = ok ? unit / UPH : 0, d8 = ok ? unit - g * UPH : 0;
            float mw[MW], M = SPKV_NEG_INF;
#pragma unroll
            for (int w = 0; w < MW; ++w) {
                mw[w] = s_m[w * 16 + g];
                M = fmaxf(M, mw[w]);
            }
            const float m_ref = (M == SPKV_NEG_INF) ? 0.f : M;
            float den = 0.f;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int w = 0; w < MW; ++w) {
                const float sc = __builtin_amdgcn_exp2f(mw[w] - m_ref);
                const float* pa = s_acc + (w * v.G + g) * kRow + d8 * 8;
                acc[0] += *reinterpret_cast<const f32x4*>(pa) * sc;
                acc[1] += *reinterpret_cast<const f32x4*>(pa + 4) * sc;
                den += s_l[w * 16 + g] * sc;
            }
            finish(g, d8, ok, M, den, acc);
        }
    }
    if (STEP) append_store<D, NT>(v, pair, ps.T, ps.L, ar, tid, s_page);
}

template <int D, int MODE, int MW>
__device__ __forceinline__ void decode_split_item(const SpkvView& v, const uint16_t* __restrict__ q,
                                                  float scale_log2e, SpkvSplit sp, int wg, float* s_mem,
                                                  int* s_page, const SpkvStepIO& io) {
    constexpr bool FUSED = MODE == kSplitFusedTwo || MODE == kSplitStep;
    const int pair = wg / sp.slots;
    const int jj = wg - pair * sp.slots;
    const PairSplit ps = pair_split(v, pair, sp);
    if (MODE == kSplitFusedTwo && jj == 0 && threadIdx.x == 0) v.pair_items[pair] = ps.groups;
    constexpr bool TICKET = MODE == kSplitMerge || MODE == kSplitStep;
    if (jj < ps.groups)       // the whole workgroup
        split_compute<D, FUSED, MW, TICKET>(v, q, scale_log2e, sp, ps, pair, jj, s_mem);
    if (MODE == kSplitMerge || MODE == kSplitStep)
        ticket_merge<D, MODE == kSplitStep, MW>(v, q, scale_log2e, sp, ps, pair, s_mem, s_page, io);
}

// Merge workgroups of 16 waves instead of 4: when pairs have more than 64 partials and the
// merge launch has at most one workgroup per compute unit (few long sequences; measured on
// 4 sequences of 128k with about 150 partials per pair: 1.1 us less per step; with 39 per
// pair, 0.5 us more; with 512 merge workgroups, 3 us more).  With equal shares, whose partial results
// begin where a load says, from 48 in the longest list on.  Step, 4 / 16 waves, us: 8 pairs of 26 MB, 76 in the longest
// 14.4 / 13.6, of 240 MB 46.1 / 45.5; 12 pairs of 40 MB, 52 16.6 / 15.6; 16 of 64 MB, 44 19.0 / 19.4; 24 of 64 MB, 29
// 18.4 / 19.4; but one dense head in eight, 16 pairs of 26 MB, 200 17.3 / 15.4, 32 of 100 MB, 100 26.2 / 25.2, 64 of
// 100 MB, 50 25.8 / 25.6.
static bool wide_merge(const SpkvView& v, const SpkvSplit& sp) {
    return (sp.runs > 0 ? sp.most > 48 : sp.slots > 64) && v.n_pairs * v.G <= 256;
}

template <int D, int MODE, int MW>
__global__ __launch_bounds__(64 * MW) void spkv_decode_split(SpkvView v, const uint16_t* __restrict__ q,
                                                             float scale_log2e, SpkvSplit sp, SpkvStepIO io) {
    extern __shared__ __attribute__((aligned(16))) float s_split[];
    __shared__ int s_page;
    decode_split_item<D, MODE, MW>(v, q, scale_log2e, sp, blockIdx.x, s_split, &s_page, io);
}

// The same with workgroups numbered without gaps (host: SpkvSplit.compact of them, one item per
// wave): id -> (pair, item) by a prefix sum of the pairs' item counts, which every wave takes for
// itself from the exact lengths.  Under the plain numbering the ids of short pairs that have no
// work lie between the items, and which compute units the dispatcher fills with how many
// items depends on the pattern of the lengths; the compute unit (or die) that gets the most sets
// the time.  Without gaps the items spread evenly whatever the lengths are, and fewer of them
// do: seven waves per compute unit (1792 items) keep enough bytes in flight, store fewer partials
// and leave room for a compute unit that is handed one more (1300 items: 2 to 19 % longer; 2944: 1 to
// 4 %).  The prefix sum costs about 1 us of every wave's start.  The host takes this numbering for
// uneven lists only (worth_gapless, with the times of both).
// n_wg comes from the host's bound of the lengths, with a workgroup more per pair in a captured
// launch; when a replayed graph has outgrown that, workgroups take a second item.
// Item `id` of all pairs' items in order: its pair and its index there; false past the last one.
// total: the number of items.  PUBLISH: the wave of id 0 stores every pair's item count.
template <bool PUBLISH>
__device__ __forceinline__ bool locate_item(const SpkvView& v, SpkvSplit sp, int id, int& total, int& pair, int& jj) {
    const int lane = threadIdx.x & 63;
    const int per_lane = (v.n_pairs + 63) >> 6;            // consecutive pairs of a lane
    const int p0 = lane * per_lane, p1 = min(p0 + per_lane, v.n_pairs);
    auto groups_of = [&](int p) -> int { return p < p1 ? pair_split(v, min(p, v.n_pairs - 1), sp).groups : 0; };
    int sum = 0;
#pragma unroll 4
    for (int i = 0; i < per_lane; ++i) sum += groups_of(p0 + i);
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    total = __builtin_amdgcn_readlane(incl, 63);
    if (PUBLISH && id == 0)
        for (int p = p0; p < p1; ++p) v.pair_items[p] = groups_of(p);
    if (id >= total) return false;
    int mine = -1, first = 0, run = incl - sum;
#pragma unroll 4
    for (int i = 0; i < per_lane; ++i) {
        const int g = groups_of(p0 + i);
        if (id >= run && id < run + g) {
            mine = p0 + i;
            first = run;
        }
        run += g;
    }
    const int src = __builtin_ctzll(__ballot(mine >= 0));
    pair = __builtin_amdgcn_readlane(mine, src);
    jj = id - __builtin_amdgcn_readlane(first, src);
    return true;
}

template <int D, bool FUSED>
__device__ __forceinline__ void decode_split_compact(const SpkvView& v, const uint16_t* __restrict__ q,
                                                     float scale_log2e, SpkvSplit sp, int wg, int n_wg) {
    int id = wg, total, pair, jj;
    do {
        if (!locate_item<FUSED>(v, sp, id, total, pair, jj)) return;
        split_compute<D, FUSED, 1, false>(v, q, scale_log2e, sp, pair_split(v, pair, sp), pair, jj, nullptr);
        id += n_wg;
    } while (id < total);
}

// (Three waves per SIMD asked for by attribute: left alone the prefix sum takes it to two.)
template <int D, bool FUSED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void spkv_decode_split_compact(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e, SpkvSplit sp) {
    decode_split_compact<D, FUSED>(v, q, scale_log2e, sp, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------ equal shares
// Large caches (host: share_split): the half-pages of all pairs, in order, are cut into SpkvSplit.runs equal
// runs, one per one-wave workgroup.  A run may begin in one pair and end in another and leaves a partial result
// in each; run i and pair p share partial slot i + p (no two overlaps have the same sum).  Every wave finds its
// run from the exact lengths, so the runs stay equal in a graph replayed on growing lists; one workgroup more
// leaves the merge every pair's slots.
// What bounds a step of this size is the rate of one compute unit, which little keeps up: a wave with one
// half-page in work and the next in flight.  More waves queue up behind each other, leave more to merge, and
// any that one compute unit has more than another work on alone at the end (hence whole multiples of the compute
// units, and no rounding to whole items per pair).  The loads behind a run's end are issued against a buffer of no
// bytes, so that what a half-page waits for is a constant number of loads in flight.
// 16 sequences of 32k, 484 MB, us a step: 82.3 as items of one pair each (2880 waves), 78.0 with 512 runs, 78.2
// with 256, 79.3 with 768, 80.3 with 1024, 81.9 with 640; three half-pages in registers 79.2.  A plain read
// of the same bytes takes 71 with 1792 workgroups, 72.7 with 2880.  The weights go in two bf16 parts
// (attend_half_page), which 512 waves have the time for (256 of them do not: 8 pairs of 156 MB 30.1 -> 32.0).
constexpr int kPairUnits = 1;    // a pair's units: its half-pages and one for what beginning it costs
__device__ __forceinline__ int list_half_pages(int n) { return (n + kHalfTokens - 1) >> 5; }
// Sum over the lanes up to and including this one.
__device__ __forceinline__ int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
    return x;
}
struct RunStart {
    int pair, L, T, hp, left;            // first half-page, its pair and lengths; units from there on
};
// All lengths in one round of loads, four pairs a lane.  run = n_runs: the workgroup of the merge's table, first
// slot | number of partial results << 16 of every pair.  False: no half-page for this workgroup.
// counts(pair): does the pair take part?
template <class Counts>
__device__ __forceinline__ bool find_run(const SpkvView& v, int run, int n_runs, RunStart& r, Counts counts) {
    constexpr int kChunks = kSharePairs / 256;
    const int lane = threadIdx.x & 63, last4 = (v.n_pairs - 1) & ~3;     // (both arrays are padded to 256 bytes)
    int4 L[kChunks], T[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
        if (c * 256 < v.n_pairs) {
            const int p = min(c * 256 + lane * 4, last4);
            L[c] = *reinterpret_cast<const int4*>(v.kept_len + p);
            T[c] = *reinterpret_cast<const int4*>(v.t_pair + p);
        }
    }
    auto units = [&](int p, int l, int t) -> int {
        const int n = p < v.n_pairs && counts(p) ? list_half_pages(l) + list_half_pages(min(t, v.w)) : 0;
        return n > 0 ? n + kPairUnits : 0;
    };
    int n[kChunks][4], before[kChunks], total = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
        if (c * 256 < v.n_pairs) {
            const int p = c * 256 + lane * 4;
            n[c][0] = units(p, L[c].x, T[c].x);
            n[c][1] = units(p + 1, L[c].y, T[c].y);
            n[c][2] = units(p + 2, L[c].z, T[c].z);
            n[c][3] = units(p + 3, L[c].w, T[c].w);
            const int sum = n[c][0] + n[c][1] + n[c][2] + n[c][3], incl = wave_scan(sum);
            before[c] = total + incl - sum;
            total += __builtin_amdgcn_readlane(incl, 63);
        }
    }
    // run i begins at unit i * share + min(i, more)
    const int share = total / n_runs, more = total - share * n_runs;
    if (run == n_runs) {
        const int longer = more * (share + 1);
        auto run_of = [&](int x) -> int { return x < longer ? x / (share + 1) : more + (x - longer) / share; };
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            if (c * 256 < v.n_pairs) {
                int at = before[c];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int p = c * 256 + lane * 4 + e;
                    int packed = 0;
                    if (n[c][e] > 0) {
                        const int r0 = run_of(at + kPairUnits);
                        packed = (run_of(at + n[c][e] - 1) - r0 + 1) << 16 | (r0 + p);
                    }
                    if (p < v.n_pairs) v.pair_items[p] = packed;
                    at += n[c][e];
                }
            }
        }
        return false;
    }
    const int x = run * share + min(run, more), len = share + (run < more ? 1 : 0);
    if (len == 0) return false;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
        if (c * 256 < v.n_pairs) {
            int at = before[c], mine = -1, first = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (x >= at && x < at + n[c][e]) {
                    mine = e;
                    first = at;
                }
                at += n[c][e];
            }
            const unsigned long long m = __ballot(mine >= 0);
            if (m != 0ull) {
                const int src = __builtin_ctzll(m), e = __builtin_amdgcn_readlane(mine, src);
                const int j = x - __builtin_amdgcn_readlane(first, src);
                r.pair = c * 256 + src * 4 + e;
                r.L = __builtin_amdgcn_readlane(e == 0 ? L[c].x : e == 1 ? L[c].y : e == 2 ? L[c].z : L[c].w, src);
                r.T = __builtin_amdgcn_readlane(e == 0 ? T[c].x : e == 1 ? T[c].y : e == 2 ? T[c].z : T[c].w, src);
                r.hp = max(0, j - kPairUnits);
                r.left = len - max(0, kPairUnits - j);
            }
        }
    }
    return true;
}

// The next pair behind `pair` that takes part, and its lengths; false: there is none.  Nearly always the one behind.
// Empty sequences, and in a multi-token call those without a token, are passed over 256 pairs a round of loads: one by
// one each pair waits for its own, and the launch for the run that crosses the gap: 64 sequences x 8 heads, 400 MB,
// drafts for the first and the last of them 137 us, 18 so (28.8 in items); 16 sequences, 200 MB 42 and 17 (25).
template <class Counts>
__device__ __forceinline__ bool next_pair(const SpkvView& v, int& pair, int& L, int& T, Counts counts) {
    if (++pair >= v.n_pairs) return false;
    L = v.kept_len[pair];
    T = v.t_pair[pair];
    if (T > 0 && counts(pair)) return true;
    const int lane = threadIdx.x & 63, last4 = (v.n_pairs - 1) & ~3;
    for (int p0 = (pair + 1) & ~3; p0 < v.n_pairs; p0 += 256) {
        const int p = p0 + lane * 4, at = min(p, last4);
        const int4 l = *reinterpret_cast<const int4*>(v.kept_len + at), t = *reinterpret_cast<const int4*>(v.t_pair + at);
        auto here = [&](int e, int n) -> bool { return p + e > pair && p + e < v.n_pairs && n > 0 && counts(p + e); };
        const int mine = here(0, t.x) ? 0 : here(1, t.y) ? 1 : here(2, t.z) ? 2 : here(3, t.w) ? 3 : 4;
        const unsigned long long m = __ballot(mine < 4);
        if (m != 0ull) {
            const int src = __builtin_ctzll(m), e = __builtin_amdgcn_readlane(mine, src);
            pair = p0 + src * 4 + e;
            L = __builtin_amdgcn_readlane(e == 0 ? l.x : e == 1 ? l.y : e == 2 ? l.z : l.w, src);
            T = __builtin_amdgcn_readlane(e == 0 ? t.x : e == 1 ? t.y : e == 2 ? t.z : t.w, src);
            return true;
        }
    }
    return false;
}

template <int D>
struct HalfPage {
    bf16x8 k[2][D / 32], v[D / 16];
};
template <int D>
__device__ __forceinline__ void load_half_page(HalfPage<D>& t, const uint16_t* base, bool wanted, int lane) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(base), 0, wanted ? 4 * kHalfTokens * D : 0, 0x00027000);
    auto get = [&](int at) -> bf16x8 {                                   // non-temporal
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + (at & 4095), at & ~4095, 2));
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int sl = 0; sl < D / 32; ++sl) t.k[i][sl] = get((i * (D / 8) + sl * 4) * 256);
#pragma unroll
    for (int db = 0; db < D / 16; ++db) t.v[db] = get(2 * kHalfTokens * D + db * 1024);
}

// KIND: the state of the cache and the columns, as in the split kernel (kSplitPlain, kSplitFusedTwo) or in
// the multi-token step (kSplitChunk: spkv_chunk_split; cu is looked at there alone).
constexpr int kSplitChunk = 4;
template <int D, int KIND>
__device__ __forceinline__ void attend_run(const SpkvView& v, const uint16_t* __restrict__ q, float scale_log2e,
                                           int run, int n_runs, const SpkvCu* cu) {
    constexpr bool FUSED = KIND == kSplitFusedTwo, CHUNK = KIND == kSplitChunk;
    constexpr int NS = D / 32, NB = D / 16, NT = D == 128 ? 2 : 4;
    constexpr int kNoVmem = 0x0f70;                // s_waitcnt vmcnt(0)
    const int lane = threadIdx.x & 63, kc = lane >> 4, n = lane & 15;
    auto counts = [&](int p) -> bool {
        if (!CHUNK) return true;
        const int b = p / v.Hkv;
        return cu->v[b + 1] > cu->v[b];
    };
    RunStart r;
    if (!find_run(v, run, n_runs, r, counts)) return;
    int pair = r.pair, L = r.L, T = r.T, left = r.left, hp0 = r.hp;
    while (true) {                                 // the run's part of pair after pair
        const int b = pair / v.Hkv, h = pair - b * v.Hkv;
        const int row0 = CHUNK ? cu->v[b] : b, n_tok = CHUNK ? cu->v[b + 1] - row0 : 1;
        const int Tw = min(T, v.w), ghp = list_half_pages(L), nhp = n_tok > 0 ? ghp + list_half_pages(Tw) : 0;
        const int hp1 = min(nhp, hp0 + left);
        if (hp1 > hp0) {
            const int cols = n_tok * v.G;          // column n: token n / G, head n % G
            const int tok = CHUNK ? n / v.G : 0;
            const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
            const float* rl = v.ring_logit + (size_t)pair * v.w;
            int pbase = hp0 >> 1, my_page = pt[min(pbase + lane, v.pt_cap - 1)];     // 64 page ids, one per lane
            bf16x8 qb[NS];
            const uint16_t* qrow = q + ((size_t)(row0 + tok) * v.Hq + (size_t)h * v.G + (CHUNK ? n - tok * v.G : n)) * D + kc * 8;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                uint4 raw = {0u, 0u, 0u, 0u};
                if (n < cols) raw = *reinterpret_cast<const uint4*>(qrow + sl * 32);
                qb[sl] = __builtin_bit_cast(bf16x8, raw);
            }
            // Step: the ring key that leaves the window and fails the gate.
            int drop_hp = -1, drop_r = -1;
            if (FUSED && hp1 > ghp && T >= v.w) {
                const int slot = T % v.w;
                if (!gate_passes(v, rl[slot], T - v.w)) {
                    drop_hp = ghp + (slot >> 5);
                    drop_r = slot & 31;
                }
            }
            // Chunk: the gates of 64 ring half-pages from g0 on, one per lane.
            const int slot0 = T >= v.w ? T % v.w : T - v.w;                // slot of age 0
            auto age_of = [&](int at) -> int { return at - slot0 + (at < slot0 ? v.w : 0); };
            int g0 = 0;
            unsigned gates = 0u;
            auto load_gates = [&](int from) {
                g0 = from;
                for (int i = 0; i < min(hp1 - ghp - from, 64); i += 2) {
                    const int at = min((from + i) * kHalfTokens + lane, Tw - 1);
                    const unsigned long long on = __ballot(gate_passes(v, rl[at], T - v.w + age_of(at)));
                    gates = lane == i ? (unsigned)on : lane == i + 1 ? (unsigned)(on >> 32) : gates;
                }
            };
            if (CHUNK && hp1 > ghp) load_gates(max(0, hp0 - ghp));
            f32x4 acc[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
            float m = SPKV_NEG_INF, l = 0.f;
            __builtin_amdgcn_s_waitcnt(kNoVmem);   // nothing of the above is waited for in the loop
            auto load = [&](HalfPage<D>& t, int hp) {
                const uint16_t* base;
                if (hp < ghp) {
                    if ((hp >> 1) >= pbase + 64) {
                        pbase = hp >> 1;
                        my_page = pt[min(pbase + lane, v.pt_cap - 1)];
                        __builtin_amdgcn_s_waitcnt(kNoVmem);
                    }
                    base = pool_page(v, __builtin_amdgcn_readlane(my_page, (hp >> 1) - pbase)) + (hp & 1) * (2 * kHalfTokens * D);
                } else {
                    const int rp = hp - ghp;
                    base = ring_page(v, pair, rp >> 1) + (rp & 1) * (2 * kHalfTokens * D);
                }
                load_half_page<D>(t, base, hp < hp1, lane);
            };
            auto attend = [&](const HalfPage<D>& t, int hp) {
                const bool ring = hp >= ghp;
                const int nvalid = !ring ? min(kHalfTokens, L - hp * kHalfTokens)
                                         : min(kHalfTokens, Tw - (hp - ghp) * kHalfTokens);
                const int masked_r = (FUSED && hp == drop_hp) ? drop_r : -1;
                const bool any_kill = nvalid < kHalfTokens || masked_r >= 0 || (CHUNK && ring);
                unsigned kill = 0u;
                if (any_kill) {
                    unsigned gate = 0u;
                    if (CHUNK && ring) {
                        if (hp - ghp >= g0 + 64) load_gates(hp - ghp);
                        gate = __builtin_amdgcn_readlane(gates, hp - ghp - g0) >> (kc * 8);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        bool out = kc * 8 + e >= nvalid || kc * 8 + e == masked_r;
                        // in the window of the chunk's token i iff its age is above i
                        if (CHUNK && ring)
                            out = out || !(((gate >> e) & 1u) || age_of((hp - ghp) * kHalfTokens + kc * 8 + e) > tok);
                        if (out) kill |= 1u << e;
                    }
                }
                attend_half_page<D, true>(t.k, t.v, qb, kill, any_kill, scale_log2e, acc, m, l);
            };
            HalfPage<D> t[NT];
            int hp = hp0;
            bool more = true;
#pragma unroll
            for (int i = 0; i < NT - 1; ++i) load(t[i], hp + i);
            while (more) {
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    if (more) {
                        load(t[(i + NT - 1) % NT], hp + NT - 1);
                        __builtin_amdgcn_sched_barrier(0);
                        attend(t[i], hp);
                        __builtin_amdgcn_sched_barrier(0);
                        more = ++hp < hp1;
                    }
                }
            }
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            if (n < cols) {
                const size_t col = (size_t)(run + pair) * (CHUNK ? 16 : v.G) + n;
                float* pa = v.part_acc + col * D + kc * 4;
#pragma unroll
                for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(pa + db * 16) = acc[db];
                if (kc == 0) {
                    v.part_ml[col * 2] = m;
                    v.part_ml[col * 2 + 1] = l;
                }
            }
        }
        left -= max(0, hp1 - hp0);
        if (left <= 0 || !next_pair(v, pair, L, T, counts)) return;
        hp0 = 0;
        left -= kPairUnits;
    }
}
template <int D, bool FUSED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_decode_shares(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e) {
    attend_run<D, FUSED ? kSplitFusedTwo : kSplitPlain>(v, q, scale_log2e, blockIdx.x, (int)gridDim.x - 1, nullptr);
}

// Fused step with the utility predictor (Eq. 1; the appendix builds it as Linear - SiLU -
// Linear per token): the hidden layer rides in the split launch, the output layer in the
// append workgroups of the second launch, so the gate logits of the new tokens cost no
// launch of their own.  The waves of the first ceil(pr.n_blocks / MW) workgroups of
// this launch compute partial sums of the hidden layer: wave (jb, tb, ks) takes 16 hidden
// units, 16 tokens and the ks-th of kPredictSplit ranges of d_model on MFMA 16x16x32 (W1 rows
// as A operand, tokens as the 16 columns) and stores part[ks][token][unit], without bias.
// The other workgroups are those of spkv_decode_split<D, true>.
__device__ __forceinline__ void predict_hidden_part(const SpkvView& v, const SpkvPredict& pr, int unit) {
    const int n_jb = pr.d_hidden / 16;
    const int ks = unit % kPredictSplit, rest = unit / kPredictSplit;
    const int jb = rest % n_jb, tb = rest / n_jb;
    const int lane = threadIdx.x & 63, kc = lane >> 4, n = lane & 15;
    const int kq = pr.d_model / kPredictSplit;            // a multiple of 32
    const int tok = tb * 16 + n;
    const bool tok_ok = tok < v.B;
    // (columns past the last token read token 0's row; their results are never stored)
    const uint16_t* wrow = pr.w1 + (size_t)(jb * 16 + n) * pr.d_model + ks * kq + kc * 8;
    const uint16_t* xrow = pr.x + (size_t)(tok_ok ? tok : 0) * pr.d_model + ks * kq + kc * 8;
    const f32x4 acc = predictor_contract(wrow, xrow, kq);
    // lane (kc, n) holds hidden units jb * 16 + 4 kc + i of token tb * 16 + n
    if (tok_ok)
        *reinterpret_cast<f32x4*>(pr.part + ((size_t)ks * v.B + tok) * pr.d_hidden + jb * 16 + 4 * kc) = acc;
}

template <int D, int MW>
__global__ __launch_bounds__(64 * MW) void spkv_decode_split_predict(SpkvView v,
                                                                const uint16_t* __restrict__ q,
                                                                float scale_log2e, SpkvSplit sp,
                                                                SpkvPredict pr) {
    extern __shared__ __attribute__((aligned(16))) float s_split[];
    const int n_pred_wg = (pr.n_blocks + MW - 1) / MW;
    if ((int)blockIdx.x >= n_pred_wg) {
        const SpkvStepIO none = {};
        decode_split_item<D, kSplitFusedTwo, MW>(v, q, scale_log2e, sp, (int)blockIdx.x - n_pred_wg,
                                                 s_split, nullptr, none);
        return;
    }
    const int unit = (int)blockIdx.x * MW + ((int)threadIdx.x >> 6);
    if (unit < pr.n_blocks) predict_hidden_part(v, pr, unit);
}

// The same under the gapless numbering.
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void spkv_decode_split_predict_compact(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e, SpkvSplit sp, SpkvPredict pr) {
    if ((int)blockIdx.x < pr.n_blocks) {
        predict_hidden_part(v, pr, blockIdx.x);
        return;
    }
    decode_split_compact<D, true>(v, q, scale_log2e, sp, (int)blockIdx.x - pr.n_blocks,
                                  (int)gridDim.x - pr.n_blocks);
}

// The same with the lists in equal shares.
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_decode_shares_predict(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e, SpkvPredict pr) {
    if ((int)blockIdx.x < pr.n_blocks)
        predict_hidden_part(v, pr, blockIdx.x);
    else
        attend_run<D, kSplitFusedTwo>(v, q, scale_log2e, (int)blockIdx.x - pr.n_blocks, (int)gridDim.x - pr.n_blocks - 1, nullptr);
}

// One wave folds the partials of one (pair, head) into a running (max, sum, acc) triple:
// with M the running max,  acc = sum_i 2^(m_i - M) acc_i,  den = sum_i 2^(m_i - M) l_i.
// The loads of successive items are independent; only the cheap rescaling is chained.
// Lane owns E = D / 64 output elements.  The wave takes items first, first + stride, ...;
// the loads of its first eight go out before `items` is looked at (slots beyond the count
// are valid memory whose contents are then ignored), so that the round trip that fetches the
// count and the one that fetches the partials overlap.
template <int D>
__device__ __forceinline__ void fold_items(const SpkvView& v, size_t slot0, int g, int first,
                                           int stride, int slots, int items, int lane, float& mw,
                                           float& den, float (&num)[D / 64]) {
    constexpr int E = D / 64, U = 8;
    mw = SPKV_NEG_INF;
    den = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) num[e] = 0.f;
    auto fold = [&](float mi, float li, const float (&a)[E]) {
        const float m_new = fmaxf(mw, mi);
        const float m_ref = (m_new == SPKV_NEG_INF) ? 0.f : m_new;   // items with no key: weight 0
        const float so = __builtin_amdgcn_exp2f(mw - m_ref), si = __builtin_amdgcn_exp2f(mi - m_ref);
        den = den * so + li * si;
#pragma unroll
        for (int e = 0; e < E; ++e) num[e] = num[e] * so + a[e] * si;
        mw = m_new;
    };
    float m0[U], l0[U], a0[U][E];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min(first + u * stride, slots - 1);
        const float* pm = v.part_ml + ((slot0 + i) * v.G + g) * 2;
        const float* pa = v.part_acc + ((slot0 + i) * v.G + g) * D + lane * E;
        m0[u] = pm[0];
        l0[u] = pm[1];
#pragma unroll
        for (int e = 0; e < E; ++e) a0[u][e] = pa[e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (first + u * stride < items) fold(m0[u], l0[u], a0[u]);
#pragma unroll 8
    for (int i = first + U * stride; i < items; i += stride) {
        const float* pm = v.part_ml + ((slot0 + i) * v.G + g) * 2;
        const float* pa = v.part_acc + ((slot0 + i) * v.G + g) * D + lane * E;
        const float mi = pm[0], li = pm[1];
        float a[E];
#pragma unroll
        for (int e = 0; e < E; ++e) a[e] = pa[e];
        fold(mi, li, a);
    }
}

// The partial results of a pair: the first slot, how many (`known`: pair_items of the split launch, which with
// shares holds both), and the slots from the first one to the last that a load may touch.
struct PartSlots {
    size_t first;
    int count, room;
};
template <bool SHARES>
__device__ __forceinline__ PartSlots part_slots(const SpkvSplit& sp, int pair, int known) {
    if (SHARES) return PartSlots{(size_t)(known & 0xffff), known >> 16, sp.slots - (known & 0xffff)};
    return PartSlots{(size_t)pair * sp.slots, known, sp.slots};
}

// Merge the partials of one (sequence, query head):
//   out = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i,  lse = (M + log2(sum)) ln 2.
// One workgroup of NWM waves per (pair, head): the waves take the items round-robin, each
// lane owns D/64 output elements, and the wave results meet in LDS.  NWM = 4, or 16 (see
// wide_merge) so that every wave still gets its items in one round of loads.
// SHARES: the partial results are those of equal shares (their slots come from a load, which the first round
// of the others need not wait for).
template <int D, int NWM, bool SHARES>
__global__ __launch_bounds__(64 * NWM) void spkv_decode_combine(SpkvView v, uint16_t* __restrict__ out,
                                                                float* __restrict__ lse, SpkvSplit sp) {
    constexpr int E = D / 64;
    const int pair = blockIdx.x / v.G, g = blockIdx.x - pair * v.G;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const PartSlots ps = part_slots<SHARES>(sp, pair, SHARES ? v.pair_items[pair] : pair_split(v, pair, sp).groups);
    __shared__ float s_m[NWM];
    __shared__ float s_den[NWM];
    __shared__ float s_acc[NWM][D];

    float mw, den, num[E];
    fold_items<D>(v, ps.first, g, wave, NWM, ps.room, ps.count, lane, mw, den, num);
#pragma unroll
    for (int e = 0; e < E; ++e) s_acc[wave][lane * E + e] = num[e];
    if (lane == 0) {
        s_m[wave] = mw;
        s_den[wave] = den;
    }
    __syncthreads();
    if (tid < D) {
        float M = s_m[0];
#pragma unroll
        for (int wv = 1; wv < NWM; ++wv) M = fmaxf(M, s_m[wv]);
        float nsum = 0.f, dsum = 0.f;
#pragma unroll
        for (int wv = 0; wv < NWM; ++wv) {
            const float sc = __builtin_amdgcn_exp2f(s_m[wv] - M);   // 0 for a wave without items
            nsum += s_acc[wv][tid] * sc;
            dsum += s_den[wv] * sc;
        }
        const size_t o = ((size_t)b * v.Hq + (size_t)h * v.G + g);
        const __bf16 r = (__bf16)(nsum / dsum);
        out[o * D + tid] = __builtin_bit_cast(uint16_t, r);
        if (lse != nullptr && tid == 0) lse[o] = (M + log2f(dsum)) * 0.6931471805599453f;
    }
}

// Second launch of the fused step: one workgroup per (sequence, query head) merges the
// partials as spkv_decode_combine does, plus one more term for the new token itself, taken
// straight from the caller's k_new / v_new (score q . k_new in fp32, weight sum 1, value
// v_new).  n_pairs further workgroups of the same launch perform the append of the new
// token exactly as spkv_append_step does, beside the merges instead of after them.  The
// item count of a pair comes from pair_items (written by the split kernel), not from the
// counters, so no merging workgroup reads what the appends are changing.
//
// PRED (step with the utility predictor): f_new is not an input.  The append workgroup of
// (sequence b, head h) first finishes the predictor for its token and head -- hidden
// activations a_j = SiLU(b1_j + sum of the kPredictSplit partial sums the split launch left),
// logit = b2_h + sum_j W2[h, j] a_j, all in fp32 -- stores the logit for the caller and
// appends with it.
template <int D, bool PRED, int NWM, bool SHARES>
__global__ __launch_bounds__(64 * NWM) void spkv_combine_append(SpkvView v, uint16_t* __restrict__ out,
                                                           float* __restrict__ lse, SpkvSplit sp,
                                                           const uint16_t* __restrict__ k_new,
                                                           const uint16_t* __restrict__ v_new,
                                                           const float* __restrict__ f_new,
                                                           const uint16_t* __restrict__ q,
                                                           float scale_log2e, SpkvPredict pr) {
    constexpr int E = D / 64;
    __shared__ int s_page;
    if ((int)blockIdx.x >= v.n_pairs * v.G) {                // the appends
        const int pair = blockIdx.x - v.n_pairs * v.G;
        const int b = pair / v.Hkv, h = pair - b * v.Hkv;
        const int T = v.t_pair[pair], L = v.kept_len[pair];
        float f_tok;
        if (PRED) {
            __shared__ float s_sum[NWM];
            float sum = 0.f;
            for (int j = threadIdx.x; j < pr.d_hidden; j += 64 * NWM) {
                float a = pr.b1 != nullptr ? pr.b1[j] : 0.f;
#pragma unroll
                for (int ks = 0; ks < kPredictSplit; ++ks)
                    a += pr.part[((size_t)ks * v.B + b) * pr.d_hidden + j];
                const unsigned wbits = pr.w2[(size_t)h * pr.d_hidden + j];
                sum += __builtin_bit_cast(float, wbits << 16) * (a / (1.f + __expf(-a)));   // SiLU
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
            __syncthreads();
            f_tok = pr.b2 != nullptr ? pr.b2[h] : 0.f;
#pragma unroll
            for (int wv = 0; wv < NWM; ++wv) f_tok += s_sum[wv];
            if (threadIdx.x == 0) pr.logits[(size_t)b * v.Hkv + h] = f_tok;
        } else {
            f_tok = f_new[(size_t)b * v.Hkv + h];
        }
        const AppendRegs<D> ar = append_load<D>(v, pair, h, b, T, L, k_new, v_new, f_tok, threadIdx.x);
        __syncthreads();
        append_store<D>(v, pair, T, L, ar, threadIdx.x, &s_page);
        return;
    }
    const int pair = blockIdx.x / v.G, g = blockIdx.x - pair * v.G;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const PartSlots ps = part_slots<SHARES>(sp, pair, v.pair_items[pair]);
    const size_t kv_row = ((size_t)b * v.Hkv + h) * D;
    const size_t q_row = ((size_t)b * v.Hq + (size_t)h * v.G + g) * D;
    // score of the new token for this head (every wave computes it; 6 shuffles)
    float dot = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned qe = q[q_row + lane * E + e], ke = k_new[kv_row + lane * E + e];
        dot += __builtin_bit_cast(float, qe << 16) * __builtin_bit_cast(float, ke << 16);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
    const float m_tok = dot * scale_log2e;
    __shared__ float s_m[NWM];
    __shared__ float s_den[NWM];
    __shared__ float s_acc[NWM][D];

    float mw, den, num[E];
    fold_items<D>(v, ps.first, g, wave, NWM, ps.room, ps.count, lane, mw, den, num);
#pragma unroll
    for (int e = 0; e < E; ++e) s_acc[wave][lane * E + e] = num[e];
    if (lane == 0) {
        s_m[wave] = mw;
        s_den[wave] = den;
    }
    __syncthreads();
    if (tid < D) {
        float M = m_tok;
#pragma unroll
        for (int wv = 0; wv < NWM; ++wv) M = fmaxf(M, s_m[wv]);
        const float w_tok = __builtin_amdgcn_exp2f(m_tok - M);
        const unsigned ve = v_new[kv_row + tid];
        float nsum = __builtin_bit_cast(float, ve << 16) * w_tok, dsum = w_tok;
#pragma unroll
        for (int wv = 0; wv < NWM; ++wv) {
            const float sc = __builtin_amdgcn_exp2f(s_m[wv] - M);
            nsum += s_acc[wv][tid] * sc;
            dsum += s_den[wv] * sc;
        }
        const size_t o = ((size_t)b * v.Hq + (size_t)h * v.G + g);
        const __bf16 r = (__bf16)(nsum / dsum);
        out[o * D + tid] = __builtin_bit_cast(uint16_t, r);
        if (lse != nullptr && tid == 0) lse[o] = (M + log2f(dsum)) * 0.6931471805599453f;
    }
}

// ------------------------------------------------------- multi-token step (chunk)
// Up to 16 new tokens per sequence attend in one pass (speculative-decoding verification,
// prompt feed in short chunks) if they fit the 16 MFMA columns: (token i, head g) pairs, col =
// i G + g, so every K/V tile is still read once per (sequence, KV head).  (Wider chunks:
// spkv_prefill_attend<..., DIRECT>; NQ, the groups of 16 columns, is 1.)
// The cache is in the state before the chunk's append.  Long-term keys are available to
// every token of the chunk (they are at least w + 1 positions behind).  A ring key of age
// a (0 = oldest, position T - w) is inside the window of chunk token i iff a > i (the window
// indicator 0 <= t - s < w with t = T + i); otherwise it counts only if its logit passes the
// gate (Eq. 3-4).  The chunk's own keys (causal, always inside the window because the
// chunk is not longer than the window) are added by spkv_chunk_combine.
//
// GAPLESS: workgroups numbered without gaps (see decode_split_compact), four
// waves per compute unit: a partial result has 16 columns here, four times a decode item's, so fewer
// items pay (16 sequences of 32k, 4 drafts: 103 us plain with 1960 items, 101.6 / 99.4 / 97.4 / 96.7
// with 1792 / 1536 / 1280 / 1024 without gaps; 40 of 2k-20k mixed 146 -> 133; 4 of 128k 56 -> 52).
template <int D, int NQ, bool GAPLESS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(GAPLESS ? 2 : 1, GAPLESS ? 2 : 10))) void spkv_chunk_split(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e, SpkvSplit sp, SpkvCu cu) {
    constexpr int NS = D / 32, NB = D / 16;
    int id = blockIdx.x, total = 0;
    do {
        int pair, j;
        if constexpr (GAPLESS) {
            if (!locate_item<true>(v, sp, id, total, pair, j)) return;
        } else {
            pair = blockIdx.x / sp.slots;
            j = blockIdx.x - pair * sp.slots;
        }
        const PairSplit ps = pair_split(v, pair, sp);
        if (!GAPLESS) {
            if (j == 0 && threadIdx.x == 0) v.pair_items[pair] = ps.items;
            if (j >= ps.items) return;
        }
        const int b = pair / v.Hkv, h = pair - b * v.Hkv;
        const int row0 = cu.v[b], n_tok = cu.v[b + 1] - row0;
        if (n_tok == 0) {
            if (!GAPLESS) return;
            id += (int)gridDim.x;
            continue;
        }
        const int cols = n_tok * v.G;
        const int hbase = ps.nhp / ps.items, hrem = ps.nhp - hbase * ps.items;
        const int hp0 = j * hbase + min(j, hrem);
        const int hp1 = hp0 + hbase + (j < hrem ? 1 : 0);
        const int lane = GAPLESS ? threadIdx.x & 63 : threadIdx.x, kc = lane >> 4, n = lane & 15;

        bf16x8 qb[NQ][NS];
        int tok_of_col[NQ];
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            const int col = c * 16 + n;
            const int i = col / v.G, g = col - i * v.G;
            tok_of_col[c] = i;
            const uint16_t* qrow = q + ((size_t)(row0 + i) * v.Hq + (size_t)h * v.G + g) * D + kc * 8;
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                uint4 raw = {0u, 0u, 0u, 0u};
                if (col < cols) raw = *reinterpret_cast<const uint4*>(qrow + sl * 32);
                qb[c][sl] = __builtin_bit_cast(bf16x8, raw);
            }
        }
        f32x4 acc[NQ][NB];
        float m[NQ], l[NQ];
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            m[c] = SPKV_NEG_INF;
            l[c] = 0.f;
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[c][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
        const float* rl = v.ring_logit + (size_t)pair * v.w;
        const int t_mod = ps.T % v.w;

        int hp = hp0;
        while (hp < hp1) {
            const int pbase = hp >> 1;
            const int my_page = pt[min(pbase + lane, v.pt_cap - 1)];
            const int hp_end = min(hp1, (pbase + 64) << 1);
            for (; hp < hp_end; ++hp) {
                const uint16_t* base;
                int nvalid;
                const bool ring = hp >= ps.ghp;
                if (!ring) {
                    const int page = __builtin_amdgcn_readlane(my_page, (hp >> 1) - pbase);
                    base = pool_page(v, page) + (hp & 1) * (2 * kHalfTokens * D);
                    nvalid = min(kHalfTokens, ps.L - hp * kHalfTokens);
                } else {
                    const int r = hp - ps.ghp;
                    base = ring_page(v, pair, r >> 1) + (r & 1) * (2 * kHalfTokens * D);
                    nvalid = min(kHalfTokens, ps.Tw - r * kHalfTokens);
                }
                // keys past the valid length (same for every column)
                unsigned kill_len = 0u;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (kc * 8 + e >= nvalid) kill_len |= 1u << e;
                // ring keys: age and gate of this lane's eight keys
                int age[8];
                unsigned gate_ok = 0u;
                if (ring) {
                    const int x0 = (hp - ps.ghp) * kHalfTokens + kc * 8;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int x = x0 + e;
                        age[e] = ps.T >= v.w ? (x - t_mod + v.w) % v.w : x + v.w - ps.T;
                        if (kc * 8 + e < nvalid && gate_passes(v, rl[x], ps.T - v.w + age[e])) gate_ok |= 1u << e;
                    }
                }
                const uint16_t* kp = base + lane * 8;
                const uint16_t* vp = base + kHalfTokens * D + lane * 8;
                bf16x8 ka[2][NS], va[NB];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int sl = 0; sl < NS; ++sl)
                        ka[t][sl] = load_stream_b128(kp + (t * (D / 8) + sl * 4) * 128);
#pragma unroll
                for (int db = 0; db < NB; ++db) va[db] = load_stream_b128(vp + db * 512);

#pragma unroll
                for (int c = 0; c < NQ; ++c) {
                    unsigned kill = kill_len;
                    if (ring) {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (!(age[e] > tok_of_col[c] || ((gate_ok >> e) & 1u))) kill |= 1u << e;
                    }
                    attend_half_page<D>(ka, va, qb[c], kill, ring || nvalid < kHalfTokens, scale_log2e,
                                        acc[c], m[c], l[c]);
                }
            }
        }

        const size_t slot = (size_t)pair * sp.slots + j;
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            float lc = l[c];
            lc += __shfl_xor(lc, 16);
            lc += __shfl_xor(lc, 32);
            const int col = c * 16 + n;
            if (col < cols) {
                float* pa = v.part_acc + ((slot * (NQ * 16) + col) * D) + kc * 4;
#pragma unroll
                for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(pa + db * 16) = acc[c][db];
                if (kc == 0) {
                    float* pm = v.part_ml + (slot * (NQ * 16) + col) * 2;
                    pm[0] = m[c];
                    pm[1] = lc;
                }
            }
        }
        id += (int)gridDim.x;
    } while (GAPLESS && id < total);
}

// The same with the lists in equal shares.
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_chunk_shares(
    SpkvView v, const uint16_t* __restrict__ q, float scale_log2e, SpkvCu cu) {
    attend_run<D, kSplitChunk>(v, q, scale_log2e, blockIdx.x, (int)gridDim.x - 1, &cu);
}

// Merge for one (pair, column = token i, head g): the split-K partials plus one term per
// chunk token j <= i taken from the caller's k / v rows (score q_i . k_j in fp32, sum 1,
// value v_j); bf16 output row cu[b] + i.  The waves share the partials and the chunk
// tokens round-robin and meet in LDS, as in spkv_decode_combine.  With f set the first n_pairs
// workgroups append the chunk meanwhile: the merge reads the caller's rows and the partials only.
template <int D>
__global__ __launch_bounds__(256) void spkv_chunk_combine(SpkvView v, const uint16_t* __restrict__ q,
                                                          const uint16_t* __restrict__ k_new,
                                                          const uint16_t* __restrict__ v_new,
                                                          uint16_t* __restrict__ out,
                                                          float* __restrict__ lse, float scale_log2e,
                                                          SpkvSplit sp, SpkvCu cu, const float* __restrict__ f) {
    constexpr int E = D / 64, cstride = 16;
    const int n_append = f != nullptr ? v.n_pairs : 0;
    if ((int)blockIdx.x < n_append) {
        append_few<D>(v, blockIdx.x, k_new, v_new, f, cu);
        return;
    }
    const int at = (int)blockIdx.x - n_append, pair = at / cstride, col = at - pair * cstride;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row0 = cu.v[b], n_tok = cu.v[b + 1] - row0;
    if (col >= n_tok * v.G) return;
    const int i = col / v.G, g = col - i * v.G;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int known = v.pair_items[pair];
    const PartSlots ps = sp.runs > 0 ? part_slots<true>(sp, pair, known) : part_slots<false>(sp, pair, known);
    __shared__ float s_m[4];
    __shared__ float s_den[4];
    __shared__ float s_acc[4][D];

    float mw = SPKV_NEG_INF, den = 0.f, num[E];
#pragma unroll
    for (int e = 0; e < E; ++e) num[e] = 0.f;
#pragma unroll 8
    for (int it = wave; it < ps.count; it += 4) {
        const size_t idx = (ps.first + it) * cstride + col;
        const float mi = v.part_ml[idx * 2], li = v.part_ml[idx * 2 + 1];
        float a[E];
#pragma unroll
        for (int e = 0; e < E; ++e) a[e] = v.part_acc[idx * D + lane * E + e];
        const float m_new = fmaxf(mw, mi);
        const float m_ref = (m_new == SPKV_NEG_INF) ? 0.f : m_new;
        const float so = __builtin_amdgcn_exp2f(mw - m_ref), si = __builtin_amdgcn_exp2f(mi - m_ref);
        den = den * so + li * si;
#pragma unroll
        for (int e = 0; e < E; ++e) num[e] = num[e] * so + a[e] * si;
        mw = m_new;
    }
    // the chunk's own tokens 0..i
    const size_t q_row = ((size_t)(row0 + i) * v.Hq + (size_t)h * v.G + g) * D;
    float qf[E];
#pragma unroll
    for (int e = 0; e < E; ++e)
        qf[e] = __builtin_bit_cast(float, (unsigned)q[q_row + lane * E + e] << 16);
    for (int jt = wave; jt <= i; jt += 4) {
        const size_t kv_row = ((size_t)(row0 + jt) * v.Hkv + h) * D;
        float dot = 0.f, vj[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            dot += qf[e] * __builtin_bit_cast(float, (unsigned)k_new[kv_row + lane * E + e] << 16);
            vj[e] = __builtin_bit_cast(float, (unsigned)v_new[kv_row + lane * E + e] << 16);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
        const float mi = dot * scale_log2e;
        const float m_new = fmaxf(mw, mi);
        const float so = __builtin_amdgcn_exp2f(mw - m_new), si = __builtin_amdgcn_exp2f(mi - m_new);
        den = den * so + si;
#pragma unroll
        for (int e = 0; e < E; ++e) num[e] = num[e] * so + vj[e] * si;
        mw = m_new;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) s_acc[wave][lane * E + e] = num[e];
    if (lane == 0) {
        s_m[wave] = mw;
        s_den[wave] = den;
    }
    __syncthreads();
    if (tid < D) {
        const float M = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));   // wave 0 has token 0
        float nsum = 0.f, dsum = 0.f;
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) {
            const float sc = __builtin_amdgcn_exp2f(s_m[wv] - M);
            nsum += s_acc[wv][tid] * sc;
            dsum += s_den[wv] * sc;
        }
        const size_t o = (size_t)(row0 + i) * v.Hq + (size_t)h * v.G + g;
        const __bf16 r = (__bf16)(nsum / dsum);
        out[o * D + tid] = __builtin_bit_cast(uint16_t, r);
        if (lse != nullptr && tid == 0) lse[o] = (M + log2f(dsum)) * 0.6931471805599453f;
    }
}

template <int D>
static hipError_t launch_chunk(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                               const uint16_t* q, uint16_t* out, float* lse, float scale_log2e,
                               SpkvSplit sp, const SpkvCu& cu, const float* f, hipStream_t s) {
    const unsigned grid = (unsigned)v.n_pairs * (unsigned)sp.slots;
    if (sp.runs > 0) spkv_chunk_shares<D><<<dim3(sp.runs + 1), dim3(64), 0, s>>>(v, q, scale_log2e, cu);
    else if (sp.compact > 0) spkv_chunk_split<D, 1, true><<<dim3(sp.compact), dim3(64), 0, s>>>(v, q, scale_log2e, sp, cu);
    else spkv_chunk_split<D, 1, false><<<dim3(grid), dim3(64), 0, s>>>(v, q, scale_log2e, sp, cu);
    spkv_chunk_combine<D><<<dim3((f != nullptr ? v.n_pairs : 0) + v.n_pairs * 16), dim3(256), 0, s>>>(
        v, q, k, vv, out, lse, scale_log2e, sp, cu, f);
    return hipGetLastError();
}

hipError_t spkv_launch_decode_chunk(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                    const uint16_t* q, uint16_t* out, float* lse, float sm_scale,
                                    SpkvSplit sp, const SpkvCu& cu, const float* f, hipStream_t s) {
    const float sl = sm_scale * 1.4426950408889634f;
    return v.D == 128 ? launch_chunk<128>(v, k, vv, q, out, lse, sl, sp, cu, f, s)
                      : launch_chunk<64>(v, k, vv, q, out, lse, sl, sp, cu, f, s);
}

int spkv_chunk_resident_items(int head_dim) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const hipError_t e =
        head_dim == 128 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, spkv_chunk_split<128, 1, false>, 64, 0)
                        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, spkv_chunk_split<64, 1, false>, 64, 0);
    if (e != hipSuccess || per_cu <= 0 || cus <= 0) return 0;
    return per_cu * cus;
}

// Launch of the split kernel for the call's merge width (1, 2 or 4 waves per workgroup).
template <int D, int MODE>
static void launch_split(const SpkvView& v, const uint16_t* q, float scale_log2e, SpkvSplit sp,
                         const SpkvStepIO& io, hipStream_t s) {
    if (sp.runs > 0 && (MODE == kSplitPlain || MODE == kSplitFusedTwo)) {
        spkv_decode_shares<D, MODE == kSplitFusedTwo><<<dim3(sp.runs + 1), dim3(64), 0, s>>>(v, q, scale_log2e);
        return;
    }
    if (sp.compact > 0 && (MODE == kSplitPlain || MODE == kSplitFusedTwo)) {
        spkv_decode_split_compact<D, MODE == kSplitFusedTwo><<<dim3(sp.compact), dim3(64), 0, s>>>(v, q, scale_log2e, sp);
        return;
    }
    const dim3 grid((unsigned)v.n_pairs * (unsigned)sp.slots);
    const size_t lds = split_lds_bytes(sp.mw, v.G, D);
    if (sp.mw == 4) spkv_decode_split<D, MODE, 4><<<grid, dim3(256), lds, s>>>(v, q, scale_log2e, sp, io);
    else if (sp.mw == 2) spkv_decode_split<D, MODE, 2><<<grid, dim3(128), lds, s>>>(v, q, scale_log2e, sp, io);
    else spkv_decode_split<D, MODE, 1><<<grid, dim3(64), 0, s>>>(v, q, scale_log2e, sp, io);
}

template <int D>
static void launch_split_predict(const SpkvView& v, const uint16_t* q, float scale_log2e,
                                 SpkvSplit sp, const SpkvPredict& pr, hipStream_t s) {
    if (sp.runs > 0) {
        spkv_decode_shares_predict<D><<<dim3(pr.n_blocks + sp.runs + 1), dim3(64), 0, s>>>(v, q, scale_log2e, pr);
        return;
    }
    if (sp.compact > 0) {
        spkv_decode_split_predict_compact<D><<<dim3(pr.n_blocks + sp.compact), dim3(64), 0, s>>>(v, q, scale_log2e, sp, pr);
        return;
    }
    const dim3 grid((unsigned)((pr.n_blocks + sp.mw - 1) / sp.mw) + (unsigned)v.n_pairs * (unsigned)sp.slots);
    const size_t lds = split_lds_bytes(sp.mw, v.G, D);
    if (sp.mw == 4) spkv_decode_split_predict<D, 4><<<grid, dim3(256), lds, s>>>(v, q, scale_log2e, sp, pr);
    else if (sp.mw == 2) spkv_decode_split_predict<D, 2><<<grid, dim3(128), lds, s>>>(v, q, scale_log2e, sp, pr);
    else spkv_decode_split_predict<D, 1><<<grid, dim3(64), 0, s>>>(v, q, scale_log2e, sp, pr);
}

// The merge of spkv_decode_attention, and of the steps (pr: with the predictor).
template <int D, int NWM>
static void launch_merge(const SpkvView& v, uint16_t* out, float* lse, SpkvSplit sp, hipStream_t s) {
    const dim3 grid(v.n_pairs * v.G), block(64 * NWM);
    if (sp.runs > 0) spkv_decode_combine<D, NWM, true><<<grid, block, 0, s>>>(v, out, lse, sp);
    else spkv_decode_combine<D, NWM, false><<<grid, block, 0, s>>>(v, out, lse, sp);
}
template <int D, bool PRED>
static void launch_merge_append(const SpkvView& v, uint16_t* out, float* lse, SpkvSplit sp, const uint16_t* k,
                                const uint16_t* vv, const float* f, const uint16_t* q, float scale_log2e,
                                const SpkvPredict& pr, hipStream_t s) {
    const dim3 grid(v.n_pairs * v.G + v.n_pairs);
    const bool wide = wide_merge(v, sp), shares = sp.runs > 0;
    if (wide && shares) spkv_combine_append<D, PRED, 16, true><<<grid, dim3(1024), 0, s>>>(v, out, lse, sp, k, vv, f, q, scale_log2e, pr);
    else if (wide) spkv_combine_append<D, PRED, 16, false><<<grid, dim3(1024), 0, s>>>(v, out, lse, sp, k, vv, f, q, scale_log2e, pr);
    else if (shares) spkv_combine_append<D, PRED, 4, true><<<grid, dim3(256), 0, s>>>(v, out, lse, sp, k, vv, f, q, scale_log2e, pr);
    else spkv_combine_append<D, PRED, 4, false><<<grid, dim3(256), 0, s>>>(v, out, lse, sp, k, vv, f, q, scale_log2e, pr);
}

hipError_t spkv_launch_decode(const SpkvView& v, const uint16_t* q, uint16_t* out, float* lse,
                              float sm_scale, SpkvSplit sp, bool split_only, bool one_launch,
                              hipEvent_t ev0, hipEvent_t ev1, hipStream_t s) {
    const float scale_log2e = sm_scale * 1.4426950408889634f;
    if (sp.mw != 1 && sp.mw != 2 && sp.mw != 4) return hipErrorInvalidValue;
    hipError_t e;
    if (one_launch && !split_only) {
        const SpkvStepIO io = {out, lse, nullptr, nullptr, nullptr};
        if (ev0 != nullptr && (e = hipEventRecord(ev0, s)) != hipSuccess) return e;
        if (v.D == 128) launch_split<128, kSplitMerge>(v, q, scale_log2e, sp, io, s);
        else launch_split<64, kSplitMerge>(v, q, scale_log2e, sp, io, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (ev1 != nullptr && (e = hipEventRecord(ev1, s)) != hipSuccess) return e;
        return hipSuccess;
    }
    const SpkvStepIO none = {};
    if (ev0 != nullptr && (e = hipEventRecord(ev0, s)) != hipSuccess) return e;
    if (v.D == 128) launch_split<128, kSplitPlain>(v, q, scale_log2e, sp, none, s);
    else launch_split<64, kSplitPlain>(v, q, scale_log2e, sp, none, s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev1 != nullptr && (e = hipEventRecord(ev1, s)) != hipSuccess) return e;
    if (split_only) return hipSuccess;
    const bool wide = wide_merge(v, sp);
    if (v.D == 128) wide ? launch_merge<128, 16>(v, out, lse, sp, s) : launch_merge<128, 4>(v, out, lse, sp, s);
    else wide ? launch_merge<64, 16>(v, out, lse, sp, s) : launch_merge<64, 4>(v, out, lse, sp, s);
    return hipGetLastError();
}

int spkv_compute_units() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

// One-wave work items the device holds at once (the registers decide, so the count is the
// same for every merge width).
int spkv_split_resident_items(int head_dim) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const hipError_t e =
        head_dim == 128
            ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, spkv_decode_split<128, kSplitStep, 1>, 64, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, spkv_decode_split<64, kSplitStep, 1>, 64, 0);
    if (e != hipSuccess || per_cu <= 0 || cus <= 0) return 0;
    return per_cu * cus;
}

hipError_t spkv_launch_decode_step(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                   const float* f, const uint16_t* q, uint16_t* out, float* lse,
                                   float sm_scale, SpkvSplit sp, bool one_launch, hipStream_t s) {
    const float scale_log2e = sm_scale * 1.4426950408889634f;
    if (sp.mw != 1 && sp.mw != 2 && sp.mw != 4) return hipErrorInvalidValue;
    if (one_launch) {
        const SpkvStepIO io = {out, lse, k, vv, f};
        if (v.D == 128) launch_split<128, kSplitStep>(v, q, scale_log2e, sp, io, s);
        else launch_split<64, kSplitStep>(v, q, scale_log2e, sp, io, s);
        return hipGetLastError();
    }
    const SpkvStepIO no_io = {};
    const SpkvPredict none = {};
    if (v.D == 128) {
        launch_split<128, kSplitFusedTwo>(v, q, scale_log2e, sp, no_io, s);
        launch_merge_append<128, false>(v, out, lse, sp, k, vv, f, q, scale_log2e, none, s);
    } else {
        launch_split<64, kSplitFusedTwo>(v, q, scale_log2e, sp, no_io, s);
        launch_merge_append<64, false>(v, out, lse, sp, k, vv, f, q, scale_log2e, none, s);
    }
    return hipGetLastError();
}

int spkv_predict_blocks(int n_tokens, int d_hidden) {
    return (d_hidden / 16) * ((n_tokens + 15) / 16) * kPredictSplit;
}

hipError_t spkv_launch_decode_step_predict(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                           const uint16_t* q, uint16_t* out, float* lse,
                                           float sm_scale, SpkvSplit sp, SpkvPredict pr,
                                           hipStream_t s) {
    const float scale_log2e = sm_scale * 1.4426950408889634f;
    if (sp.mw != 1 && sp.mw != 2 && sp.mw != 4) return hipErrorInvalidValue;
    pr.n_blocks = spkv_predict_blocks(v.B, pr.d_hidden);
    if (v.D == 128) {
        launch_split_predict<128>(v, q, scale_log2e, sp, pr, s);
        launch_merge_append<128, true>(v, out, lse, sp, k, vv, nullptr, q, scale_log2e, pr, s);
    } else {
        launch_split_predict<64>(v, q, scale_log2e, sp, pr, s);
        launch_merge_append<64, true>(v, out, lse, sp, k, vv, nullptr, q, scale_log2e, pr, s);
    }
    return hipGetLastError();
}
