// Device-side helpers shared by the kernel files: vector types, streaming loads, page
// addressing, the gate, page allocation, the single-token append (used by the write kernel
// and by the fused decode step), the work partition and one half-page of flash decoding on
// MFMA operands held in registers.
#pragma once
#include <algorithm>

#include "spkv_internal.h"


typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

#define SPKV_NEG_INF (-__builtin_inff())

// ------------------------------------------------------------------ small helpers
__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// 128-bit streaming load of 8 bf16.  K/V tiles are read once per decode step and never
// again before the whole cache has gone by, so they are loaded non-temporal: the lines
// bypass L2 / Infinity Cache retention instead of evicting the little that is reused
// (queries, page tables, partials).  Measured on MI355X: about 12 % more read bandwidth
// than plain loads for this access pattern.
__device__ __forceinline__ bf16x8 load_stream_b128(const uint16_t* p) {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    const u32x4 r = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return __builtin_bit_cast(bf16x8, r);
}

// Stores that other compute dies (each has its own L2) may read later in the SAME launch:
// written through to device scope, so that waiting for the wave's outstanding stores is all
// it takes to make them visible -- no write-back of the whole L2 (a device-scope release fence
// costs that, and thousands of them per launch were measured at +200 us).
// (The s_nop: a store of more than 8 bytes reads its data registers up to two cycles after it
// issues, and the compiler, which keeps that distance for its own stores, does not look into
// an asm statement -- without it the next instruction may overwrite the data.)
__device__ __forceinline__ void store_device_b128(float* p, f32x4 x) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(x) : "memory");
}
__device__ __forceinline__ void store_device_b32(float* p, float x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits for every vector memory operation of this wave, the stores above included.
__device__ __forceinline__ void wait_all_vmem() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }

__device__ __forceinline__ int mbcnt64(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

__device__ __forceinline__ uint16_t* ring_page(const SpkvView& v, int pair, int rp) {
    return v.ring + ((size_t)pair * v.n_ring_pages + rp) * (size_t)spkv_page_elems(v.D);
}

__device__ __forceinline__ uint16_t* pool_page(const SpkvView& v, int page) {
    return v.pool + (size_t)page * (size_t)spkv_page_elems(v.D);
}

// The gate of the pair at position pos with utility logit f: Eq. 2 on the logit, or one of
// the first n_sink positions of the sequence (optional always-kept attention sinks, the
// "fixed attention sinks" variant of the ablations; n_sink = 0 is the paper's method).
__device__ __forceinline__ bool gate_passes(const SpkvView& v, float f, int pos) {
    return f >= v.theta || pos < v.n_sink;
}

// One pool page for the caller: a recycled one if the stack of released pages has any,
// else the next never-used one; -1 if the pool is exhausted.  Pushes onto the stack happen
// only in spkv_release_sequence, never in the same launch as pops, and a failed pop puts
// its decrement back, so the counter is exact between launches.
__device__ __forceinline__ int alloc_page(const SpkvView& v) {
    const int idx = atomicSub(v.free_top, 1) - 1;
    if (idx >= 0) return v.free_pages[idx];
    atomicAdd(v.free_top, 1);
    const int page = atomicAdd(v.pool_next, 1);
    return page < v.n_pages ? page : -1;
}

// `need` pages at once, for one thread of a workgroup that then hands them out: one atomic on
// the bump counter (and one on the stack of recycled pages only when it holds any) instead of
// one or three per page -- every atomic of a launch goes to the same two addresses, and they
// are served one after the other.  Page i of the batch: batch_page(v, pb, i); -1 past the pool.
struct PageBatch {
    int stack_lo, from_stack, pool_base;
};
// recycled: the stack's entries as they were when the launch had begun.
__device__ __forceinline__ PageBatch alloc_page_batch(const SpkvView& v, int need, int recycled) {
    PageBatch pb = {0, 0, 0};
    if (need <= 0) return pb;
    // no page is pushed in a launch that pops, so a stack seen empty stays empty
    if (recycled > 0) {
        const int top = atomicSub(v.free_top, need);
        const int take = min(max(top, 0), need);
        if (take < need) atomicAdd(v.free_top, need - take);     // put back what was not there
        pb.from_stack = take;
        pb.stack_lo = top - take;
    }
    const int rest = need - pb.from_stack;
    if (rest > 0) pb.pool_base = atomicAdd(v.pool_next, rest);
    return pb;
}
__device__ __forceinline__ PageBatch alloc_page_batch(const SpkvView& v, int need) {
    return alloc_page_batch(v, need, __hip_atomic_load(v.free_top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ int batch_page(const SpkvView& v, const PageBatch& pb, int i) {
    if (i < pb.from_stack) return v.free_pages[pb.stack_lo + i];
    const int page = pb.pool_base + (i - pb.from_stack);
    return page < v.n_pages ? page : -1;
}

// The half-page in which a list ends is read whole: its keys past the end are masked, but a weight of
// zero would still turn an infinite value into a NaN.  Whoever lengthens a list from `from` to `to`
// entries therefore clears the values behind its end if this call began that half-page (page: the one it
// lies in) -- bytes that no row of the call touches, so in any order with the rows -- and a prune those behind
// its new end.  Pages then need no clearing when they are handed out again, whatever they held.  nt threads, this one tid.
__device__ __forceinline__ bool ends_in_new_half_page(int from, int to) {
    return to > from && (to & (kHalfTokens - 1)) != 0 && (to & ~(kHalfTokens - 1)) >= from;
}
template <int D>
__device__ __forceinline__ void clear_list_end(uint16_t* page, int to, int tid, int nt) {
    const int a = to & (kPageTokens - 1), end = (a | (kHalfTokens - 1)) + 1, whole = (a + 7) & ~7;
    for (int i = tid; i < (whole - a) * D; i += nt) page[spkv_v_off(D, a + i / D, i % D)] = 0;
    for (int i = tid; i < (end - whole) / 8 * D; i += nt)
        *reinterpret_cast<uint4*>(page + spkv_v_off(D, whole + i / D * 8, i % D)) = make_uint4(0u, 0u, 0u, 0u);
}

// ------------------------------------------------------------------ memory -> LDS copies
// One wave-wide 16-byte load from global memory straight into LDS: lane i's 16 bytes at
// `src` land at LDS byte address lds_row + 16 i (lds_row wave-uniform).  The load counts
// as a vector memory load in flight until its data is in LDS.  (No memory clobber: the
// compiler would then stop treating the page table as read-only and turn its scalar lookups
// into vector loads that wait for these copies.  What orders the copies against the LDS
// reads is the workgroup barrier, which neither the asm nor the reads may cross.)
__device__ __forceinline__ void load_row_to_lds(const uint16_t* src, unsigned lds_row) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(src), "s"(lds_row)
                 : "m0");
}

// The same for data that no other workgroup reads (non-temporal: its lines do not push out of
// the L2 what is shared).
__device__ __forceinline__ void load_row_to_lds_once(const uint16_t* src, unsigned lds_row) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :
                 : "v"(src), "s"(lds_row)
                 : "m0");
}

// The same for one dword per lane: lane i's 4 bytes land at lds_row + 4 i.
__device__ __forceinline__ void load_word_to_lds(const float* src, unsigned lds_row) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :
                 : "v"(src), "s"(lds_row)
                 : "m0");
}

// The same with a wave-uniform base and a byte offset per lane.
__device__ __forceinline__ void load_row_to_lds(const char* base, unsigned voff, unsigned lds_row) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(base), "s"(lds_row)
                 : "m0");
}

// Waits until at most N of this wave's vector memory loads are still in flight (they
// complete in the order issued).
template <int N>
__device__ __forceinline__ void wait_loads_but() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N));
}

// ------------------------------------------------------------------ utility predictor
// Hidden layer of the predictor (Eq. 1) for 16 hidden units x 16 tokens over kq (a multiple
// of 32) elements of d_model: lane (kc, n) passes its row of W1 (unit n) and of the tokens'
// hidden states (token n), both offset by kc * 8 elements; it gets the sums of units
// 4 kc .. 4 kc + 3 for token n.  Loads go out eight steps at a time so that the memory
// round trips overlap (the tail repeats the last step's loads and skips its MFMAs).
__device__ __forceinline__ f32x4 predictor_contract(const uint16_t* __restrict__ wrow,
                                                    const uint16_t* __restrict__ xrow, int kq) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < kq; k0 += 256) {
        uint4 a[8], bv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = min(k0 + u * 32, kq - 32);
            a[u] = *reinterpret_cast<const uint4*>(wrow + k);
            bv[u] = *reinterpret_cast<const uint4*>(xrow + k);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u * 32 < kq)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u]),
                                                              __builtin_bit_cast(bf16x8, bv[u]),
                                                              acc, 0, 0, 0);
    }
    return acc;
}

// ------------------------------------------------- write path, one token per sequence
// Appendix "Inference Kernels": write the new pair into the next ring slot; if the slot
// held a pair (window full), that pair leaves the window: keep it (append to the head's
// long-term pages, allocating a page with one atomic when a page boundary is crossed) if
// its stored logit passes the gate, else drop it.  One workgroup of D threads per
// (sequence, KV head); thread d moves V element d, threads < D/8 move one 16-byte K chunk.
// Append of one token to one (sequence, head), shared by spkv_append_step (workgroup of D
// threads) and spkv_combine_append (256 or 1024 threads, the first D of them move data), in two
// halves so that a caller can put other work between the loads and the stores.
// `row` indexes the new token in k/vv, f_new is its logit for this head; T and L are the
// pair's counters as read by every thread before any of them is updated.
// NT = threads that take part (a multiple of 64); thread tid moves V elements tid,
// tid + NT, ... (one per thread when NT >= D).
// Between the halves lies a barrier of the workgroup (the caller's): the second one changes the
// counters, the ring's row and its logit, which a late wave of the first must not find changed.
template <int D, int NT = D>
struct AppendRegs {
    static constexpr int VPT = (D + NT - 1) / NT;
    float f_old, f_new;
    int page_entry;
    uint16_t v_new[VPT], v_old[VPT];
    uint4 k_new, k_old;
};

// Everything the counters address, issued together (the outgoing row is read before it is
// known whether it is kept: 2 + 16 bytes per thread).
template <int D, int NT = D>
__device__ __forceinline__ AppendRegs<D, NT> append_load(const SpkvView& v, int pair, int h, int row,
                                                         int T, int L, const uint16_t* __restrict__ k,
                                                         const uint16_t* __restrict__ vv,
                                                         float f_new, int tid) {
    AppendRegs<D, NT> r;
    constexpr int VPT = AppendRegs<D, NT>::VPT;
    const bool kmover = tid < D / 8;
    const int slot = T % v.w;
    const uint16_t* rp = ring_page(v, pair, slot >> 6);
    const int rk = slot & 63;
    const bool full = T >= v.w;
    const int lp = L >> 6, gk = L & 63;
    const size_t src = ((size_t)row * v.Hkv + h) * D;
    r.f_old = full ? v.ring_logit[(size_t)pair * v.w + slot] : 0.f;
    r.page_entry = (gk != 0 && lp < v.pt_cap) ? v.page_table[(size_t)pair * v.pt_cap + lp] : -1;
    r.f_new = f_new;
    r.k_new = make_uint4(0u, 0u, 0u, 0u);
    r.k_old = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int d = tid + j * NT;
        r.v_new[j] = 0;
        r.v_old[j] = 0;
        if (d < D) {
            r.v_new[j] = vv[src + d];
            if (full) r.v_old[j] = rp[spkv_v_off(D, rk, d)];
        }
    }
    if (kmover) {
        r.k_new = *reinterpret_cast<const uint4*>(k + src + tid * 8);
        if (full) r.k_old = *reinterpret_cast<const uint4*>(rp + spkv_k_off(D, rk, tid * 8));
    }
    return r;
}

template <int D, int NT = D>
__device__ __forceinline__ void append_store(const SpkvView& v, int pair, int T, int L,
                                             const AppendRegs<D, NT>& r, int tid, int* s_page) {
    constexpr int VPT = AppendRegs<D, NT>::VPT;
    const bool kmover = tid < D / 8;
    const int slot = T % v.w;
    uint16_t* rp = ring_page(v, pair, slot >> 6);
    const int rk = slot & 63;
    const bool full = T >= v.w;
    const int lp = L >> 6, gk = L & 63;
    const bool have_page = gk != 0 && lp < v.pt_cap;
    if (full && gate_passes(v, r.f_old, T - v.w)) {               // Eq. 2 on the logit
        int page = r.page_entry;
        if (!have_page) {                                         // first pair of a new page
            if (tid == 0) {
                const int np = lp < v.pt_cap ? alloc_page(v) : -1;
                if (np >= 0) v.page_table[(size_t)pair * v.pt_cap + lp] = np;
                else *v.err_flag = 1;
                *s_page = np;
            }
            __syncthreads();
            page = *s_page;
        }
        if (page >= 0) {
            uint16_t* gp = pool_page(v, page);
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                const int d = tid + j * NT;
                if (d < D) gp[spkv_v_off(D, gk, d)] = r.v_old[j];
            }
            if (kmover) *reinterpret_cast<uint4*>(gp + spkv_k_off(D, gk, tid * 8)) = r.k_old;
            if (tid < NT && ends_in_new_half_page(L, L + 1)) clear_list_end<D>(gp, L + 1, tid, NT);
            if (tid == 0) {
                v.pos_pool[(size_t)page * kPageTokens + gk] = T - v.w;
                v.logit_pool[(size_t)page * kPageTokens + gk] = r.f_old;
                v.kept_len[pair] = L + 1;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const int d = tid + j * NT;
        if (d < D) rp[spkv_v_off(D, rk, d)] = r.v_new[j];
    }
    if (kmover) *reinterpret_cast<uint4*>(rp + spkv_k_off(D, rk, tid * 8)) = r.k_new;
    if (tid == 0) {
        v.ring_logit[(size_t)pair * v.w + slot] = r.f_new;
        v.t_pair[pair] = T + 1;
        if (gate_passes(v, r.f_new, T)) v.gate_on[pair] += 1;
    }
}

// Lane (r = lane / 16, c = lane % 16) moves chunk c of one row into row dk of page dp.
template <int D>
__device__ __forceinline__ void store_row_chunk(uint16_t* dp, int dk, int c, uint4 kk, uint4 vv) {
    *reinterpret_cast<uint4*>(dp + spkv_k_off(D, dk, c * 8)) = kk;
    uint16_t* vd = dp + spkv_v_off(D, dk, c * 8);      // element e of the chunk is 8 e further
    const unsigned w[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) vd[e * 8] = (uint16_t)(w[e >> 1] >> ((e & 1) * 16));
}

// Append of up to kFewTokens tokens (and at most w, so that none enters and leaves the window within
// the call) to one (sequence, head) by a workgroup of 256 threads: chunk c = tid % 16 of leaving row and
// of new row tid / 16.  Every wave judges all leaving rows for itself, so the only barriers are the one
// between reading the ring and writing it and the one that hands out a page.  Bound by dependent round
// trips, three of them: counters (the new rows travel beside), ring rows, logits and page id, stores.
constexpr int kFewTokens = 16;
template <int D>
__device__ __forceinline__ void append_few(const SpkvView& v, int pair, const uint16_t* __restrict__ k,
                                           const uint16_t* __restrict__ vv, const float* __restrict__ f,
                                           const SpkvCu& cu) {
    const int b = pair / v.Hkv, h = pair - b * v.Hkv, row0 = cu.v[b], n = cu.v[b + 1] - row0;
    if (n == 0) return;
    __shared__ int s_few_page;
    const int tid = threadIdx.x, lane = tid & 63, r = tid >> 4, c = tid & 15;
    const int T = v.t_pair[pair], L = v.kept_len[pair];
    const bool mover = c < D / 8;
    uint4 k_new = {0u, 0u, 0u, 0u}, v_new = k_new, k_old = k_new, v_old = k_new;
    if (r < n && mover) {
        const size_t src = ((size_t)(row0 + r) * v.Hkv + h) * D + c * 8;
        k_new = *reinterpret_cast<const uint4*>(k + src);
        v_new = *reinterpret_cast<const uint4*>(vv + src);
    }
    const float f_new = lane < n ? f[((size_t)row0 + lane) * v.Hkv + h] : 0.f;      // lane j: token j
    const int r0 = max(0, T - v.w), nr = max(0, min(T, max(0, T + n - v.w)) - r0);
    const float f_old = lane < nr ? v.ring_logit[(size_t)pair * v.w + (r0 + lane) % v.w] : 0.f;
    const int lp = L >> 6, gk = L & 63;
    int page = gk != 0 && lp < v.pt_cap ? v.page_table[(size_t)pair * v.pt_cap + lp] : -1;
    if (r < nr && mover) {
        const int slot = (r0 + r) % v.w, sk = slot & 63;
        const uint16_t* sp = ring_page(v, pair, slot >> 6);
        const uint16_t* vs = sp + spkv_v_off(D, sk, c * 8);
        k_old = *reinterpret_cast<const uint4*>(sp + spkv_k_off(D, sk, c * 8));
        v_old.x = (unsigned)vs[0] | ((unsigned)vs[8] << 16);
        v_old.y = (unsigned)vs[16] | ((unsigned)vs[24] << 16);
        v_old.z = (unsigned)vs[32] | ((unsigned)vs[40] << 16);
        v_old.w = (unsigned)vs[48] | ((unsigned)vs[56] << 16);
    }
    const unsigned long long mask = __ballot(lane < nr && gate_passes(v, f_old, r0 + lane));
    const int kept = __popcll(mask), on = __popcll(__ballot(lane < n && gate_passes(v, f_new, T + lane)));
    const int first = (L + kPageTokens - 1) / kPageTokens, last = (L + kept + kPageTokens - 1) / kPageTokens;
    if (last > first) {                                  // at most one page (kept <= 16)
        if (tid == 0) {
            const int np = first < v.pt_cap ? alloc_page(v) : -1;
            if (np >= 0) v.page_table[(size_t)pair * v.pt_cap + first] = np;
            else *v.err_flag = 1;
            s_few_page = np;
        }
    }
    __syncthreads();                                     // the leaving rows have been read
    const int new_page = last > first ? s_few_page : 0;
    if (tid == 0) {
        if (new_page >= 0) v.kept_len[pair] = L + kept;
        v.t_pair[pair] = T + n;
        v.gate_on[pair] += on;
    }
    if (new_page < 0) return;
    if (ends_in_new_half_page(L, L + kept))
        clear_list_end<D>(pool_page(v, (L + kept) >> 6 >= first ? new_page : page), L + kept, tid, 256);
    const float lg_old = __shfl(f_old, r), lg_new = __shfl(f_new, r);      // (all lanes here)
    if (r < nr && ((mask >> r) & 1ull)) {
        const int gi = L + __popcll(mask & ((1ull << r) - 1)), dk = gi & 63;
        if ((gi >> 6) >= first) page = new_page;
        if (mover) store_row_chunk<D>(pool_page(v, page), dk, c, k_old, v_old);
        if (c == 0) {
            v.pos_pool[(size_t)page * kPageTokens + dk] = r0 + r;
            v.logit_pool[(size_t)page * kPageTokens + dk] = lg_old;
        }
    }
    if (r < n) {
        const int slot = (T + r) % v.w;
        if (mover) store_row_chunk<D>(ring_page(v, pair, slot >> 6), slot & 63, c, k_new, v_new);
        if (c == 0) v.ring_logit[(size_t)pair * v.w + slot] = lg_new;
    }
}

// ------------------------------------------------------------------ work partition
// Work unit: a half-page (32 keys).  Pair p has ceil(L/32) long-term half-pages followed
// by ceil(min(T, w)/32) ring half-pages.  The host picks hp_per_item (about total half-
// pages / target item count, from its upper bound of the lengths) and the slot count per
// pair; every pair is then cut evenly into ceil(n / hp_per_item) items from its exact
// device-side lengths, so that the split-K grid is balanced over the kept lengths
// whatever their spread.  Both decode kernels derive the same partition from (L, T).
//
// With sp.mw > 1 (single-token decode kernels only) mw one-wave items share a workgroup and
// merge their results there: the pair gets min(ceil(n / (mw hp_per_item)), slots) workgroups,
// one partial slot each, and is cut evenly into min(groups * mw, n) items.
struct PairSplit {
    int nhp;    // half-pages of the pair
    int ghp;    // of which long-term
    int groups; // partial slots in use (= items for mw = 1)
    int items;  // work items the pair is cut into
    int L, T, Tw;
};

__device__ __forceinline__ PairSplit pair_split(const SpkvView& v, int pair, SpkvSplit sp) {
    PairSplit r;
    r.L = v.kept_len[pair];
    r.T = v.t_pair[pair];
    r.Tw = min(r.T, v.w);
    r.ghp = (r.L + kHalfTokens - 1) >> 5;
    r.nhp = r.ghp + ((r.Tw + kHalfTokens - 1) >> 5);
    const int per = sp.hp_per_item * sp.mw;
    r.groups = min((r.nhp + per - 1) / per, sp.slots);
    r.items = min(r.groups * sp.mw, r.nhp);
    return r;
}

// ------------------------------------------------------------------- split-K decode
// One half-page (32 keys) of flash decoding on the MFMA operands already in registers:
//   S[key][head]   = K[key][:] . Q[head][:]          2 x D/32 MFMA 16x16x32 (bf16 -> fp32)
//   online softmax in the log2 domain (running max m, sum l), weights rounded to bf16
//   O[d][head]    += V[key][d] * P[key][head]        D/16 MFMA 16x16x32
// Bit e of `kill` excludes this lane's key r = 8 kc + e (for the column this lane holds);
// `any_kill` is the wave-uniform "some lane has a bit set".
// TWO: the weights as two bf16 parts, 16 bits of each.  (With one part the largest weight of an item, the
// reference of the others, is the only one without an error, and the longer the items the fewer of those there
// are: 16 sequences of 32k, 2-norm of the error against 64 bits 2.16e-3 with 2880 items, 2.23e-3 with 512 runs, 1.66e-3,
// the rounding of the outputs, with two parts.)
template <int D, bool TWO = false>
__device__ __forceinline__ void attend_half_page(const bf16x8 (&ka)[2][D / 32],
                                                 const bf16x8 (&va)[D / 16],
                                                 const bf16x8 (&qb)[D / 32], unsigned kill,
                                                 bool any_kill, float scale_log2e,
                                                 f32x4 (&acc)[D / 16], float& m, float& l) {
    constexpr int NS = D / 32, NB = D / 16;
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[0][sl], qb[sl], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[1][sl], qb[sl], s1, 0, 0, 0);
    }
    // Lane (kc, n) now holds, for head n, the keys r = 8 kc + 4 t + i of the half-page.
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = s0[i] * scale_log2e;
        x[4 + i] = s1[i] * scale_log2e;
    }
    if (any_kill) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if ((kill >> e) & 1u) x[e] = SPKV_NEG_INF;
    }
    float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                     fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx);
    // m_new is -inf only while every key seen so far was excluded; a finite reference then
    // keeps exp2(-inf - ref) = 0 instead of exp2(-inf + inf) = NaN.
    const float m_ref = (m_new == SPKV_NEG_INF) ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m - m_ref);
    f32x8 p;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(x[e] - m_ref);
        psum += p[e];
    }
    l = l * alpha + psum;
    if (__ballot(m_new != m) != 0ull) {
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] *= alpha;
    }
    m = m_new;
    const bf16x8 pb = __builtin_convertvector(p, bf16x8);
#pragma unroll
    for (int db = 0; db < NB; ++db)
        acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[db], pb, acc[db], 0, 0, 0);
    if (TWO) {
        const bf16x8 pl = __builtin_convertvector(p - __builtin_convertvector(pb, f32x8), bf16x8);
#pragma unroll
        for (int db = 0; db < NB; ++db)
            acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[db], pl, acc[db], 0, 0, 0);
    }
}

// Eight V rows held in LDS (s_rows[row][d]) leave as 16-byte units: eight consecutive keys
// of one head-dim element, rows dk0 .. dk0 + 7 of page (or half-page) dp.  Lane l takes elements
// l and 64 + l, so that a store covers runs of 256 bytes (two neighbouring units per lane, half
// of every 64-byte piece per store, were a third more store requests).
template <int D>
__device__ __forceinline__ void store_v_units(uint16_t* dp, int dk0, const uint16_t (*s_rows)[D],
                                              int lane) {
#pragma unroll
    for (int d = lane; d < D; d += 64) {
        unsigned w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            w[r] = (unsigned)s_rows[2 * r][d] | ((unsigned)s_rows[2 * r + 1][d] << 16);
        *reinterpret_cast<uint4*>(dp + spkv_v_off(D, dk0, d)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// ----------------------------------------------------------- staging rows of a prefill call
// One workgroup of 256 threads per (staging half-page sh, pair): wave wv fills rows 8 wv .. 8 wv + 7.  Rows
// without a position (before the sequence start, past the chunk) are zero, so that a
// masked key never meets a non-finite V element.  Reads the ring and the token count as they were before
// the append: at most beside the launch of it that leaves both alone (spkv_stage_ring).
// With st.bias set (soft gating) it also stores log2 u = log2 sigmoid(f) of every new row,
// divided by the score scale.
template <int D>
__device__ __forceinline__ void stage_half_page(const SpkvView& v, const uint16_t* __restrict__ k,
                                                const uint16_t* __restrict__ vv, const float* __restrict__ f,
                                                const SpkvCu& cu, const SpkvStage& st, int pair, int sh) {
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row0 = cu.v[b], n = cu.v[b + 1] - row0;
    if (n == 0 || sh * kHalfTokens >= v.w + n) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15;
    const int T0 = v.t_pair[pair];
    __shared__ __attribute__((aligned(16))) uint16_t s_v[4][8][D];
    uint16_t* dp = st.stage + ((size_t)pair * st.shp + sh) * (size_t)(2 * kHalfTokens * D);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int row = pass * 4 + (lane >> 4);
        const int u = sh * kHalfTokens + wave * 8 + row;
        if (c < D / 8) {
            uint4 kk = {0u, 0u, 0u, 0u}, vl = {0u, 0u, 0u, 0u};
            if (u >= v.w) {
                const int j = u - v.w;
                if (j < n) {
                    const size_t src = ((size_t)(row0 + j) * v.Hkv + h) * D + c * 8;
                    kk = *reinterpret_cast<const uint4*>(k + src);
                    vl = *reinterpret_cast<const uint4*>(vv + src);
                }
            } else {
                const int s = T0 - v.w + u;
                if (s >= 0) {
                    const int slot = s % v.w;
                    const uint16_t* sp = ring_page(v, pair, slot >> 6);
                    const int sk = slot & 63;
                    kk = *reinterpret_cast<const uint4*>(sp + spkv_k_off(D, sk, c * 8));
                    const uint16_t* vs = sp + spkv_v_off(D, sk, c * 8);
                    unsigned wd[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        wd[e] = (unsigned)vs[(2 * e) * 8] | ((unsigned)vs[(2 * e + 1) * 8] << 16);
                    vl = make_uint4(wd[0], wd[1], wd[2], wd[3]);
                }
            }
            *reinterpret_cast<uint4*>(dp + spkv_k_off(D, wave * 8 + row, c * 8)) = kk;
            *reinterpret_cast<uint4*>(&s_v[wave][row][c * 8]) = vl;
        }
        if (st.bias != nullptr && c == 0) {
            float lb = 0.f;
            if (u >= v.w && u - v.w < n) {
                // log u = log sigmoid(f) = -softplus(-f) (Eq. 1 and the soft gate), in log2
                const float x = f[((size_t)row0 + (u - v.w)) * v.Hkv + h];
                const float ls = x < -20.f ? x : -log1pf(__expf(-x));
                lb = ls * 1.4426950408889634f * st.bias_unit;
            }
            st.bias[((size_t)pair * st.shp + sh) * kHalfTokens + wave * 8 + row] = lb;
        }
    }
    __builtin_amdgcn_wave_barrier();
    store_v_units<D>(dp, wave * 8, s_v[wave], lane);
}
