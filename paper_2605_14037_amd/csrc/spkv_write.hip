// Write path of the SP-KV cache on gfx950: zero fill and copies, the append of one token per
// sequence (fused gate + evict + ring write), the bulk append (ballot + mbcnt stream
// compaction in stable order), sequence release and the read-back of kept positions.
//
// Gate: Eq. 2 of the paper taken on the logit, z = 1[f >= theta].  The window ring holds
// exactly the keys with 0 <= t - s < w and the long-term pages exactly the gated-on keys with
// t - s >= w (Eq. 3-4), so the two sets are disjoint and their union is what Eq. 5 attends to.
#include "spkv_device.h"

// ------------------------------------------------------------------------ zero fill
__global__ __launch_bounds__(256) void spkv_fill_zero(uint4* p, size_t n16) {
    const uint4 z = {0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = z;
}

hipError_t spkv_launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    spkv_fill_zero<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(static_cast<uint4*>(p), n16);
    return hipGetLastError();
}

// Back to the empty cache in one launch: everything before the pool (counters, ring, tables) and the
// counters behind it.  The pages keep what they held (clear_list_end): 16 sequences of 32k tokens, half
// of a 0.9 GB arena in use, 64 us with the pages cleared, 6 without.
__global__ __launch_bounds__(256) void spkv_reset(uint4* arena, size_t n16, size_t tail16, size_t tail_n16) {
    const uint4 z = {0u, 0u, 0u, 0u};
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < n16; i += step) arena[i] = z;
    for (size_t i = i0; i < tail_n16; i += step) arena[tail16 + i] = z;
}

// Offsets and sizes in bytes, multiples of 256.
hipError_t spkv_launch_reset(void* arena, size_t pool, size_t tail, size_t tail_bytes, hipStream_t s) {
    const unsigned blocks = (unsigned)std::min<size_t>((std::max(pool, tail_bytes) / 16 + 255) / 256, 256 * 8);
    spkv_reset<<<dim3(blocks), dim3(256), 0, s>>>(static_cast<uint4*>(arena), pool / 16, tail / 16, tail_bytes / 16);
    return hipGetLastError();
}

// --------------------------------------------------------------- lengths to the host
// The ticket tells the host that the lengths have arrived without an event: asking an event while
// any stream of the process is being captured ends that capture.  One workgroup; every thread's
// lengths are out at system scope before the barrier, the ticket after it.
__device__ __forceinline__ void copy_lengths(const int32_t* __restrict__ len, int n, const SpkvLengthCopy& to) {
    for (int p = threadIdx.x; p < n; p += blockDim.x) to.host[p] = len[p];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(to.host + n, to.ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ __launch_bounds__(256) void spkv_copy_lengths(const int32_t* __restrict__ len, int n, int32_t* to_host,
                                                         int32_t ticket) {
    copy_lengths(len, n, SpkvLengthCopy{to_host, ticket});
}

hipError_t spkv_launch_copy_lengths(const SpkvView& v, SpkvLengthCopy to, hipStream_t s) {
    spkv_copy_lengths<<<dim3(1), dim3(256), 0, s>>>(v.kept_len, v.n_pairs, to.host, to.ticket);
    return hipGetLastError();
}

// ------------------------------------------------------------- plain copy (reference)
__global__ __launch_bounds__(256) void spkv_plain_copy(uint4* __restrict__ d,
                                                       const uint4* __restrict__ s, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16;
         i += (size_t)gridDim.x * blockDim.x)
        d[i] = s[i];
}

hipError_t spkv_launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    spkv_plain_copy<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(
        static_cast<uint4*>(dst), static_cast<const uint4*>(src), n16);
    return hipGetLastError();
}

// ------------------------------------------------- plain streaming read (reference)
// The memory side of the decode kernel and nothing else: one-wave workgroups, each reading
// its share of the launch's 16 KB chunks with sixteen non-temporal 1 KB wave-wide loads per
// chunk (the half-page access pattern) and storing 1 KB at the end (as a work item stores its
// partial result).  Chunk c of the launch lies in run c / chunks_per_run; run i of the launch
// is run ((first_run + i) * stride) mod total_runs of the region, so with a stride coprime to
// total_runs successive launches read distinct, scattered runs.
__global__ __launch_bounds__(64) void spkv_plain_read(const uint16_t* __restrict__ src,
                                                      long long total_runs, int chunks_per_run,
                                                      long long first_run, long long n_chunks,
                                                      long long stride, uint4* __restrict__ sink) {
    const long long g = blockIdx.x, n = gridDim.x;
    const long long c0 = g * n_chunks / n, c1 = (g + 1) * n_chunks / n;
    const int lane = threadIdx.x;
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (long long c = c0; c < c1; ++c) {
        const long long i = c / chunks_per_run;
        const int within = (int)(c - i * chunks_per_run);
        const long long run = (long long)(((unsigned long long)(first_run + i) * (unsigned long long)stride) %
                                          (unsigned long long)total_runs);
        const uint16_t* base = src + ((size_t)run * chunks_per_run + within) * 8192 + lane * 8;
        u32x4 x[16];
#pragma unroll
        for (int t = 0; t < 16; ++t)
            x[t] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + t * 512));
#pragma unroll
        for (int t = 0; t < 16; ++t) acc ^= x[t];
    }
    sink[(size_t)g * 64 + lane] = make_uint4(acc.x, acc.y, acc.z, acc.w);
}

hipError_t spkv_launch_read(const void* src, long long total_runs, int chunks_per_run,
                            long long first_run, long long n_runs, long long stride,
                            int n_workgroups, void* sink, hipStream_t s) {
    spkv_plain_read<<<dim3((unsigned)n_workgroups), dim3(64), 0, s>>>(
        static_cast<const uint16_t*>(src), total_runs, chunks_per_run, first_run,
        n_runs * chunks_per_run, stride, static_cast<uint4*>(sink));
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void spkv_copy_rows(int32_t* __restrict__ dst,
                                                      const int32_t* __restrict__ src, int rows,
                                                      int src_width, int dst_width) {
    const size_t n = (size_t)rows * src_width;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const size_t r = i / src_width, c = i - r * src_width;
        dst[r * dst_width + c] = src[i];
    }
}

hipError_t spkv_launch_copy_rows(int32_t* dst, const int32_t* src, int rows, int src_width,
                                 int dst_width, hipStream_t s) {
    const size_t n = (size_t)rows * src_width;
    if (n == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 256 * 16);
    spkv_copy_rows<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(dst, src, rows, src_width, dst_width);
    return hipGetLastError();
}

template <int D>
__global__ __launch_bounds__(D) void spkv_append_step(SpkvView v, const uint16_t* __restrict__ k,
                                                      const uint16_t* __restrict__ vv,
                                                      const float* __restrict__ f, SpkvCu cu) {
    const int pair = blockIdx.x;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row = cu.v[b];
    if (cu.v[b + 1] - row == 0) return;
    __shared__ int s_page;
    const int T = v.t_pair[pair];
    const int L = v.kept_len[pair];
    const AppendRegs<D> r =
        append_load<D>(v, pair, h, row, T, L, k, vv, f[(size_t)row * v.Hkv + h], threadIdx.x);
    __syncthreads();
    append_store<D>(v, pair, T, L, r, threadIdx.x, &s_page);
}

hipError_t spkv_launch_append_step(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                   const float* f, const SpkvCu& cu, hipStream_t s) {
    if (v.D == 128)
        spkv_append_step<128><<<dim3(v.n_pairs), dim3(128), 0, s>>>(v, k, vv, f, cu);
    else
        spkv_append_step<64><<<dim3(v.n_pairs), dim3(64), 0, s>>>(v, k, vv, f, cu);
    return hipGetLastError();
}

// ----------------------------------------------------- write path, many tokens (bulk)
// For (sequence, head) with n new tokens, T_old stored: positions that leave the window
// are [max(0, T_old - w), T_old + n - w).  Those below T_old sit in the ring (<= w of
// them, handled by spkv_bulk_ring); the others are new tokens j in [0, n - w) that enter
// and leave the window within this call (handled per 256-token segment, one token per
// thread).  The last min(n, w) new tokens land in the ring.  Long-term order is ascending
// position: ring-evicted first, then new tokens; ranks come from ballot + mbcnt prefix
// sums inside a wave, popcounts across the four waves of a segment, and a scan of the
// per-segment counts across segments.
//
// Rows are moved 16 at a time per workgroup: 16 lanes per row, each lane one 16-byte K
// chunk and the 8 V elements of the same head-dim range (loads coalesced per row; the V
// elements go out as 2-byte stores at 16-byte stride, which is what the page layout asks).

// Per-pair scratch written by spkv_bulk_ring for spkv_bulk_scatter.
struct BulkInfo {
    int32_t T_old;        // tokens held before this call
    int32_t new_base;     // long-term index of the first kept NEW token (after ring-evicted ones)
    int32_t ok;           // 0: capacity error, the call writes nothing more for this pair
    int32_t pad;
    SpanOrder order;      // entry `pair` of the order of the attention's spans, written by spkv_bulk_scatter
    int32_t pad2[2];
};
static_assert(sizeof(BulkInfo) == kSpanOrderStride * 4, "order entries lie in the scratch of the pairs");

// Stage 1: per (segment, pair): how many of the segment's new tokens pass the gate, and how
// many of those also leave the window within this call (j < n - w).
__global__ __launch_bounds__(256) void spkv_bulk_count(SpkvView v, const float* __restrict__ f,
                                                       SpkvCu cu) {
    const int pair = blockIdx.y, seg = blockIdx.x;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int n = cu.v[b + 1] - cu.v[b];
    const int n_ev = max(0, n - v.w);
    const int j = seg * kSegTokens + (int)threadIdx.x;
    if (seg * kSegTokens >= n) return;
    __shared__ int s_ev[4], s_on[4];
    const bool on = j < n && gate_passes(v, f[((size_t)cu.v[b] + j) * v.Hkv + h], v.t_pair[pair] + j);
    const int c_on = __popcll(__ballot(on));
    const int c_ev = __popcll(__ballot(on && j < n_ev));
    if (lane_id() == 0) {
        s_on[threadIdx.x >> 6] = c_on;
        s_ev[threadIdx.x >> 6] = c_ev;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        v.seg_count[(size_t)pair * v.n_seg_cap + seg] = s_ev[0] + s_ev[1] + s_ev[2] + s_ev[3];
        v.seg_on[(size_t)pair * v.n_seg_cap + seg] = s_on[0] + s_on[1] + s_on[2] + s_on[3];
    }
}

// Block-wide exclusive scan of one int per thread (256 threads); returns the exclusive
// prefix and the block total.  s_w: 4 ints of shared memory.
__device__ __forceinline__ int block_excl_scan(int x, int* s_w, int& total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    __syncthreads();
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int woff = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < wave) woff += s_w[i];
        total += s_w[i];
    }
    return woff + incl - x;
}

// Stage 2: one workgroup per pair.  Counts the pairs leaving the ring that are kept,
// turns the segment counts into offsets, allocates every page the call needs with one
// allocation per page, publishes the new lengths, then moves the kept ring rows.
//
// prefix (may be null; used by the prefill attention): for the new token i of the call, at
// position t = T_old + i, prefix[(row of token i) * H_kv + h] = number of long-term entries,
// after this call, whose position is <= t - w -- the entries available to query t outside
// its window (the list is in ascending position, so they are a prefix of it).  Stage 2
// writes the tokens whose t - w is a ring position, stage 3 the others; tokens with
// t - w < 0 get no entry (their count is 0).
//
// SMALL: every sequence brings at most min(w, 256) tokens, so no new token leaves the window
// within the call and this launch is the whole append: it also counts the gate-on tokens from
// the logits (stage 1's job otherwise) and, once the kept rows have left the ring, writes
// the new tokens into it (stage 3's job otherwise).
//
// COUNT: chunks of at most kCountSegs segments per sequence -- this launch also does stage 1's
// job for its pair (the per-segment counts from the logits, every wave's popcounts parked in
// LDS), so that the call is two launches instead of three.  Bound by dependent round trips, so only three are
// left: logits, counters and the stack of pages together, ring logits, the pool's atomic; counts, offsets and
// lengths go from one barrier's popcounts to every wave's registers.  16 sequences x 4096 tokens 11.3 -> 9.7 us
// (counts and offsets through memory, the counters before the logits, six barriers more before).
constexpr int kCountSegs = 16;
//
// MOVE = false: the kept ring rows are moved by stage 3 (ring_in_one_workgroup).
// SMALL = false leaves the ring and the token counts alone (stage 3 writes both).
template <int D, bool SMALL, bool COUNT, bool MOVE>
__device__ __forceinline__ void bulk_ring(const SpkvView& v, const SpkvCu& cu, int32_t* prefix,
                                          const uint16_t* __restrict__ k, const uint16_t* __restrict__ vv,
                                          const float* __restrict__ f, int pair) {
    const int b = pair / v.Hkv;
    const int n = cu.v[b + 1] - cu.v[b];
    if (n == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hh = pair - b * v.Hkv, nseg_all = (n + kSegTokens - 1) / kSegTokens;
    // COUNT: every segment's logit of this thread and what thread 0 needs to count and to take pages, before
    // anything is waited for
    float fv[COUNT ? kCountSegs : 1];
    int on_before = 0, recycled = 0;
    if (COUNT) {
#pragma unroll
        for (int sg = 0; sg < kCountSegs; ++sg) {
            const int j = sg * kSegTokens + tid;
            fv[sg] = (sg < nseg_all && j < n) ? f[((size_t)cu.v[b] + j) * v.Hkv + hh] : 0.f;
        }
        if (tid == 0) {
            on_before = v.gate_on[pair];
            recycled = __hip_atomic_load(v.free_top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    const int T_old = v.t_pair[pair], T_new = T_old + n, L_old = v.kept_len[pair];
    const int r0 = max(0, T_old - v.w);
    const int r1 = min(T_old, max(0, T_new - v.w));
    const int nr = max(0, r1 - r0);
    const int n_ev = max(0, n - v.w);
    const int nseg = (n_ev + kSegTokens - 1) / kSegTokens;
    const float* rl = v.ring_logit + (size_t)pair * v.w;
    int32_t* sc = v.seg_count + (size_t)pair * v.n_seg_cap;
    __shared__ int s_w[4];
    __shared__ BulkInfo s_bi;
    __shared__ uint16_t s_list[256];
    __shared__ int s_seg[COUNT ? kCountSegs : 1][4][2];

    // the ring logits of the first 256 leaving positions travel with the segments' logits
    const float rl_first = tid < nr ? rl[(r0 + tid) % v.w] : 0.f;
    const int end_page = (COUNT && (L_old & (kPageTokens - 1)) != 0) ? v.page_table[(size_t)pair * v.pt_cap + (L_old >> 6)] : -1;
    if (COUNT) {          // stage 1 for this pair: per segment and wave, kept-and-leaving / gate-on
#pragma unroll
        for (int sg = 0; sg < kCountSegs; ++sg) {
            if (sg < nseg_all) {
                const int j = sg * kSegTokens + tid;
                const bool on = j < n && gate_passes(v, fv[sg], T_old + j);
                const int c_on = __popcll(__ballot(on));
                const int c_ev = __popcll(__ballot(on && j < n_ev));
                if (lane == 0) {
                    s_seg[sg][wave][0] = c_ev;
                    s_seg[sg][wave][1] = c_on;
                }
            }
        }
    }

    // (a) how many ring pairs are kept
    int cnt = 0;
    for (int base = 0; base < nr; base += 256) {
        const int idx = base + tid;
        const bool flag = idx < nr && gate_passes(v, base == 0 ? rl_first : rl[(r0 + idx) % v.w], r0 + idx);
        cnt += __popcll(__ballot(flag));
    }
    if (lane == 0) s_w[wave] = cnt;
    __syncthreads();
    const int ring_kept = s_w[0] + s_w[1] + s_w[2] + s_w[3];

    // (b) segment counts -> exclusive offsets
    int carry = 0;
    if (COUNT) {          // by every wave, of (segment, wave) pairs, one a lane: nothing goes through memory
        const bool counted = lane < 4 * nseg_all;
        int incl = counted ? s_seg[lane >> 2][lane & 3][0] : 0, on = counted ? s_seg[lane >> 2][lane & 3][1] : 0;
        const int mine = incl;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
            on += __shfl_xor(on, o);
        }
        carry = __builtin_amdgcn_readlane(incl, 63);
        if (wave == 0 && counted && (lane & 3) == 0) sc[lane >> 2] = incl - mine;
        if (tid == 0) v.gate_on[pair] = on_before + on;
    }
    for (int base = 0; !COUNT && base < nseg; base += 256) {
        const int i = base + tid;
        const int c = i < nseg ? sc[i] : 0;
        int tot;
        const int ex = block_excl_scan(c, s_w, tot);
        if (i < nseg) sc[i] = carry + ex;
        carry += tot;
    }
    const int total_new = ring_kept + carry;

    // gate-on count of the call (Eq. 8 numerator), summed here so that no kernel needs
    // same-address atomics
    if (!COUNT) {
        int on = 0;
        if (SMALL) {
            const bool flag = tid < n && gate_passes(v, f[((size_t)cu.v[b] + tid) * v.Hkv + hh], T_old + tid);
            on = flag ? 1 : 0;
        } else {
            const int32_t* so = v.seg_on + (size_t)pair * v.n_seg_cap;
            for (int i = tid; i < nseg_all; i += 256) on += so[i];
        }
        for (int o = 32; o > 0; o >>= 1) on += __shfl_xor(on, o);
        __syncthreads();
        if (lane == 0) s_w[wave] = on;
        __syncthreads();
        if (tid == 0) v.gate_on[pair] += s_w[0] + s_w[1] + s_w[2] + s_w[3];
    }

    // (c) pages: all the call's pages of this pair in one allocation; the table entries are
    //     visible to the whole workgroup after the barrier and to stage 3 after the launch
    const int first = (L_old + kPageTokens - 1) / kPageTokens;
    const int last = (L_old + total_new + kPageTokens - 1) / kPageTokens;
    const int need = last <= v.pt_cap ? last - first : 0;
    int bad = last > v.pt_cap ? 1 : 0;
    __shared__ PageBatch s_pb;
    if (tid == 0) s_pb = COUNT ? alloc_page_batch(v, need, recycled) : alloc_page_batch(v, need);
    __syncthreads();
    for (int i = tid; i < need; i += 256) {
        const int page = batch_page(v, s_pb, i);
        if (page < 0) bad = 1;
        else v.page_table[(size_t)pair * v.pt_cap + first + i] = page;
    }
    // (the bump allocator's pages ascend: the last one of the batch is past the pool if any is)
    const int any_bad = COUNT ? (bad != 0 || (need > s_pb.from_stack && s_pb.pool_base + (need - s_pb.from_stack) > v.n_pages))
                              : __syncthreads_or(bad);
    if (tid == 0) {
        if (any_bad) *v.err_flag = 1;
        s_bi.T_old = T_old;
        s_bi.new_base = L_old + ring_kept;
        s_bi.ok = any_bad ? 0 : 1;
        *reinterpret_cast<BulkInfo*>(v.bulk_info + (size_t)pair * 8) = s_bi;
        if (!any_bad) v.kept_len[pair] = L_old + total_new;
        if (SMALL) v.t_pair[pair] = T_new;
    }
    if (!COUNT || MOVE) {
        __threadfence_block();
        __syncthreads();
    }
    if (any_bad) return;
    const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
    if (ends_in_new_half_page(L_old, L_old + total_new)) {
        const int lp = (L_old + total_new) >> 6;
        const int page = !COUNT ? pt[lp] : lp >= first ? batch_page(v, s_pb, lp - first) : end_page;
        clear_list_end<D>(pool_page(v, page), L_old + total_new, tid, 256);
    }

    // (d) move the kept ring rows, 256 ring positions at a time; without MOVE only their ranks are
    //     wanted, for the prefix counts
    if (!MOVE && prefix == nullptr) return;
    int done = 0;
    for (int base = 0; base < nr; base += 256) {
        const int idx = base + tid;
        const bool flag = idx < nr && gate_passes(v, base == 0 ? rl_first : rl[(r0 + idx) % v.w], r0 + idx);
        int tot;
        const int rank = block_excl_scan(flag ? 1 : 0, s_w, tot);
        if (MOVE && flag) s_list[rank] = (uint16_t)tid;
        if (prefix != nullptr && idx < nr) {
            const int i = r0 + idx + v.w - T_old;      // the new token whose t - w is this position
            prefix[((size_t)cu.v[b] + i) * v.Hkv + (pair - b * v.Hkv)] = L_old + done + rank + (flag ? 1 : 0);
        }
        __syncthreads();
        if (!MOVE) {
            done += tot;
            continue;
        }
        const int c = lane & 15;
        // four rows per lane at a time: all their loads go out before the first store
        for (int rb = wave * 4; rb < tot; rb += 64) {
            uint4 kk[4], vl[4];
            int sv[4], page[4];
            float lg[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = rb + u * 16 + (lane >> 4);
                sv[u] = -1;
                if (r < tot && c < D / 8) {
                    const int s = r0 + base + s_list[r];
                    const int slot = s % v.w;
                    const uint16_t* sp = ring_page(v, pair, slot >> 6);
                    const int sk = slot & 63;
                    kk[u] = *reinterpret_cast<const uint4*>(sp + spkv_k_off(D, sk, c * 8));
                    const uint16_t* vs = sp + spkv_v_off(D, sk, c * 8);
                    unsigned w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = (unsigned)vs[(2 * e) * 8] | ((unsigned)vs[(2 * e + 1) * 8] << 16);
                    vl[u] = make_uint4(w[0], w[1], w[2], w[3]);
                    page[u] = pt[(L_old + done + r) >> 6];
                    lg[u] = rl[slot];
                    sv[u] = s;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (sv[u] >= 0) {
                    const int gi = L_old + done + rb + u * 16 + (lane >> 4);
                    store_row_chunk<D>(pool_page(v, page[u]), gi & 63, c, kk[u], vl[u]);
                    if (c == 0) {
                        v.pos_pool[(size_t)page[u] * kPageTokens + (gi & 63)] = sv[u];
                        v.logit_pool[(size_t)page[u] * kPageTokens + (gi & 63)] = lg[u];
                    }
                }
            }
        }
        done += tot;
        __syncthreads();
    }
    if (SMALL) {        // the new tokens into the ring slots the oldest pairs have just left
        const int h = pair - b * v.Hkv, row0 = cu.v[b], c = lane & 15;
        for (int rb = wave * 4; rb < n; rb += 16) {
            const int jj = rb + (lane >> 4);
            if (jj < n && c < D / 8) {
                const int slot = (T_old + jj) % v.w;
                const size_t src = ((size_t)(row0 + jj) * v.Hkv + h) * D + c * 8;
                const uint4 kk = *reinterpret_cast<const uint4*>(k + src);
                const uint4 vl = *reinterpret_cast<const uint4*>(vv + src);
                store_row_chunk<D>(ring_page(v, pair, slot >> 6), slot & 63, c, kk, vl);
                if (c == 0)
                    v.ring_logit[(size_t)pair * v.w + slot] = f[((size_t)row0 + jj) * v.Hkv + h];
            }
        }
    }
}

template <int D, bool SMALL, bool COUNT, bool MOVE>
__global__ __launch_bounds__(256) void spkv_bulk_ring(SpkvView v, SpkvCu cu, int32_t* prefix,
                                                      const uint16_t* __restrict__ k,
                                                      const uint16_t* __restrict__ vv,
                                                      const float* __restrict__ f) {
    bulk_ring<D, SMALL, COUNT, MOVE>(v, cu, prefix, k, vv, f, blockIdx.x);
}
// Stage 2 of a prefill call and, in further workgroups, its staging rows: neither writes what the other
// reads (ring, ring logits, token counts; lists and tables).  Both wait for memory most of their time.
// Two launches / one, us a prompt with its attention: one sequence of 1000 tokens in pieces of 270
// 193 / 173, two of 600 48 / 44, one of 16k in pieces of 4096 720 / 693, four of 3k-19k 1660 / 1621.
template <int D, bool COUNT, bool MOVE>
__global__ __launch_bounds__(256) void spkv_stage_ring(SpkvView v, SpkvCu cu, int32_t* prefix,
                                                       const uint16_t* __restrict__ k,
                                                       const uint16_t* __restrict__ vv,
                                                       const float* __restrict__ f, SpkvStage st) {
    const int id = (int)blockIdx.x - v.n_pairs;
    if (id < 0) {
        bulk_ring<D, false, COUNT, MOVE>(v, cu, prefix, k, vv, f, blockIdx.x);
    } else {
        const int pair = id / st.hps;
        stage_half_page<D>(v, k, vv, f, cu, st, pair, id - pair * st.hps);
    }
}

// The last min(n, w) tokens of the call go into the ring: a wave takes units of eight consecutive
// slots s0 .. s0 + 7 -- one 16-byte V unit per head-dim element.  Slot s receives the newest position
// p < T_new with p mod w = s if the call brought it (p >= T_new - min(n, w)).  A unit whose eight
// slots are all written goes out as whole 16-byte units, transposed through LDS; otherwise the
// written rows go one by one.
template <int D>
struct RingUnit {
    int s0, age0;            // first slot; tokens between slot s0's newest position and the last one
    bool all;
    float logit;             // lanes 0-7: of slot s0 + lane
    uint4 k[2], v[2];        // rows lane / 16 and 4 + lane / 16
};
// token index (row of the call) landing in slot s0 + r, or -1
__device__ __forceinline__ int ring_token(int s0, int age0, int r, int n, int w) {
    const int age = age0 >= r ? age0 - r : age0 - r + w;
    return s0 + r < w && age < min(n, w) ? n - 1 - age : -1;
}
template <int D>
__device__ __forceinline__ RingUnit<D> load_ring_unit(const SpkvView& v, const uint16_t* __restrict__ k,
                                                      const uint16_t* __restrict__ vv,
                                                      const float* __restrict__ f, int h, int row0,
                                                      int n, int T_old, int s0, int lane) {
    const int c = lane & 15;
    RingUnit<D> u;
    u.s0 = s0;
    u.all = s0 < v.w;
    u.age0 = s0 < v.w ? (T_old + n - 1 - s0 + v.w) % v.w : 0;
    u.logit = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) u.all = u.all && ring_token(s0, u.age0, r, n, v.w) >= 0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int j = ring_token(s0, u.age0, pass * 4 + (lane >> 4), n, v.w);
        u.k[pass] = make_uint4(0u, 0u, 0u, 0u);
        u.v[pass] = make_uint4(0u, 0u, 0u, 0u);
        if (j >= 0 && c < D / 8) {
            const size_t src = ((size_t)(row0 + j) * v.Hkv + h) * D + c * 8;
            u.k[pass] = *reinterpret_cast<const uint4*>(k + src);
            u.v[pass] = *reinterpret_cast<const uint4*>(vv + src);
        }
    }
    if (lane < 8) {
        const int j = ring_token(s0, u.age0, lane, n, v.w);
        if (j >= 0) u.logit = f[((size_t)row0 + j) * v.Hkv + h];
    }
    return u;
}
template <int D>
__device__ __forceinline__ void store_ring_unit(const SpkvView& v, const RingUnit<D>& u, int pair, int n,
                                                uint16_t (*s_rows)[D], int lane) {
    if (u.s0 >= v.w) return;
    const int c = lane & 15, dk0 = u.s0 & 63;
    uint16_t* dp = ring_page(v, pair, u.s0 >> 6);
    if (lane < 8 && ring_token(u.s0, u.age0, lane, n, v.w) >= 0)
        v.ring_logit[(size_t)pair * v.w + u.s0 + lane] = u.logit;
    if (u.all) {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int row = pass * 4 + (lane >> 4);
            if (c < D / 8) {
                *reinterpret_cast<uint4*>(dp + spkv_k_off(D, dk0 + row, c * 8)) = u.k[pass];
                *reinterpret_cast<uint4*>(&s_rows[row][c * 8]) = u.v[pass];
            }
        }
        __builtin_amdgcn_wave_barrier();
        store_v_units<D>(dp, dk0, s_rows, lane);
        __builtin_amdgcn_wave_barrier();
    } else {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int r = pass * 4 + (lane >> 4);
            if (ring_token(u.s0, u.age0, r, n, v.w) >= 0 && c < D / 8)
                store_row_chunk<D>(dp, dk0 + r, c, u.k[pass], u.v[pass]);
        }
    }
}

// One wave, a lane per pair: its group, rank by length in the group, and the spans of the group before it.
// The heads of a sequence are dealt to the groups by length, back and forth.
__device__ __forceinline__ void order_spans(const SpkvView& v, const SpkvCu& cu, SpanCut cut) {
    const int p = threadIdx.x, b = min(p, v.n_pairs - 1) / v.Hkv;
    const int len = p < v.n_pairs ? v.kept_len[p] : -1;
    const int spans = p < v.n_pairs ? (cu.v[b + 1] - cu.v[b] + cut.tokens - 1) / cut.tokens : 0;
    int rank = 0;
    for (int o = 0; o < v.n_pairs; ++o) {
        const int l = __builtin_amdgcn_readlane(len, o);
        rank += o >= b * v.Hkv && o < (b + 1) * v.Hkv && (l > len || (l == len && o < p)) ? 1 : 0;
    }
    const int round = rank / cut.groups, at = rank - round * cut.groups;
    const int group = ((round + b) & 1) != 0 ? cut.groups - 1 - at : at;
    int entry = 0, before = 0;
    for (int o = 0; o < v.n_pairs; ++o) {
        const int l = __builtin_amdgcn_readlane(len, o), n = __builtin_amdgcn_readlane(spans, o);
        const int g = __builtin_amdgcn_readlane(group, o);
        const bool ahead = g == group && (l > len || (l == len && o < p));
        entry += g < group || ahead ? 1 : 0;
        before += ahead ? n : 0;
    }
    if (p < v.n_pairs)
        *reinterpret_cast<SpanOrder*>(v.bulk_info + kSpanOrderAt + (size_t)entry * kSpanOrderStride) =
            SpanOrder{before, p | group << 16};
}

// Stage 3: per (kScatterSegs segments = 512 tokens, pair).  Thread i owns token j0 + i: gate flag,
// rank (mbcnt inside the wave + the popcounts of the lower waves + the offset from stage 2); the
// kept tokens' indices are compacted into LDS and their rows moved in groups of eight consecutive
// destination rows (whole 16-byte V units, transposed through LDS), two groups per wave at a
// time so that all their loads are in flight together; rows before the first and after the
// last whole group go one by one, their V elements as 2-byte stores.  The last workgroup of a
// pair (ring_here) moves the kept rows that leave the ring in the
// same way and then writes the last min(n, w) tokens of the call into the ring, two units' loads
// at a time; without it (ring_in_one_workgroup) workgroups of their own write the slots, eight per
// wave, and stage 2 has moved the rows.  The first workgroup sends the lengths, which stage 2 has
// settled, to the host (`to`) before its own work: the host has them while this launch runs and need
// not wait for the stream to know what the next call may take.
// cut.tokens > 0: one row of workgroups more, of which the first leaves the order of the attention's spans.
// Bound by the requests in flight of a few dependent rounds (logits, rows, stores) more than by
// bytes: 16 sequences x 4096 tokens, 8 heads of 128, a fifth of the pairs kept (77 MB read, 70
// written) 50 us with 256 tokens per workgroup, one group at a time and V units stored in
// pairs; 46 us now with the leaving ring rows, whose move took 7 of the 18 us of stage 2.
// 256 tokens per workgroup 52 us, 1024 tokens 49.  Workgroups are numbered pair by pair: with the heads of a
// token (whose logits share a line) on one XCD, whole prompts of 16 sequences of 32k take 514 us instead of 520 in
// pieces of 4096 and 1009 instead of 1026 of 1024, but 701 instead of 680 of 2048, 8 sequences 338 / 330, 3 heads of
// 64 201 / 194, 5 heads of 128 258 / 248.
constexpr int kScatterSegs = 2, kScatterThreads = kScatterSegs * kSegTokens;

template <int D>
__global__ __launch_bounds__(kScatterThreads) void spkv_bulk_scatter(SpkvView v, const uint16_t* __restrict__ k,
                                                                     const uint16_t* __restrict__ vv,
                                                                     const float* __restrict__ f, SpkvCu cu,
                                                                     int32_t* prefix, int quads, int ring_here,
                                                                     SpanCut cut, SpkvLengthCopy to) {
    constexpr int NW = kScatterThreads / 64;
    if ((int)blockIdx.y == v.n_pairs) {
        if (blockIdx.x == 0 && threadIdx.x < 64) order_spans(v, cu, cut);
        return;
    }
    if (to.host != nullptr && blockIdx.x == 0 && blockIdx.y == 0) copy_lengths(v.kept_len, v.n_pairs, to);
    const int pair = blockIdx.y, quad = blockIdx.x;
    const int b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int row0 = cu.v[b];
    const int n = cu.v[b + 1] - row0;
    const int j0 = quad * kScatterThreads;
    if (n == 0 || (quad < quads && j0 >= n)) return;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_ev = max(0, n - v.w);
    const int j = j0 + tid;
    const float fj = (quad < quads && j < n) ? f[((size_t)row0 + j) * v.Hkv + h] : 0.f;
    const int seg_off = (quad < quads && j0 < n_ev) ? v.seg_count[(size_t)pair * v.n_seg_cap + quad * kScatterSegs] : 0;
    const BulkInfo bi = *reinterpret_cast<const BulkInfo*>(v.bulk_info + (size_t)pair * 8);
    if (quad == 0 && tid == 0) v.t_pair[pair] = bi.T_old + n;
    if (bi.ok == 0) return;
    __shared__ int s_cnt[2][NW];
    __shared__ uint16_t s_list[2 * kScatterThreads];
    __shared__ __attribute__((aligned(16))) uint16_t s_v[NW][8][D];
    if (quad >= quads && ring_here == 0) {      // the ring part of the grid (ring_here = 0): independent of the segments
        const int s0 = (quad - quads) * (NW * 8) + wave * 8;
        store_ring_unit<D>(v, load_ring_unit<D>(v, k, vv, f, h, row0, n, bi.T_old, s0, lane), pair, n, s_v[wave], lane);
        return;
    }
    // rows leaving the ring: positions r0 .. r0 + nr - 1, thread i looks at r0 + i
    const float* rl = v.ring_logit + (size_t)pair * v.w;
    const int r0 = max(0, bi.T_old - v.w);
    const bool ring_wg = quad >= quads;
    const int nr = ring_wg ? max(0, min(bi.T_old, max(0, bi.T_old + n - v.w)) - r0) : 0;
    const bool rev = tid < nr && gate_passes(v, rl[(r0 + tid) % v.w], r0 + tid);
    const bool ev = !ring_wg && j < n_ev && gate_passes(v, fj, bi.T_old + j);
    const unsigned long long rmask = __ballot(rev), mask = __ballot(ev);
    if (lane == 0) {
        s_cnt[0][wave] = __popcll(rmask);
        s_cnt[1][wave] = __popcll(mask);
    }
    __syncthreads();
    int roff = 0, woff = 0, n_ring = 0, n_new = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int a0 = s_cnt[0][i], a1 = s_cnt[1][i];
        if (i < wave) {
            roff += a0;
            woff += a1;
        }
        n_ring += a0;
        n_new += a1;
    }
    constexpr unsigned kFromRing = 0x8000u;
    if (rev) s_list[roff + mbcnt64(rmask)] = (uint16_t)(kFromRing | (unsigned)tid);
    if (ev) s_list[n_ring + woff + mbcnt64(mask)] = (uint16_t)tid;
    if (prefix != nullptr && !ring_wg && j < n_ev)       // token j leaves the window of token j + w
        prefix[((size_t)row0 + j + v.w) * v.Hkv + h] =
            bi.new_base + seg_off + woff + mbcnt64(mask) + (ev ? 1 : 0);
    __syncthreads();

    const int total = n_ring + n_new;
    // chunk c of the row of a list entry (nothing for lanes past the row)
    struct Row {
        uint4 k, v;
    };
    auto load_row = [&](unsigned e) -> Row {
        Row r = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u)};
        if (c >= D / 8) return r;
        if (e & kFromRing) {
            const int slot = (r0 + (int)(e & 0x7fffu)) % v.w;
            const uint16_t* sp = ring_page(v, pair, slot >> 6);
            const uint16_t* vs = sp + spkv_v_off(D, slot & 63, c * 8);
            r.k = *reinterpret_cast<const uint4*>(sp + spkv_k_off(D, slot & 63, c * 8));
            r.v.x = (unsigned)vs[0] | ((unsigned)vs[8] << 16);
            r.v.y = (unsigned)vs[16] | ((unsigned)vs[24] << 16);
            r.v.z = (unsigned)vs[32] | ((unsigned)vs[40] << 16);
            r.v.w = (unsigned)vs[48] | ((unsigned)vs[56] << 16);
        } else {
            const size_t src = ((size_t)(row0 + j0 + (int)e) * v.Hkv + h) * D + c * 8;
            r.k = *reinterpret_cast<const uint4*>(k + src);
            r.v = *reinterpret_cast<const uint4*>(vv + src);
        }
        return r;
    };
    auto store_meta = [&](unsigned e, int page, int dk) {
        const bool ring = (e & kFromRing) != 0u;
        const int i = (int)(e & 0x7fffu);
        v.pos_pool[(size_t)page * kPageTokens + dk] = ring ? r0 + i : bi.T_old + j0 + i;
        v.logit_pool[(size_t)page * kPageTokens + dk] =
            ring ? rl[(r0 + i) % v.w] : f[((size_t)row0 + j0 + i) * v.Hkv + h];
    };
    const int lr = lane >> 4;                  // a lane's row of four
    auto store_group = [&](int e0, int page, int dk0, const Row& a, const Row& b2) {
        uint16_t* dp = pool_page(v, page);
        if (c < D / 8) {
            *reinterpret_cast<uint4*>(dp + spkv_k_off(D, dk0 + lr, c * 8)) = a.k;
            *reinterpret_cast<uint4*>(dp + spkv_k_off(D, dk0 + 4 + lr, c * 8)) = b2.k;
            *reinterpret_cast<uint4*>(&s_v[wave][lr][c * 8]) = a.v;
            *reinterpret_cast<uint4*>(&s_v[wave][4 + lr][c * 8]) = b2.v;
        }
        __builtin_amdgcn_wave_barrier();
        store_v_units<D>(dp, dk0, s_v[wave], lane);
        if (lane < 8) store_meta(s_list[e0 + lane], page, dk0 + lane);
        __builtin_amdgcn_wave_barrier();
    };
    if (total > 0) {
        const int g0 = ring_wg ? bi.new_base - n_ring : bi.new_base + seg_off;
        const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
        const int gend = g0 + total;
        const int ga = min(gend, (g0 + 7) & ~7);   // destination indices [ga, gb) are whole
        const int gb = max(ga, gend & ~7);         // groups of 8 aligned to 8: whole V units

        for (int G8 = ga + wave * 8; G8 < gb; G8 += 2 * NW * 8) {
            const int G2 = G8 + NW * 8;
            const bool two = G2 < gb;
            const int e1 = G8 - g0, e2 = two ? G2 - g0 : e1;
            const int page1 = pt[G8 >> 6], page2 = two ? pt[G2 >> 6] : 0;
            const Row a0 = load_row(s_list[e1 + lr]), a1 = load_row(s_list[e1 + 4 + lr]);
            const Row b0 = load_row(s_list[e2 + lr]), b1 = load_row(s_list[e2 + 4 + lr]);
            store_group(e1, page1, G8 & 63, a0, a1);
            if (two) store_group(e2, page2, G2 & 63, b0, b1);
        }
        // The rows before the first and after the last whole group, one row per 16 lanes.
        const int n_head = ga - g0, n_tail = gend - gb;
        for (int rb = wave * 4; rb < n_head + n_tail; rb += NW * 4) {
            const int x = rb + (lane >> 4);
            if (x < n_head + n_tail && c < D / 8) {
                const int r = x < n_head ? x : (gb - g0) + (x - n_head);
                const int gi = g0 + r, page = pt[gi >> 6];
                const Row a = load_row(s_list[r]);
                store_row_chunk<D>(pool_page(v, page), gi & 63, c, a.k, a.v);
                if (c == 0) store_meta(s_list[r], page, gi & 63);
            }
        }
    }
    if (ring_wg) {            // the rows that leave have been read: the new ones take their slots
        __syncthreads();
        for (int s0 = wave * 8; s0 < v.w; s0 += 2 * NW * 8) {       // two units' loads in flight
            const RingUnit<D> a = load_ring_unit<D>(v, k, vv, f, h, row0, n, bi.T_old, s0, lane);
            if (s0 + NW * 8 < v.w) {
                const RingUnit<D> a2 = load_ring_unit<D>(v, k, vv, f, h, row0, n, bi.T_old, s0 + NW * 8, lane);
                store_ring_unit<D>(v, a, pair, n, s_v[wave], lane);
                store_ring_unit<D>(v, a2, pair, n, s_v[wave], lane);
            } else {
                store_ring_unit<D>(v, a, pair, n, s_v[wave], lane);
            }
        }
    }
}

// One workgroup per pair for the ring (a thread per slot), or stage 2 moves the leaving rows and a
// workgroup per 64 slots writes the new ones.  The one workgroup works through its slots one
// round after the other, which pays where other workgroups fill the chip meanwhile: short rings, and
// longer ones beside several segments of many pairs.  Prompts of 4096 tokens, us per prompt, stage 2 /
// one workgroup (8 KV heads of 128): in pieces of 270 and a ring of 256, 8 pairs 460 / 503, 256 pairs
// 746 / 900; ring of 64, 128 pairs 410 / 392; in pieces of 700 and a ring of 128, 64 pairs 235 / 219;
// ring of 512, 8 pairs 292 / 300, 128 pairs 413 / 380.
static bool ring_in_one_workgroup(const SpkvView& v, int n_max) {
    if (v.w > kScatterThreads) return false;
    return v.w <= 64 || (n_max > kScatterThreads && (v.w <= 128 || v.n_pairs >= 64));
}

bool spkv_append_stages(const SpkvView& v, int n_max) {        // (a launch counts its threads in 32 bits)
    return spkv_append_copies_lengths(v, n_max) &&
           (int64_t)v.n_pairs * (1 + ((int64_t)v.w + n_max + kHalfTokens - 1) / kHalfTokens) <= INT32_MAX / 256;
}
bool spkv_append_copies_lengths(const SpkvView& v, int n_max) { return n_max > v.w || n_max > kSegTokens; }

template <int D>
__global__ __launch_bounds__(256) void spkv_append_few(SpkvView v, const uint16_t* __restrict__ k,
                                                       const uint16_t* __restrict__ vv,
                                                       const float* __restrict__ f, SpkvCu cu) {
    append_few<D>(v, blockIdx.x, k, vv, f, cu);
}

hipError_t spkv_launch_append_bulk(const SpkvView& v, const uint16_t* k, const uint16_t* vv,
                                   const float* f, const SpkvCu& cu, int n_max, int32_t* prefix,
                                   SpanCut cut, const SpkvStage& st, SpkvLengthCopy to, hipStream_t s) {
    if (n_max <= kFewTokens && n_max <= v.w && prefix == nullptr) {
        if (v.D == 128) spkv_append_few<128><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v, k, vv, f, cu);
        else spkv_append_few<64><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v, k, vv, f, cu);
        return hipGetLastError();
    }
    if (!spkv_append_copies_lengths(v, n_max)) {    // short chunks: one launch
        if (v.D == 128) spkv_bulk_ring<128, true, false, true><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v, cu, prefix, k, vv, f);
        else spkv_bulk_ring<64, true, false, true><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v, cu, prefix, k, vv, f);
        return hipGetLastError();
    }
    const int segs_all = (n_max + kSegTokens - 1) / kSegTokens;
    const int quads = (n_max + kScatterThreads - 1) / kScatterThreads;
    const bool ring_here = ring_in_one_workgroup(v, n_max);
    const dim3 grid3(quads + (ring_here ? 1 : (v.w + kScatterThreads / 8 - 1) / (kScatterThreads / 8)), v.n_pairs + (cut.tokens > 0 ? 1 : 0));
    const bool fold = segs_all <= kCountSegs;       // the per-pair launch counts for itself
    if (!fold) spkv_bulk_count<<<dim3(segs_all, v.n_pairs), dim3(256), 0, s>>>(v, f, cu);
    auto stage2 = [&](auto kernel) { kernel<<<dim3(v.n_pairs), dim3(256), 0, s>>>(v, cu, prefix, k, vv, f); };
    const dim3 grid2((unsigned)v.n_pairs * (unsigned)(1 + st.hps));
    auto staged = [&](auto kernel) { kernel<<<grid2, dim3(256), 0, s>>>(v, cu, prefix, k, vv, f, st); };
    if (v.D == 128) {
        if (st.stage != nullptr && fold) ring_here ? staged(spkv_stage_ring<128, true, false>) : staged(spkv_stage_ring<128, true, true>);
        else if (st.stage != nullptr) ring_here ? staged(spkv_stage_ring<128, false, false>) : staged(spkv_stage_ring<128, false, true>);
        else if (fold) ring_here ? stage2(spkv_bulk_ring<128, false, true, false>) : stage2(spkv_bulk_ring<128, false, true, true>);
        else ring_here ? stage2(spkv_bulk_ring<128, false, false, false>) : stage2(spkv_bulk_ring<128, false, false, true>);
        spkv_bulk_scatter<128><<<grid3, dim3(kScatterThreads), 0, s>>>(v, k, vv, f, cu, prefix, quads, ring_here, cut, to);
    } else {
        if (st.stage != nullptr && fold) ring_here ? staged(spkv_stage_ring<64, true, false>) : staged(spkv_stage_ring<64, true, true>);
        else if (st.stage != nullptr) ring_here ? staged(spkv_stage_ring<64, false, false>) : staged(spkv_stage_ring<64, false, true>);
        else if (fold) ring_here ? stage2(spkv_bulk_ring<64, false, true, false>) : stage2(spkv_bulk_ring<64, false, true, true>);
        else ring_here ? stage2(spkv_bulk_ring<64, false, false, false>) : stage2(spkv_bulk_ring<64, false, false, true>);
        spkv_bulk_scatter<64><<<grid3, dim3(kScatterThreads), 0, s>>>(v, k, vv, f, cu, prefix, quads, ring_here, cut, to);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ prune after a raise
// After the threshold has been raised (Sec. 2.1: tau can be chosen after training, per
// deployment): every long-term entry whose stored logit no longer passes the gate is dropped
// and the list closed up, in place and in order.  One workgroup per (sequence, KV head)
// walks its list 256 entries at a time: flags, ranks by a block scan, then the kept rows
// move down 16 at a time -- read into registers, barrier, written.  A row's destination
// index never exceeds its own index and rows go in ascending order, so no write lands on a
// row that is still to be read.  Pages the shorter list no longer reaches go back onto the
// stack of recycled pages (pushes only: no page is allocated in this launch).
template <int D>
__global__ __launch_bounds__(256) void spkv_prune(SpkvView v) {
    const int pair = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15;
    const int L = v.kept_len[pair];
    int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
    __shared__ int s_w[4];
    __shared__ uint16_t s_list[256];
    __shared__ int s_base;
    int out = 0;                                           // entries kept so far (uniform)
    for (int seg0 = 0; seg0 < L; seg0 += 256) {
        const int idx = seg0 + tid;
        bool keep = false;
        if (idx < L) {
            const size_t e = (size_t)pt[idx >> 6] * kPageTokens + (idx & 63);
            keep = gate_passes(v, v.logit_pool[e], v.pos_pool[e]);
        }
        int tot;
        const int rank = block_excl_scan(keep ? 1 : 0, s_w, tot);
        if (keep) s_list[rank] = (uint16_t)tid;
        __syncthreads();
        for (int rb = 0; rb < tot; rb += 16) {
            const int r = rb + wave * 4 + (lane >> 4);
            const bool mine = r < tot && c < D / 8;
            uint4 kk = {0u, 0u, 0u, 0u};
            unsigned w[4] = {0u, 0u, 0u, 0u};
            int pos = 0;
            float lg = 0.f;
            if (mine) {
                const int si = seg0 + s_list[r];
                const int sp_page = pt[si >> 6], sk = si & 63;
                const uint16_t* sp = pool_page(v, sp_page);
                kk = *reinterpret_cast<const uint4*>(sp + spkv_k_off(D, sk, c * 8));
                const uint16_t* vs = sp + spkv_v_off(D, sk, c * 8);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = (unsigned)vs[(2 * e) * 8] | ((unsigned)vs[(2 * e + 1) * 8] << 16);
                pos = v.pos_pool[(size_t)sp_page * kPageTokens + sk];
                lg = v.logit_pool[(size_t)sp_page * kPageTokens + sk];
            }
            __syncthreads();                               // every row of the group has been read
            if (mine) {
                const int di = out + r;
                const int dp_page = pt[di >> 6], dk = di & 63;
                store_row_chunk<D>(pool_page(v, dp_page), dk, c, kk, make_uint4(w[0], w[1], w[2], w[3]));
                if (c == 0) {
                    v.pos_pool[(size_t)dp_page * kPageTokens + dk] = pos;
                    v.logit_pool[(size_t)dp_page * kPageTokens + dk] = lg;
                }
            }
            __syncthreads();                               // ... and written, before the next group reads
        }
        out += tot;
    }
    const int np_old = (L + kPageTokens - 1) / kPageTokens, np_new = (out + kPageTokens - 1) / kPageTokens;
    const int n_free = np_old - np_new;
    if (tid == 0) s_base = n_free > 0 ? atomicAdd(v.free_top, n_free) : 0;
    __syncthreads();
    for (int i = tid; i < n_free; i += 256) v.free_pages[s_base + i] = pt[np_new + i];
    if (out < L && (out & (kHalfTokens - 1)) != 0)         // dropped rows behind the new end (every row has moved)
        clear_list_end<D>(pool_page(v, pt[out >> 6]), out, tid, 256);
    if (tid == 0) v.kept_len[pair] = out;
}

hipError_t spkv_launch_prune(const SpkvView& v, hipStream_t s) {
    if (v.D == 128) spkv_prune<128><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v);
    else spkv_prune<64><<<dim3(v.n_pairs), dim3(256), 0, s>>>(v);
    return hipGetLastError();
}

// ---------------------------------------------------------------- release a sequence
// One workgroup per KV head of the sequence: its pages go onto the stack of recycled pages
// and its counters back to zero.  Further ones clear the values of its ring: while the next
// owner's window fills, the half-page that ends it is read whole, and a weight of zero would turn an
// infinity among the old ones into a NaN (keys are masked by selection).
__host__ __device__ __forceinline__ int ring_half_pages(const SpkvView& v) { return (v.w + kHalfTokens - 1) / kHalfTokens; }
__global__ __launch_bounds__(256) void spkv_release_sequence(SpkvView v, int b) {
    const int pair = b * v.Hkv + blockIdx.x;
    const int tid = threadIdx.x;
    if (blockIdx.y > 0) {
        for (int hp = blockIdx.y - 1; hp < ring_half_pages(v); hp += gridDim.y - 1) {
            uint4* values = reinterpret_cast<uint4*>(ring_page(v, pair, hp >> 1) + ((hp & 1) * 2 + 1) * kHalfTokens * v.D);
            for (int i = tid; i < kHalfTokens * v.D / 8; i += 256) values[i] = make_uint4(0u, 0u, 0u, 0u);
        }
        return;
    }
    const int np = (v.kept_len[pair] + kPageTokens - 1) / kPageTokens;
    __shared__ int s_base;
    if (tid == 0) s_base = np > 0 ? atomicAdd(v.free_top, np) : 0;
    __syncthreads();
    for (int i = tid; i < np; i += 256)
        v.free_pages[s_base + i] = v.page_table[(size_t)pair * v.pt_cap + i];
    if (tid == 0) {
        v.kept_len[pair] = 0;
        v.t_pair[pair] = 0;
        v.gate_on[pair] = 0;
    }
}

hipError_t spkv_launch_release_sequence(const SpkvView& v, int b, hipStream_t s) {
    spkv_release_sequence<<<dim3(v.Hkv, 1 + std::min(ring_half_pages(v), 256)), dim3(256), 0, s>>>(v, b);
    return hipGetLastError();
}

// ------------------------------------------------------------ kept positions (debug)
__global__ __launch_bounds__(256) void spkv_gather_positions(SpkvView v, int pair) {
    const int L = v.kept_len[pair];
    for (int gi = blockIdx.x * blockDim.x + threadIdx.x; gi < L; gi += gridDim.x * blockDim.x) {
        const int page = v.page_table[(size_t)pair * v.pt_cap + (gi >> 6)];
        v.pos_scratch[gi] = v.pos_pool[(size_t)page * kPageTokens + (gi & 63)];
    }
}

hipError_t spkv_launch_gather_positions(const SpkvView& v, int pair, hipStream_t s) {
    spkv_gather_positions<<<dim3(64), dim3(256), 0, s>>>(v, pair);
    return hipGetLastError();
}

