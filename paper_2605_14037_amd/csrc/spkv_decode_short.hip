// Single-token decode of caches with short lists: one workgroup per (sequence, KV head) reads the
// whole pair, merges in LDS and finishes -- no partial results in memory, no second launch.
#include "spkv_device.h"

// Waves per workgroup: 16 at head_dim 64; at 128 two half-pages in flight per wave need 218 registers.
constexpr int short_waves(int head_dim) { return head_dim == 64 ? 16 : 8; }

// Half-page hp of the pair goes to wave hp mod NW, the next one's loads out before the current one is
// worked on; the arithmetic is that of the split kernel (attend_half_page).  The waves meet in LDS,
// D / P output dimensions at a time (P = 1, 2, 4 for groups of up to 4, 8, 16 heads).
// STEP (spkv_decode_step): the cache is in the state before the append of the newest token, whose own
// term is added in the merge and which is appended once every wave has read what it needs of the
// ring; the pair leaving the window is left out unless it passes the gate.
// Bound by dependent round trips: counters and page ids together, tiles, then the merge and the stores.
// One sequence of 2k, 2 KV heads of 64, 19 half-pages the longer list: 6.0 us a step replayed from a
// graph, 6.9 as a split and a merge launch (13.4 -> 10.0 issued call by call).  A further round of half-pages
// costs 1 us while one compute unit reads from the L2, 2 from behind it, so longer lists are
// left to the split kernel, which spreads a pair over the chip (short_lists, with the times of both).
template <int D, int P, bool STEP>
__global__ __launch_bounds__(64 * short_waves(D)) void spkv_decode_short(SpkvView v, const uint16_t* __restrict__ q,
                                                                      float scale_log2e, SpkvStepIO io) {
    constexpr int NW = short_waves(D), NS = D / 32, NB = D / 16, DP = D / P;
    constexpr int kRow = DP + 16;                         // no bank conflicts between a wave's rows
    __shared__ __attribute__((aligned(16))) float s_acc[NW * 4 * P * kRow];
    __shared__ float s_m[NW][16], s_l[NW][16], s_tok[16];
    __shared__ int s_page;
    const int pair = blockIdx.x, b = pair / v.Hkv, h = pair - b * v.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, kc = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t* pt = v.page_table + (size_t)pair * v.pt_cap;
    int pbase = 0, my_page = pt[min(lane, v.pt_cap - 1)];        // with the counters, not after them
    const int L = v.kept_len[pair], T = v.t_pair[pair];
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
    const int Tw = min(T, v.w), ghp = (L + kHalfTokens - 1) >> 5, nhp = ghp + ((Tw + kHalfTokens - 1) >> 5);

    struct Tile {
        bf16x8 k[2][NS], v[NB];
    };
    auto load = [&](Tile& t, int hp) {
        const uint16_t* base;
        if (hp < ghp) {
            const int lp = hp >> 1;
            if (lp >= pbase + 64) {
                pbase = lp;
                my_page = pt[min(pbase + lane, v.pt_cap - 1)];
            }
            base = pool_page(v, __builtin_amdgcn_readlane(my_page, lp - pbase)) + (hp & 1) * (2 * kHalfTokens * D);
        } else {
            const int r = hp - ghp;
            base = ring_page(v, pair, r >> 1) + (r & 1) * (2 * kHalfTokens * D);
        }
        const uint16_t* kp = base + lane * 8;
        const uint16_t* vp = base + kHalfTokens * D + lane * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) t.k[i][sl] = load_stream_b128(kp + (i * (D / 8) + sl * 4) * 128);
#pragma unroll
        for (int db = 0; db < NB; ++db) t.v[db] = load_stream_b128(vp + db * 512);
    };
    Tile t0, t1;                         // two half-pages of the wave in flight
    int hp = wave;
    if (hp < nhp) load(t0, hp);
    int drop_hp = -1, drop_r = -1;       // the ring key that leaves the window and fails the gate
    if (STEP && T >= v.w) {
        const int slot = T % v.w;
        if (!gate_passes(v, v.ring_logit[(size_t)pair * v.w + slot], T - v.w)) {
            drop_hp = ghp + (slot >> 5);
            drop_r = slot & 31;
        }
    }
    f32x4 acc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = SPKV_NEG_INF, l = 0.f;
    auto attend = [&](const Tile& t) {
        const int nvalid = hp < ghp ? min(kHalfTokens, L - hp * kHalfTokens)
                                    : min(kHalfTokens, Tw - (hp - ghp) * kHalfTokens);
        const int masked_r = (STEP && hp == drop_hp) ? drop_r : -1;
        const bool any_kill = nvalid < kHalfTokens || masked_r >= 0;
        unsigned kill = 0u;
        if (any_kill) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (kc * 8 + e >= nvalid || kc * 8 + e == masked_r) kill |= 1u << e;
        }
        attend_half_page<D>(t.k, t.v, qb, kill, any_kill, scale_log2e, acc, m, l);
        hp += NW;
    };
    while (hp < nhp) {
        if (hp + NW < nhp) load(t1, hp + NW);
        attend(t0);
        if (hp >= nhp) break;
        if (hp + NW < nhp) load(t0, hp + NW);
        attend(t1);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);

    AppendRegs<D> ar;
    const size_t kv_row = ((size_t)b * v.Hkv + h) * D;
    if (STEP) {
        // the append's loads travel while the waves meet
        ar = append_load<D>(v, pair, h, b, T, L, io.k_new, io.v_new, io.f_new[(size_t)b * v.Hkv + h], tid);
        for (int g = wave; g < v.G; g += NW) {            // score of the new token in fp32, a head per wave
            const size_t q_row = ((size_t)b * v.Hq + (size_t)h * v.G + g) * D;
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < D / 64; ++e) {
                const unsigned qe = q[q_row + lane * (D / 64) + e], ke = io.k_new[kv_row + lane * (D / 64) + e];
                dot += __builtin_bit_cast(float, qe << 16) * __builtin_bit_cast(float, ke << 16);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
            if (lane == 0) s_tok[g] = dot * scale_log2e;
        }
    }
    if (kc == 0) {
        s_m[wave][n] = m;
        s_l[wave][n] = l;
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (p > 0) __syncthreads();
        if (n < v.G) {
            float* pa = s_acc + (wave * v.G + n) * kRow + kc * 4;
#pragma unroll
            for (int i = 0; i < NB / P; ++i) *reinterpret_cast<f32x4*>(pa + i * 16) = acc[p * (NB / P) + i];
        }
        __syncthreads();
        for (int e = tid; e < v.G * DP; e += 64 * NW) {
            const int g = e / DP, dd = e - g * DP, d = p * DP + dd;
            float M = STEP ? s_tok[g] : SPKV_NEG_INF;
#pragma unroll
            for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w][g]);
            const float m_ref = (M == SPKV_NEG_INF) ? 0.f : M;      // no key at all: every weight 0
            float num = 0.f, den = 0.f;
            if (STEP) {
                den = __builtin_amdgcn_exp2f(s_tok[g] - m_ref);
                num = __builtin_bit_cast(float, (unsigned)io.v_new[kv_row + d] << 16) * den;
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float sc = __builtin_amdgcn_exp2f(s_m[w][g] - m_ref);
                num += sc * s_acc[(w * v.G + g) * kRow + dd];
                den += sc * s_l[w][g];
            }
            const size_t o = (size_t)b * v.Hq + (size_t)h * v.G + g;
            const __bf16 r = (__bf16)(num / den);
            io.out[o * D + d] = __builtin_bit_cast(uint16_t, r);
            if (io.lse != nullptr && d == 0) io.lse[o] = (M + log2f(den)) * 0.6931471805599453f;
        }
    }
    if (STEP) append_store<D>(v, pair, T, L, ar, tid, &s_page);
}

template <int D, bool STEP>
static hipError_t launch_short(const SpkvView& v, const uint16_t* q, float scale_log2e, const SpkvStepIO& io,
                               hipStream_t s) {
    const dim3 grid(v.n_pairs), block(64 * short_waves(D));
    if (v.G <= 4) spkv_decode_short<D, 1, STEP><<<grid, block, 0, s>>>(v, q, scale_log2e, io);
    else if (v.G <= 8) spkv_decode_short<D, 2, STEP><<<grid, block, 0, s>>>(v, q, scale_log2e, io);
    else spkv_decode_short<D, 4, STEP><<<grid, block, 0, s>>>(v, q, scale_log2e, io);
    return hipGetLastError();
}

int spkv_short_waves(int head_dim) { return short_waves(head_dim); }

hipError_t spkv_launch_decode_short(const SpkvView& v, const uint16_t* q, float sm_scale, const SpkvStepIO& io,
                                    hipStream_t s) {
    const float sl = sm_scale * 1.4426950408889634f;
    if (io.k_new != nullptr)
        return v.D == 128 ? launch_short<128, true>(v, q, sl, io, s) : launch_short<64, true>(v, q, sl, io, s);
    return v.D == 128 ? launch_short<128, false>(v, q, sl, io, s) : launch_short<64, false>(v, q, sl, io, s);
}
