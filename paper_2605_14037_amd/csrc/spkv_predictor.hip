// Utility predictor of the SP-KV gate (Eq. 1) on gfx950.
#include "spkv_device.h"

// ------------------------------------------------------------------ utility predictor
// Eq. 1 with the predictor of the paper's listing: Linear(d_model, d_hidden) - SiLU -
// Linear(d_hidden, n_kv_heads), pre-sigmoid.  Hidden layer: one workgroup per (16 hidden
// units, 16 tokens); its four waves split d_model, each running MFMA 16x16x32 with the W1
// rows as A operand (rows = hidden units, contraction over d_model) and the tokens as the
// 16 columns; partial sums meet in LDS, bias and SiLU are applied in fp32.
__global__ __launch_bounds__(256) void spkv_predictor_hidden(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ w1,
                                                             const float* __restrict__ b1,
                                                             float* __restrict__ act, int n_tokens,
                                                             int d_model, int d_hidden) {
    const int j0 = blockIdx.x * 16, t0 = blockIdx.y * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kc = lane >> 4, n = lane & 15;
    const int kq = d_model / 4;                       // this wave's share of d_model
    const uint16_t* wrow = w1 + (size_t)(j0 + n) * d_model + wave * kq + kc * 8;
    const bool tok_ok = t0 + n < n_tokens;
    const uint16_t* xrow = x + (size_t)(tok_ok ? t0 + n : 0) * d_model + wave * kq + kc * 8;
    // (columns past the last token read token 0's row; their results are never stored)
    const f32x4 acc = predictor_contract(wrow, xrow, kq);   // kq is a multiple of 32 (d_model of 128)
    // lane (kc, n) holds hidden units j0 + 4 kc + i of token t0 + n
    __shared__ float s_part[4][16][17];
#pragma unroll
    for (int i = 0; i < 4; ++i) s_part[wave][4 * kc + i][n] = acc[i];
    __syncthreads();
    const int jj = tid >> 4, tt = tid & 15;
    if (t0 + tt < n_tokens) {
        float h = s_part[0][jj][tt] + s_part[1][jj][tt] + s_part[2][jj][tt] + s_part[3][jj][tt];
        if (b1 != nullptr) h += b1[j0 + jj];
        act[(size_t)(t0 + tt) * d_hidden + j0 + jj] = h / (1.f + __expf(-h));     // SiLU
    }
}

// Output layer: one wave per (token, KV head): logits = b2 + W2[h, :] . act[t, :].
__global__ __launch_bounds__(64) void spkv_predictor_out(const float* __restrict__ act,
                                                         const uint16_t* __restrict__ w2,
                                                         const float* __restrict__ b2,
                                                         float* __restrict__ logits, int d_hidden,
                                                         int n_kv_heads) {
    const int t = blockIdx.x / n_kv_heads, h = blockIdx.x - t * n_kv_heads;
    float sum = 0.f;
    for (int j = threadIdx.x; j < d_hidden; j += 64) {
        const unsigned wbits = w2[(size_t)h * d_hidden + j];
        sum += __builtin_bit_cast(float, wbits << 16) * act[(size_t)t * d_hidden + j];
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (threadIdx.x == 0) logits[(size_t)t * n_kv_heads + h] = sum + (b2 != nullptr ? b2[h] : 0.f);
}

// Many tokens (prompt processing): the whole predictor in one launch, register-tiled.  One
// workgroup per 64 tokens; wave wv owns hidden units 64 wv .. 64 wv + 63, so d_hidden / 64
// waves cover the hidden layer.  Each wave keeps a 64 x 64 (hidden x token) tile of fp32 sums
// in 16 MFMA accumulators and walks d_model in steps of 32: four 16-byte loads of W1 rows and
// four of token rows per lane feed 16 MFMAs (the operands of the next step are loaded before
// the MFMAs of the current one).  Bias and SiLU are applied in registers, the output layer is
// taken per wave over its 64 hidden units (16 products per lane, head and token group, then a
// sum over the four lane groups), and the waves' partial logits meet in LDS.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void spkv_predictor_tiled(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ w1,
                                                             const float* __restrict__ b1,
                                                             const uint16_t* __restrict__ w2,
                                                             const float* __restrict__ b2,
                                                             float* __restrict__ logits, int n_tokens,
                                                             int d_model, int d_hidden, int n_kv_heads) {
    extern __shared__ float s_logit[];                     // [waves][64 tokens][n_kv_heads]
    const int tid = threadIdx.x, lane = tid & 63, kc = lane >> 4, n = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = d_hidden / 64;
    const int t0 = blockIdx.x * 64, j0 = wv * 64;
    const uint16_t* wrow[4];
    const uint16_t* xrow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        wrow[i] = w1 + (size_t)(j0 + i * 16 + n) * d_model + kc * 8;
        // (columns past the last token read the last token's row; their results are not stored)
        xrow[i] = x + (size_t)min(t0 + i * 16 + n, n_tokens - 1) * d_model + kc * 8;
    }
    f32x4 acc[4][4];
#pragma unroll
    for (int hs = 0; hs < 4; ++hs)
#pragma unroll
        for (int ts = 0; ts < 4; ++ts) acc[hs][ts] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // KS steps of 32 along d_model per iteration; the operands of the next iteration are
    // loaded before the MFMAs of the current one (d_model is a multiple of 128)
    constexpr int KS = 2;
    uint4 a[KS][4], b[KS][4];
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[u][i] = *reinterpret_cast<const uint4*>(wrow[i] + u * 32);
            b[u][i] = *reinterpret_cast<const uint4*>(xrow[i] + u * 32);
        }
    for (int k = KS * 32; k <= d_model; k += KS * 32) {
        uint4 an[KS][4], bn[KS][4];
        const int kn = min(k, d_model - KS * 32);          // the last iteration reloads its own operands
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                an[u][i] = *reinterpret_cast<const uint4*>(wrow[i] + kn + u * 32);
                bn[u][i] = *reinterpret_cast<const uint4*>(xrow[i] + kn + u * 32);
            }
        __builtin_amdgcn_sched_barrier(0);     // keep the loads ahead of the MFMAs
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
            for (int hs = 0; hs < 4; ++hs)
#pragma unroll
                for (int ts = 0; ts < 4; ++ts)
                    acc[hs][ts] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, a[u][hs]), __builtin_bit_cast(bf16x8, b[u][ts]),
                        acc[hs][ts], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[u][i] = an[u][i];
                b[u][i] = bn[u][i];
            }
    }
    // lane (kc, n) holds hidden units j0 + 16 hs + 4 kc + i of tokens t0 + 16 ts + n
#pragma unroll
    for (int hs = 0; hs < 4; ++hs)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float bias = b1 != nullptr ? b1[j0 + hs * 16 + 4 * kc + i] : 0.f;
#pragma unroll
            for (int ts = 0; ts < 4; ++ts) {
                const float h = acc[hs][ts][i] + bias;
                acc[hs][ts][i] = h / (1.f + __expf(-h));                           // SiLU
            }
        }
    for (int hd = 0; hd < n_kv_heads; ++hd) {
        float w[4][4];
#pragma unroll
        for (int hs = 0; hs < 4; ++hs)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned bits = w2[(size_t)hd * d_hidden + j0 + hs * 16 + 4 * kc + i];
                w[hs][i] = __builtin_bit_cast(float, bits << 16);
            }
#pragma unroll
        for (int ts = 0; ts < 4; ++ts) {
            float p = 0.f;
#pragma unroll
            for (int hs = 0; hs < 4; ++hs)
#pragma unroll
                for (int i = 0; i < 4; ++i) p += w[hs][i] * acc[hs][ts][i];
            p += __shfl_xor(p, 16);
            p += __shfl_xor(p, 32);
            if (kc == 0) s_logit[((size_t)wv * 64 + ts * 16 + n) * n_kv_heads + hd] = p;
        }
    }
    __syncthreads();
    for (int o = tid; o < 64 * n_kv_heads; o += 64 * n_waves) {
        const int tok = o / n_kv_heads, hd = o - tok * n_kv_heads;
        if (t0 + tok >= n_tokens) continue;
        float sum = b2 != nullptr ? b2[hd] : 0.f;
        for (int w8 = 0; w8 < n_waves; ++w8) sum += s_logit[((size_t)w8 * 64 + tok) * n_kv_heads + hd];
        logits[(size_t)(t0 + tok) * n_kv_heads + hd] = sum;
    }
}

// Many tokens, d_hidden <= 256: the operands staged through LDS.  A workgroup takes TT tokens
// and the whole hidden layer (so every token row is fetched once from memory, whatever
// d_hidden is): TT / 64 x NHW waves, each with a 64 x 64 (hidden x token) tile of fp32 sums in
// four MFMA 32x32x16 accumulators.  Blocks of 64 elements of d_model -- 128 bytes of every W1
// row and token row -- are copied straight into LDS, eight lanes per row, two blocks ahead of
// the one in use (ring of three), and a wave waits only for its own copies of the next block,
// not for the newest.  The token rows are copied non-temporal, so that they do not push W1 out of
// the L2 (292 MB come from behind it, of which the tokens are 268; worth 2 % of the time).
// Chunk c (16 bytes) of row r lies at position c ^ ((r >> 1) & 7) of the row: the sixteen rows
// an operand read touches at a time then cover all 64 banks once.
// What bounds it, 32 768 tokens of 4096 -> 256 -> 8: the rows' way into LDS beside the products
// (by counters the matrix units are busy 48 % of the SIMD time; waves wait 26 % of their time for
// copies and the barrier and 44 % for an issue slot).  115 us with 64-token workgroups, two
// stages in LDS and 16x16x32 products, 78 us now.  Stages half as wide and five ahead: 100 us
// (the copies are bound by rows, not by latency).  The epilogue's loads go out together: one by
// one, behind a branch each, they were 9 us of every call.
// Every workgroup takes the blocks of d_model in the same order: equal hidden states have equal logits to the
// last bit wherever they stand in a launch, and copies of a prompt keep the same tokens.  (With blocks in an
// order of its own per workgroup, 32 768 tokens of 4096 with 64 units take 51 us instead of 66: token rows 8 KB apart
// are on few memory channels when all read the same 128 bytes of them.)
// Sums of kGemmFlush stages are added up outside the MFMA accumulators: the relative error
// against 64 bits is 5.7e-8 (one chain over d_model: 1.55e-7) for 2 us.
constexpr int kGemmK = 64;           // elements of d_model per stage
constexpr int kGemmBufs = 3;         // stages in LDS: one in use, two on their way
constexpr int kGemmFlush = 8;        // stages summed in the MFMA accumulators before they are added up
constexpr int kGemmHeads = 32;       // KV heads per pass of the output layer

template <int NHW, int TT>
__global__ __launch_bounds__(TT * NHW) void spkv_predictor_gemm(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w1, const float* __restrict__ b1,
    const uint16_t* __restrict__ w2, const float* __restrict__ b2, float* __restrict__ logits,
    int n_tokens, int d_model, int d_hidden, int n_kv_heads) {
    constexpr int NW = NHW * (TT / 64);                    // waves
    constexpr int kRows = NHW * 64 + TT;                   // rows of a stage: W1 rows, then token rows
    constexpr int kRowBytes = kGemmK * 2, kStageBytes = kRows * kRowBytes;
    constexpr int kCopies = kRows / 8 / NW;                // 1 KB copies (8 rows) per wave and stage
    constexpr int kWCopies = NHW * 8 / NW;                 // of which the first are W1 rows
    static_assert(kRows % (8 * NW) == 0 && NHW * 8 % NW == 0, "whole copies per wave");
    __shared__ __attribute__((aligned(16))) unsigned char s_raw[kGemmBufs * kStageBytes];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, n = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wh = wv % NHW, wt = wv / NHW;                // hidden units 64 wh .., tokens 64 wt ..
    const int t0 = blockIdx.x * TT;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)s_raw;
    const int n_stages = d_model / kGemmK;                 // at least 2 (d_model is a multiple of 128)
    // this wave's copies: rows 8 i .. 8 i + 7 for i = wv, wv + NW, ...  (rows past d_hidden or
    // past the last token repeat the last one; their results are not used)
    const uint16_t* src[kCopies];
#pragma unroll
    for (int u = 0; u < kCopies; ++u) {
        const int r = (wv + u * NW) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        src[u] = (u < kWCopies ? w1 + (size_t)min(r, d_hidden - 1) * d_model
                               : x + (size_t)min(t0 + r - NHW * 64, n_tokens - 1) * d_model) + c * 8;
    }
    // copies u0 .. u1 - 1 of stage st (past the end: the last stage again, never used, so that
    // the count of copies in flight stays the same)
    auto copy_stage = [&](int st, int buf, int u0, int u1) {
        const int k0 = min(st, n_stages - 1) * kGemmK;
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            if (u < u0 || u >= u1) continue;
            const unsigned dst = lds0 + (unsigned)(buf * kStageBytes + (wv + u * NW) * 1024);
            if (u < kWCopies) load_row_to_lds(src[u] + k0, dst);
            else load_row_to_lds_once(src[u] + k0, dst);
        }
    };
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    f32x16 sum[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) sum[i][j] = acc[i][j];
    copy_stage(0, 0, 0, kCopies);
    copy_stage(1, 1, 0, kCopies);
    wait_loads_but<kCopies>();                             // stage 0 has landed
    __syncthreads();
    // byte offsets of this lane's operand rows inside a stage, and their swizzle
    const int ra = (wh * 64 + n) * kRowBytes, rb = (NHW * 64 + wt * 64 + n) * kRowBytes, sw = (n >> 1) & 7;
    bf16x8 a[2][2], b[2][2];
    auto operands = [&](const unsigned char* tile, int u) {
        const int c = ((2 * u + half) ^ sw) << 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[u & 1][i] = *reinterpret_cast<const bf16x8*>(tile + ra + i * 32 * kRowBytes + c);
            b[u & 1][i] = *reinterpret_cast<const bf16x8*>(tile + rb + i * 32 * kRowBytes + c);
        }
    };
    auto products = [&](int u) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u & 1][i], b[u & 1][j], acc[i][j], 0, 0, 0);
    };
    operands(s_raw, 0);
    int buf = 0;
    for (int st = 0; st < n_stages; ++st) {
        const unsigned char* tile = s_raw + buf * kStageBytes;
        const int nbuf = buf >= 1 ? buf - 1 : kGemmBufs - 1;       // stage st + 2 goes where st - 1 was
        buf = buf == kGemmBufs - 1 ? 0 : buf + 1;
        // Four MFMA steps of 16.  The operands of a step are read during the step before it, the
        // next stage's copies go out a third at a time between them (all at once they hold up
        // the waves' own reads), and the barrier stands before the last step, so that the first
        // operands of the next stage are on their way while the last products of this one run.
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            operands(tile, u + 1);
            copy_stage(st + 2, nbuf, u * kCopies / 3, (u + 1) * kCopies / 3);
            products(u);
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_loads_but<kCopies>();                         // all but the newest: stage st + 1 has landed
        __syncthreads();
        operands(s_raw + buf * kStageBytes, 0);
        products(3);
        __builtin_amdgcn_sched_barrier(0);
        if ((st + 1) % kGemmFlush == 0 || st + 1 == n_stages) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    sum[i][j] += acc[i][j];
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
                }
        }
    }
    wait_loads_but<0>();                                   // LDS is written again below
    // lane (half, n) holds hidden units j0 + 32 i + 8 g + 4 half + e (register 4 g + e) of tokens
    // t0 + 64 wt + 32 j + n
    const int j0 = wh * 64;
    float bias[2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {                     // (units past d_hidden: any value)
            const int unit = min(j0 + i * 32 + (r >> 2) * 8 + half * 4 + (r & 3), d_hidden - 1);
            bias[i][r] = b1 != nullptr ? b1[unit] : 0.f;
        }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const bool real = j0 + i * 32 + (r >> 2) * 8 + half * 4 < d_hidden;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float h = sum[i][j][r] + bias[i][r];
                const float act = h / (1.f + __expf(-h));                          // SiLU
                sum[i][j][r] = real ? act : 0.f;
            }
        }
    // Output layer, kGemmHeads heads at a time: their W2 rows go to LDS in one round of loads
    uint16_t* s_w2 = reinterpret_cast<uint16_t*>(s_raw);                           // [heads][NHW * 64]
    float* s_logit = reinterpret_cast<float*>(s_raw + kGemmHeads * NHW * 128);     // [NHW][heads][TT]
    static_assert(kGemmHeads * NHW * 128 + NHW * kGemmHeads * TT * 4 <= kGemmBufs * kStageBytes, "LDS");
    for (int h0 = 0; h0 < n_kv_heads; h0 += kGemmHeads) {
        const int nh = min(kGemmHeads, n_kv_heads - h0);
        __syncthreads();
        for (int e = tid; e < nh * NHW * 32; e += 64 * NW) {       // pairs of hidden units
            const int hd = e / (NHW * 32), u2 = (e - hd * (NHW * 32)) * 2;
            reinterpret_cast<unsigned*>(s_w2)[e] =
                u2 < d_hidden ? *reinterpret_cast<const unsigned*>(w2 + (size_t)(h0 + hd) * d_hidden + u2) : 0u;
        }
        __syncthreads();
        for (int hd = 0; hd < nh; ++hd) {
            float p[2] = {0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {                      // four consecutive hidden units
                    float t[2] = {0.f, 0.f};                       // (short chains: half the rounding error)
                    const uint2 w = *reinterpret_cast<const uint2*>(s_w2 + hd * (NHW * 64) + j0 + i * 32 + g * 8 + half * 4);
                    const float wf[4] = {__builtin_bit_cast(float, w.x << 16), __builtin_bit_cast(float, w.x & 0xffff0000u),
                                         __builtin_bit_cast(float, w.y << 16), __builtin_bit_cast(float, w.y & 0xffff0000u)};
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[j] += wf[e] * sum[i][j][g * 4 + e];
                    p[0] += t[0];
                    p[1] += t[1];
                }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                p[j] += __shfl_xor(p[j], 32);
                if (half == 0) s_logit[(wh * kGemmHeads + hd) * TT + wt * 64 + j * 32 + n] = p[j];
            }
        }
        __syncthreads();
        for (int o = tid; o < TT * nh; o += 64 * NW) {
            const int tok = o / nh, hd = o - tok * nh;
            if (t0 + tok >= n_tokens) continue;
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < NHW; ++w) t += s_logit[(w * kGemmHeads + hd) * TT + tok];
            logits[(size_t)(t0 + tok) * n_kv_heads + h0 + hd] = t + (b2 != nullptr ? b2[h0 + hd] : 0.f);
        }
    }
}

template <int NHW, int TT>
static hipError_t launch_predictor_gemm(const uint16_t* x, const uint16_t* w1, const float* b1,
                                        const uint16_t* w2, const float* b2, float* logits, int n_tokens,
                                        int d_model, int d_hidden, int n_kv_heads, hipStream_t s) {
    spkv_predictor_gemm<NHW, TT><<<dim3((n_tokens + TT - 1) / TT), dim3(TT * NHW), 0, s>>>(
        x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads);
    return hipGetLastError();
}

hipError_t spkv_launch_predictor(const uint16_t* x, const uint16_t* w1, const float* b1,
                                 const uint16_t* w2, const float* b2, float* logits, float* act,
                                 int n_tokens, int d_model, int d_hidden, int n_kv_heads,
                                 hipStream_t s) {
    // The staged kernel takes about the same time for any number of tokens up to a workgroup per
    // compute unit (d_model 1024: 18 us, 4096: 42, 50 with 256 units), the pair of launches below
    // grows with tokens x (units + what reading a token and storing its heads costs, which weighs
    // the more the shorter the rows are).  Pair / staged on either side of the line, us, 8 heads:
    // 4096 tokens of 4096, 16 / 48 units 19 / 33 against 42, 96 units 55 / 42; 6000 of 4096, 32
    // units 36 / 42, 48 units 51 / 42; 4096 of 1024, 32 units 15 / 18, 64 units 20 / 18; 6000 of
    // 1024, 16 units 18 / 17; one head: 12 000 of 4096, 16 units 29 / 40, 32 units 50 / 41.  Up to
    // 512 elements per row one launch is faster because it is one (11 us against 13).
    // 128 tokens per workgroup halve the fetches of W1 once 64 would need a second round (16 384
    // tokens: 58 us with 64 each; 20 000: 65 us with 128, 100 with 64).
    const int64_t units = (int64_t)n_tokens * d_hidden;
    const bool staged = units >= 350000 ||
                        (n_tokens >= 4096 &&
                         (d_model <= 512 ||
                          units * d_model + n_tokens * (4000 + 4500LL * n_kv_heads) >= 300000LL * d_model));
    if (staged && d_hidden <= 256) {
        const bool wide = n_tokens > 16384;
        if (d_hidden <= 64) return wide ? launch_predictor_gemm<1, 128>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s)
                                        : launch_predictor_gemm<1, 64>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s);
        if (d_hidden <= 128) return wide ? launch_predictor_gemm<2, 128>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s)
                                         : launch_predictor_gemm<2, 64>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s);
        return wide ? launch_predictor_gemm<4, 128>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s)
                    : launch_predictor_gemm<4, 64>(x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads, s);
    }
    // Wider hidden layers (up to 512 units): the register-tiled kernel, about 120 us per
    // workgroup for d_model = 4096 (32 768 tokens: 242 us).
    if (n_tokens >= 4096 && d_hidden > 256 && d_hidden % 64 == 0 && d_hidden <= 512 && n_kv_heads <= 64) {
        const int n_waves = d_hidden / 64;
        const size_t lds = (size_t)n_waves * 64 * n_kv_heads * sizeof(float);
        spkv_predictor_tiled<<<dim3((n_tokens + 63) / 64), dim3(64 * n_waves), lds, s>>>(
            x, w1, b1, w2, b2, logits, n_tokens, d_model, d_hidden, n_kv_heads);
        return hipGetLastError();
    }
    spkv_predictor_hidden<<<dim3(d_hidden / 16, (n_tokens + 15) / 16), dim3(256), 0, s>>>(
        x, w1, b1, act, n_tokens, d_model, d_hidden);
    spkv_predictor_out<<<dim3(n_tokens * n_kv_heads), dim3(64), 0, s>>>(act, w2, b2, logits, d_hidden,
                                                                        n_kv_heads);
    return hipGetLastError();
}

