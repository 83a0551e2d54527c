// K2 (canonical): the reward model's chains on the matrix cores, for one to three
// hidden layers of one width (64, 128 or 256).
//
// The canonical score of a pair (Section 4.1, the batched forward of Alg. 4) is
// a fixed sequence of fmaf roundings: layer 1 resumed from the instance partial
// over the five request/pair columns, each unit of a later layer from its bias
// over the activations before it in ascending order, the head from its bias over
// the last activations in ascending order (the chains of canonical_score).  The fp32
// matrix-core instruction v_mfma_f32_32x32x1_2b_f32 takes one input k per
// instruction and rounds each of its multiply-adds once, exactly as fmaf does
// (denormals kept), so stepping k in the chain's order reproduces every chain
// bit for bit: these scores equal the vector-ALU scorer's.
//
// A workgroup of H / 64 waves scores 32 pairs; wave p has the units 64 p ..
// 64 p + 63 of each layer.  Both blocks of an instruction hold the same 32 pairs
// (columns) and together the wave's units (rows): lane l gives the A operand of
// unit 64 p + l, and lanes l and l + 32 give the same pair's B operand.
// Accumulator register i of lane l then holds unit
// 64 p + 32 (i / 16) + 8 (i % 16 / 4) + 4 (l / 32) + i % 4, pair l % 32.
//   layer 1: the accumulators start at the instance partials; five steps with
//            A = W1's column for that derived input, B = the pair's input;
//            ReLU (and bf16 rounding) into the workgroup's LDS tile [pair][k];
//   others:  accumulators from the bias; per k one coalesced 256-byte read of the
//            wave's part of W^T row k (A, held eight k ahead) and one LDS read of
//            four k of the pair's activations (B); ReLU (and bf16 rounding) into
//            the tile once every wave has read it;
//   head:    a lane per pair runs the chain over the tile's row.
// What bounds it is the fp32 matrix rate, 64 cycles per instruction.  A wave per
// 32 pairs with all of a layer in its registers leaves one wave per SIMD at
// H = 256, whose loads and epilogues nothing covers; split, four share a SIMD,
// and a few pairs (a small batch, the band) finish in a quarter of the chain.
// 524,288 pairs of two layers of 256: 749 us with a wave per 32 pairs, 857 with a
// group of 32 a workgroup (a load per matrix instruction keeps the address unit
// as busy as the matrix cores), 725 with two groups.  256 listed pairs: 44 and 21.
// 60,000 pairs of three layers of 128: 110 layer by layer, 56 here.
#include <type_traits>

#include "k_common.h"

namespace ls {

namespace {

typedef float f32x32_t __attribute__((ext_vector_type(32)));

constexpr int kChainPairs = 32;   // pairs per group (a workgroup has one or two)

struct ChainModel {
    const float* w1t;             // [d][H]
    const float* wt[2];           // later hidden layers, [H][H] (input-major)
    const float* b[2];
    const float *wh, *bh;         // head
    int d_inst, mids;             // mids: hidden layers after the first
};

// LDS row stride of the activation tile: h1 rounded to 4, plus 4 when that is a
// multiple of 8 (16-byte reads of 32 rows without bank conflicts).
__host__ __device__ constexpr int chain_ldh(int h1) { return ((h1 + 3) & ~3) + ((((h1 + 3) >> 2) & 1) ? 0 : 4); }

template <bool BF>
__device__ __forceinline__ float act(float z) {
    const float a = relu(z);
    return BF ? bf16_rne_num(a) : a;
}

}  // namespace

// LIST: score the pairs list[0 .. *count) (pair indices r * N + i), with
// persistent workgroups that take 32 NG list entries at a time; otherwise every
// pair, 32 NG per workgroup (more than chain_groups() launches: in turns).
template <bool BF, int H, int NG, bool LIST>
__device__ __forceinline__ void chain_body(const ChainModel& M, const float* __restrict__ mu,
                                           const float* __restrict__ isig, const float* __restrict__ part_t,
                                           int32_t R, int32_t N, const int64_t* __restrict__ req_off,
                                           const int32_t* __restrict__ prompt_len,
                                           const int32_t* __restrict__ overlap, int block_tokens,
                                           const int64_t* __restrict__ list, const uint32_t* __restrict__ count,
                                           float* __restrict__ scores) {
    static_assert(H % 64 == 0 && H <= 256, "a wave per 64 units");
    constexpr int LDH = chain_ldh(H);
    constexpr int NP = NG * kChainPairs;
    extern __shared__ __align__(16) float hl[];          // [NP][LDH]
    const int lane = threadIdx.x & 63, col = lane & 31, hi = lane >> 5;
    const int u0 = 64 * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // the wave's first unit
    const int64_t cnt = LIST ? (int64_t)*count : (int64_t)R * N;
    float* __restrict__ row = hl + col * LDH;                          // group n's: row + n * 32 LDH
    const int64_t turn = (int64_t)gridDim.x * NP;
    for (int64_t e0 = (int64_t)blockIdx.x * NP; e0 < cnt; e0 += turn) {
        float xt[NG][5];
        int32_t inst[NG];
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            const int64_t e = e0 + 32 * n + col < cnt ? e0 + 32 * n + col : cnt - 1;   // past the end: a valid pair
            const int64_t q = LIST ? list[e] : e;
            const int64_t r = q / N;
            inst[n] = (int32_t)(q - r * N);
            float x[5];
            derived_columns(prompt_len[r], req_off[r + 1] - req_off[r], overlap[q], block_tokens, x);
            normalise_tail<BF>(x, mu, isig, M.d_inst, xt[n]);
        }
        // this lane's g-th four consecutive units
        auto unit4 = [&](int g) { return u0 + 32 * (g >> 2) + 8 * (g & 3) + 4 * hi; };
        f32x32_t acc[NG];
        auto store = [&]() {
#pragma unroll
            for (int n = 0; n < NG; ++n)
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    *reinterpret_cast<float4*>(row + n * kChainPairs * LDH + unit4(g)) =
                        make_float4(act<BF>(acc[n][4 * g]), act<BF>(acc[n][4 * g + 1]), act<BF>(acc[n][4 * g + 2]),
                                    act<BF>(acc[n][4 * g + 3]));
        };
        // a layer's first weights go out before the layer ahead of it is done
        constexpr int G = 8;                                           // inputs per group
        const float* __restrict__ wt = nullptr;                        // W^T[k][u0 + lane] = wt[k * H]
        auto load = [&](float (&w)[G], int k0) {
#pragma unroll
            for (int g = 0; g < G; ++g) w[g] = wt[(int64_t)(k0 + g) * H];
        };
        float wa[G], wb[G];
        if (M.mids > 0) {
            wt = M.wt[0] + u0 + lane;
            load(wa, 0);
        }
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int i = 0; i < 32; ++i)
                acc[n][i] = part_t[(uint32_t)(unit4(i >> 2) + (i & 3)) * (uint32_t)N + (uint32_t)inst[n]];
        {
            const float* __restrict__ w1 = M.w1t + (int64_t)M.d_inst * H + u0 + lane;
            float a[5];
#pragma unroll
            for (int c = 0; c < 5; ++c) a[c] = w1[c * H];
#pragma unroll
            for (int c = 0; c < 5; ++c)
#pragma unroll
                for (int n = 0; n < NG; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x1f32(a[c], xt[n][c], acc[n], 0, 0, 0);
        }
        store();
        auto step = [&](const float (&w)[G], int k0) {
            float4 b[NG][G / 4];
#pragma unroll
            for (int n = 0; n < NG; ++n)
#pragma unroll
                for (int g = 0; g < G / 4; ++g)
                    b[n][g] = *reinterpret_cast<const float4*>(row + n * kChainPairs * LDH + k0 + 4 * g);
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int n = 0; n < NG; ++n) {
                    const float4 v = b[n][k >> 2];
                    const float bv = (k & 3) == 0 ? v.x : (k & 3) == 1 ? v.y : (k & 3) == 2 ? v.z : v.w;
                    acc[n] = __builtin_amdgcn_mfma_f32_32x32x1f32(w[k], bv, acc[n], 0, 0, 0);
                }
        };
        static_assert(H % (2 * G) == 0, "whole double groups");
#pragma unroll 1
        for (int l = 0; l < M.mids; ++l) {
            const float* __restrict__ bias = M.b[l];
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const float v = bias[unit4(i >> 2) + (i & 3)];
#pragma unroll
                for (int n = 0; n < NG; ++n) acc[n][i] = v;
            }
            __syncthreads();
#pragma unroll 1
            for (int k0 = 0; k0 < H; k0 += 2 * G) {
                load(wb, k0 + G);
                step(wa, k0);
                if (k0 + 2 * G < H) load(wa, k0 + 2 * G);
                step(wb, k0 + G);
            }
            if (l + 1 < M.mids) {
                wt = M.wt[l + 1] + u0 + lane;
                load(wa, 0);
            }
            __syncthreads();
            store();
        }
        __syncthreads();
        // head: units in ascending order
        if (threadIdx.x < NP && e0 + (int)threadIdx.x < cnt) {
            const float* __restrict__ h = hl + (int)threadIdx.x * LDH;
            float t = M.bh[0];
#pragma unroll 4
            for (int u = 0; u < H; u += 4) {
                const float4 v = *reinterpret_cast<const float4*>(h + u);
                t = __builtin_fmaf(M.wh[u], v.x, t);
                t = __builtin_fmaf(M.wh[u + 1], v.y, t);
                t = __builtin_fmaf(M.wh[u + 2], v.z, t);
                t = __builtin_fmaf(M.wh[u + 3], v.w, t);
            }
            const int64_t e = e0 + (int)threadIdx.x;
            scores[LIST ? list[e] : e] = t;
        }
        if (e0 + turn < cnt) __syncthreads();                          // the tile is the next group's
    }
}

// Every pair, 32 NG per workgroup.
template <bool BF, int H, int NG>
__global__ __launch_bounds__(H) __attribute__((amdgpu_waves_per_eu(4 / NG))) void score_chain_mfma_kernel(
    ChainModel M, const float* __restrict__ mu, const float* __restrict__ isig, const float* __restrict__ part_t,
    int32_t R, int32_t N, const int64_t* __restrict__ req_off, const int32_t* __restrict__ prompt_len,
    const int32_t* __restrict__ overlap, int block_tokens, float* __restrict__ scores) {
    chain_body<BF, H, NG, false>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, nullptr, nullptr,
                             scores);
}

// The candidate band's rescoring (bf16 models of two layers of 256): the pairs
// list[0 .. *count), persistent workgroups.
template <int H, int NG>
__global__ __launch_bounds__(H) __attribute__((amdgpu_waves_per_eu(4 / NG))) void rescore_chain_mfma_kernel(
    ChainModel M, const float* __restrict__ mu, const float* __restrict__ isig, const float* __restrict__ part_t,
    int32_t R, int32_t N, const int64_t* __restrict__ req_off, const int32_t* __restrict__ prompt_len,
    const int32_t* __restrict__ overlap, int block_tokens, const int64_t* __restrict__ list,
    const uint32_t* __restrict__ count, float* __restrict__ scores) {
    chain_body<true, H, NG, true>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, list, count, scores);
}

// Two layers of up to 128 units: a wave scores 32 pairs by itself, with all of
// layer 2's passes in its accumulators and the head in lanes 0-31, which take
// units 4-7 of every 8 from lanes 32-63 by a lane shuffle.  No barriers; the tile
// leaves LDS for two waves per SIMD and the kernels hold their registers to that.
// (131,072 pairs of h = 128: 62.5 us; a workgroup of two waves 67.6.  Small
// batches and short lists were not compared.)
template <bool BF, int H1, int H2, bool LIST>
__device__ __forceinline__ void wave_body(const PairModel& M, const float* __restrict__ mu,
                                           const float* __restrict__ isig, const float* __restrict__ part_t,
                                           int32_t R, int32_t N, const int64_t* __restrict__ req_off,
                                           const int32_t* __restrict__ prompt_len,
                                           const int32_t* __restrict__ overlap, int block_tokens,
                                           const int64_t* __restrict__ list, const uint32_t* __restrict__ count,
                                           float* __restrict__ scores) {
    static_assert(H1 % 64 == 0 && H2 % 64 == 0 && H1 <= 128 && H2 <= 128, "64-unit passes");
    constexpr int P1 = H1 / 64, P2 = H2 / 64, LDH = chain_ldh(H1);
    extern __shared__ __align__(16) float hl[];          // [kChainPairs][LDH]
    const int lane = threadIdx.x, col = lane & 31, hi = lane >> 5;
    const int64_t cnt = LIST ? (int64_t)*count : (int64_t)R * N;
    for (int64_t e0 = (int64_t)blockIdx.x * kChainPairs; e0 < cnt; e0 += (int64_t)gridDim.x * kChainPairs) {
    // the model's bases, opaque to the optimiser: their loads stay inside the
    // loop instead of holding b2, w3, W1 columns, W2T rows and partial addresses
    // in registers across tasks
    // (an opaque zero offset: the pointers keep their global address space)
    uint32_t z0 = 0;
    asm volatile("" : "+s"(z0));
    const float *w1b = M.w1 + z0, *w2b = M.w2t + z0, *b2b = M.b2 + z0, *w3b = M.w3 + z0, *ptb = part_t + z0;
    const uint32_t Nb = (uint32_t)N + z0;
    const int64_t e = e0 + col < cnt ? e0 + col : cnt - 1;       // lanes past the end score a valid pair
    const int64_t q = LIST ? list[e] : e;
    const int64_t r = q / N;
    const int32_t inst = (int32_t)(q - r * N);
    float x[5], xt[5];
    derived_columns(prompt_len[r], req_off[r + 1] - req_off[r], overlap[q], block_tokens, x);
    normalise_tail<BF>(x, mu, isig, M.d_inst, xt);

    // layer 1, one 64-unit pass at a time, into the activation tile
    float* __restrict__ row = hl + col * LDH;
#pragma unroll
    for (int p = 0; p < P1; ++p) {
        f32x32_t acc;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int u = 64 * p + 32 * (i >> 4) + 8 * ((i & 15) >> 2) + 4 * hi + (i & 3);
            acc[i] = ptb[(uint32_t)u * Nb + (uint32_t)inst];
        }
        const float* __restrict__ w1 = w1b + (int64_t)(64 * p + lane) * M.d + M.d_inst;
        float a[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) a[c] = w1[c];
#pragma unroll
        for (int c = 0; c < 5; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x1f32(a[c], xt[c], acc, 0, 0, 0);
#pragma unroll
        for (int g = 0; g < 8; ++g) {          // registers 4 g .. 4 g + 3: four consecutive units
            const int u = 64 * p + 32 * (g >> 2) + 8 * (g & 3) + 4 * hi;
            *reinterpret_cast<float4*>(row + u) =
                make_float4(act<BF>(acc[4 * g]), act<BF>(acc[4 * g + 1]), act<BF>(acc[4 * g + 2]),
                            act<BF>(acc[4 * g + 3]));
        }
    }

    // layer 2: every pass at once
    f32x32_t acc[P2];
#pragma unroll
    for (int p = 0; p < P2; ++p)
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[p][i] = b2b[64 * p + 32 * (i >> 4) + 8 * ((i & 15) >> 2) + 4 * hi + (i & 3)];
    const float* __restrict__ w2 = w2b + lane;              // W2T[k][64 p + lane] = w2[k * H2 + 64 p]
    constexpr int G = 8;                                    // inputs per group
    auto load = [&](float (&w)[G][P2], int k0) {
#pragma unroll
        for (int e = 0; e < G; ++e)
#pragma unroll
            for (int p = 0; p < P2; ++p) w[e][p] = w2[(int64_t)(k0 + e) * H2 + 64 * p];
    };
    auto step = [&](const float (&w)[G][P2], int k0) {
        float4 b[G / 4];
#pragma unroll
        for (int g = 0; g < G / 4; ++g) b[g] = *reinterpret_cast<const float4*>(row + k0 + 4 * g);
#pragma unroll
        for (int e = 0; e < G; ++e) {
            const float4 v = b[e >> 2];
            const float bv = (e & 3) == 0 ? v.x : (e & 3) == 1 ? v.y : (e & 3) == 2 ? v.z : v.w;
#pragma unroll
            for (int p = 0; p < P2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x1f32(w[e][p], bv, acc[p], 0, 0, 0);
        }
    };
    static_assert(H1 % (2 * G) == 0, "whole double groups");
    float wa[G][P2], wb[G][P2];
    load(wa, 0);
#pragma unroll 1
    for (int k0 = 0; k0 < H1; k0 += 2 * G) {
        load(wb, k0 + G);
        step(wa, k0);
        if (k0 + 2 * G < H1) load(wa, k0 + 2 * G);
        step(wb, k0 + G);
    }

    // head: units in ascending order; lanes 0-31 hold units 0-3 of every 8, and
    // take units 4-7 from lanes 32-63
    float t = M.b3[0];
#pragma unroll
    for (int p = 0; p < P2; ++p)
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int u = 64 * p + 32 * (g >> 2) + 8 * (g & 3);
            float lo[4], up[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float h = act<BF>(acc[p][4 * g + e]);
                lo[e] = h;
                up[e] = __shfl_xor(h, 32);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) t = __builtin_fmaf(w3b[u + e], lo[e], t);
#pragma unroll
            for (int e = 0; e < 4; ++e) t = __builtin_fmaf(w3b[u + 4 + e], up[e], t);
        }
    if (hi == 0 && e0 + col < cnt) scores[q] = t;
    }
}

// Every pair, one group of 32 per workgroup.
template <bool BF, int H1, int H2>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void score_wave_mfma_kernel(
    PairModel M, const float* __restrict__ mu, const float* __restrict__ isig, const float* __restrict__ part_t,
    int32_t R, int32_t N, const int64_t* __restrict__ req_off, const int32_t* __restrict__ prompt_len,
    const int32_t* __restrict__ overlap, int block_tokens, float* __restrict__ scores) {
    wave_body<BF, H1, H2, false>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, nullptr,
                                  nullptr, scores);
}

// The candidate band's rescoring (bf16 models): the pairs list[0 .. *count), persistent waves.
template <int H1, int H2>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void rescore_wave_mfma_kernel(
    PairModel M, const float* __restrict__ mu, const float* __restrict__ isig, const float* __restrict__ part_t,
    int32_t R, int32_t N, const int64_t* __restrict__ req_off, const int32_t* __restrict__ prompt_len,
    const int32_t* __restrict__ overlap, int block_tokens, const int64_t* __restrict__ list,
    const uint32_t* __restrict__ count, float* __restrict__ scores) {
    wave_body<true, H1, H2, true>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, list, count,
                                 scores);
}

uint32_t chain_groups(int64_t pairs, int per_group, int threads) {
    const int64_t want = (pairs + per_group - 1) / per_group, most = (int64_t)UINT32_MAX / threads;
    return (uint32_t)(want < most ? want : most);
}

namespace {

template <bool BF, int H, int NG>
hipError_t launch_chain(const ChainModel& M, const float* mu, const float* isig, const float* part_t, int32_t R,
                        int32_t N, const int64_t* req_off, const int32_t* prompt_len, const int32_t* overlap,
                        int block_tokens, const int64_t* list, const uint32_t* count, int n_cu, float* scores,
                        hipStream_t s) {
    const size_t lds = sizeof(float) * NG * kChainPairs * chain_ldh(H);
    if (list) {
        // persistent: as many workgroups as fill every CU with four waves a SIMD and as its LDS holds
        const int fit = (int)((160u << 10) / lds), per_cu = fit < 1024 / H ? fit : 1024 / H;
        if constexpr (BF && H == 256)
            hipLaunchKernelGGL((rescore_chain_mfma_kernel<H, NG>), dim3((uint32_t)(n_cu * per_cu)), dim3(H), lds, s, M,
                               mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, list, count, scores);
        else
            return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((score_chain_mfma_kernel<BF, H, NG>),
                           dim3(chain_groups((int64_t)R * N, NG * kChainPairs, H)), dim3(H), lds, s, M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, scores);
    }
    return hipGetLastError();
}

template <bool BF, int H1, int H2>
hipError_t launch_wave(const PairModel& M, const float* mu, const float* isig, const float* part_t, int32_t R,
                        int32_t N, const int64_t* req_off, const int32_t* prompt_len, const int32_t* overlap,
                        int block_tokens, const int64_t* list, const uint32_t* count, int n_cu, float* scores,
                        hipStream_t s) {
    const size_t lds = sizeof(float) * kChainPairs * chain_ldh(H1);
    if (list) {
        // persistent: as many single-wave workgroups as the LDS lets every CU hold
        const int per_cu = (int)((160u << 10) / lds) < 8 ? (int)((160u << 10) / lds) : 8;
        if constexpr (BF)
            hipLaunchKernelGGL((rescore_wave_mfma_kernel<H1, H2>), dim3((uint32_t)(n_cu * per_cu)), dim3(64), lds, s, M,
                               mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, list, count, scores);
        else
            return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((score_wave_mfma_kernel<BF, H1, H2>),
                           dim3(chain_groups((int64_t)R * N, kChainPairs, 64)), dim3(64), lds, s, M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, block_tokens, scores);
    }
    return hipGetLastError();
}

template <bool BF>
hipError_t dispatch_chain(const ModelDims& m, const ChainModel& M, const float* mu, const float* isig,
                          const float* part_t, int32_t R, int32_t N, const int64_t* req_off, const int32_t* prompt_len,
                          const int32_t* overlap, const int64_t* list, const uint32_t* count, int n_cu, float* scores,
                          hipStream_t s) {
    const int bt = m.block_tokens;
    // two groups a workgroup share each weight read, once they leave every CU two workgroups; fewer pairs spread out
    // (a list holds about R pairs)
    const bool two = (list ? (int64_t)R : (int64_t)R * N) >= (int64_t)n_cu * 128;
    if (m.h[0] == 64)
        return two ? launch_chain<BF, 64, 2>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                             scores, s)
                   : launch_chain<BF, 64, 1>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                             scores, s);
    if (m.h[0] == 128)
        return two ? launch_chain<BF, 128, 2>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                             scores, s)
                   : launch_chain<BF, 128, 1>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                             scores, s);
    return two ? launch_chain<BF, 256, 2>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                         scores, s)
               : launch_chain<BF, 256, 1>(M, mu, isig, part_t, R, N, req_off, prompt_len, overlap, bt, list, count, n_cu,
                                         scores, s);
}

}  // namespace

bool chain_mfma_supported(const ModelDims& m) {
    for (int l = 1; l < m.L; ++l)
        if (m.h[l] != m.h[0]) return false;
    return m.d == m.d_inst + 5 && (m.h[0] == 64 || m.h[0] == 128 || m.h[0] == 256);
}

// The kernels index the instance partials [h][N] in 32 bits.
bool chain_scores(const ModelDims& m, int32_t N) {
    return m.mfma_chains && chain_mfma_supported(m) && (int64_t)m.h[0] * N <= (int64_t)UINT32_MAX + 1;
}

bool scores_by_layer(const ModelDims& m, int32_t N) { return m.L != 2 && !chain_scores(m, N); }

hipError_t launch_score_chain_mfma(const ModelDims& m, const float* compute, const float* mu, const float* inv_sigma,
                                   const float* part_t, int32_t R, int32_t N, const int64_t* req_off,
                                   const int32_t* prompt_len, const int32_t* overlap, const int64_t* list,
                                   const uint32_t* count, int n_cu, float* scores, hipStream_t s) {
    if ((int64_t)R * N <= 0) return hipSuccess;
    if (!chain_scores(m, N) || (list == nullptr) != (count == nullptr)) return hipErrorInvalidValue;
    ChainModel M{};
    M.w1t = compute + m.c_wt[0];
    M.mids = m.L - 1;
    for (int l = 1; l < m.L; ++l) {
        M.wt[l - 1] = compute + m.c_wt[l];
        M.b[l - 1] = compute + m.c_bl[l];
    }
    M.wh = compute + m.c_wt[m.L];
    M.bh = compute + m.c_bl[m.L];
    M.d_inst = m.d_inst;
    if (m.L == 2 && m.h[0] <= 128) {
        const PairModel W{compute + m.c_w1, compute + m.c_w2t, compute + m.c_b2, compute + m.c_w3, compute + m.c_b3,
                          m.d, m.d_inst, m.h1, m.h2};
        auto wave = [&](auto bf) {
            constexpr bool BF = decltype(bf)::value;
            return m.h1 == 64 ? launch_wave<BF, 64, 64>(W, mu, inv_sigma, part_t, R, N, req_off, prompt_len, overlap,
                                                        m.block_tokens, list, count, n_cu, scores, s)
                              : launch_wave<BF, 128, 128>(W, mu, inv_sigma, part_t, R, N, req_off, prompt_len, overlap,
                                                          m.block_tokens, list, count, n_cu, scores, s);
        };
        return m.bf16 ? wave(std::true_type{}) : wave(std::false_type{});
    }
    if (m.bf16)
        return dispatch_chain<true>(m, M, mu, inv_sigma, part_t, R, N, req_off, prompt_len, overlap, list, count, n_cu,
                                    scores, s);
    return dispatch_chain<false>(m, M, mu, inv_sigma, part_t, R, N, req_off, prompt_len, overlap, list, count, n_cu,
                                 scores, s);
}

}  // namespace ls
