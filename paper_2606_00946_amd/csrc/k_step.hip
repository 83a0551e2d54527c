// K4 for small batches: one SGD step in two launches (Section 4.3.2, the
// minibatches of a retraining round and updates on few logged samples).
//
// At a few hundred samples the step's work is small and what costs is the chain
// of dependent launches: the layer-by-layer step runs 20 to 27 kernels of 2 to
// 15 us each.  Here
//   step_rows     takes a few samples per workgroup through the whole network,
//                 forward and back: normalisation, every layer, the loss
//                 gradient, every hidden layer's gradient.  Activations stay in
//                 LDS; the weights stream from L2, each read once per workgroup
//                 and layer; what the weight gradients need goes to memory
//                 sample-major.
//   step_weights  takes a 16 x 16 tile of one layer's weights per workgroup: the
//                 gradient as fp32 matrix-core products over the samples, then
//                 the SGD step of that tile's masters and compute copies.
// The forward and the hidden gradients are the canonical chains (bias or zero
// first, inputs ascending, one fmaf each) in the order of the layer-by-layer
// kernels, so their values are the same to the bit; only the sums over the
// batch (weight gradients, loss) have an order of their own, fixed by B, the loss
// and the bias gradients in 64 bits.
//
// Measured (us per step, before -> now): 3 x 128 fp32 with dropout 135 -> 22 at
// B = 256, 169 -> 29 at 1,000, 341 -> 83 at 8,192; 64-256-256 bf16 119 -> 30, 174
// -> 41 and 166 -> 139.  step_rows is 18 of the 22 us.
#include <algorithm>

#include "k_policy.h"

namespace ls {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kStepWidth = 256;               // widest layer (inputs and units)
constexpr int kStepRow = kStepWidth + 4;      // LDS row of one sample's activations

struct StepLayer {
    int in, out;
    int64_t mw, mb, wt, bl;                   // masters W [out][in] and b, compute copy W^T [in][out] and b
    float *a, *dl;                            // sample-major [B][out]
};

struct StepArgs {
    int L, d, B, hl;
    StepLayer layer[4];                       // the hidden layers, then the head
    int64_t c_w1;                             // row-major first layer of two-layer compute copies, or -1
    int n_master, n_compute;                  // floats
    const float* mu;
    const float* isig;
    float* master;
    float* compute;
    const int32_t* code;                      // row b: ax/ay row code[b], or bx/by row -code[b] - 1; null: ax/ay row b
    const float *ax, *ay, *bx, *by;
    float* xn;                                // sample-major [B][d]
    float *g, *e2;                            // [B]
    float lr;
    float* grad_out;
    float* loss_out;                          // mean squared error of this step, or null
    double* acc;                              // running sum of step losses, or null
    int acc_reset;                            // the sum starts with this step
    DropArgs D;
};

__device__ __forceinline__ float step_drop(const DropArgs& D, int layer, int64_t b, int j, float v) {
    if (D.thr53 == 0) return v;
    const uint64_t c = ((((D.step * 4u + (uint64_t)layer) << 24) | (uint64_t)b) << 10) | (uint64_t)j;
    const bool drop = (mix64(D.seed + (c + 1u) * 0x9e3779b97f4a7c15ull) >> 11) < D.thr53;
    return drop ? 0.0f : __fmul_rn(v, D.scale);
}

// SP fma chains over inputs 0 .. K - 1 in ascending order, all with the same
// weights w[k * ld] (rounded to bf16 first where QW: masters), inputs from LDS
// rows xs + i * kStepRow (one address across the wave: broadcasts), the weights
// a group of kStepPre inputs ahead.  What bounds it at small batches is the rate
// at which a CU takes a wave's addresses, about 16 cycles per load of one word a
// lane (55 cycles per input with four waves).  Where a thread has one sample the
// group is 32 inputs, else 16.  Tried and no better: a ring of 64 ahead that runs
// on over the stages, immediate row offsets, and the weights through LDS in 64 KB
// chunks of 16-byte loads (21 cycles per input, but 3,000 per chunk to fetch and
// store it; 118 against 83 us a step at 8,192).
template <bool QW, int SP, int kStepPre>
__device__ __forceinline__ void step_chain(float (&acc)[SP], const float* __restrict__ w, int64_t ld, int K,
                                           const float* xs) {
    float wa[kStepPre], wb[kStepPre];
    auto load = [&](float (&q)[kStepPre], int k0) {
#pragma unroll
        for (int e = 0; e < kStepPre; ++e) q[e] = w[(int64_t)(k0 + e < K ? k0 + e : K - 1) * ld];
    };
    auto full = [&](const float (&q)[kStepPre], int k0) {
#pragma unroll
        for (int e = 0; e < kStepPre; e += 4) {
            float4 x[SP];
#pragma unroll
            for (int i = 0; i < SP; ++i) x[i] = *reinterpret_cast<const float4*>(xs + i * kStepRow + k0 + e);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float wv = QW ? bf16_rne(q[e + j]) : q[e + j];
#pragma unroll
                for (int i = 0; i < SP; ++i) {
                    const float xv = j == 0 ? x[i].x : j == 1 ? x[i].y : j == 2 ? x[i].z : x[i].w;
                    acc[i] = __builtin_fmaf(wv, xv, acc[i]);
                }
            }
        }
    };
    auto tail = [&](const float (&q)[kStepPre], int k0) {
#pragma unroll
        for (int e = 0; e < kStepPre; ++e) {
            if (k0 + e >= K) break;
            const float wv = QW ? bf16_rne(q[e]) : q[e];
#pragma unroll
            for (int i = 0; i < SP; ++i) acc[i] = __builtin_fmaf(wv, xs[i * kStepRow + k0 + e], acc[i]);
        }
    };
    load(wa, 0);
    int k0 = 0;
    for (; k0 + 2 * kStepPre <= K; k0 += 2 * kStepPre) {
        load(wb, k0 + kStepPre);
        full(wa, k0);
        load(wa, k0 + 2 * kStepPre);
        full(wb, k0 + kStepPre);
    }
    if (k0 < K) {
        load(wb, k0 + kStepPre);
        if (k0 + kStepPre <= K) full(wa, k0);
        else tail(wa, k0);
        tail(wb, k0 + kStepPre);
    }
}

// G groups of T / G threads; a thread is unit (tid % (T / G)) of its group's SP
// samples, so a workgroup takes G * SP samples.
template <bool BF, int T, int G, int SP, int PRE>
__global__ __launch_bounds__(T) void step_rows_kernel(StepArgs P) {
    constexpr int W = T / G, S = G * SP;
    __shared__ __align__(16) float xs[2][S * kStepRow];
    __shared__ float gs[S];
    __shared__ __align__(16) float w3[kStepWidth];
    const int tid = (int)threadIdx.x, unit = tid % W, grp = tid / W;
    const int64_t b0 = (int64_t)blockIdx.x * S;
    // Every XCD's L2 starts a step without the weights, which the last step's tiles left in memory: a workgroup reads
    // one word of each 128-byte line of its share of them, an eighth of the workgroups (consecutive ones go to
    // different XCDs) taking all (25.1 -> 24.0 us a step at B = 256 of 3 x 128, 29.9 -> 29.1 at 1,000).
    uint32_t touched = 0;
    {
        const int share = (int)(gridDim.x + 7) / 8, mine = (int)blockIdx.x / 8;
        const int lc = (P.n_compute + 31) / 32, lines = lc + (P.n_master + 31) / 32;
#pragma unroll 4
        for (int q = mine * T + tid; q < lines; q += share * T)
            touched |= __float_as_uint(q < lc ? P.compute[32 * q] : P.master[32 * (q - lc)]);
    }
    for (int e = tid; e < S * P.d; e += T) {
        const int i = e / P.d, c = e - i * P.d;
        const int64_t b = b0 + i;
        float v = 0.0f;
        if (b < P.B) {
            const int32_t code = P.code ? P.code[b] : (int32_t)b;
            const float raw = code >= 0 ? P.ax[(int64_t)code * P.d + c] : P.bx[(-(int64_t)code - 1) * P.d + c];
            v = __fmul_rn(__fsub_rn(raw, P.mu[c]), P.isig[c]);
            if (BF) v = bf16_rne(v);
            P.xn[b * P.d + c] = v;
        }
        xs[0][i * kStepRow + c] = v;
    }
    for (int k = tid; k < P.hl; k += T) w3[k] = P.compute[P.layer[P.L].wt + k];
    asm volatile("" ::"v"(touched));
    __syncthreads();
    // forward; bit i of mask[l]: this thread's unit of sample i is on (z > 0)
    uint32_t mask[3] = {0u, 0u, 0u};
    int cur = 0;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        if (l >= P.L) break;
        const int K = P.layer[l].in, O = P.layer[l].out;
        const int o = unit < O ? unit : O - 1;
        float acc[SP];
        const float bias = P.compute[P.layer[l].bl + o];
#pragma unroll
        for (int i = 0; i < SP; ++i) acc[i] = bias;
        step_chain<false, SP, PRE>(acc, P.compute + P.layer[l].wt + o, O, K, xs[cur] + grp * SP * kStepRow);
        if (unit < O) {
#pragma unroll
            for (int i = 0; i < SP; ++i) {
                const int64_t b = b0 + grp * SP + i;
                if (acc[i] > 0.0f) mask[l] |= 1u << i;
                float v = step_drop(P.D, l, b, unit, relu(acc[i]));
                if (BF) v = bf16_rne(v);
                xs[cur ^ 1][(grp * SP + i) * kStepRow + unit] = v;
                if (b < P.B) P.layer[l].a[b * O + unit] = v;
            }
        }
        cur ^= 1;
        __syncthreads();
    }
    // head, loss and its gradient: a lane per sample
    if (tid < S) {
        const int64_t b = b0 + tid;
        float t = P.compute[P.layer[P.L].bl];
        const float* x = xs[cur] + tid * kStepRow;
        int k = 0;
        for (; k + 16 <= P.hl; k += 16) {
            float4 xv[4], wv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                xv[e] = *reinterpret_cast<const float4*>(x + k + 4 * e);
                wv[e] = *reinterpret_cast<const float4*>(w3 + k + 4 * e);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t = __builtin_fmaf(wv[e].x, xv[e].x, t);
                t = __builtin_fmaf(wv[e].y, xv[e].y, t);
                t = __builtin_fmaf(wv[e].z, xv[e].z, t);
                t = __builtin_fmaf(wv[e].w, xv[e].w, t);
            }
        }
        for (; k < P.hl; ++k) t = __builtin_fmaf(w3[k], x[k], t);
        float gv = 0.0f;
        if (b < P.B) {
            const int32_t code = P.code ? P.code[b] : (int32_t)b;
            const float y = code >= 0 ? P.ay[code] : P.by[-(int64_t)code - 1];
            const float err = t - y;
            gv = (2.0f * err) / (float)P.B;
            if (BF) gv = bf16_rne(gv);
            P.g[b] = gv;
            P.e2[b] = err * err;
        }
        gs[tid] = gv;
    }
    __syncthreads();
    // backward: the last hidden layer from the head, the others through W^T
    // (masters, row-major: consecutive threads read consecutive inputs)
#pragma unroll
    for (int l = 2; l >= 0; --l) {
        if (l >= P.L) continue;
        const int O = P.layer[l].out;
        float v[SP];
        if (l == P.L - 1) {
            const float wj = w3[unit < O ? unit : 0];
#pragma unroll
            for (int i = 0; i < SP; ++i) v[i] = gs[grp * SP + i] * wj;
        } else {
#pragma unroll
            for (int i = 0; i < SP; ++i) v[i] = 0.0f;
            step_chain<BF, SP, PRE>(v, P.master + P.layer[l + 1].mw + (unit < O ? unit : O - 1), O, P.layer[l + 1].out,
                                    xs[cur] + grp * SP * kStepRow);
        }
        if (unit < O) {
#pragma unroll
            for (int i = 0; i < SP; ++i) {
                const int64_t b = b0 + grp * SP + i;
                float q = step_drop(P.D, l, b, unit, ((mask[l] >> i) & 1u) ? v[i] : 0.0f);
                if (BF) q = bf16_rne(q);
                xs[cur ^ 1][(grp * SP + i) * kStepRow + unit] = q;
                if (b < P.B) P.layer[l].dl[b * O + unit] = q;
            }
        }
        cur ^= 1;
        if (l > 0) __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// A workgroup per 16 x 16 tile of one layer's weights; eight waves share the
// samples, four consecutive ones per v_mfma_f32_16x16x4_f32 step, groups of
// four dealt to the waves in turn and, within a wave, to four accumulators: four
// independent matrix-core chains of B / 128 instructions, B / 32 products each
// (256 at B = 8,192; the split-K kernel of larger batches sums 64 and then its
// chunks in sequence, and its errors against 64 bits are larger throughout:
// 1.7e-7 against 5e-8 there).  Each operand is read straight from the
// sample-major arrays, 64 bytes per row.  The workgroups of a layer's first
// input tile also sum its bias gradient, in 64 bits: one fp32 sum of B / 32 terms
// a lane was off by up to 64 units in the last place where they have one sign.
// The last workgroup reduces the loss.
// ---------------------------------------------------------------------------
constexpr int kStepWaves = 8;

template <bool BF>
__global__ __launch_bounds__(64 * kStepWaves) void step_weights_kernel(StepArgs P) {
    __shared__ __align__(16) float red[kStepWaves][256];
    __shared__ double redb[kStepWaves][16];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // which layer and tile
    int t = (int)blockIdx.x, l = 0, O = 0, K = 0, tk = 1;
    for (; l <= P.L; ++l) {
        O = P.layer[l].out;
        K = P.layer[l].in;
        tk = (K + 15) / 16;
        const int n = ((O + 15) / 16) * tk;
        if (t < n) break;
        t -= n;
    }
    if (l > P.L) {                                        // the loss
        double* sum = reinterpret_cast<double*>(&red[0][0]);
        double v = 0.0;
        for (int b = tid; b < P.B; b += 64 * kStepWaves) v += (double)P.e2[b];
        sum[tid] = v;
        __syncthreads();
        for (int w = 32 * kStepWaves; w > 0; w >>= 1) {
            if (tid < w) sum[tid] += sum[tid + w];
            __syncthreads();
        }
        if (tid == 0) {
            const double loss = sum[0] / (double)P.B;
            if (P.loss_out) *P.loss_out = (float)loss;
            if (P.acc) *P.acc = (P.acc_reset ? 0.0 : *P.acc) + loss;
        }
        return;
    }
    const int o0 = 16 * (t / tk), k0 = 16 * (t % tk);
    const float* __restrict__ A = l == P.L ? P.g : P.layer[l].dl;
    const float* __restrict__ X = l == 0 ? P.xn : P.layer[l - 1].a;
    const int r = lane & 15, q = lane >> 4;
    const bool ov = o0 + r < O, kv = k0 + r < K;
    const float* __restrict__ ap = A + (ov ? o0 + r : 0);
    const float* __restrict__ xp = X + (kv ? k0 + r : 0);
    const int groups = (P.B + 3) / 4;
    f32x4_t acc[4] = {};
    double bs = 0.0;
    for (int g0 = wave; g0 < groups; g0 += 4 * kStepWaves) {
        float av[4], xv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int b = 4 * (g0 + j * kStepWaves) + q;
            const int bc = b < P.B ? b : P.B - 1;
            av[j] = ap[(int64_t)bc * O];
            xv[j] = xp[(int64_t)bc * K];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = 4 * (g0 + j * kStepWaves) + q < P.B;
            const float a = in && ov ? av[j] : 0.0f, x = in && kv ? xv[j] : 0.0f;
            if (k0 == 0) bs += (double)a;
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, x, acc[j], 0, 0, 0);
        }
    }
    // accumulator register i of lane (q, r): row 4 q + i, column r
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][(4 * q + i) * 16 + r] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
    if (k0 == 0) {
        bs += __shfl_xor(bs, 16);
        bs += __shfl_xor(bs, 32);
        if (q == 0) redb[wave][r] = bs;
    }
    __syncthreads();
    auto apply = [&](int64_t p, float gr) -> float {
        const float w = (float)((double)P.master[p] - (double)P.lr * (double)gr);
        P.master[p] = w;
        if (P.grad_out) P.grad_out[p] = gr;
        return w;
    };
    if (tid < 256) {
        const int o = o0 + (tid >> 4), k = k0 + (tid & 15);
        if (o < O && k < K) {
            float v[kStepWaves];
#pragma unroll
            for (int w = 0; w < kStepWaves; ++w) v[w] = red[w][tid];
            const float gr = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            const float w = apply(P.layer[l].mw + (int64_t)o * K + k, gr);
            const float c = BF ? bf16_rne(w) : w;
            P.compute[P.layer[l].wt + (int64_t)k * O + o] = c;
            if (l == 0 && P.c_w1 >= 0) P.compute[P.c_w1 + (int64_t)o * K + k] = c;
        }
    } else if (tid < 272 && k0 == 0) {
        const int o = o0 + tid - 256;
        if (o < O) {
            double v[kStepWaves];
#pragma unroll
            for (int w = 0; w < kStepWaves; ++w) v[w] = redb[w][tid - 256];
            const double gr = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            P.compute[P.layer[l].bl + o] = apply(P.layer[l].mb + o, (float)gr);
        }
    }
}

int step_width(const ModelDims& m) {
    int w = m.d;
    for (int l = 0; l < m.L; ++l) w = std::max(w, m.h[l]);
    return w;
}

template <bool BF, int T, int G>
void launch_rows(const StepArgs& P, int sp, hipStream_t s) {
    const dim3 grid((uint32_t)((P.B + G * sp - 1) / (G * sp))), block(T);
    if (sp == 1) hipLaunchKernelGGL((step_rows_kernel<BF, T, G, 1, 32>), grid, block, 0, s, P);
    else if (sp == 2) hipLaunchKernelGGL((step_rows_kernel<BF, T, G, 2, 16>), grid, block, 0, s, P);
    else hipLaunchKernelGGL((step_rows_kernel<BF, T, G, 4, 16>), grid, block, 0, s, P);
}

template <bool BF>
void launch_rows_of(const StepArgs& P, int width, int sp, hipStream_t s) {
    // up to 256 samples of 65 to 128 units go one to a workgroup of two waves: half the loads of a CU per input (22.2
    // us a step at B = 256 of 3 x 128, 23.6 with two samples on four waves; at 512 it is 28.2 against 25.7)
    if (width <= 64) launch_rows<BF, 256, 4>(P, sp, s);
    else if (width <= 128 && P.B <= 256)
        hipLaunchKernelGGL((step_rows_kernel<BF, 128, 1, 1, 32>), dim3((uint32_t)P.B), dim3(128), 0, s, P);
    else if (width <= 128) launch_rows<BF, 256, 2>(P, sp, s);
    else launch_rows<BF, 256, 1>(P, sp, s);
}

}  // namespace

// The first models to cross over do so here: three layers of 256 with 256 inputs
// in bf16, 254 us layer by layer and 253 in two launches at B = 8,192; 64-256-256
// in bf16 151 and 136; in fp32, and at 128 units, two launches still take less than
// half there (37-128-128-128: 321 and 88).
constexpr int kStepMaxBatch = 8192;

// One narrow hidden layer in bf16 crosses earlier.  From 7,681 samples in
// multiples of eight its layer-by-layer step stores bf16 and runs on the matrix
// cores (16 workgroups of 512 samples), and with so few units most of the two-launch
// step's lanes idle: 16-8 39 us layer by layer and 45 in two launches at 8,192,
// 64-32 47 and 51, 130-8 53 and 66, 200-32 68 and 75.  Between 65 and 128 inputs
// the lines meet at 16 units (128-8 52 and 55, 128-32 58 and 56).
static bool step_layers_win(const ModelDims& m, int32_t B) {
    const int width = step_width(m);
    return m.bf16 && m.L == 1 && m.h[0] <= (width > 64 && width <= 128 ? 16 : 32) && B > 7680 && B % 8 == 0 &&
           m.mfma_chains;
}

bool step_fused(const ModelDims& m, int32_t B) {
    return B <= kStepMaxBatch && step_width(m) <= kStepWidth && !step_layers_win(m, B);
}

int64_t step_workspace_bytes(const ModelDims& m, int32_t B) {
    auto up = [](int64_t n) { return (n + 63) & ~int64_t(63); };
    int64_t n = up((int64_t)m.d * B) + 2 * up(B);
    for (int l = 0; l < m.L; ++l) n += 2 * up((int64_t)m.h[l] * B);
    return n * (int64_t)sizeof(float);
}

hipError_t launch_step_fused(const ModelDims& m, float* master, float* compute, const float* mu, const float* isig,
                             int32_t B, const StepRows& rows, float lr, const StepLoss& loss, float* grad_out,
                             void* workspace, const DropArgs& drop, hipStream_t s) {
    StepArgs P{};
    P.L = m.L; P.d = m.d; P.B = B; P.hl = m.hl;
    float* w = reinterpret_cast<float*>(workspace);
    auto take = [&](int64_t n) { float* p = w; w += (n + 63) & ~int64_t(63); return p; };
    for (int l = 0; l <= m.L; ++l) {
        StepLayer& Y = P.layer[l];
        Y.in = m.in_of(l); Y.out = m.out_of(l);
        Y.mw = m.m_w[l]; Y.mb = m.m_b[l]; Y.wt = m.c_wt[l]; Y.bl = m.c_bl[l];
        if (l < m.L) { Y.a = take((int64_t)Y.out * B); Y.dl = take((int64_t)Y.out * B); }
    }
    P.c_w1 = m.L == 2 ? m.c_w1 : -1;
    P.n_master = (int)m.n_params;
    P.n_compute = (int)m.n_compute;
    P.mu = mu; P.isig = isig; P.master = master; P.compute = compute;
    P.code = rows.code; P.ax = rows.ax; P.ay = rows.ay; P.bx = rows.bx; P.by = rows.by;
    P.xn = take((int64_t)m.d * B);
    P.g = take(B);
    P.e2 = take(B);
    P.lr = lr; P.grad_out = grad_out;
    P.loss_out = loss.step; P.acc = loss.acc; P.acc_reset = loss.reset;
    P.D = drop;
    const int width = step_width(m);
    const int G = width <= 64 ? 4 : width <= 128 ? 2 : 1;
    // samples per thread: one while the workgroups it makes are about one a CU (24 us at B = 256 of the 3 x 128
    // model, 26 with two, all 16 inputs ahead; 22 now), two up to three a CU (30.5 at B = 1,000; 33 with one, 34
    // with four), then four (83 at B = 8,192; 115 with two, 158 with one): each weight read then serves more samples
    const int sp = B <= 256 * G ? 1 : B <= 768 * G ? 2 : 4;
    if (m.bf16) launch_rows_of<true>(P, width, sp, s);
    else launch_rows_of<false>(P, width, sp, s);
    int tiles = 0;
    for (int l = 0; l <= m.L; ++l) tiles += ((m.out_of(l) + 15) / 16) * ((m.in_of(l) + 15) / 16);
    const bool want_loss = loss.step || loss.acc;
    const dim3 grid((uint32_t)(tiles + (want_loss ? 1 : 0))), block(64 * kStepWaves);
    if (m.bf16) hipLaunchKernelGGL(step_weights_kernel<true>, grid, block, 0, s, P);
    else hipLaunchKernelGGL(step_weights_kernel<false>, grid, block, 0, s, P);
    return hipGetLastError();
}

}  // namespace ls
