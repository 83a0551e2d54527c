// Admission of FIFO evictions to the replay pool (Section 4.3.2, Training-data
// selection) for pools of up to kWalkSlots members.
//
// The rule is sequential: each candidate's decision depends on the ones before
// it.  But every distance it can ask for -- pool to pool, candidate to pool,
// candidate to candidate -- is known before a chunk of candidates is decided,
// and so is each point's short list of nearest original members.  So per chunk
//   dist_kernel   all three distance tables, 64 x 64 tiles over the whole GPU;
//   top_kernel    per point (member or candidate) its kTop nearest original
//                 members, ascending;
//   walk_kernel   one workgroup decides the candidates in order.  Its threads
//                 hold the members' nearest-neighbour distances in registers; a
//                 nearest neighbour that has to be found again is the first
//                 entry of the point's list that is still a member, or the
//                 nearest admitted candidate, whichever is nearer: one wave, a
//                 few hundred values, instead of the pool's whole row;
//   apply_kernel  the chunk's result: rows and embeddings of the slots that
//                 changed hands, and the distances the next chunk needs.
// What bounds the walk is latency: three barriers and one round of dependent
// global reads per admission.  A push of 1,000 rows into full pools of 5,000
// (256 units): 14.8 ms when one workgroup searched whole rows with its state in
// LDS, 1.28 ms now; the first push of 1,000 on new rows, 903 of them admitted,
// 34.7 and 9.0 ms (12.2 when one wave searched a whole row by itself).
//
// Distances are compared as the bit patterns of non-negative doubles, which
// order like the numbers; a NaN's pattern is above infinity's, so it is never
// nearer than anything, and a candidate all of whose distances are NaN does
// not enter a full pool.
#include "ls_internal.h"

namespace ls {

namespace {

constexpr int kWalkThreads = 1024;
constexpr int kWalkOwn = 6;                            // members per thread
constexpr int kWalkSlots = kWalkThreads * kWalkOwn;    // 6,144
constexpr int kWalkChunk = 512;                        // candidates decided per launch
constexpr int kWalkLook = 8;                           // candidates whose distance is found ahead
constexpr int kWalkFull = 8;                           // whole rows searched between two barriers
constexpr int kTop = 12;                               // entries of a point's list
constexpr uint64_t kInfBits = 0x7ff0000000000000ull;
constexpr uint64_t kNoBits = ~0ull;                    // no value

// ---------------------------------------------------------------------------
// Squared distances, summed over units in ascending order by one thread each.
// Tiles of 64 x 64, a thread 4 x 4 of them, 16 units of both sides in LDS at a
// time.  What bounds it is the fp64 rate (a subtraction, a product and a sum per
// unit and pair; the sums keep their separate roundings).  A table of a set with
// itself computes the tiles on and above the diagonal and writes both halves:
// (a - b)^2 is (b - a)^2 to the bit.
// ---------------------------------------------------------------------------
constexpr int kTile = 64, kTileJ = 16;

struct DistJob {
    const double *A, *B;
    int32_t na, nb;
    double *out, *outT;                                // [na][ldo], [nb][ldt] (or null)
    int64_t ldo, ldt;
    int32_t sym;                                       // A is B: out alone, its diagonal infinite
    int32_t tiles;
};

struct DistJobs {
    DistJob job[3];
};

__global__ __launch_bounds__(256) void dist_kernel(DistJobs J, int H) {
    __shared__ double sa[kTileJ][kTile + 2], sb[kTileJ][kTile + 2];
    int t = (int)blockIdx.x, which = 0;
    while (which < 2 && t >= J.job[which].tiles) t -= J.job[which++].tiles;
    const DistJob& q = J.job[which];
    int ta, tb;
    if (q.sym) {                                       // tile t of the triangle ta <= tb, by columns
        tb = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while ((tb + 1) * (tb + 2) / 2 <= t) ++tb;
        while (tb * (tb + 1) / 2 > t) --tb;
        ta = t - tb * (tb + 1) / 2;
    } else {
        const int nt = (q.nb + kTile - 1) / kTile;
        ta = t / nt;
        tb = t - ta * nt;
    }
    const int32_t a0 = ta * kTile, b0 = tb * kTile;
    const int tid = (int)threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int lr = tid >> 2, lq = 4 * (tid & 3);
    const double* __restrict__ pa = q.A + (int64_t)(a0 + lr < q.na ? a0 + lr : q.na - 1) * H;
    const double* __restrict__ pb = q.B + (int64_t)(b0 + lr < q.nb ? b0 + lr : q.nb - 1) * H;
    double acc[4][4] = {};
    double ra[4], rb[4];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = j0 + lq + e;
            ra[e] = pa[j < H ? j : H - 1];
            rb[e] = pb[j < H ? j : H - 1];
        }
    };
    fetch(0);
    for (int j0 = 0; j0 < H; j0 += kTileJ) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sa[lq + e][lr] = ra[e];
            sb[lq + e][lr] = rb[e];
        }
        __syncthreads();
        if (j0 + kTileJ < H) fetch(j0 + kTileJ);
        const int jn = H - j0 < kTileJ ? H - j0 : kTileJ;
        auto unit = [&](int j) {
            double a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = sa[j][ty + 16 * u];
                b[u] = sb[j][tx + 16 * u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double e = a[u] - b[v];
                    acc[u][v] += e * e;
                }
        };
        if (jn == kTileJ) {
#pragma unroll 4
            for (int j = 0; j < kTileJ; ++j) unit(j);
        } else {
            for (int j = 0; j < jn; ++j) unit(j);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int32_t a = a0 + ty + 16 * u;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int32_t b = b0 + tx + 16 * v;
            if (a >= q.na || b >= q.nb) continue;
            if (q.sym) {
                q.out[(int64_t)a * q.ldo + b] = a == b ? INFINITY : acc[u][v];
                if (ta != tb) q.out[(int64_t)b * q.ldo + a] = acc[u][v];
            } else {
                q.out[(int64_t)a * q.ldo + b] = acc[u][v];
                if (q.outT) q.outT[(int64_t)b * q.ldt + a] = acc[u][v];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// wave-wide minimum of bit patterns
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_min(uint64_t v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
    const uint64_t o = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
    return o < v ? o : v;
}

// over each row of 16 lanes: lane xor 1, xor 2, then the mirrored half row and row
__device__ __forceinline__ uint64_t row_min(uint64_t v) {
    v = dpp_min<0xB1>(v);
    v = dpp_min<0x4E>(v);
    v = dpp_min<0x141>(v);
    return dpp_min<0x140>(v);
}

__device__ __forceinline__ uint64_t wave_min(uint64_t v) {
    v = row_min(v);
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)v, off);
        v = o < v ? o : v;
    }
    return v;
}

__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// lowest `slot` among the lanes whose bit is set (at least one)
__device__ __forceinline__ int32_t lowest_slot(uint64_t m, int32_t slot) {
    int32_t best = __builtin_amdgcn_readlane(slot, (int)__builtin_ctzll(m));
    for (m &= m - 1; m != 0; m &= m - 1) {
        const int32_t s = __builtin_amdgcn_readlane(slot, (int)__builtin_ctzll(m));
        best = s < best ? s : best;
    }
    return best;
}

// The walk shares data between waves in LDS alone (what it reads from memory
// does not change), so its barriers order LDS only and leave loads in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// A workgroup per point: rows [0, n) are the members (row of D, itself left
// out), the rest the candidates (row of dcp).  Ties in any order: only the
// values decide.  A thread offers the two nearest of its 24, so a round is one
// reduction; a list ends (-2: more may follow, -1: nothing does) when a thread
// has given both, and the walk then searches the whole row, all waves a part each,
// when none of the entries is a member any more.  5,512 points: 49 us (151 with every
// thread offering all of its own).
// ---------------------------------------------------------------------------
constexpr int kTopThreads = 256;
constexpr int kTopOwn = kWalkSlots / kTopThreads;      // 24

__global__ __launch_bounds__(kTopThreads) void top_kernel(const uint64_t* __restrict__ D,
                                                          const uint64_t* __restrict__ dcp, int32_t n, int32_t cap,
                                                          uint64_t* __restrict__ top_d, int32_t* __restrict__ top_i) {
    __shared__ uint64_t sv[2][kTopThreads / 64];
    __shared__ int32_t cut[2];                         // a thread has given both: its next is not known
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t p = (int32_t)blockIdx.x;
    const uint64_t* __restrict__ row = p < n ? D + (int64_t)p * cap : dcp + (int64_t)(p - n) * cap;
    uint64_t x[kTopOwn];
#pragma unroll
    for (int u = 0; u < kTopOwn; ++u) {
        const int32_t j = tid + u * kTopThreads;
        x[u] = j < n ? row[j] : kNoBits;
        if (j == p || x[u] > kInfBits) x[u] = kNoBits;
    }
    // this thread's two nearest, and whether there are more
    uint64_t m1 = kNoBits, m2 = kNoBits;
    int32_t i1 = -1, i2 = -1, found = 0;
#pragma unroll
    for (int u = 0; u < kTopOwn; ++u) {
        const int32_t j = tid + u * kTopThreads;
        found += x[u] != kNoBits ? 1 : 0;
        if (x[u] < m1) {
            m2 = m1;
            i2 = i1;
            m1 = x[u];
            i1 = j;
        } else if (x[u] < m2) {
            m2 = x[u];
            i2 = j;
        }
    }
    int given = 0;                                     // entries this thread has put on the list
    if (tid < 2) cut[tid] = 0;
    int r = 0, rest = -1;
    for (; r < kTop; ++r) {
        const uint64_t w = wave_min(m1);
        if (lane == 0) sv[r & 1][wv] = w;
        __syncthreads();
        if (cut[(r & 1) ^ 1]) {                        // uniform: of the round before
            rest = -2;
            break;
        }
        uint64_t best = sv[r & 1][0];
        int from = 0;
#pragma unroll
        for (int k = 1; k < kTopThreads / 64; ++k) {
            const uint64_t o = sv[r & 1][k];
            if (o < best) {
                best = o;
                from = k;
            }
        }
        if (best == kNoBits) break;                    // uniform: nothing left
        if (wv == from && lane == (int)__builtin_ctzll(__ballot(m1 == best))) {
            top_d[(int64_t)p * kTop + r] = best;
            top_i[(int64_t)p * kTop + r] = i1;
            m1 = m2;
            i1 = i2;
            m2 = kNoBits;
            if (++given == 2 && found > 2) cut[r & 1] = 1;
        }
    }
    if (tid >= r && tid < kTop) {
        top_d[(int64_t)p * kTop + tid] = kNoBits;
        top_i[(int64_t)p * kTop + tid] = rest;
    }
}

// ---------------------------------------------------------------------------
// The walk.  Slot k belongs to thread k % 1024.  org[k] is the candidate of
// this chunk that holds slot k (-1: the member it started with, or none).
// ---------------------------------------------------------------------------
struct WalkArgs {
    const uint64_t *D, *dcp, *dpc, *dcc, *top_d;       // [n][cap], [nch][cap], [n][nch], [nch][nch], [n + nch][kTop]
    const int32_t* top_i;
    int32_t n, cap, nch;
    int32_t* origin;                                   // [cap]
    int32_t* admitted;
};

__global__ __launch_bounds__(kWalkThreads) void walk_kernel(WalkArgs W) {
    __shared__ int32_t org[kWalkSlots];
    __shared__ int32_t redo[kWalkSlots + 1], res_i[kWalkSlots + 1];
    __shared__ uint64_t res_d[kWalkSlots + 1];
    __shared__ int32_t slot_of[kWalkChunk];            // the slot a candidate holds, or -1
    __shared__ uint64_t near[kWalkChunk];              // this candidate's distances to the chunk's
    __shared__ uint64_t look_d[kWalkLook], wmin_v[kWalkThreads / 64];
    __shared__ int32_t wmin_s[kWalkThreads / 64];
    __shared__ int32_t n_redo, n_full;
    __shared__ int32_t full[kWalkSlots + 1 + kWalkLook];   // points whose list holds no member any more
    __shared__ uint64_t part_v[kWalkFull][kWalkThreads / 64];
    __shared__ int32_t part_s[kWalkFull][kWalkThreads / 64];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t n0 = W.n, cap = W.cap, nch = W.nch;
    int32_t n = n0, taken = 0;
    uint64_t nnd[kWalkOwn], x[kWalkOwn];
    int32_t nni[kWalkOwn], own[kWalkOwn];              // nearest neighbour's slot; org of the own slots
    auto load_row = [&](int32_t c) {
#pragma unroll
        for (int u = 0; u < kWalkOwn; ++u) {
            const int32_t k = tid + u * kWalkThreads;
            x[u] = W.dcp[(int64_t)c * cap + (k < n0 ? k : 0)];     // a slot without a member: not used
        }
        return tid < nch ? W.dcc[(int64_t)c * nch + tid] : 0ull;
    };
#pragma unroll
    for (int u = 0; u < kWalkOwn; ++u) {
        const int32_t k = tid + u * kWalkThreads;
        own[u] = -1;
        nnd[u] = kNoBits;
        nni[u] = -1;
        if (k < n0) {
            const uint64_t v = W.top_d[(int64_t)k * kTop];
            nnd[u] = v < kInfBits ? v : kInfBits;
            nni[u] = W.top_i[(int64_t)k * kTop];
        }
        org[k] = -1;
    }
    if (tid < kWalkChunk) slot_of[tid] = -1;
    if (tid == 0) n_redo = n_full = 0;
    // the pool's smallest nearest-neighbour distance, lowest slot on ties
    uint64_t pool_v = kNoBits;
    int32_t pool_s = -1;
    auto pool_publish = [&]() {
        uint64_t v = nnd[0];
        int32_t s = tid;
#pragma unroll
        for (int u = 1; u < kWalkOwn; ++u)
            if (nnd[u] < v) {
                v = nnd[u];
                s = tid + u * kWalkThreads;
            }
        const uint64_t w = wave_min(v);
        s = lowest_slot(__ballot(v == w), s);
        if (lane == 0) {
            wmin_v[wv] = w;
            wmin_s[wv] = s;
        }
    };
    auto pool_collect = [&]() {
        const uint64_t v = wmin_v[lane & 15];
        const int32_t s = wmin_s[lane & 15];
        pool_v = uniform(row_min(v));
        pool_s = lowest_slot(__ballot(v == pool_v) & 0xffffull, s);
    };
    // nearest member of one point, by one wave: value and slot, kNoBits and -1 without any.
    // `a` >= 0: candidate a, else the member that slot k started with.
    // Returns whether the whole row is wanted too: every listed member has been replaced and there may be others.
    auto nearest = [&](int32_t k, int32_t a, int32_t upto, uint64_t& bv, int32_t& bs) -> bool {
        const int64_t p = a >= 0 ? (int64_t)n0 + a : (int64_t)k;
        const uint64_t* __restrict__ brow = a >= 0 ? W.dcc + (int64_t)a * nch : W.dpc + (int64_t)k * nch;
        uint64_t tv = kNoBits;
        int32_t ti = -1;
        if (lane < kTop) {
            tv = W.top_d[p * kTop + lane];
            ti = W.top_i[p * kTop + lane];
        }
        constexpr int E = kWalkChunk / 64;
        uint64_t b[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t q = lane + 64 * e;
            b[e] = 64 * e < upto ? brow[q < nch ? q : nch - 1] : kNoBits;      // uniform: later ones not decided
        }
        uint64_t v = kNoBits;
        int32_t s = -1;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t q = lane + 64 * e;
            const int32_t sq = slot_of[q];
            if (q < nch && q != a && sq >= 0 && b[e] <= kInfBits && b[e] < v) {
                v = b[e];
                s = sq;
            }
        }
        const uint64_t w = wave_min(v);
        bv = w;
        bs = -1;
        if (w != kNoBits) bs = __builtin_amdgcn_readlane(s, (int)__builtin_ctzll(__ballot(v == w)));
        const uint64_t live = __ballot(ti >= 0 && org[ti >= 0 ? ti : 0] < 0);
        if (live != 0) {
            const int f = (int)__builtin_ctzll(live);
            const uint64_t fv = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(tv >> 32), f) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tv, f);
            if (fv < bv) {
                bv = fv;
                bs = __builtin_amdgcn_readlane(ti, f);
            }
            return false;
        }
        return __builtin_amdgcn_readlane(ti, kTop - 1) != -1;
    };
    __syncthreads();
    uint64_t next = 0;                                 // this thread's entry of the next candidate's dcc row
    int32_t have = -1;                                 // the candidate whose row is in x and near
    int32_t slot = -1, nr = -1;                        // the slot last taken; members listed (-1: none taken)
    int32_t c = 0;
    for (;;) {
        // a wave per point: the listed members, the new one (nr), then the next candidates, whose distances hold
        // until one of them is admitted
        for (int32_t r = wv; r <= nr + kWalkLook; r += kWalkThreads / 64) {
            const bool member = r <= nr;
            const int32_t a = c + (r - nr - 1);
            if (!member && a >= nch) break;
            const int32_t k = !member ? -1 : r < nr ? __builtin_amdgcn_readfirstlane(redo[r]) : slot;
            uint64_t v;
            int32_t s;
            const bool whole = nearest(k, member ? __builtin_amdgcn_readfirstlane(org[k]) : a, c, v, s);
            if (lane == 0) {
                if (whole) full[atomicAdd(&n_full, 1)] = r;
                if (member) {
                    res_d[r] = v < kInfBits ? v : kInfBits;
                    res_i[r] = s;
                } else {
                    look_d[a - c] = v;
                }
            }
        }
        lds_barrier();
        // whole rows, every wave a part of each
        const int32_t nf = __builtin_amdgcn_readfirstlane(n_full);
        for (int32_t f0 = 0; f0 < nf; f0 += kWalkFull) {
            const int32_t nb = nf - f0 < kWalkFull ? nf - f0 : kWalkFull;
            for (int32_t f = 0; f < nb; ++f) {
                const int32_t r = __builtin_amdgcn_readfirstlane(full[f0 + f]);
                const int32_t k = r < nr ? __builtin_amdgcn_readfirstlane(redo[r]) : slot;
                const int32_t a = r <= nr ? __builtin_amdgcn_readfirstlane(org[k]) : c + (r - nr - 1);
                const uint64_t* __restrict__ row = a >= 0 ? W.dcp + (int64_t)a * cap : W.D + (int64_t)k * cap;
                uint64_t y[kWalkOwn], v = kNoBits;
                int32_t s = -1;
#pragma unroll
                for (int u = 0; u < kWalkOwn; ++u) {
                    const int32_t j = tid + u * kWalkThreads;
                    y[u] = row[j < n0 ? j : n0 - 1];
                }
#pragma unroll
                for (int u = 0; u < kWalkOwn; ++u) {
                    const int32_t j = tid + u * kWalkThreads;
                    if (j < n0 && (a >= 0 || j != k) && own[u] < 0 && y[u] <= kInfBits && y[u] < v) {
                        v = y[u];
                        s = j;
                    }
                }
                const uint64_t w = wave_min(v);
                s = lowest_slot(__ballot(v == w), s);
                if (lane == 0) {
                    part_v[f][wv] = w;
                    part_s[f][wv] = s;
                }
            }
            lds_barrier();
            if (wv < nb) {
                const int32_t r = __builtin_amdgcn_readfirstlane(full[f0 + wv]);
                const uint64_t v = part_v[wv][lane & 15];
                const int32_t s = part_s[wv][lane & 15];
                const uint64_t w = uniform(row_min(v));
                const int32_t best = lowest_slot(__ballot(v == w) & 0xffffull, s);
                if (lane == 0) {
                    if (r <= nr) {
                        if (w < res_d[r]) {
                            res_d[r] = w;
                            res_i[r] = best;
                        }
                    } else if (w < look_d[r - nr - 1]) {
                        look_d[r - nr - 1] = w;
                    }
                }
            }
            lds_barrier();
        }
        if (tid == 0 && nf > 0) n_full = 0;
        if (nr >= 0) {
#pragma unroll
            for (int u = 0; u < kWalkOwn; ++u) {
                const int32_t k = tid + u * kWalkThreads;
                const int32_t q = k == slot ? nr : -2 - nni[u];
                if (q >= 0) {
                    nnd[u] = res_d[q];
                    nni[u] = res_i[q];
                }
            }
            if (tid == 0) n_redo = 0;
            if (tid < nch) near[tid] = next;
            have = c;
        }
        pool_publish();
        lds_barrier();
        pool_collect();
        // the next candidate that enters
        const int32_t look0 = c;
        bool enters = false;
        while (c < nch && c - look0 < kWalkLook) {
            const uint64_t v = uniform(look_d[c - look0]);
            enters = n < cap || (v <= kInfBits && v > pool_v);
            if (enters) break;
            ++c;
        }
        if (c >= nch) break;
        if (!enters) {
            lds_barrier();                             // every look_d read
            nr = -1;
            slot = -1;
            continue;
        }
        slot = n < cap ? n : pool_s;
        if (have != c) {
            next = load_row(c);
            lds_barrier();                             // the last reads of near
            if (tid < nch) near[tid] = next;
            lds_barrier();
        }
        // members whose neighbour leaves are listed; the others may be nearer to the new one
#pragma unroll
        for (int u = 0; u < kWalkOwn; ++u) {
            const int32_t k = tid + u * kWalkThreads;
            if (k == slot) {
                if (own[u] >= 0) slot_of[own[u]] = -1;
                own[u] = c;
                org[k] = c;
                slot_of[c] = k;
            } else if (k < n) {
                const uint64_t v = own[u] >= 0 ? near[own[u]] : x[u];
                if (nni[u] == slot) {
                    const int32_t q = atomicAdd(&n_redo, 1);
                    redo[q] = k;
                    nni[u] = -(q + 2);
                } else if (v < nnd[u]) {
                    nnd[u] = v;
                    nni[u] = slot;
                }
            }
        }
        if (n < cap) ++n;
        ++taken;
        ++c;
        if (c < nch) next = load_row(c);
        lds_barrier();
        nr = __builtin_amdgcn_readfirstlane(n_redo);
    }
#pragma unroll
    for (int u = 0; u < kWalkOwn; ++u) {
        const int32_t k = tid + u * kWalkThreads;
        if (k < cap) W.origin[k] = own[u];
    }
    if (tid == 0) *W.admitted += taken;
}

// ---------------------------------------------------------------------------
// After a chunk, a workgroup per slot: the row and embedding of a slot that
// changed hands, and (`next`) its row of D and the columns of D that did.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void apply_kernel(const int32_t* __restrict__ origin, int32_t n, int32_t cap,
                                                    int32_t nch, int H, int d, const double* __restrict__ cemb,
                                                    const float* __restrict__ cx, const float* __restrict__ cy,
                                                    const double* __restrict__ dcp, const double* __restrict__ dpc,
                                                    const double* __restrict__ dcc, double* __restrict__ emb,
                                                    float* __restrict__ rx, float* __restrict__ ry,
                                                    double* __restrict__ D, int next) {
    const int32_t k = (int32_t)blockIdx.x;
    const int tid = (int)threadIdx.x;
    const int32_t ok = origin[k];
    if (ok >= 0) {
        for (int j = tid; j < d; j += 256) rx[(int64_t)k * d + j] = cx[(int64_t)ok * d + j];
        if (tid == 0) ry[k] = cy[ok];
    }
    if (!next) return;
    if (ok >= 0)
        for (int j = tid; j < H; j += 256) emb[(int64_t)k * H + j] = cemb[(int64_t)ok * H + j];
    for (int32_t j = tid; j < n; j += 256) {
        const int32_t oj = origin[j];
        double v;
        if (ok >= 0) v = j == k ? INFINITY : oj >= 0 ? dcc[(int64_t)ok * nch + oj] : dcp[(int64_t)ok * cap + j];
        else if (oj >= 0) v = dpc[(int64_t)k * nch + oj];
        else continue;
        D[(int64_t)k * cap + j] = v;
    }
}

DistJob dist_job(const double* A, int32_t na, const double* B, int32_t nb, double* out, int64_t ldo, double* outT,
                 int64_t ldt, int sym) {
    const int ta = (na + kTile - 1) / kTile, tb = (nb + kTile - 1) / kTile;
    return {A, B, na, nb, out, outT, ldo, ldt, sym, na < 1 || nb < 1 ? 0 : sym ? ta * (ta + 1) / 2 : ta * tb};
}

void launch_dist(const DistJobs& J, int H, hipStream_t s) {
    const int tiles = J.job[0].tiles + J.job[1].tiles + J.job[2].tiles;
    if (tiles > 0) hipLaunchKernelGGL(dist_kernel, dim3((uint32_t)tiles), dim3(256), 0, s, J, H);
}

int64_t up256(int64_t b) { return (b + 255) & ~int64_t(255); }

}  // namespace

bool admission_walks(int32_t cap) { return cap <= kWalkSlots; }

int32_t admission_walk_chunk(int32_t nc) { return nc < kWalkChunk ? nc : kWalkChunk; }

// dcp, dpc, dcc, the lists, the slots' origins
int64_t admission_walk_bytes(int32_t cap, int32_t nc) {
    const int64_t ch = admission_walk_chunk(nc);
    return 2 * up256(ch * cap * 8) + up256(ch * ch * 8) + up256((cap + ch) * kTop * 8) + up256((cap + ch) * kTop * 4) +
           up256((int64_t)cap * 4);
}

// Embeddings are in emb (n0 members) and cemb (nc candidates); *admitted is cleared.
hipError_t launch_admission_walk(int32_t n0, int32_t nc, int H, int d, int32_t cap, const float* cx, const float* cy,
                                 const double* cemb, double* emb, float* rx, float* ry, double* D, int32_t* admitted,
                                 void* workspace, hipStream_t s) {
    const int32_t chunk = admission_walk_chunk(nc);
    char* w = reinterpret_cast<char*>(workspace);
    auto take = [&](int64_t bytes) {
        char* p = w;
        w += up256(bytes);
        return p;
    };
    double* dcp = reinterpret_cast<double*>(take((int64_t)chunk * cap * 8));
    double* dpc = reinterpret_cast<double*>(take((int64_t)chunk * cap * 8));
    double* dcc = reinterpret_cast<double*>(take((int64_t)chunk * chunk * 8));
    uint64_t* top_d = reinterpret_cast<uint64_t*>(take(((int64_t)cap + chunk) * kTop * 8));
    int32_t* top_i = reinterpret_cast<int32_t*>(take(((int64_t)cap + chunk) * kTop * 4));
    int32_t* origin = reinterpret_cast<int32_t*>(take((int64_t)cap * 4));
    int32_t n = n0;
    for (int32_t c0 = 0; c0 < nc; c0 += chunk) {
        const int32_t nch = nc - c0 < chunk ? nc - c0 : chunk;
        const double* ce = cemb + (int64_t)c0 * H;
        DistJobs J;
        J.job[0] = dist_job(emb, c0 == 0 ? n : 0, emb, n, D, cap, nullptr, 0, 1);    // later chunks: kept by apply_kernel
        J.job[1] = dist_job(ce, nch, emb, n, dcp, cap, dpc, nch, 0);
        J.job[2] = dist_job(ce, nch, ce, nch, dcc, nch, nullptr, 0, 1);
        launch_dist(J, H, s);
        hipLaunchKernelGGL(top_kernel, dim3((uint32_t)(n + nch)), dim3(kTopThreads), 0, s,
                           reinterpret_cast<const uint64_t*>(D), reinterpret_cast<const uint64_t*>(dcp), n, cap, top_d,
                           top_i);
        WalkArgs W{reinterpret_cast<const uint64_t*>(D), reinterpret_cast<const uint64_t*>(dcp),
                   reinterpret_cast<const uint64_t*>(dpc), reinterpret_cast<const uint64_t*>(dcc), top_d, top_i,
                   n, cap, nch, origin, admitted};
        hipLaunchKernelGGL(walk_kernel, dim3(1), dim3(kWalkThreads), 0, s, W);
        n = n + nch < cap ? n + nch : cap;
        hipLaunchKernelGGL(apply_kernel, dim3((uint32_t)n), dim3(256), 0, s, origin, n, cap, nch, H, d, ce,
                           cx + (int64_t)c0 * d, cy + c0, dcp, dpc, dcc, emb, rx, ry, D, c0 + nch < nc ? 1 : 0);
    }
    return hipGetLastError();
}

// The tables of the admission that keeps its state in memory (k_buffer.hip).
void launch_distances(const double* A, int32_t na, const double* B, int32_t nb, int H, double* out, int64_t ldo,
                      bool sym, hipStream_t s) {
    DistJobs J{};
    J.job[0] = dist_job(A, na, B, nb, out, ldo, nullptr, 0, sym ? 1 : 0);
    launch_dist(J, H, s);
}

}  // namespace ls
