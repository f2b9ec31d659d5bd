// mpnn.hip — the learned initial partition: a three-layer message-passing
// network that proposes the k-way assignment of the coarsest graph (the slot
// of the paper's initial partitioning, §III-B), its training loss and
// hand-written backward pass, and Adam.
//
// Inference is bit-reproducible: weights are used rounded to bfloat16 (nearest,
// ties to even) as binary32 values; every sum is a chain of fused
// multiply-adds in a fixed order (neighbours in CSR order from 0, then inputs
// in index order from the bias, self inputs before aggregated ones); the
// reciprocal of a weighted degree and the two ratio features are formed in
// binary64 and rounded once. Nothing else is fused: contraction is off for
// this file. Training kernels use the same forward; their gradients are
// plain binary32 (atomics in the weight-gradient reductions).
//
// Network (per vertex v):
//   X[v]  = (c(v)/c_max, deg(v)/max_deg, y_8[v][0..15]),
//           y_0 = seeded +-1 probes, y_{t+1}[v] = (y_t[v] + (sum_u w(v,u) y_t[u]) / d(v)) / 2
//   h_l   = ReLU(b_l + Ws_l h_{l-1}[v] + Wn_l m_l[v]),  m_l[v] = (sum_u w(v,u) h_{l-1}[u]) / d(v)
//   z[v]  = bh + Wh h_3[v];  block(v) = argmax z[v] (ties -> lowest)
// d(v) is the weighted degree; a vertex without neighbours keeps y and gets m = 0.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>

#include "mpnn.hpp"
#include "prims.hpp"

#pragma clang fp contract(off)

namespace gp {

int32_t mpnn_param_count(int32_t k) {
    return (2 * kMpHid * kMpFeat + kMpHid) + 2 * (2 * kMpHid * kMpHid + kMpHid) + kMpHid * k + k;
}

namespace {

constexpr int kMB = 256;  // block size of the network kernels

// splitmix64 (Steele, Lea & Flood 2014): finaliser of x + golden gamma.
__device__ __forceinline__ uint64_t splitmix(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Round to the nearest bfloat16 (ties to even); NaN stays a quiet NaN.
__global__ void k_bf16(const float *__restrict__ in, float *__restrict__ out, int32_t count) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        uint32_t u = __float_as_uint(in[i]);
        if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu) != 0) u = (u & 0xffff0000u) | 0x00400000u;
        else u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
        out[i] = __uint_as_float(u);
    }
}

// Aggregation over neighbours, acc <- fma(w(v,u), X[u][c], acc) over the CSR
// row in order: one chain per (row, column), so a row's time is bound by its
// degree times the latency of a fused multiply-add, as long as its operands are
// there. Rows up to kWideRow entries: a lane per column (16, 32 or 64 lanes per
// row) that gets the neighbours' ids from its row's lanes, loaded together, and
// requests 16 neighbours' values at once. Wider rows: a workgroup per row and
// slice of kSlice columns; four waves fetch the next kStage neighbours' slices
// and stage them in LDS while kSlice lanes of the fifth run their chains over
// those staged before. At 50,000 vertices and 3M entries (the widest row has
// 12,600) a walk step took 1.29 ms with a thread per (row, column) that loaded
// id and value one after the other and staging without overlap, and takes 0.09
// ms so, 17 cycles per step of the widest row. Rows of 97 to 192 entries cost
// less in lanes (a walk step 96 -> 91 us, a 64-column layer 335 -> 258 us),
// wider ones less staged (122 us with lanes up to 512).
constexpr int kWideRow = 192;
constexpr int kSlice = 16;
constexpr int kStage = 256;
constexpr int kGatherBlock = kWave + kStage;  // one wave for the chains, the others fetch and stage
constexpr int kStagePitch = kStage + 4;  // a lane's four values lie in banks of their own

struct WideFlag {
    const int32_t *xadj;
    __device__ bool operator()(int64_t v) const { return xadj[v + 1] - xadj[v] > kWideRow; }
};
struct WideEmit {
    int32_t *wide;
    __device__ void operator()(int64_t v, int32_t pos) const { wide[pos] = (int32_t)v; }
};

// 1/d(v) (binary64 reciprocal rounded once) and the maxima of c and deg. A
// workgroup per wide row (the first `wblocks` of them), 16 lanes per other row:
// a lane per row walked a hub's weights alone (1.34 ms at 50,000 vertices and
// 3.3M entries). Bound: one read of the weights.
__global__ __launch_bounds__(kMB) void k_vstats(int32_t n, const int32_t *__restrict__ wide,
                                                const int32_t *__restrict__ nwide, int32_t wblocks,
                                                const int32_t *__restrict__ xadj,
                                                const int32_t *__restrict__ adjwgt, const int32_t *__restrict__ vwgt,
                                                bool active_only, float *__restrict__ rinv, int32_t *__restrict__ mx) {
    __shared__ int32_t tmp[kMB / kWave + 1];
    __shared__ int64_t t64[kMB / kWave + 1];
    constexpr int GL = 16;
    int32_t cm = 0, dm = 0;
    if ((int32_t)blockIdx.x < wblocks) {
        const int32_t m = *nwide;
        for (int32_t r = blockIdx.x; r < m; r += wblocks) {
            const int32_t v = wide[r], b = xadj[v], e = xadj[v + 1];
            int64_t s = 0;
            if (adjwgt) {
                for (int32_t i0 = b + threadIdx.x; i0 < e; i0 += 4 * kMB) {
                    int32_t x[4];
#pragma unroll
                    for (int j = 0; j < 4; j++) x[j] = i0 + j * kMB < e ? adjwgt[i0 + j * kMB] : 0;
                    s += (int64_t)x[0] + x[1] + x[2] + x[3];
                }
                s = block_sum<kMB>(s, t64);
            } else {
                s = e - b;
            }
            if (threadIdx.x == 0) rinv[v] = (float)(1.0 / (double)s);
            cm = max(cm, vwgt ? vwgt[v] : 1);
            dm = max(dm, e - b);
        }
    } else {
        const int gl = threadIdx.x % GL;
        for (int32_t v0 = (blockIdx.x - wblocks) * (kMB / GL); v0 < n; v0 += (gridDim.x - wblocks) * (kMB / GL)) {
            const int32_t v = v0 + threadIdx.x / GL;
            const int32_t b = v < n ? xadj[v] : 0, e = v < n ? xadj[v + 1] : 0;
            if (v >= n || e - b > kWideRow) continue;
            const int32_t s = e - b;
            if (adjwgt) {  // each weight fits 31 bits, their sum may not
                int64_t t = 0;
                for (int32_t i = b + gl; i < e; i += GL) t += adjwgt[i];
#pragma unroll
                for (int d = GL / 2; d > 0; d >>= 1) t += __shfl_xor(t, d, GL);
                if (gl == 0) rinv[v] = t > 0 ? (float)(1.0 / (double)t) : 0.0f;
            } else if (gl == 0) {
                rinv[v] = s > 0 ? (float)(1.0 / (double)s) : 0.0f;
            }
            if (!active_only || e > b) {
                cm = max(cm, vwgt ? vwgt[v] : 1);
                dm = max(dm, e - b);
            }
        }
    }
    cm = block_max<kMB>(cm, tmp);
    dm = block_max<kMB>(dm, tmp);
    if (threadIdx.x == 0) {
        if (cm > __hip_atomic_load(&mx[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&mx[0], cm);
        if (dm > __hip_atomic_load(&mx[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&mx[1], dm);
    }
}

// The first `wblocks` workgroups take the wide rows, the others the rest.
// WALK: out[v][c] = (X[v][c] + acc * rinv[v]) / 2 (X[v][c] without neighbours),
// else out[v][c] = acc * rinv[v] (0 without neighbours).
template <int COLS, bool WALK>
__global__ __launch_bounds__(kGatherBlock) void k_gather(int32_t n, const int32_t *__restrict__ wide,
                                                         const int32_t *__restrict__ nwide, int32_t wblocks,
                                                         const int32_t *__restrict__ xadj,
                                                         const int32_t *__restrict__ adjncy,
                                                         const int32_t *__restrict__ adjwgt,
                                                         const float *__restrict__ rinv, const float *__restrict__ X,
                                                         float *__restrict__ out) {
    __shared__ __align__(16) float sx[2][kSlice * kStagePitch + 16];  // + 16: the chains read ahead
    __shared__ __align__(16) float sw[2][kStage + 16];
    if ((int32_t)blockIdx.x < wblocks) {
        constexpr int SL = (COLS + kSlice - 1) / kSlice;
        const int32_t items = *nwide * SL;
        const bool chain = threadIdx.x < kWave;      // the first wave
        const int32_t t = (int32_t)threadIdx.x - kWave;  // the others: neighbour t of each chunk
        for (int32_t it = blockIdx.x; it < items; it += wblocks) {
            const int32_t v = wide[it / SL], c0 = it % SL * kSlice;
            const int32_t cols = min(kSlice, COLS - c0);
            const int32_t b = xadj[v], e = xadj[v + 1], nch = (e - b + kStage - 1) / kStage;
            float acc = 0.0f, wv = 0.0f, x[kSlice];
            int32_t nu = 0, nw = 1;
            // ids and weights are requested two chunks before their values are staged
            const auto fetch_id = [&](int32_t q) {
                nu = q < e ? adjncy[q] : 0;
                nw = q < e && adjwgt ? adjwgt[q] : 1;
            };
            const auto fetch = [&]() {
                wv = (float)nw;
                const float *r = X + (int64_t)nu * COLS + c0;
                if constexpr (COLS % 4 == 0) {
#pragma unroll
                    for (int j = 0; j < kSlice / 4; j++) {
                        const float4 f = reinterpret_cast<const float4 *>(r)[j];
                        x[4 * j] = f.x;
                        x[4 * j + 1] = f.y;
                        x[4 * j + 2] = f.z;
                        x[4 * j + 3] = f.w;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < kSlice; j++) x[j] = r[j < cols ? j : 0];
                }
            };
            const auto stage = [&](int buf) {
                sw[buf][t] = wv;
#pragma unroll
                for (int j = 0; j < kSlice; j++) sx[buf][j * kStagePitch + t] = x[j];
            };
            if (!chain) {
                fetch_id(b + t);
                fetch();
                fetch_id(b + kStage + t);
                stage(0);
                if (nch > 1) {
                    fetch();
                    fetch_id(b + 2 * kStage + t);
                }
            }
            __syncthreads();
            for (int32_t ch = 0; ch < nch; ch++) {
                if (!chain) {
                    if (ch + 1 < nch) {
                        stage((ch + 1) & 1);
                        if (ch + 2 < nch) {
                            fetch();
                            fetch_id(b + (ch + 3) * kStage + t);
                        }
                    }
                } else if (threadIdx.x < kSlice) {
                    const float *xc = sx[ch & 1] + threadIdx.x * kStagePitch, *wc = sw[ch & 1];
                    const float4 *xs = reinterpret_cast<const float4 *>(xc);
                    const float4 *ws = reinterpret_cast<const float4 *>(wc);
                    const int32_t len = min(kStage, e - b - ch * kStage);
                    // 32 steps at a time; each half's operands are read while the other half runs
                    float4 xa[4], wa[4], xb[4], wb[4];
                    const auto load = [&](float4 (&xr)[4], float4 (&wr)[4], int32_t g) {
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            xr[j] = xs[4 * g + j];
                            wr[j] = ws[4 * g + j];
                        }
                    };
                    const auto steps = [&](const float4 (&xr)[4], const float4 (&wr)[4]) {
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            acc = __builtin_fmaf(wr[j].x, xr[j].x, acc);
                            acc = __builtin_fmaf(wr[j].y, xr[j].y, acc);
                            acc = __builtin_fmaf(wr[j].z, xr[j].z, acc);
                            acc = __builtin_fmaf(wr[j].w, xr[j].w, acc);
                        }
                    };
                    const int32_t pairs = len / 32;
                    load(xa, wa, 0);
                    for (int32_t p = 0; p < pairs; p++) {
                        load(xb, wb, 2 * p + 1);
                        __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the steps
                        steps(xa, wa);
                        __builtin_amdgcn_sched_barrier(0);
                        load(xa, wa, 2 * p + 2);  // past the chunk after its last pair: not used
                        __builtin_amdgcn_sched_barrier(0);
                        steps(xb, wb);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    for (int32_t q = pairs * 32; q < len; q++) acc = __builtin_fmaf(wc[q], xc[q], acc);
                }
                __syncthreads();
            }
            if ((int32_t)threadIdx.x < cols) {
                const int64_t i = (int64_t)v * COLS + c0 + threadIdx.x;
                out[i] = WALK ? (X[i] + acc * rinv[v]) * 0.5f : acc * rinv[v];
            }
        }
        return;
    }
    // ---- rows of at most kWideRow entries
    constexpr int GL = COLS <= 16 ? 16 : (COLS <= 32 ? 32 : 64), NG = kGatherBlock / GL;
    constexpr int UB = 16;
    const int32_t c = threadIdx.x % GL, grp = threadIdx.x / GL;
    const int32_t cc = c < COLS ? c : 0;
    for (int32_t v0 = (blockIdx.x - wblocks) * NG; v0 < n; v0 += (gridDim.x - wblocks) * NG) {
        const int32_t v = v0 + grp;
        const int32_t b = v < n ? xadj[v] : 0;
        int32_t e = v < n ? xadj[v + 1] : 0;
        const bool mine = v < n && e - b <= kWideRow;
        if (!mine) e = b;
        float acc = 0.0f;
        const int32_t chunks = wave_max((e - b + GL - 1) / GL);
        int32_t u = b + c < e ? adjncy[b + c] : 0;
        float w = b + c < e && adjwgt ? (float)adjwgt[b + c] : 1.0f;
        for (int32_t ch = 0; ch < chunks; ch++) {
            const int32_t nq = b + (ch + 1) * GL + c;
            const int32_t nu = nq < e ? adjncy[nq] : 0;
            const float nw = nq < e && adjwgt ? (float)adjwgt[nq] : 1.0f;
#pragma unroll
            for (int s0 = 0; s0 < GL; s0 += UB) {
                const int32_t left = e - (b + ch * GL + s0);  // entries of the row from here on
                if (__ballot(left > 0) == 0) break;
                float xv[UB], ws[UB];
#pragma unroll
                for (int j = 0; j < UB; j++) {
                    xv[j] = X[(int64_t)__shfl(u, s0 + j, GL) * COLS + cc];
                    ws[j] = __shfl(w, s0 + j, GL);
                }
#pragma unroll
                for (int j = 0; j < UB; j++) {
                    const float f = __builtin_fmaf(ws[j], xv[j], acc);
                    acc = j < left ? f : acc;
                }
            }
            u = nu;
            w = nw;
        }
        if (mine && c < COLS) {
            const int64_t i = (int64_t)v * COLS + c;
            if (WALK) {
                const float self = X[i];
                out[i] = e > b ? (self + acc * rinv[v]) * 0.5f : self;
            } else {
                out[i] = e > b ? acc * rinv[v] : 0.0f;
            }
        }
    }
}

struct ActiveFlag {
    const int32_t *xadj;
    __device__ bool operator()(int64_t v) const { return xadj[v + 1] > xadj[v]; }
};
struct RankEmit {
    int32_t *rank;
    __device__ void operator()(int64_t v, int32_t pos) const { rank[v] = pos; }
};

// y_0[v][j] = -1 if the top bit of splitmix(splitmix(seed) ^ (16 id + j)) is set, else +1
__global__ void k_probes(int32_t n, uint64_t seed, const int32_t *__restrict__ rank, float *__restrict__ Y) {
    const uint64_t base = splitmix(seed);
    const int64_t N = (int64_t)n * kMpProbe;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = (int32_t)(i / kMpProbe), j = (int32_t)(i % kMpProbe);
        const uint64_t id = rank ? (uint64_t)rank[v] : (uint64_t)v;
        Y[i] = (splitmix(base ^ (id * kMpProbe + (uint64_t)j)) >> 63) ? -1.0f : 1.0f;
    }
}

__global__ void k_features(int32_t n, const int32_t *__restrict__ xadj, const int32_t *__restrict__ vwgt,
                           const int32_t *__restrict__ mx, const float *__restrict__ Y, float *__restrict__ X) {
    const double cmax = (double)mx[0];
    const int32_t dmax = mx[1];
    const int64_t N = (int64_t)n * kMpFeat;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = (int32_t)(i / kMpFeat), f = (int32_t)(i % kMpFeat);
        float x;
        if (f == 0) x = (float)((double)(vwgt ? vwgt[v] : 1) / cmax);
        else if (f == 1) x = dmax > 0 ? (float)((double)(xadj[v + 1] - xadj[v]) / (double)dmax) : 0.0f;
        else x = Y[(int64_t)v * kMpProbe + (f - 2)];
        X[i] = x;
    }
}

// Hidden layers: O[v][o] = ReLU(b[o] + sum_i Ws[o][i] H[v][i] + sum_i Wn[o][i] M[v][i]),
// lane o of a wave is output o, weights transposed in LDS. A wave takes VB
// vertices at a time, so a weight read from LDS serves VB chains, and their
// inputs (the same for all lanes) come through scalar loads. Bound: the LDS
// reads; 71 us a layer of 64 inputs at 50,000 vertices with one vertex per wave, 44 so.
template <int DIN>
__global__ __launch_bounds__(kMB) void k_hidden(int32_t n, const float *__restrict__ H, const float *__restrict__ M,
                                                const float *__restrict__ Ws, const float *__restrict__ Wn,
                                                const float *__restrict__ bias, float *__restrict__ O) {
    constexpr int VB = 4, NW = kMB / kWave;
    __shared__ float sWs[DIN * kMpHid], sWn[DIN * kMpHid];
    for (int32_t t = threadIdx.x; t < DIN * kMpHid; t += kMB) {
        const int32_t o = t / DIN, i = t % DIN;
        sWs[i * kMpHid + o] = Ws[t];
        sWn[i * kMpHid + o] = Wn[t];
    }
    __syncthreads();
    const int lane = lane_id();
    const float bo = bias[lane];
    const int32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * NW + threadIdx.x / kWave);
    for (int32_t v0 = wave * VB; v0 < n; v0 += gridDim.x * NW * VB) {
        float acc[VB];
        const float *h[VB], *m[VB];
#pragma unroll
        for (int j = 0; j < VB; j++) {
            const int64_t v = min(v0 + j, n - 1);
            acc[j] = bo;
            h[j] = H + v * DIN;
            m[j] = M + v * DIN;
        }
#pragma unroll 8
        for (int i = 0; i < DIN; i++) {
            const float w = sWs[i * kMpHid + lane];
#pragma unroll
            for (int j = 0; j < VB; j++) acc[j] = __builtin_fmaf(w, h[j][i], acc[j]);
        }
#pragma unroll 8
        for (int i = 0; i < DIN; i++) {
            const float w = sWn[i * kMpHid + lane];
#pragma unroll
            for (int j = 0; j < VB; j++) acc[j] = __builtin_fmaf(w, m[j][i], acc[j]);
        }
#pragma unroll
        for (int j = 0; j < VB; j++)
            if (v0 + j < n) O[(int64_t)(v0 + j) * kMpHid + lane] = acc[j] > 0.0f ? acc[j] : 0.0f;
    }
}

// The head: Z[v][o] = b[o] + sum_i W[o][i] H[v][i] with the weights staged
// transposed in LDS (lane o reads consecutive words). `dp` lanes (a power of
// two >= dout) serve one vertex.
__global__ __launch_bounds__(kMB) void k_head(int32_t n, int32_t din, int32_t dout, int32_t dp,
                                              const float *__restrict__ H, const float *__restrict__ W,
                                              const float *__restrict__ bias, float *__restrict__ O) {
    __shared__ float sW[kMpHid * kMpHid], sb[kMpHid];
    for (int32_t t = threadIdx.x; t < din * dout; t += kMB) {
        const int32_t o = t / din, i = t % din;
        sW[i * dout + o] = W[t];
    }
    for (int32_t t = threadIdx.x; t < dout; t += kMB) sb[t] = bias[t];
    __syncthreads();
    const int32_t o = threadIdx.x % dp, vpb = kMB / dp;
    if (o >= dout) return;
    for (int64_t v = (int64_t)blockIdx.x * vpb + threadIdx.x / dp; v < n; v += (int64_t)gridDim.x * vpb) {
        const float *h = H + v * din;
        float acc = sb[o];
        for (int32_t i = 0; i < din; i++) acc = __builtin_fmaf(sW[i * dout + o], h[i], acc);
        O[v * dout + o] = acc;
    }
}

__global__ void k_argmax(int32_t n, int32_t k, const float *__restrict__ Z, const int32_t *__restrict__ xadj,
                         bool active_only, int32_t *__restrict__ part, int32_t *__restrict__ nonfinite) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const float *z = Z + (int64_t)v * k;
        int32_t best = 0;
        bool fin = isfinite(z[0]);
        for (int32_t c = 1; c < k; c++) {
            fin &= isfinite(z[c]);
            if (z[c] > z[best]) best = c;
        }
        if (part) part[v] = best;
        if (nonfinite && !fin && (!active_only || xadj[v + 1] > xadj[v])) atomicOr(nonfinite, 1);
    }
}

// ------------------------------------------------------------------ decoding
// Every vertex ranks the blocks by logit (highest first, ties -> lower block);
// round r offers each unplaced vertex's r-th block, and the offers to block t
// are admitted in ascending vertex id while B[t] + (weight of all offers to t
// up to and including v) <= lmax; leftovers go one by one, ascending, to the
// lightest block.

// pref[v][rank] = block; part[v] = -1 (unplaced) or -2 (takes no part)
__global__ void k_prefs(int32_t n, int32_t k, const float *__restrict__ Z, const int32_t *__restrict__ xadj,
                        bool active_only, uint8_t *__restrict__ pref, int32_t *__restrict__ part) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const float *z = Z + (int64_t)v * k;
        for (int32_t c = 0; c < k; c++) {
            const float zc = z[c];
            int32_t rank = 0;
            for (int32_t d = 0; d < k; d++) rank += (z[d] > zc) || (z[d] == zc && d < c);
            pref[(int64_t)v * k + rank] = (uint8_t)c;
        }
        part[v] = (active_only && xadj[v + 1] == xadj[v]) ? -2 : -1;
    }
}

constexpr int kDB = 1024;

// one workgroup per block t: admit round r's offers to t in ascending id
__global__ __launch_bounds__(kDB) void k_decode_round(int32_t n, int32_t k, int32_t r, const uint8_t *__restrict__ pref,
                                                      const int32_t *__restrict__ vwgt, int64_t lmax,
                                                      int64_t *__restrict__ B, int32_t *__restrict__ part) {
    __shared__ int64_t tmp[kDB / kWave + 1];
    const int32_t t = blockIdx.x;
    int64_t run = B[t], admitted = 0;
    for (int32_t base = 0; base < n; base += kDB) {
        const int32_t v = base + threadIdx.x;
        int64_t c = 0;
        // only this workgroup changes part[v] for offers to t in this round
        if (v < n && part[v] == -1 && pref[(int64_t)v * k + r] == t) c = vwgt ? vwgt[v] : 1;
        int64_t total;
        const int64_t excl = block_excl_scan<kDB>(c, tmp, &total);
        const bool ok = c > 0 && run + excl + c <= lmax;
        if (ok) part[v] = t;
        admitted += block_sum<kDB>(ok ? c : (int64_t)0, tmp);
        run += total;
    }
    if (threadIdx.x == 0) B[t] += admitted;
}

// unplaced vertices, ascending, each into the currently lightest block. One
// workgroup reads the assignment in 256-vertex chunks; thread 0 then places
// that chunk's unplaced vertices in order (block weights in LDS).
constexpr int kLeftBlock = 256;
__global__ __launch_bounds__(kLeftBlock) void k_decode_leftover(int32_t n, int32_t k,
                                                                const int32_t *__restrict__ vwgt,
                                                                int64_t *__restrict__ B, int32_t *__restrict__ part) {
    __shared__ int64_t sB[kMpMaxK];
    __shared__ uint8_t sleft[kLeftBlock];
    if (blockIdx.x != 0) return;
    for (int32_t t = threadIdx.x; t < k; t += kLeftBlock) sB[t] = B[t];
    for (int32_t v0 = 0; v0 < n; v0 += kLeftBlock) {
        const int32_t v = v0 + threadIdx.x;
        uint8_t left = 0;
        if (v < n) {
            const int32_t p = part[v];
            if (p == -2) part[v] = 0;  // takes no part: any valid block id
            left = p == -1;
        }
        sleft[threadIdx.x] = left;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int32_t i = 0; i < kLeftBlock; i++) {
                if (!sleft[i]) continue;
                int32_t b = 0;
                for (int32_t t = 1; t < k; t++)
                    if (sB[t] < sB[b]) b = t;
                part[v0 + i] = b;
                sB[b] += vwgt ? vwgt[v0 + i] : 1;
            }
        }
        __syncthreads();
    }
    for (int32_t t = threadIdx.x; t < k; t += kLeftBlock) B[t] = sB[t];
}

// ------------------------------------------------------------------ training

// S = softmax(Z): `kp` lanes (a power of two >= k) per vertex.
__global__ __launch_bounds__(kMB) void k_softmax(int32_t n, int32_t k, int32_t kp, const float *__restrict__ Z,
                                                 float *__restrict__ S) {
    const int32_t c = threadIdx.x % kp, vpb = kMB / kp;
    for (int64_t v = (int64_t)blockIdx.x * vpb + threadIdx.x / kp; v < n; v += (int64_t)gridDim.x * vpb) {
        const float z = c < k ? Z[v * k + c] : -INFINITY;
        float m = z;
        for (int32_t d = kp / 2; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, kp));
        const float x = c < k ? __expf(z - m) : 0.0f;
        float s = x;
        for (int32_t d = kp / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, kp);
        if (c < k) S[v * k + c] = x * (1.0f / s);
    }
}

constexpr float kPClip = 1e-6f;

// Edge term of the loss: for every directed edge (v,u), p = <S_v, S_u> and
// BCE against [t_v == t_u], weighted by w(v,u)/Omega. gS[v] collects the
// gradient w.r.t. S_v from both directions of each edge (2 * dl/dp * S_u).
// One workgroup per vertex, `kp` lanes (a power of two >= k) per edge, so a row
// takes kMB / kp edges at a time: with kp lanes per vertex the widest row set
// the time (277 us at 835 vertices and 28,000 entries, 24 us so).
__global__ __launch_bounds__(kMB) void k_edge_loss(int32_t n, int32_t k, int32_t kp, const int32_t *__restrict__ xadj,
                                                   const int32_t *__restrict__ adjncy,
                                                   const int32_t *__restrict__ adjwgt,
                                                   const int32_t *__restrict__ target, const float *__restrict__ S,
                                                   const int64_t *__restrict__ omega, float *__restrict__ gS,
                                                   double *__restrict__ loss) {
    __shared__ float sg[kMB];
    __shared__ double sl[kMB / kWave + 1];
    const float inv_omega = *omega > 0 ? (float)(1.0 / (double)*omega) : 0.0f;
    const int32_t c = threadIdx.x % kp, grp = threadIdx.x / kp, ng = kMB / kp;
    double lsum = 0.0;
    for (int64_t v = blockIdx.x; v < n; v += gridDim.x) {
        const float sv = c < k ? S[v * k + c] : 0.0f;
        const int32_t tv = target[v];
        const int32_t b = xadj[v], e = xadj[v + 1];
        float g = 0.0f, l = 0.0f;
        for (int32_t q = b + grp; q < e; q += ng) {
            const int32_t u = adjncy[q];
            const float su = c < k ? S[(int64_t)u * k + c] : 0.0f;
            float p = sv * su;
            for (int32_t d = kp / 2; d > 0; d >>= 1) p += __shfl_xor(p, d, kp);
            const float w = (adjwgt ? (float)adjwgt[q] : 1.0f) * inv_omega;
            const bool y = target[u] == tv;
            const float pc = fminf(fmaxf(p, kPClip), 1.0f - kPClip);
            l += w * -(y ? __logf(pc) : __logf(1.0f - pc));
            const bool inside = p > kPClip && p < 1.0f - kPClip;
            const float dldp = inside ? (y ? -1.0f / pc : 1.0f / (1.0f - pc)) : 0.0f;
            g += 2.0f * w * dldp * su;
        }
        if (c == 0) lsum += l;
        sg[threadIdx.x] = g;
        __syncthreads();
        for (int32_t h = ng / 2; h > 0; h >>= 1) {  // ng is a power of two
            if (grp < h) sg[threadIdx.x] += sg[threadIdx.x + h * kp];
            __syncthreads();
        }
        if ((int32_t)threadIdx.x < k) gS[v * k + threadIdx.x] = sg[threadIdx.x];
        __syncthreads();
    }
    lsum = block_sum<kMB>(lsum, sl);
    if (threadIdx.x == 0 && lsum != 0.0) atomicAdd(loss, lsum);
}

// Q[c] = sum_v c(v) S[v][c], products and sums in binary64: the balance term is
// the difference of Q / C and 1 / k, so what is lost here grows by the ratio of
// the two (binary32 sums per workgroup, added up in the order in which lanes came,
// moved the balance loss by up to 2e-5 from call to call at k = 2). `kp` lanes (a
// power of two >= k) per vertex.
__global__ __launch_bounds__(kMB) void k_colsum(int32_t n, int32_t k, int32_t kp, const float *__restrict__ S,
                                                const int32_t *__restrict__ vwgt, double *__restrict__ Q) {
    __shared__ double part[kMB];
    const int32_t c = threadIdx.x % kp, grp = threadIdx.x / kp, vpb = kMB / kp;
    double s = 0.0;
    if (c < k)
        for (int64_t v = (int64_t)blockIdx.x * vpb + grp; v < n; v += (int64_t)gridDim.x * vpb)
            s += (double)S[v * k + c] * (vwgt ? (double)vwgt[v] : 1.0);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int32_t h = vpb / 2; h > 0; h >>= 1) {  // vpb is a power of two
        if (grp < h) part[threadIdx.x] += part[threadIdx.x + h * kp];
        __syncthreads();
    }
    if ((int32_t)threadIdx.x < k) atomicAdd(&Q[threadIdx.x], part[threadIdx.x]);
}

// dZ = S * (g - <S, g>) with g = gS + balance term 2 lam k (Q_c/C - 1/k) c(v)/C;
// `kp` lanes (a power of two >= k) per vertex.
__global__ __launch_bounds__(kMB) void k_softmax_back(int32_t n, int32_t k, int32_t kp, const float *__restrict__ S,
                                                      const float *__restrict__ gS, const double *__restrict__ Q,
                                                      const int64_t *__restrict__ C, float lam,
                                                      const int32_t *__restrict__ vwgt, float *__restrict__ dZ) {
    const int32_t c = threadIdx.x % kp, vpb = kMB / kp;
    const double invC = 1.0 / (double)*C;
    const float bal = c < k ? (float)(2.0 * lam * k * (Q[c] * invC - 1.0 / k)) : 0.0f;
    for (int64_t v = (int64_t)blockIdx.x * vpb + threadIdx.x / kp; v < n; v += (int64_t)gridDim.x * vpb) {
        const float cv = (float)((vwgt ? (double)vwgt[v] : 1.0) * invC);
        const float s = c < k ? S[v * k + c] : 0.0f;
        const float g = c < k ? gS[v * k + c] + bal * cv : 0.0f;
        float dot = s * g;
        for (int32_t d = kp / 2; d > 0; d >>= 1) dot += __shfl_xor(dot, d, kp);
        if (c < k) dZ[v * k + c] = s * (g - dot);
    }
}

// C = total vertex weight (whole numbers: any order)
__global__ __launch_bounds__(kMB) void k_vsum(int32_t n, const int32_t *__restrict__ vwgt, int64_t *__restrict__ C) {
    __shared__ int64_t tmp[kMB / kWave + 1];
    int64_t s = 0;
    for (int64_t v = (int64_t)blockIdx.x * kMB + threadIdx.x; v < n; v += (int64_t)gridDim.x * kMB)
        s += vwgt ? vwgt[v] : 1;
    s = block_sum<kMB>(s, tmp);
    if (threadIdx.x == 0) atomicAdd((unsigned long long *)C, (unsigned long long)s);
}

constexpr int kWgChunk = 16;
constexpr int kWgTile = 4;                             // outputs x inputs of one thread
constexpr int kWgPitch = kMpHid + kWgTile;
static_assert(kMpMaxK <= kMpHid, "a chunk's rows of A fit kWgPitch");

// gW[o][i] += sum_v A[v][o] B[v][i]; gb[o] += sum_v A[v][o] (when gb != null),
// for one or two matrices B (blockIdx.y) with the same A. A workgroup stages
// kWgChunk rows of A and B in LDS; a thread keeps a 4 x 4 tile of the sums in
// registers (eight LDS words per sixteen products), one atomic per entry and
// workgroup at the end. A workgroup takes kWgRows rows at a time: the fewer
// workgroups, the fewer atomics, and the fewer binary32 sums meet in the gradient.
// (Its error against binary64 is that of the untiled kernel before: 0.80 to 1.25 of
// it on 12 graphs of 300 to 1500 vertices, 0.99 on average, as repeats differ.)
constexpr int kWgPer = 4, kWgRows = kWgPer * kWgChunk;
struct WGrad {
    const float *B;
    float *gW, *gb;
};
__global__ __launch_bounds__(kMB) void k_wgrad(int32_t n, int32_t dout, int32_t din, const float *__restrict__ A,
                                               WGrad first, WGrad second) {
    __shared__ __align__(16) float sA[kWgChunk * kWgPitch], sB[kWgChunk * kWgPitch];
    const WGrad w = blockIdx.y == 0 ? first : second;
    const int32_t o0 = threadIdx.x / (kMpHid / kWgTile) * kWgTile, i0 = threadIdx.x % (kMpHid / kWgTile) * kWgTile;
    float acc[kWgTile][kWgTile] = {}, bsum = 0.0f;
    for (int64_t i = 0, base = (int64_t)blockIdx.x * kWgRows; base < n;
         i++, base = ((int64_t)blockIdx.x + i / kWgPer * gridDim.x) * kWgRows + i % kWgPer * kWgChunk) {
        const int32_t rows = (int32_t)min<int64_t>(kWgChunk, n - base);
        __syncthreads();
        for (int32_t t = threadIdx.x; t < kWgChunk * kMpHid; t += kMB) {
            const int32_t r = t / kMpHid, x = t % kMpHid;
            sA[r * kWgPitch + x] = r < rows && x < dout ? A[(base + r) * dout + x] : 0.0f;
            sB[r * kWgPitch + x] = r < rows && x < din ? w.B[(base + r) * din + x] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kWgChunk; q++) {
            const float4 x = *reinterpret_cast<const float4 *>(sA + q * kWgPitch + o0);
            const float4 y = *reinterpret_cast<const float4 *>(sB + q * kWgPitch + i0);
            const float xa[4] = {x.x, x.y, x.z, x.w}, ya[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
            for (int o = 0; o < kWgTile; o++)
#pragma unroll
                for (int i = 0; i < kWgTile; i++) acc[o][i] = __builtin_fmaf(xa[o], ya[i], acc[o][i]);
            if (threadIdx.x < kMpHid) bsum += sA[q * kWgPitch + threadIdx.x];
        }
    }
#pragma unroll
    for (int o = 0; o < kWgTile; o++)
#pragma unroll
        for (int i = 0; i < kWgTile; i++)
            if (o0 + o < dout && i0 + i < din) atomicAdd(&w.gW[(o0 + o) * din + i0 + i], acc[o][i]);
    if (w.gb && (int32_t)threadIdx.x < dout) atomicAdd(&w.gb[threadIdx.x], bsum);
}

// out1[v][i] = sum_o W1[o][i] D[v][o]; out2 likewise with W2 (when given).
// mask (when given): out1[v][i] = 0 where !(mask[v][i] > 0) (the ReLU below).
__global__ __launch_bounds__(kMB) void k_dense_t(int32_t n, int32_t dout, int32_t din, const float *__restrict__ D,
                                                 const float *__restrict__ W1, const float *__restrict__ W2,
                                                 const float *__restrict__ mask, float *__restrict__ out1,
                                                 float *__restrict__ out2) {
    __shared__ float s1[kMpHid * kMpMaxK], s2[kMpHid * kMpMaxK];
    for (int32_t t = threadIdx.x; t < din * dout; t += kMB) {
        s1[t] = W1[t];
        if (W2) s2[t] = W2[t];
    }
    __syncthreads();
    const int64_t N = (int64_t)n * din;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < N; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = t / din;
        const int32_t i = (int32_t)(t % din);
        const float *d = D + v * dout;
        float a = 0.0f, b = 0.0f;
        for (int32_t o = 0; o < dout; o++) {
            a += s1[o * din + i] * d[o];
            if (W2) b += s2[o * din + i] * d[o];
        }
        out1[t] = mask && !(mask[t] > 0.0f) ? 0.0f : a;
        if (W2) out2[t] = b;
    }
}

// out[u][i] = (out[u][i] + sum_{v in N(u)} w(u,v) dM[v][i] / d(v)) [mask[u][i] > 0]:
// the transpose of the aggregation, then the ReLU of the layer below. One
// workgroup per row, a lane per column, the row's entries dealt to the waves 16
// at a time (88 us with a lane per output at 835 vertices, 9 us so).
__global__ __launch_bounds__(kMB) void k_aggregate_t(int32_t n, const int32_t *__restrict__ xadj,
                                                     const int32_t *__restrict__ adjncy,
                                                     const int32_t *__restrict__ adjwgt,
                                                     const float *__restrict__ rinv, const float *__restrict__ dM,
                                                     const float *__restrict__ mask, float *__restrict__ out) {
    constexpr int NW = kMB / kWave, UB = 16;
    __shared__ float part[NW][kMpHid];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    for (int32_t u = blockIdx.x; u < n; u += gridDim.x) {
        const int32_t b = xadj[u], e = xadj[u + 1];
        float acc = 0.0f;
        for (int32_t q0 = b + w * UB; q0 < e; q0 += NW * UB) {
            const int32_t q = q0 + (lane & (UB - 1));
            const int32_t v = q < e ? adjncy[q] : 0;
            const float f = q < e ? (adjwgt ? (float)adjwgt[q] : 1.0f) * rinv[v] : 0.0f;
            float x[UB];
#pragma unroll
            for (int j = 0; j < UB; j++) x[j] = dM[(int64_t)__shfl(v, j, kWave) * kMpHid + lane];
#pragma unroll
            for (int j = 0; j < UB; j++) {
                const float t = __builtin_fmaf(__shfl(f, j, kWave), x[j], acc);
                acc = q0 + j < e ? t : acc;
            }
        }
        part[w][lane] = acc;
        __syncthreads();
        if (w == 0) {
            const int64_t i = (int64_t)u * kMpHid + lane;
            float t = out[i];
#pragma unroll
            for (int j = 0; j < NW; j++) t += part[j][lane];
            out[i] = mask[i] > 0.0f ? t : 0.0f;
        }
        __syncthreads();
    }
}

__global__ void k_adam(int32_t count, float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

int pow2_at_least(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

struct Net {  // offsets of the parameter blocks
    int64_t ws[3], wn[3], b[3], wh, bh;
    explicit Net(int32_t k) {
        int64_t o = 0;
        const int din[3] = {kMpFeat, kMpHid, kMpHid};
        for (int l = 0; l < 3; l++) {
            ws[l] = o;
            o += (int64_t)kMpHid * din[l];
            wn[l] = o;
            o += (int64_t)kMpHid * din[l];
            b[l] = o;
            o += kMpHid;
        }
        wh = o;
        o += (int64_t)kMpHid * k;
        bh = o;
        (void)k;
    }
};

// the rows above kWideRow entries (device list and count)
struct WideRows {
    int32_t *list = nullptr, *count = nullptr;
};
int wide_rows(const DevGraph &g, WideRows &w, Scratch &sc) {
    GP_TRY(sc.alloc(&w.list, g.n));
    GP_TRY(sc.alloc(&w.count, 1));
    GP_HIP(hipMemsetAsync(w.count, 0, sizeof(int32_t), sc.stream()));
    return compact(WideFlag{g.xadj}, WideEmit{w.list}, g.n, nullptr, w.count, sc);
}

// at most this many: each has more than kWideRow of the entries
int64_t wide_most(const DevGraph &g) { return std::min<int64_t>(g.n, (int64_t)g.nnz / (kWideRow + 1)); }

template <int COLS, bool WALK>
int gather(const DevGraph &g, const WideRows &w, const float *rinv, const float *X, float *out, hipStream_t s) {
    constexpr int GL = COLS <= 16 ? 16 : (COLS <= 32 ? 32 : 64);
    const int64_t most = wide_most(g) * ((COLS + kSlice - 1) / kSlice);
    const unsigned wb = most > 0 ? grid_for(most, 1, 4096) : 0;
    hipLaunchKernelGGL((k_gather<COLS, WALK>), dim3(wb + grid_for(g.n, kGatherBlock / GL, 1 << 15)), dim3(kGatherBlock), 0, s, g.n,
                       w.list, w.count, (int32_t)wb, g.xadj, g.adjncy, g.adjwgt, rinv, X, out);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

// X: [n][18] features; rinv (may be null): receives 1/d(v)
int features(const DevGraph &g, uint64_t seed, bool active_only, float *X, float *rinv, const WideRows &wide,
             Scratch &sc) {
    hipStream_t s = sc.stream();
    const int32_t n = g.n;
    float *r = rinv, *Ya = nullptr, *Yb = nullptr;
    int32_t *mx = nullptr, *rank = nullptr, *cnt = nullptr;
    if (!r) GP_TRY(sc.alloc(&r, n));
    GP_TRY(sc.alloc(&Ya, (size_t)n * kMpProbe));
    GP_TRY(sc.alloc(&Yb, (size_t)n * kMpProbe));
    GP_TRY(sc.alloc(&mx, 2));
    GP_HIP(hipMemsetAsync(mx, 0, sizeof(int32_t) * 2, s));
    const unsigned wb = wide_most(g) > 0 ? grid_for(wide_most(g), 1, 512) : 0;
    hipLaunchKernelGGL(k_vstats, dim3(wb + grid_for(n, kMB / 16, 1024)), dim3(kMB), 0, s, n, wide.list, wide.count,
                       (int32_t)wb, g.xadj, g.adjwgt, g.vwgt, active_only, r, mx);
    GP_LAUNCH_CHECK();
    if (active_only) {
        GP_TRY(sc.alloc(&rank, n));
        GP_TRY(sc.alloc(&cnt, 1));
        GP_HIP(hipMemsetAsync(rank, 0, sizeof(int32_t) * (size_t)n, s));
        GP_TRY(compact(ActiveFlag{g.xadj}, RankEmit{rank}, n, nullptr, cnt, sc));
    }
    hipLaunchKernelGGL(k_probes, dim3(grid_for((int64_t)n * kMpProbe, 256, 1 << 16)), dim3(256), 0, s, n, seed, rank,
                       Ya);
    GP_LAUNCH_CHECK();
    for (int t = 0; t < kMpWalk; t++) {
        GP_TRY((gather<kMpProbe, true>(g, wide, r, Ya, Yb, s)));
        std::swap(Ya, Yb);
    }
    hipLaunchKernelGGL(k_features, dim3(grid_for((int64_t)n * kMpFeat, 256, 1 << 16)), dim3(256), 0, s, n, g.xadj,
                       g.vwgt, mx, Ya, X);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

struct Acts {  // forward activations kept for the backward pass
    float *X = nullptr, *rinv = nullptr, *H[3] = {}, *M[3] = {}, *Z = nullptr, *Wt = nullptr;
};

int run_forward(const DevGraph &g, int32_t k, const float *params, uint64_t seed, bool active_only, Acts &a,
                Scratch &sc) {
    hipStream_t s = sc.stream();
    const int32_t n = g.n, P = mpnn_param_count(k);
    GP_TRY(sc.alloc(&a.X, (size_t)n * kMpFeat));
    GP_TRY(sc.alloc(&a.rinv, n));
    GP_TRY(sc.alloc(&a.Wt, P));
    for (int l = 0; l < 3; l++) {
        GP_TRY(sc.alloc(&a.H[l], (size_t)n * kMpHid));
        GP_TRY(sc.alloc(&a.M[l], (size_t)n * (l == 0 ? kMpFeat : kMpHid)));
    }
    GP_TRY(sc.alloc(&a.Z, (size_t)n * k));
    hipLaunchKernelGGL(k_bf16, dim3(grid_for(P, 256, 256)), dim3(256), 0, s, params, a.Wt, P);
    GP_LAUNCH_CHECK();
    WideRows wide;
    GP_TRY(wide_rows(g, wide, sc));
    GP_TRY(features(g, seed, active_only, a.X, a.rinv, wide, sc));
    const Net net(k);
    const float *in = a.X;
    const unsigned gh = grid_for(n, 4 * (kMB / kWave), 2048);
    for (int l = 0; l < 3; l++) {
        const float *ws = a.Wt + net.ws[l], *wn = a.Wt + net.wn[l], *bl = a.Wt + net.b[l];
        if (l == 0) {
            GP_TRY((gather<kMpFeat, false>(g, wide, a.rinv, in, a.M[l], s)));
            hipLaunchKernelGGL(k_hidden<kMpFeat>, dim3(gh), dim3(kMB), 0, s, n, in, a.M[l], ws, wn, bl, a.H[l]);
        } else {
            GP_TRY((gather<kMpHid, false>(g, wide, a.rinv, in, a.M[l], s)));
            hipLaunchKernelGGL(k_hidden<kMpHid>, dim3(gh), dim3(kMB), 0, s, n, in, a.M[l], ws, wn, bl, a.H[l]);
        }
        GP_LAUNCH_CHECK();
        in = a.H[l];
    }
    const int32_t kp = pow2_at_least(k);
    hipLaunchKernelGGL(k_head, dim3(grid_for(n, kMB / kp, 2048)), dim3(kMB), 0, s, n, kMpHid, k, kp, in,
                       a.Wt + net.wh, a.Wt + net.bh, a.Z);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

}  // namespace

int mpnn_features(const DevGraph &g, uint64_t seed, bool active_only, float *X, float *rinv, Scratch &sc) {
    if (g.n == 0) return GP_OK;
    WideRows wide;
    GP_TRY(wide_rows(g, wide, sc));
    return features(g, seed, active_only, X, rinv, wide, sc);
}

int mpnn_forward(const DevGraph &g, int32_t k, const float *params, uint64_t seed, bool active_only, float *Z,
                 int32_t *part, int32_t *nonfinite_dev, Scratch &sc) {
    if (g.n == 0) return GP_OK;
    Acts a;
    GP_TRY(run_forward(g, k, params, seed, active_only, a, sc));
    hipStream_t s = sc.stream();
    if (Z) GP_HIP(hipMemcpyAsync(Z, a.Z, sizeof(float) * (size_t)g.n * k, hipMemcpyDeviceToDevice, s));
    if (part || nonfinite_dev) {
        hipLaunchKernelGGL(k_argmax, dim3(grid_for(g.n, 256, 4096)), dim3(256), 0, s, g.n, k, a.Z, g.xadj,
                           active_only, part, nonfinite_dev);
        GP_LAUNCH_CHECK();
    }
    return GP_OK;
}

int mpnn_decode(const DevGraph &g, int32_t k, const float *Z, int64_t lmax, bool active_only, int32_t *part,
                Scratch &sc) {
    hipStream_t s = sc.stream();
    const int32_t n = g.n;
    if (n == 0) return GP_OK;
    uint8_t *pref = nullptr;
    int64_t *B = nullptr;
    GP_TRY(sc.alloc(&pref, (size_t)n * k));
    GP_TRY(sc.alloc(&B, k));
    GP_HIP(hipMemsetAsync(B, 0, sizeof(int64_t) * (size_t)k, s));
    hipLaunchKernelGGL(k_prefs, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, n, k, Z, g.xadj, active_only, pref,
                       part);
    GP_LAUNCH_CHECK();
    for (int32_t r = 0; r < k; r++) {
        hipLaunchKernelGGL(k_decode_round, dim3(k), dim3(kDB), 0, s, n, k, r, pref, g.vwgt, lmax, B, part);
        GP_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_decode_leftover, dim3(1), dim3(kLeftBlock), 0, s, n, k, g.vwgt, B, part);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

int mpnn_backward(const DevGraph &g, int32_t k, const float *params, uint64_t seed, const int32_t *target,
                  float lam, float *grad, double *loss_host, Scratch &sc) {
    hipStream_t s = sc.stream();
    const int32_t n = g.n, P = mpnn_param_count(k);
    GP_HIP(hipMemsetAsync(grad, 0, sizeof(float) * (size_t)P, s));
    if (n == 0) {
        if (loss_host) loss_host[0] = loss_host[1] = 0.0;
        return GP_OK;
    }
    Acts a;
    GP_TRY(run_forward(g, k, params, seed, false, a, sc));
    const int32_t kp = pow2_at_least(k);
    float *S = nullptr, *gS = nullptr, *dZ = nullptr, *dA = nullptr, *dB = nullptr, *dM = nullptr;
    double *acc = nullptr;  // [0] edge loss, [1..k] Q
    int64_t *tot = nullptr;  // Omega (sum of all directed edge weights), C (total vertex weight)
    GP_TRY(sc.alloc(&S, (size_t)n * k));
    GP_TRY(sc.alloc(&gS, (size_t)n * k));
    GP_TRY(sc.alloc(&dZ, (size_t)n * k));
    GP_TRY(sc.alloc(&dA, (size_t)n * kMpHid));
    GP_TRY(sc.alloc(&dB, (size_t)n * kMpHid));
    GP_TRY(sc.alloc(&dM, (size_t)n * kMpHid));
    GP_TRY(sc.alloc(&acc, (size_t)k + 4));
    tot = reinterpret_cast<int64_t *>(acc + k + 2);
    GP_HIP(hipMemsetAsync(acc, 0, sizeof(double) * ((size_t)k + 4), s));
    if (g.nnz > 0)
        hipLaunchKernelGGL(k_vsum, dim3(grid_for(g.nnz, kMB * 16, 256)), dim3(kMB), 0, s, g.nnz, g.adjwgt, tot);
    hipLaunchKernelGGL(k_vsum, dim3(grid_for(n, kMB * 16, 256)), dim3(kMB), 0, s, n, g.vwgt, tot + 1);
    const unsigned gk = grid_for(n, kMB / kp, 4096);
    hipLaunchKernelGGL(k_softmax, dim3(gk), dim3(kMB), 0, s, n, k, kp, a.Z, S);
    GP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_edge_loss, dim3(grid_for(n, 1, 1024)), dim3(kMB), 0, s, n, k, kp, g.xadj, g.adjncy,
                       g.adjwgt, target, S, tot, gS, acc);
    GP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_colsum, dim3(grid_for(n, (kMB / kp) * 8, 256)), dim3(kMB), 0, s, n, k, kp, S, g.vwgt,
                       acc + 1);
    GP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_softmax_back, dim3(gk), dim3(kMB), 0, s, n, k, kp, S, gS, acc + 1, tot + 1, lam, g.vwgt, dZ);
    GP_LAUNCH_CHECK();
    const Net net(k);
    const unsigned gw = grid_for(n, kWgRows, 512);
    // head
    hipLaunchKernelGGL(k_wgrad, dim3(gw), dim3(kMB), 0, s, n, k, kMpHid, dZ,
                       WGrad{a.H[2], grad + net.wh, grad + net.bh}, WGrad{});
    GP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_dense_t, dim3(grid_for((int64_t)n * kMpHid, 256, 4096)), dim3(kMB), 0, s, n, k, kMpHid, dZ,
                       a.Wt + net.wh, (const float *)nullptr, a.H[2], dA, (float *)nullptr);
    GP_LAUNCH_CHECK();
    for (int l = 2; l >= 0; l--) {
        const int32_t din = l == 0 ? kMpFeat : kMpHid;
        const float *Hin = l == 0 ? a.X : a.H[l - 1];
        hipLaunchKernelGGL(k_wgrad, dim3(gw, 2), dim3(kMB), 0, s, n, kMpHid, din, dA,
                           WGrad{Hin, grad + net.ws[l], grad + net.b[l]}, WGrad{a.M[l], grad + net.wn[l], nullptr});
        GP_LAUNCH_CHECK();
        if (l == 0) break;
        hipLaunchKernelGGL(k_dense_t, dim3(grid_for((int64_t)n * din, 256, 4096)), dim3(kMB), 0, s, n, kMpHid, din,
                           dA, a.Wt + net.ws[l], a.Wt + net.wn[l], (const float *)nullptr, dB, dM);
        GP_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_aggregate_t, dim3(grid_for(n, 1, 8192)), dim3(kMB), 0, s, n, g.xadj, g.adjncy, g.adjwgt,
                           a.rinv, dM, a.H[l - 1], dB);
        GP_LAUNCH_CHECK();
        std::swap(dA, dB);
    }
    if (loss_host) {
        std::vector<double> h((size_t)k + 4);
        GP_HIP(hipMemcpyAsync(h.data(), acc, sizeof(double) * ((size_t)k + 4), hipMemcpyDeviceToHost, s));
        GP_HIP(hipStreamSynchronize(s));
        int64_t total;
        std::memcpy(&total, &h[k + 3], sizeof(total));
        const double C = (double)total;
        double bal = 0.0;
        for (int32_t c = 0; c < k; c++) {
            const double d = h[1 + c] / C - 1.0 / k;
            bal += d * d;
        }
        loss_host[0] = h[0];
        loss_host[1] = lam * k * bal;
    }
    return GP_OK;
}

int mpnn_adam(float *params, float *m, float *v, const float *grad, int32_t count, int32_t step, float lr, float b1,
              float b2, float eps, hipStream_t s) {
    const float c1 = 1.0f - std::pow(b1, (float)step), c2 = 1.0f - std::pow(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(count, 256, 1024)), dim3(256), 0, s, count, params, m, v, grad, lr, b1,
                       b2, eps, c1, c2);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

}  // namespace gp
