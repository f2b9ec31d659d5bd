// admit.hpp — admission of a round's proposals (§IV-A: a move happens only if
// the target is still feasible), included by lp.hip.
//
// The rule: the proposers to a target t are taken in ascending vertex id and
// admitted while W[t] + (weight of the proposers so far) <= cap(t), W at the
// round start. Weights are >= 1, so the admitted proposers of a target are
// exactly those below one vertex id; nothing has to be sorted to find it.
//
// Few labels against the vertices (k_dadm_*, up to 12,288 labels): per tile of
// consecutive vertices the proposed weight per target, a prefix over the tiles per
// target, and with it the one tile in which the target's room ends. Every tile
// before that admits, every tile after it refuses, and one workgroup per target
// takes that tile in order.
//
// More labels (k_sadm_*), as in clustering: the proposed weights are added to W at
// once. A target still within its bound admits everything. The proposers of the
// others (contested targets, usually few) are gathered per target, and one wave or
// workgroup per contested target finds the id where its room ends: by counting
// smaller ids for up to 64 proposers, else by a radix selection over the ids
// with weight histograms.
//
// Bound: one read of the proposals (4 bytes a vertex) in each of two kernels
// and the movers' own gathers. Before this form the movers were compacted,
// sorted by target and scanned (about 17 launches a round): on a 101 x 97 x 89
// weighted grid, k = 32, that took 6.6 ms of a 14 ms level.
//
// Atomics on one cache line from many workgroups take about 11 ns each here
// (they cross the XCDs), so counts and weight changes go through one store per
// workgroup and a sum in the last kernel, or through an LDS hash first. (By
// targets that is what a few hundred or thousand labels cost: nearly every
// proposer adds to a target that all tiles propose to. R-MAT-20, 3000 blocks: 226 us
// a round in its tally, apply and select.)
#pragma once
#include "lp.hpp"

namespace gp {

namespace {

// per-group round bookkeeping: gs[q] = {moves this round, previous moves, done, rounds_run, rounds seen}
struct GroupState {
    int32_t moves, prev, done, rounds_run, seen;
    int64_t total;
};

__device__ __forceinline__ int64_t vweight(const int32_t *vwgt, int32_t v) {
    return vwgt ? (int64_t)vwgt[v] : (int64_t)1;
}

constexpr int kDadmBlock = 256;
constexpr int kDadmChunk = 4096;     // vertices a workgroup takes at a time: 16 consecutive ones per thread
constexpr int kDenseAdm = 256, kDadmSome = 2048, kDadmMany = 8192, kDadmLabels = 12288;  // labels of the tiled form's variants
// (12,288 labels: a tile's sums are 24 bytes a vertex, which keeps a round's buffers
// within those of the sorted movers)
constexpr int kDadmMaxTiles = 2048;  // tiles of a round (larger graphs take more chunks per tile)
constexpr int kSadmBlock = 512;
constexpr int kSadmPer = 4;
constexpr int kSadmTile = kSadmBlock * kSadmPer;
constexpr int kSadmSlots = 2 * kSadmTile;  // LDS hash: a tile's targets leave it half empty
constexpr int kSadmLog = 12;
static_assert((1 << kSadmLog) == kSadmSlots, "LDS hash size");
constexpr int kSelBlock = 1024;
constexpr int kSelBits = 12;  // digit of the radix selection: two passes for up to 2^24 vertices
constexpr int kSelBins = 1 << kSelBits;

struct AdmitCtx {
    int32_t n, nlabels;
    int32_t *prop;  // [n] proposed label, -1: none; all -1 again after the round
    const int32_t *vwgt;
    int64_t *W;
    int64_t U;
    const int64_t *capv;
    int32_t *labels;
    uint8_t *lab8;
    LPDev *dev;
    const int32_t *group;
    GroupState *gs;
    uint8_t *act;  // active-set rounds: a refused vertex owes at least one evaluation
    uint8_t *todo;  // set by the movers' marks (refinement), null: none
    // the round's movers: tile i owns entries [i * tile, i * tile + tcnt[i])
    int32_t tile, ntiles;
    int32_t *mv;      // vertex
    int32_t *old;     // its label before the move, -1: refused
    int32_t *tcnt;    // [ntiles]
    int32_t *tmoves;  // [ncol] admitted movers per workgroup
    // few labels: by tiles
    int32_t ncol;        // workgroups of the apply kernel: one per label, then one per tile
    int64_t *part;       // [nlabels * ntiles] proposed weight of a tile, then the tile's weight change
    int32_t *cut;        // [nlabels] tile in which the label's room ends (ntiles: none)
    int64_t *cutroom;    // [nlabels] room left before that tile
    // more labels: by targets
    int32_t *cpos, *segv, *segp;  // [n] position among the target's proposers; their vertices and list entries
    int32_t *ccnt;                // [nlabels] proposers of a contested target, then their first slot; 0 between rounds
    int32_t *ct, *ctS;            // contested targets, their proposers
    int64_t *ctW;                 // W of a contested target with everything proposed
    int32_t *nct;                 // [2] contested targets, slots given out
    int vbits;
};

__device__ __forceinline__ int64_t cap_of(const AdmitCtx &c, int32_t t) { return c.capv ? c.capv[t] : c.U; }

// gs[q].moves counts the lanes with `moved` (one atomic when all are of one group); every lane calls it.
__device__ __forceinline__ void count_group(const AdmitCtx &c, int32_t v, bool moved) {
    const uint64_t mm = __ballot(moved);
    if (!mm) return;
    const int32_t q = moved ? c.group[v] : 0;
    const int32_t q0 = __shfl(q, __ffsll((unsigned long long)mm) - 1, kWave);
    if (__ballot(moved && q != q0) == 0) {
        if (lane_id() == 0) atomicAdd(&c.gs[q0].moves, (int32_t)__popcll(mm));
    } else if (moved) {
        atomicAdd(&c.gs[q].moves, 1);
    }
}

__device__ __forceinline__ void refuse(const AdmitCtx &c, int32_t v) {
    if (c.act && c.act[v] == 0) c.act[v] = 1;  // refused by capacity: evaluated again
}

// ---------------------------------------------------------------- few labels: by tiles

// The proposals of vertices v0 .. v0 + 15, -1 past the last vertex.
__device__ __forceinline__ void load16(const AdmitCtx &c, int64_t v0, int32_t (&t)[16]) {
    const int32_t *p = c.prop + v0;
    if (v0 + 16 > c.n) {
#pragma unroll
        for (int i = 0; i < 16; i++) t[i] = v0 + i < c.n ? p[i] : -1;
        return;
    }
    const int4 *q = reinterpret_cast<const int4 *>(p);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int4 x = q[i];
        t[4 * i] = x.x;
        t[4 * i + 1] = x.y;
        t[4 * i + 2] = x.z;
        t[4 * i + 3] = x.w;
    }
}

template <int LMAX>
__global__ __launch_bounds__(kDadmBlock) void k_dadm_tally(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ unsigned long long h[LMAX];
    for (int32_t i = threadIdx.x; i < c.nlabels; i += kDadmBlock) h[i] = 0;
    __syncthreads();
    const int32_t tile = blockIdx.x;
    for (int32_t o = 0; o < c.tile; o += kDadmChunk) {
        const int64_t v0 = (int64_t)tile * c.tile + o + threadIdx.x * 16;
        if (v0 >= c.n) break;
        int32_t t[16];
        load16(c, v0, t);
#pragma unroll
        for (int i = 0; i < 16; i++)
            if (t[i] >= 0) atomicAdd(&h[t[i]], (unsigned long long)vweight(c.vwgt, (int32_t)v0 + i));
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < c.nlabels; i += kDadmBlock) c.part[(int64_t)i * c.ntiles + tile] = (int64_t)h[i];
    if (threadIdx.x == 0) c.tcnt[tile] = 0;
}

// One workgroup per label: the first tile in which its proposers exceed the room.
__global__ __launch_bounds__(256) void k_dadm_cut(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ int64_t t64[256 / kWave + 1];
    __shared__ int32_t t32[256 / kWave + 1];
    const int32_t t = blockIdx.x;
    const int64_t room = cap_of(c, t) - c.W[t];
    const int64_t *x = c.part + (int64_t)t * c.ntiles;
    const int32_t per = (c.ntiles + 255) / 256;
    const int32_t i0 = threadIdx.x * per, i1 = min(i0 + per, c.ntiles);
    int64_t s = 0;
    for (int32_t i = i0; i < i1; i++) s += x[i];
    int64_t run = block_excl_scan<256>(s, t64, (int64_t *)nullptr);
    int32_t at = INT_MAX;
    for (int32_t i = i0; i < i1; i++) {
        if (run + x[i] > room) {
            at = i;
            break;
        }
        run += x[i];
    }
    const int32_t first = block_min<256>(at, t32);
    if (at == first && at != INT_MAX) {
        c.cut[t] = at;
        c.cutroom[t] = room - run;
    }
    if (threadIdx.x == 0 && first == INT_MAX) c.cut[t] = c.ntiles;
}

// The tiles' workgroups (one per tile) and the labels' (one per label, for the
// tile in which its room ends). Up to kDadmSome labels in one launch, with the
// weight changes of both in LDS. With more labels in a launch each: a label's
// workgroup has few movers then and adds their weights to W itself, without the
// LDS, whose clearing alone would be most of the launch (rgg of 16,385 vertices,
// 5000 blocks, 25 rounds: 2811 us with it, 1444 by targets).
template <int LMAX, bool TILES, bool LABELS>
__global__ __launch_bounds__(kDadmBlock) void k_dadm_apply(AdmitCtx c) {
    if (c.dev->done) return;
    constexpr bool LDS = TILES, CUTS = LDS && LMAX <= kDadmSome;
    __shared__ unsigned long long dw[LDS ? LMAX : 1];
    __shared__ int32_t scut[CUTS ? LMAX : 1];
    __shared__ int64_t t64[kDadmBlock / kWave + 1];
    __shared__ int32_t t32[kDadmBlock / kWave + 1];
    __shared__ int32_t sbase;
    const int32_t col = blockIdx.x + (LABELS ? 0 : c.nlabels);
    const bool ordered = LABELS && (!TILES || col < c.nlabels);  // takes the label's last tile in order
    const int32_t tile = ordered ? c.cut[col] : col - c.nlabels;
    if constexpr (LDS) {
        for (int32_t i = threadIdx.x; i < c.nlabels; i += kDadmBlock) {
            dw[i] = 0;
            if (CUTS && !ordered) scut[i] = c.cut[i];
        }
        __syncthreads();
    }
    int64_t gain = 0;  // without LDS: the weight this thread's movers bring to the label
    int32_t moves = 0;
    if (tile < c.ntiles) {
        const int64_t room = ordered ? c.cutroom[col] : 0;
        int64_t run = 0;
        for (int32_t o = 0; o < c.tile; o += kDadmChunk) {
            const int64_t v0 = (int64_t)tile * c.tile + o + threadIdx.x * 16;
            if ((int64_t)tile * c.tile + o >= c.n) break;  // uniform
            int32_t t[16];
            load16(c, v0, t);
            uint32_t adm = 0, mine = 0;  // bit i: vertex v0 + i is admitted; decided here
            if (ordered) {
                int64_t s = 0;
#pragma unroll
                for (int i = 0; i < 16; i++)
                    if (t[i] == col) s += vweight(c.vwgt, (int32_t)v0 + i);
                int64_t tot;
                int64_t pre = run + block_excl_scan<kDadmBlock>(s, t64, &tot);
                run += tot;
#pragma unroll
                for (int i = 0; i < 16; i++)
                    if (t[i] == col) {
                        pre += vweight(c.vwgt, (int32_t)v0 + i);
                        mine |= 1u << i;
                        if (pre <= room) adm |= 1u << i;
                    }
            } else {
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const int32_t cut = t[i] < 0 ? tile : CUTS ? scut[t[i]] : c.cut[t[i]];
                    if (tile != cut) {
                        mine |= 1u << i;
                        if (tile < cut) adm |= 1u << i;
                    }
                }
            }
            const int32_t cnt = __popc(adm);
            int32_t tot;
            int32_t at = block_excl_scan<kDadmBlock>(cnt, t32, &tot);
            if (tot) {  // uniform
                if (threadIdx.x == 0) sbase = atomicAdd(&c.tcnt[tile], tot);
                __syncthreads();
                at += tile * c.tile + sbase;
                __syncthreads();
            }
            moves += cnt;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                if (!((mine >> i) & 1)) continue;
                const int32_t v = (int32_t)v0 + i;
                c.prop[v] = -1;
                if (!((adm >> i) & 1)) {
                    refuse(c, v);
                    continue;
                }
                const int32_t from = c.labels[v];
                const unsigned long long w = (unsigned long long)vweight(c.vwgt, v);
                c.labels[v] = t[i];
                if (c.lab8) c.lab8[v] = (uint8_t)t[i];
                c.mv[at] = v;
                c.old[at] = from;
                at++;
                if constexpr (LDS) {
                    atomicAdd(&dw[t[i]], w);
                    atomicAdd(&dw[from], (unsigned long long)(-(long long)w));
                } else {
                    gain += (int64_t)w;
                    atomicAdd((unsigned long long *)&c.W[from], (unsigned long long)(-(long long)w));
                }
            }
            if (c.group)
                for (int i = 0; i < 16; i++) count_group(c, (int32_t)v0 + i, (adm >> i) & 1);
        }
    }
    moves = block_sum<kDadmBlock>(moves, t32);
    if (threadIdx.x == 0) c.tmoves[col] = moves;
    if constexpr (LDS) {
        __syncthreads();
        for (int32_t i = threadIdx.x; i < c.nlabels; i += kDadmBlock) {
            const unsigned long long x = dw[i];
            if (!ordered) c.part[(int64_t)i * c.ntiles + tile] = (int64_t)x;
            else if (x) atomicAdd((unsigned long long *)&c.W[i], x);
        }
    } else {
        gain = block_sum<kDadmBlock>(gain, t64);
        if (threadIdx.x == 0 && gain) atomicAdd((unsigned long long *)&c.W[col], (unsigned long long)gain);
    }
}

template <int LMAX>
inline void launch_tiled_as(const AdmitCtx &c, hipStream_t s) {
    const dim3 tiles(c.ntiles), labels(c.nlabels), all(c.ncol), block(kDadmBlock);
    hipLaunchKernelGGL(k_dadm_tally<LMAX>, tiles, block, 0, s, c);
    hipLaunchKernelGGL(k_dadm_cut, labels, dim3(256), 0, s, c);
    if constexpr (LMAX <= kDadmSome) {
        hipLaunchKernelGGL((k_dadm_apply<LMAX, true, true>), all, block, 0, s, c);
    } else {
        hipLaunchKernelGGL((k_dadm_apply<LMAX, true, false>), tiles, block, 0, s, c);
        hipLaunchKernelGGL((k_dadm_apply<1, false, true>), labels, block, 0, s, c);
    }
}
inline void launch_tiled(const AdmitCtx &c, hipStream_t s) {
    if (c.nlabels <= kDenseAdm) launch_tiled_as<kDenseAdm>(c, s);
    else if (c.nlabels <= kDadmSome) launch_tiled_as<kDadmSome>(c, s);
    else if (c.nlabels <= kDadmMany) launch_tiled_as<kDadmMany>(c, s);
    else launch_tiled_as<kDadmLabels>(c, s);
}

// ---------------------------------------------------------------- round end

// Round bookkeeping by one workgroup: `extra` + the sum of tmoves[0 .. cols) moves.
__device__ __forceinline__ void round_end(const AdmitCtx &c, int32_t extra, int32_t cols, int32_t *t32) {
    int32_t m = 0;
    for (int32_t i = threadIdx.x; i < cols; i += 256) m += c.tmoves[i];
    m = block_sum<256>(m, t32);
    if (threadIdx.x != 0) return;
    LPDev *d = c.dev;
    const int32_t r = d->round;
    d->round = r + 1;
    if (d->done) return;
    m += extra;
    d->rounds_run = r + 1;
    d->total_moves += m;
    if (r >= 1 && m == 0 && d->prev_moves == 0) d->done = 1;
    d->prev_moves = m;
    d->round_moves = 0;
}

// One workgroup per label sums its weight changes; the first also ends the round.
// Only the first reads the stop flag, because it is the one that sets it: a wave
// of another workgroup could see it before or after. The others need no test:
// the round that sets the flag moved nothing and left all zeros in part, and the
// rounds after it write none.
__global__ __launch_bounds__(256) void k_dadm_end(AdmitCtx c) {
    __shared__ int64_t t64[256 / kWave + 1];
    __shared__ int32_t t32[256 / kWave + 1];
    const int32_t t = blockIdx.x;
    int64_t s = 0;
    for (int32_t i = threadIdx.x; i < c.ntiles; i += 256) s += c.part[(int64_t)t * c.ntiles + i];
    s = block_sum<256>(s, t64);
    if (threadIdx.x == 0 && s) c.W[t] += s;
    if (t == 0) round_end(c, 0, c.dev->done ? 0 : c.ncol, t32);
}

// ---------------------------------------------------------------- more labels: by targets

// Slot of label t in an LDS table of keys (-1: empty), inserting it.
__device__ __forceinline__ uint32_t adm_slot(int32_t *key, int32_t t) {
    uint32_t h = ((uint32_t)t * 0x9E3779B1u) >> (32 - kSadmLog);
    for (;;) {
        const int32_t k = key[h];
        if (k == t) return h;
        if (k == -1) {
            const int32_t p = atomicCAS(&key[h], -1, t);
            if (p == -1 || p == t) return h;
        }
        h = (h + 1) & (kSadmSlots - 1);
    }
}

// W[target] += weight of its proposers.
__global__ __launch_bounds__(kSadmBlock) void k_sadm_tally(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ int32_t key[kSadmSlots];
    __shared__ unsigned long long val[kSadmSlots];
    const int64_t v0 = (int64_t)blockIdx.x * kSadmTile + threadIdx.x;
    int32_t t[kSadmPer];
    bool any = false;
#pragma unroll
    for (int q = 0; q < kSadmPer; q++) {
        const int64_t v = v0 + q * kSadmBlock;
        t[q] = v < c.n ? c.prop[v] : -1;
        any |= t[q] >= 0;
    }
    if (!__syncthreads_or(any)) return;
    for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock) {
        key[i] = -1;
        val[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSadmPer; q++)
        if (t[q] >= 0)
            atomicAdd(&val[adm_slot(key, t[q])], (unsigned long long)vweight(c.vwgt, (int32_t)(v0 + q * kSadmBlock)));
    __syncthreads();
    for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock)
        if (key[i] >= 0) atomicAdd((unsigned long long *)&c.W[key[i]], val[i]);
}

// Proposers of targets within their bound move; those of contested targets
// get a position among the target's proposers.
__global__ __launch_bounds__(kSadmBlock) void k_sadm_apply(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ int32_t key[kSadmSlots];
    __shared__ int32_t cnt[kSadmSlots];
    __shared__ int32_t t32[kSadmBlock / kWave + 1];
    __shared__ int32_t snew, sbase;
    const int32_t tile = blockIdx.x;
    const int64_t v0 = (int64_t)tile * kSadmTile + threadIdx.x;
    int32_t t[kSadmPer];
    int32_t mine = 0;
#pragma unroll
    for (int q = 0; q < kSadmPer; q++) {
        const int64_t v = v0 + q * kSadmBlock;
        t[q] = v < c.n ? c.prop[v] : -1;
        mine += t[q] >= 0;
    }
    int32_t tot;
    int32_t at = tile * kSadmTile + block_excl_scan<kSadmBlock>(mine, t32, &tot);
    if (threadIdx.x == 0) c.tcnt[tile] = tot;
    if (!tot) {  // uniform
        if (threadIdx.x == 0) c.tmoves[tile] = 0;
        return;
    }
    int64_t w[kSadmPer], cap[kSadmPer];
#pragma unroll
    for (int q = 0; q < kSadmPer; q++) {
        w[q] = t[q] >= 0 ? c.W[t[q]] : 0;
        cap[q] = t[q] >= 0 ? cap_of(c, t[q]) : 0;
    }
    bool con = false;
#pragma unroll
    for (int q = 0; q < kSadmPer; q++) con |= w[q] > cap[q];
    const bool contested = __syncthreads_or(con);
    if (contested) {
        for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock) {
            key[i] = -1;
            cnt[i] = 0;
        }
        if (threadIdx.x == 0) snew = 0;
        __syncthreads();
    }
    int32_t moves = 0;
    int32_t pos[kSadmPer];
    uint32_t slot[kSadmPer];
    const int32_t at0 = at;
#pragma unroll
    for (int q = 0; q < kSadmPer; q++) {
        const int32_t v = (int32_t)(v0 + q * kSadmBlock);
        const bool go = t[q] >= 0 && w[q] <= cap[q];
        if (go) {
            c.old[at] = c.labels[v];
            c.labels[v] = t[q];
            if (c.lab8) c.lab8[v] = (uint8_t)t[q];
            c.prop[v] = -1;
            moves++;
        } else if (t[q] >= 0) {
            slot[q] = adm_slot(key, t[q]);
            pos[q] = atomicAdd(&cnt[slot[q]], 1);
            c.old[at] = -1;
        }
        if (t[q] >= 0) c.mv[at++] = v;
        if (c.group) count_group(c, v, go);
    }
    if (contested) {
        __syncthreads();
        // the tile's proposers of each contested target, after those of the tiles before it in time
        int32_t fresh = 0;
        for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock)
            if (key[i] >= 0) {
                const int32_t b = atomicAdd(&c.ccnt[key[i]], cnt[i]);
                cnt[i] = b;
                fresh += b == 0;
            }
        int32_t nf = fresh ? atomicAdd(&snew, fresh) : 0;
        __syncthreads();
        if (threadIdx.x == 0 && snew) sbase = atomicAdd(&c.nct[0], snew);
        __syncthreads();
        for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock)
            if (key[i] >= 0 && cnt[i] == 0) {
                const int32_t j = sbase + nf++;
                c.ct[j] = key[i];
                c.ctW[j] = c.W[key[i]];
            }
        at = at0;
#pragma unroll
        for (int q = 0; q < kSadmPer; q++) {
            if (t[q] < 0) continue;
            if (w[q] > cap[q]) c.cpos[at] = cnt[slot[q]] + pos[q];
            at++;
        }
    }
    moves = block_sum<kSadmBlock>(moves, t32);
    if (threadIdx.x == 0) c.tmoves[tile] = moves;
}

// Slots of the contested targets' proposers, in any order of targets.
__global__ __launch_bounds__(256) void k_sadm_offsets(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ int32_t t32[256 / kWave + 1];
    __shared__ int32_t sbase;
    const int32_t m = c.nct[0];
    for (int32_t i0 = blockIdx.x * 256; i0 < m; i0 += gridDim.x * 256) {
        const int32_t i = i0 + threadIdx.x;
        const int32_t t = i < m ? c.ct[i] : -1, s = t >= 0 ? c.ccnt[t] : 0;
        int32_t tot;
        const int32_t ex = block_excl_scan<256>(s, t32, &tot);
        if (threadIdx.x == 0) sbase = atomicAdd(&c.nct[1], tot);
        __syncthreads();
        if (t >= 0) {
            c.ctS[i] = s;
            c.ccnt[t] = sbase + ex;
        }
        __syncthreads();
    }
}

// The admitted movers' weight leaves their old labels; the contested
// targets' proposers go to their slots.
__global__ __launch_bounds__(kSadmBlock) void k_sadm_scatter(AdmitCtx c) {
    if (c.dev->done) return;
    __shared__ int32_t key[kSadmSlots];
    __shared__ unsigned long long val[kSadmSlots];
    const int32_t tile = blockIdx.x, m = c.tcnt[tile];
    if (m == 0) return;  // uniform
    for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock) {
        key[i] = -1;
        val[i] = 0;
    }
    __syncthreads();
    const int32_t p1 = tile * kSadmTile + m;
    for (int32_t p = tile * kSadmTile + threadIdx.x; p < p1; p += kSadmBlock) {
        const int32_t v = c.mv[p], from = c.old[p];
        if (from >= 0) {
            atomicAdd(&val[adm_slot(key, from)], (unsigned long long)vweight(c.vwgt, v));
        } else {
            const int32_t s = c.ccnt[c.prop[v]] + c.cpos[p];
            c.segv[s] = v;
            c.segp[s] = p;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSadmSlots; i += kSadmBlock)
        if (key[i] >= 0) atomicAdd((unsigned long long *)&c.W[key[i]], (unsigned long long)(-(long long)val[i]));
}

__device__ __forceinline__ void sadm_move(const AdmitCtx &c, int32_t v, int32_t p, int32_t t, int64_t w) {
    const int32_t from = c.labels[v];
    c.labels[v] = t;
    if (c.lab8) c.lab8[v] = (uint8_t)t;
    c.old[p] = from;
    atomicAdd((unsigned long long *)&c.W[from], (unsigned long long)(-w));
}

// Contested targets: W[t] (with everything proposed) minus what the proposers
// from some id on weigh has to be within the bound; find that id.
__global__ __launch_bounds__(kSelBlock) void k_sadm_select(AdmitCtx c) {
    if (c.dev->done) return;
    constexpr int NW = kSelBlock / kWave, PER = kSelBins / kSelBlock, U4 = 4;
    __shared__ unsigned long long h[kSelBins];
    __shared__ int64_t t64[NW + 1];
    __shared__ int32_t t32[NW + 1];
    __shared__ int64_t s_room;
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    const int32_t m = c.nct[0];
    int32_t moves = 0;
    // ---- more than 64 proposers: one workgroup per target
    for (int32_t i = blockIdx.x; i < m; i += gridDim.x) {
        const int32_t t = c.ct[i], s = c.ctS[i];
        if (s <= kWave) continue;  // uniform
        const int32_t *sv = c.segv + c.ccnt[t], *sp = c.segp + c.ccnt[t];
        int64_t room = 0;    // for the proposers with the digits found so far
        int32_t prefix = 0;  // those digits
        const int top = ((c.vbits + kSelBits - 1) / kSelBits - 1) * kSelBits;
        for (int shift = top; shift >= 0; shift -= kSelBits) {
#pragma unroll
            for (int q = 0; q < PER; q++) h[threadIdx.x + q * kSelBlock] = 0;
            __syncthreads();
            for (int32_t j0 = threadIdx.x; j0 < s; j0 += U4 * kSelBlock) {
                int32_t v[U4];
#pragma unroll
                for (int q = 0; q < U4; q++) v[q] = j0 + q * kSelBlock < s ? sv[j0 + q * kSelBlock] : -1;
#pragma unroll
                for (int q = 0; q < U4; q++)
                    if (v[q] >= 0 && (int32_t)((int64_t)v[q] >> (shift + kSelBits)) == prefix)
                        atomicAdd(&h[(v[q] >> shift) & (kSelBins - 1)], (unsigned long long)vweight(c.vwgt, v[q]));
            }
            __syncthreads();
            // the first bin whose inclusive prefix exceeds the room
            int64_t x[PER], own = 0;
#pragma unroll
            for (int q = 0; q < PER; q++) {
                x[q] = (int64_t)h[threadIdx.x * PER + q];
                own += x[q];
            }
            int64_t sum;
            int64_t run = block_excl_scan<kSelBlock>(own, t64, &sum);
            if (shift == top) room = cap_of(c, t) - c.ctW[i] + sum;  // below sum: the target is contested
            int32_t bin = INT_MAX;
#pragma unroll
            for (int q = 0; q < PER; q++) {
                if (bin == INT_MAX) {
                    if (run + x[q] > room) bin = threadIdx.x * PER + q;
                    else run += x[q];
                }
            }
            const int32_t first = block_min<kSelBlock>(bin, t32);
            if (bin == first) s_room = room - run;  // one thread: the bins are distinct
            __syncthreads();
            prefix = (int32_t)(((uint32_t)prefix << kSelBits) | (uint32_t)first);
            room = s_room;
            __syncthreads();
        }
        int64_t rej = 0;  // ids below `prefix` are admitted
        for (int32_t j = threadIdx.x; j - lane < s; j += kSelBlock) {
            const bool valid = j < s;
            const int32_t v = valid ? sv[j] : 0;
            const bool go = valid && v < prefix;
            if (valid) {
                const int64_t w = vweight(c.vwgt, v);
                c.prop[v] = -1;
                if (go) {
                    sadm_move(c, v, sp[j], t, w);
                    moves++;
                } else {
                    rej += w;
                    refuse(c, v);
                }
            }
            if (c.group) count_group(c, v, go);
        }
        rej = block_sum<kSelBlock>(rej, t64);
        if (threadIdx.x == 0) {
            atomicAdd((unsigned long long *)&c.W[t], (unsigned long long)(-rej));
            c.ccnt[t] = 0;
        }
        __syncthreads();
    }
    // ---- at most 64 proposers: one wave per target
    for (int32_t i = blockIdx.x * NW + wid; i < m; i += gridDim.x * NW) {
        const int32_t t = c.ct[i], s = c.ctS[i];
        if (s > kWave) continue;  // taken above
        const bool valid = lane < s;
        const int32_t j = c.ccnt[t] + lane;
        const int32_t v = valid ? c.segv[j] : INT_MAX;
        const int64_t w = valid ? vweight(c.vwgt, v) : 0;
        const int64_t room = cap_of(c, t) - c.ctW[i] + wave_sum(w);
        int64_t pre = w;
        for (int q = 0; q < s; q++) {
            const int32_t vq = __shfl(v, q, kWave);
            const int64_t wq = __shfl(w, q, kWave);
            if (vq < v) pre += wq;
        }
        const bool go = valid && pre <= room;
        if (valid) {
            c.prop[v] = -1;
            if (go) {
                sadm_move(c, v, c.segp[j], t, w);
                moves++;
            } else {
                refuse(c, v);
            }
        }
        if (c.group) count_group(c, valid ? v : 0, go);
        const int64_t rej = wave_sum(valid && !go ? w : (int64_t)0);
        if (lane == 0) {
            atomicAdd((unsigned long long *)&c.W[t], (unsigned long long)(-rej));
            c.ccnt[t] = 0;
        }
    }
    moves = wave_sum(moves);
    if (lane == 0 && moves) atomicAdd(&c.dev->round_moves, moves);
}

__global__ __launch_bounds__(256) void k_sadm_end(AdmitCtx c) {
    __shared__ int32_t t32[256 / kWave + 1];
    const bool stopped = c.dev->done;
    const int32_t extra = stopped ? 0 : c.dev->round_moves;
    round_end(c, extra, stopped ? 0 : c.ntiles, t32);
    if (threadIdx.x < 2) c.nct[threadIdx.x] = 0;
}

}  // namespace

}  // namespace gp
