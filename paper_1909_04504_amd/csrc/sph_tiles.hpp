// LDS-staged cell tiles for the 3D pair passes (summation scheme).
//
// The cell grid (Sec. 2.2) is cut into boxes of tw x th x td cells.  A
// workgroup takes one box: its targets are the particles of the box's cells,
// its candidates those of the union box (the box grown by the stencil reach S
// on every side), which holds every neighbour of every target.  The union is
// staged in LDS once per workgroup; the targets then find their neighbours,
// and later gather their neighbours' records, from LDS instead of from
// cache-resident global memory.
//
//  * Frame: a staged position is the fixed-point offset of the particle from
//    its cell centre plus its union cell's index times 2^27, so the
//    separation of two staged particles is the same exact integer as the
//    cell-relative one of pair_geom; the pair terms are bitwise those of the
//    global passes.  A float copy, relative to the union centre, filters
//    candidates outside a band around (2h)^2 (its error is below a tenth of
//    the band); the exact predicate decides inside the band.
//  * Walk order: rows (z, y) in stencil order, x cells ascending, slots
//    ascending -- the order of walk_pairs -- so the lists, their counts and
//    every sum are those of the global passes.  Rows whose y/z distance from
//    the target leaves no room for a neighbour are skipped and the others are
//    clipped in x to the cells the support can reach (with a margin of 1e-4 of
//    R^2 and of a cell), which drops only candidates the predicate rejects.
//  * Lists: entries are 16-bit union indices, written by each lane in
//    octets (16 bytes, one store per eight entries) into tiles of 64 sorted
//    slots: entry k of slot i at ((i/64) cap/8 + k/8) 64 + i%64 octets.  They
//    are only meaningful to the tile passes of the same grid.
//  * Targets the tile passes cannot take -- more neighbours than the list
//    capacity, or a tile whose union does not fit in LDS (then every target's
//    count is set to kTileOverflow) -- are left to the fallback kernels, which
//    walk the cells in global memory with the same arithmetic.  A build that
//    leaves any such target stores its epoch in the workspace's fallback
//    word; the fallback kernels exit at once when the word holds another
//    epoch.  In FP64, where the staging holds fewer particles, a fluid denser
//    than the mean of its grid may overflow most tiles: the sort, or the
//    packing of a sorted state, looks at some of them (tile_probe), and where
//    they would, the tile passes leave every target to the fallback, whose
//    density pass writes the global-format lists as it walks.
#pragma once

#include "sph_kernels.hpp"

namespace sph {

// Sizes of one pass's workgroup: threads (waves of 64) that set tiles up and
// stage them, union cells (two per thread), target cells and staged particles
// per tile.
template <int THREADS, int CELLS, int TCELLS, int CAP>
struct TileCfg {
    static constexpr int kThreads = THREADS, kCells = CELLS, kTCells = TCELLS, kCap = CAP;
    static_assert(CELLS <= 2 * THREADS && TCELLS <= THREADS, "cells per thread");
};
using CfgF = TileCfg<512, 1024, 160, 3072>;  // mixed precision
using CfgD = TileCfg<256, 512, 64, 2000>;    // FP64
template <typename T> struct TileCfgOf;
template <> struct TileCfgOf<float> { using type = CfgF; };
template <> struct TileCfgOf<double> { using type = CfgD; };
template <bool B> struct BoolC { static constexpr bool value = B; };
constexpr uint32_t kTileOverflow = 0xffffffffu;  // count of a target left to the fallback
constexpr int kFallbackBlocks = 1024;            // grid of the fallback kernels (grid-stride)


// Per-workgroup bookkeeping in LDS.
template <typename CFG>
struct TileMeta {
    uint32_t off[CFG::kCells + 1];  // union index of each cell's first particle; off[ncu] = total
    uint32_t gs[CFG::kCells];       // global slot of each cell's first particle
    uint32_t tpre[CFG::kTCells + 1];  // targets before each target cell
    int tc[CFG::kTCells];             // union index of each target cell
    int ntcells;
    uint32_t total, ntargets;
    uint32_t wsum[CFG::kThreads / 64];
};

// Exclusive scan of two counts per thread (cells 2t, 2t+1) over the
// CFG::kThreads threads tid of the set-up (further threads of the workgroup
// take part in the barriers only); returns the offset of cell 2t, total in
// *total.
template <typename CFG>
__device__ __forceinline__ uint32_t tile_scan2(uint32_t a, uint32_t b, TileMeta<CFG>& M,
                                               uint32_t* total, int tid) {
    const int lane = tid & 63, w = tid >> 6;
    const uint32_t v = a + b;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63 && tid < CFG::kThreads) M.wsum[w] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < CFG::kThreads / 64; ++k) {
        before += k < w ? M.wsum[k] : 0u;
        all += M.wsum[k];
    }
    __syncthreads();  // wsum is reused by the next scan
    *total = all;
    return before + incl - v;
}

// Whether the tile's box holds no particle: the keys of its cells lie
// between those of its first and last corner cells (row-major and Z-order
// keys both grow with each coordinate), so an empty slot range between them
// means empty cells.  Two loads per workgroup, before any other work.
__device__ __forceinline__ bool tile_empty(const Grid& G, const Tiles& TL, const int c0[3],
                                           const uint32_t* __restrict__ cstart,
                                           const uint32_t* __restrict__ cend) {
    __shared__ uint32_t se[2];
    if (threadIdx.x == 0) {
        const int a[3] = {c0[0], c0[1], c0[2]};
        const int b[3] = {min(c0[0] + TL.tw, G.nc[0]) - 1, min(c0[1] + TL.th, G.nc[1]) - 1,
                          min(c0[2] + TL.td, G.nc[2]) - 1};
        se[0] = cstart[cell_key(a, G)];
        se[1] = cend[cell_key(b, G)];
    }
    __syncthreads();
    return se[1] <= se[0];
}

// Cell ranges of the union, their scan, and the target cells, in two
// halves: tile_setup_loads issues each thread's loads (union cells 2t and
// 2t + 1), tile_setup_finish forms the counts, the scans and the target
// cells from them (so that a pass can have the loads in flight while it
// works on another tile).
struct SetupLoads {
    uint32_t s[2], e[2];
    bool in[2];
};
__device__ __forceinline__ SetupLoads tile_setup_loads(const Grid& G, const Tiles& TL,
                                                       const int c0[3],
                                                       const uint32_t* __restrict__ cstart,
                                                       const uint32_t* __restrict__ cend,
                                                       int tid) {
    const int ncu = TL.uw * TL.uh * TL.ud;
    SetupLoads r;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c = 2 * tid + q;
        r.s[q] = r.e[q] = 0;
        r.in[q] = false;
        if (c < ncu) {
            int uc[3];
            union_coords(TL, c, uc);
            const int gx = tile_axis(G, 0, c0[0], uc[0], TL.S);
            const int gy = tile_axis(G, 1, c0[1], uc[1], TL.S);
            const int gz = tile_axis(G, 2, c0[2], uc[2], TL.S);
            if (gx >= 0 && gy >= 0 && gz >= 0) {
                const int gc[3] = {gx, gy, gz};
                const uint32_t key = cell_key(gc, G);
                r.s[q] = cstart[key];
                r.e[q] = cend[key];
                r.in[q] = true;
            }
        }
    }
    return r;
}
// Returns the number of union particles (every thread).
template <typename CFG>
__device__ __forceinline__ uint32_t tile_setup_finish(const Grid& G, const Tiles& TL,
                                                      const int c0[3], int n,
                                                      const SetupLoads& r, TileMeta<CFG>& M,
                                                      int tid) {
    const int ncu = TL.uw * TL.uh * TL.ud;
    uint32_t cnt[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c = 2 * tid + q;
        cnt[q] = 0;
        if (c < ncu) {
            uint32_t s = 0;
            if (r.in[q]) {
                s = r.s[q];
                const uint32_t e = r.e[q] < (uint32_t)n ? r.e[q] : (uint32_t)n;
                cnt[q] = e > s ? e - s : 0u;
            }
            M.gs[c] = s;
        }
    }
    uint32_t total;
    const uint32_t o = tile_scan2(cnt[0], cnt[1], M, &total, tid);
    {
        const int c = 2 * tid;
        if (c < ncu) M.off[c] = o;
        if (c + 1 < ncu) M.off[c + 1] = o + cnt[0];
    }
    if (tid == 0) {
        M.off[ncu] = total;
        M.total = total;
    }
    __syncthreads();
    // target cells: the box's cells inside the grid, each its own slot range
    // (with Z-order keys the cells of a row are not adjacent); thread r
    // takes target cell r, and a workgroup scan gives their offsets
    const int twc = min(TL.tw, G.nc[0] - c0[0]);
    const int thc = min(TL.th, G.nc[1] - c0[1]);
    const int tdc = min(TL.td, G.nc[2] - c0[2]);
    const int ntc = twc * thc * tdc;
    const int rr = tid;
    uint32_t tcnt = 0;
    int tcell = 0;
    if (rr < ntc) {
        // rr < kTCells, twc thc <= 144: exact FP32 quotients
        const int z = small_quot(rr, __builtin_amdgcn_rcpf((float)(twc * thc)));
        const int rem = rr - z * (twc * thc);
        const int y = small_quot(rem, __builtin_amdgcn_rcpf((float)twc));
        const int x = rem - y * twc;
        tcell = (TL.S + x) + TL.uw * ((TL.S + y) + TL.uh * (TL.S + z));
        tcnt = M.off[tcell + 1] - M.off[tcell];
    }
    uint32_t ntargets;
    const uint32_t tpre = tile_scan2(tcnt, 0u, M, &ntargets, tid);
    if (rr < ntc) {
        M.tc[rr] = tcell;
        M.tpre[rr] = tpre;
    }
    if (tid == 0) {
        M.tpre[ntc] = ntargets;
        M.ntcells = ntc;
        M.ntargets = ntargets;
    }
    __syncthreads();
    return total;
}
template <typename CFG>
__device__ __forceinline__ uint32_t tile_setup(const Grid& G, const Tiles& TL, const int c0[3],
                                               const uint32_t* __restrict__ cstart,
                                               const uint32_t* __restrict__ cend, int n,
                                               TileMeta<CFG>& M, int tid) {
    return tile_setup_finish(G, TL, c0, n, tile_setup_loads(G, TL, c0, cstart, cend, tid), M, tid);
}

// Target t of the tile: its union index, global slot and union cell coords.
template <typename CFG>
__device__ __forceinline__ void tile_target(const Tiles& TL, const TileMeta<CFG>& M, uint32_t t,
                                            uint32_t* ui, uint32_t* gi, int uc[3]) {
    // the target cell: the last r with tpre[r] <= t (binary search)
    int lo = 0, hi = M.ntcells;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (M.tpre[mid] <= t) lo = mid; else hi = mid;
    }
    const int c = M.tc[lo];
    const uint32_t k = t - M.tpre[lo];
    *ui = M.off[c] + k;
    *gi = M.gs[c] + k;
    union_coords(TL, c, uc);
}

// Octet k8 (entries 8 k8 .. 8 k8 + 7) of slot i's list.
__device__ __forceinline__ size_t tile_octet(uint32_t i, uint32_t cap, uint32_t k8) {
    return ((size_t)(i >> 6) * (cap >> 3) + k8) * 64 + (i & 63);
}

// Marks every target of the tile for the fallback (its union does not fit):
// in its count, and in its first octet, where the mark outlives the count
// (kNoIndex is no union index).
constexpr uint32_t kNoIndex = 0xffffu;
template <typename CFG>
__device__ __forceinline__ void tile_mark_overflow(const TileMeta<CFG>& M,
                                                   uint32_t* __restrict__ ncnt,
                                                   uint4* __restrict__ list, uint32_t cap) {
    for (int r = 0; r < M.ntcells; ++r) {
        const uint32_t len = M.tpre[r + 1] - M.tpre[r];
        for (uint32_t k = threadIdx.x; k < len; k += CFG::kThreads) {
            const uint32_t i = M.gs[M.tc[r]] + k;
            ncnt[i] = kTileOverflow;
            list[tile_octet(i, cap, 0)] = make_uint4(~0u, ~0u, ~0u, ~0u);
        }
    }
}

// Stages the union's records: store(u, load(j), ux, uy, uz) for union
// particle u held in global slot j of union cell (ux, uy, uz).  The cell of
// every union index is noted first (tile_cellof), so that each thread then
// loads its particles at indices t, t + kThreads, ... with all loads in flight
// (tile_stage_loads; kCap <= 8 kThreads: a single round) and
// stores them (tile_stage_store).  cellof: kCap entries of LDS, the
// union cell of each staged particle (left unset when the union does not
// fit; NT: the workgroup's threads).
template <typename CFG, int NT = CFG::kThreads>
__device__ __forceinline__ void tile_cellof(const Tiles& TL, const TileMeta<CFG>& M,
                                            uint16_t* cellof) {
    const int ncu = TL.uw * TL.uh * TL.ud;
    if (M.total <= (uint32_t)CFG::kCap)
        for (int c = threadIdx.x; c < ncu; c += NT)
            for (uint32_t u = M.off[c]; u < M.off[c + 1]; ++u) cellof[u] = (uint16_t)c;
    __syncthreads();
}
template <typename CFG, typename P>
struct StageRegs {
    static constexpr int kQ = (CFG::kCap + CFG::kThreads - 1) / CFG::kThreads;
    static_assert(kQ <= 8, "staging registers");
    P v[kQ];
};
template <typename CFG, typename P, typename Load>
__device__ __forceinline__ void tile_stage_loads(const TileMeta<CFG>& M, const uint16_t* cellof,
                                                 Load&& load, StageRegs<CFG, P>& R, int tid) {
    const uint32_t total = M.total;
#pragma unroll
    for (int q = 0; q < StageRegs<CFG, P>::kQ; ++q) {
        const uint32_t u = (uint32_t)(tid + q * CFG::kThreads);
        if (u < total) {
            const int c = cellof[u];
            R.v[q] = load(M.gs[c] + (u - M.off[c]));
        }
    }
}
template <typename CFG, typename P, typename Store>
__device__ __forceinline__ void tile_stage_store(const Tiles& TL, const TileMeta<CFG>& M,
                                                 const uint16_t* cellof,
                                                 const StageRegs<CFG, P>& R, Store&& store,
                                                 int tid) {
    const uint32_t total = M.total;
#pragma unroll
    for (int q = 0; q < StageRegs<CFG, P>::kQ; ++q) {
        const uint32_t u = (uint32_t)(tid + q * CFG::kThreads);
        if (u < total) {
            int uc[3];
            union_coords(TL, cellof[u], uc);
            store(u, R.v[q], uc[0], uc[1], uc[2]);
        }
    }
}
template <typename CFG, typename Load, typename Store>
__device__ __forceinline__ void tile_stage(const Tiles& TL, TileMeta<CFG>& M, uint16_t* cellof,
                                           Load&& load, Store&& store) {
    tile_cellof(TL, M, cellof);
    using P = decltype(load(0u));
    StageRegs<CFG, P> R;
    const int tid = (int)threadIdx.x;
    tile_stage_loads(M, cellof, load, R, tid);
    tile_stage_store(TL, M, cellof, R, store, tid);
}

// Union-frame record: cell-relative fixed point plus the union cell times 2^27.
__device__ __forceinline__ int4 tile_rec(const int4& r, int ux, int uy, int uz) {
    int4 p;
    p.x = ux * (1 << kFixBits) + r.x;
    p.y = uy * (1 << kFixBits) + r.y;
    p.z = uz * (1 << kFixBits) + r.z;
    p.w = r.w;
    return p;
}

__device__ __forceinline__ uint32_t half_of(const uint4& v, int e) {
    const uint32_t w = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
    return (e & 1) ? (w >> 16) : (w & 0xffffu);
}

// The first two octets of slot i's list, fetched before its count is known
// (both within the slot's cap / 8 octets, so always in bounds), for
// tile_list_loop.
struct ListHead {
    uint4 o0, o1;
};
__device__ __forceinline__ ListHead tile_list_head(const uint4* __restrict__ list, uint32_t i,
                                                  uint32_t cap) {
    const uint4* __restrict__ base = list + tile_octet(i, cap, 0);
    return ListHead{base[0], base[cap >= 16 ? 64 : 0]};
}

// Calls body(load(u)) for the cnt entries u of slot i's list, in order
// (head: tile_list_head of the slot).  The loads of a full octet's eight
// entries are issued together and the next octet is fetched meanwhile; the
// last, partial octet goes entry by entry.  Octet fetches are unconditional,
// their index clamped to the list's last octet, so that the rotating octets
// stay in registers (a conditional fetch makes the compiler keep them in
// scratch memory and wait on every fetch at the top of the loop).  Two
// octets per iteration, for a longer fetch distance, measured slower (the
// larger code and register count cost more than the latency they hide).
template <int kGroup = 8, typename Load, typename Body>
__device__ __forceinline__ void tile_list_loop(const uint4* __restrict__ list, uint32_t i,
                                               uint32_t cap, uint32_t cnt, const ListHead& head,
                                               Load&& load, Body&& body) {
    static_assert(kGroup == 8 || kGroup == 4, "whole or half octets");
    using P = decltype(load(0u));
    const uint32_t nfull = cnt >> 3, rest = cnt & 7u;
    const uint32_t noct = nfull + (rest ? 1u : 0u);
    if (noct == 0) return;
    const uint32_t last = noct - 1;
    // octet k8 of the slot is 64 k8 uint4 after its first
    const uint4* __restrict__ base = list + tile_octet(i, cap, 0);
    uint4 nxt = head.o0;
    uint4 nxt2 = head.o1;
    for (uint32_t k8 = 0; k8 < nfull; ++k8) {
        const uint4 cur = nxt;
        nxt = nxt2;
        nxt2 = base[(size_t)min(k8 + 2, last) * 64];
#pragma unroll
        for (int h = 0; h < 8; h += kGroup) {
            P p[kGroup];
#pragma unroll
            for (int e = 0; e < kGroup; ++e) p[e] = load(half_of(cur, h + e));
#pragma unroll
            for (int e = 0; e < kGroup; ++e) body(p[e]);
        }
    }
    if (rest) {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if ((uint32_t)e < rest) body(load(half_of(nxt, e)));
    }
}

// Calls body(load(u), k) for the entries u = entry k of slot i's list in
// whole half octets, the last one completed by entries k >= cnt that are the
// target itself (body sees to it that they add nothing): no entry by entry
// tail, whose reads nothing covers.
template <typename Load, typename Body>
__device__ __forceinline__ void tile_list_whole(const uint4* __restrict__ list, uint32_t i,
                                                uint32_t cap, uint32_t cnt, const ListHead& head,
                                                Load&& load, Body&& body) {
    using P = decltype(load(0u));
    if (cnt == 0) return;
    const uint32_t last = (cnt - 1) >> 3;
    const uint4* __restrict__ base = list + tile_octet(i, cap, 0);
    uint4 nxt = head.o0, nxt2 = head.o1;
    for (uint32_t k = 0; k < cnt; k += 8) {
        const uint4 cur = nxt;
        nxt = nxt2;
        nxt2 = base[(size_t)min((k >> 3) + 2, last) * 64];
        P p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = load(half_of(cur, e));
#pragma unroll
        for (int e = 0; e < 4; ++e) body(p[e], k + (uint32_t)e);
        if (k + 4 < cnt) {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = load(half_of(cur, 4 + e));
#pragma unroll
            for (int e = 0; e < 4; ++e) body(p[e], k + 4 + (uint32_t)e);
        }
    }
}

// Per-thread FP64 values summed over the workgroup (wave butterflies, then
// the waves in order) into part[q * stride + b].
template <int NV, int NT>
__device__ __forceinline__ void tile_block_sum(double v[NV], double* __restrict__ part, int b,
                                               int stride) {
    __shared__ double sh[NV][NT / 64];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double x = v[q];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
        v[q] = x;
    }
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < NV; ++q) sh[q][threadIdx.x >> 6] = v[q];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int q = 0; q < NV; ++q) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w) s += sh[q][w];
            part[(int64_t)q * stride + b] = s;
        }
}

// Workgroup sum of a per-thread count into the tile's interaction counter.
template <int NT>
__device__ __forceinline__ void tile_count(uint32_t cnt, unsigned long long* __restrict__ pairs,
                                           int blk) {
    __shared__ uint32_t wc[NT / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
    if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < NT / 64; ++w) t += wc[w];
        add_pairs(pairs, blk, t);
    }
}

// Float copy of a staged record, relative to the centre of the union's cell
// TL.cen, for the build's filter (w: the particle's union cell).  FP64
// records are absolute: w L moves one to the image of its union cell (w grid
// lengths away) and the union centre is subtracted before the conversion, so
// that the copy's error is below a tenth of the filter's band as in mixed
// precision.  *far: more than 4 cells outside its cell (a particle clamped
// into an edge cell from far outside, or not finite; mixed-precision records
// are clamped there): the copy is not accurate enough then, and the tile is
// left to the fallback.
__device__ __forceinline__ float4 filt_copy(const int4& r, const int uc[3], const int[3],
                                            const Grid&, const Tiles& TL,
                                            const PairConst<float>& C, bool*) {
    const int4 p = tile_rec(r, uc[0], uc[1], uc[2]);
    float4 f;
    f.x = (float)(p.x - TL.cen[0] * (1 << kFixBits)) * C.fix_scale_f[0];
    f.y = (float)(p.y - TL.cen[1] * (1 << kFixBits)) * C.fix_scale_f[1];
    f.z = (float)(p.z - TL.cen[2] * (1 << kFixBits)) * C.fix_scale_f[2];
    return f;
}
__device__ __forceinline__ float4 filt_copy(const double4& r, const int uc[3], const int c0[3],
                                            const Grid& G, const Tiles& TL,
                                            const PairConst<double>&, bool* far) {
    const double x[3] = {r.x, r.y, r.z};
    float f[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // grid lengths between the union cell and its cell inside the grid
        int w = 0, c = c0[k] - TL.S + uc[k];
        while (c < 0) { c += G.nc[k]; --w; }
        while (c >= G.nc[k]) { c -= G.nc[k]; ++w; }
        const double centre =
            G.lo[k] + ((double)(c0[k] - TL.S + TL.cen[k]) + 0.5) * G.cs[k];
        f[k] = (float)((x[k] + (double)w * G.L[k]) - centre);
        *far |= !(fabsf(f[k] - (float)(uc[k] - TL.cen[k]) * TL.csf[k]) <= 4.f * TL.csf[k]);
    }
    float4 o;
    o.x = f[0];
    o.y = f[1];
    o.z = f[2];
    return o;
}
// Periodic image of a tile's union cell coordinate u along axis k (the
// stencil_axis wrap of every target that reaches it).
__device__ __forceinline__ int tile_wrap(const Grid& G, int k, int c0, int u, int S) {
    const int c = c0 - S + u;
    return c < 0 ? -1 : (c >= G.nc[k] ? 1 : 0);
}
// Exact predicate of target record ri (global slot record of union cell ut)
// and candidate record rj of union cell uj: the geometry of pair_geom.
__device__ __forceinline__ bool tile_exact(const int4& ri, const int ut[3], const int4& rj,
                                           const int uj[3], const int[3], const Grid&,
                                           const Tiles&, const PairConst<float>& C) {
    const Geom<float> g =
        pair_geom<3>(tile_rec(ri, ut[0], ut[1], ut[2]), tile_rec(rj, uj[0], uj[1], uj[2]), 0, 0,
                     0, 0, 0, 0, C);
    return geom_r2d(g, C) < C.R2_d;
}
__device__ __forceinline__ bool tile_exact(const double4& ri, const int[3], const double4& rj,
                                           const int uj[3], const int c0[3], const Grid& G,
                                           const Tiles& TL, const PairConst<double>& C) {
    const Geom<double> g =
        pair_geom<3>(ri, rj, 0, 0, 0, tile_wrap(G, 0, c0[0], uj[0], TL.S),
                     tile_wrap(G, 1, c0[1], uj[1], TL.S), tile_wrap(G, 2, c0[2], uj[2], TL.S), C);
    return pair_accept(g, C);
}
// Whether a target lies inside its cell (its rows may then be clipped): the
// fixed-point offset itself, or the float copy's (FP64; the margin is far
// below the clip's).
__device__ __forceinline__ bool tile_inside(const int4& r, const float4&, const int[3],
                                            const Tiles&) {
    const int half = 1 << (kFixBits - 1);
    return abs(r.x) <= half && abs(r.y) <= half && abs(r.z) <= half;
}
__device__ __forceinline__ bool tile_inside(const double4&, const float4& f, const int uc[3],
                                            const Tiles& TL) {
    auto in = [&](float v, int k) {
        return fabsf(v - (float)(uc[k] - TL.cen[k]) * TL.csf[k]) <= 0.50001f * TL.csf[k];
    };
    return in(f.x, 0) && in(f.y, 1) && in(f.z, 2);
}

// Octet k8 of a thread's ring of RING entries.
template <int RING>
__device__ __forceinline__ uint4 ring_octet(const uint2* myring, uint32_t k8) {
    const uint32_t o = 2 * (k8 & (uint32_t)(RING / 8 - 1));
    const uint2 lo = myring[o], hi = myring[o + 1];
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}
// The neighbours of one target (float copy pf, union cell uc) among the staged
// union, in walk order: their union indices go through the ring, and their
// number is returned.  group(before, now) is called after each group of at
// most four with the counts; entries it leaves in the ring are the caller's.
// exact(u) is the predicate inside the band.  Entries are appended without
// branches: every candidate is written at the next free place and the count
// advances only for accepted ones.
// VALU issue and the LDS bound it (busy 97% and 90% of the 256^3 cube's build),
// so the groups must fill the lanes: with half-size cells the rows of a stencil
// plane form a queue in registers, and a lane that ends a row goes on with its
// next one while others are still in theirs.  A wave of the 256^3 cube then
// takes 101 groups instead of the 134 of lanes that wait for the longest row
// (73 if nothing waited; one queue over all planes would take 85, but 25
// registers to shift): build 5.90 -> 5.27 ms.  With whole cells the rows are
// longer and the lanes of a cell read them together; the queue's reads meet
// more bank conflicts there (75^3 quintic lattice: build 0.39 against 0.36
// ms), so each row is a loop of its own.
template <int S, int RING, typename T, typename CFG, typename Exact, typename Group>
__device__ __forceinline__ uint32_t tile_candidates(const Tiles& TL, const TileMeta<CFG>& M,
                                                    const float4* Pf, const PairConst<T>& C,
                                                    const float4& pf, const int uc[3], bool clip,
                                                    uint2* myring, Exact&& exact,
                                                    Group&& group) {
    // the octets are read back as uint2: the halves may alias them
    typedef uint16_t __attribute__((may_alias)) Half;
    Half* const my = (Half*)myring;
    const float cxf = (float)TL.cen[0], cyf = (float)TL.cen[1], czf = (float)TL.cen[2];
    uint32_t cnt = 0;
    // the (2S+1)^2 stencil rows in walk order (z planes, then y rows).  A
    // plane's distance is taken once for its rows, and the x range in cell
    // units from px_c, the target's x in cells shifted by the union centre
    // and 1/2 (the clip keeps its margins: roundings of these forms move it
    // by far less than clip_pad)
    constexpr int NR = 2 * S + 1;
    constexpr int NQ = S == 2 ? NR : 1;  // rows of a queue
    const float px_c = pf.x * TL.inv_csf[0] + (cxf + 0.5f);
#pragma unroll 1
    for (int iz = 0; iz < NR; ++iz) {
        const int uz = uc[2] + iz - S;
        const float dz =
            fmaxf(fabsf(pf.z - ((float)uz - czf) * TL.csf[2]) - 0.5f * TL.csf[2], 0.f);
        const float w2z = TL.rclip2 - dz * dz;
        if (clip && !(w2z > 0.f)) continue;
        const int planec = TL.uw * TL.uh * uz;
#pragma unroll 1
        for (int iy0 = 0; iy0 < NR; iy0 += NQ) {
            // rows with candidates, their first union index and end in the
            // two halves of a word (0: none)
            uint32_t rq[NQ] = {};
#pragma unroll
            for (int iq = NQ - 1; iq >= 0; --iq) {
                const int uy = uc[1] + iy0 + iq - S;
                const float dy =
                    fmaxf(fabsf(pf.y - ((float)uy - cyf) * TL.csf[1]) - 0.5f * TL.csf[1], 0.f);
                const float w2 = w2z - dy * dy;
                int xa = uc[0] - S, xb = uc[0] + S;
                if (clip) {
                    const float wc =
                        (__builtin_amdgcn_sqrtf(fmaxf(w2, 0.f)) + TL.clip_pad) * TL.inv_csf[0];
                    xa = max(xa, (int)floorf(px_c - wc));
                    xb = min(xb, (int)floorf(px_c + wc));
                }
                if (clip && !(w2 > 0.f)) xb = xa - 1;
                const int rowc = planec + TL.uw * uy;
                const uint32_t ua = M.off[rowc + xa];
                const uint32_t ue = M.off[rowc + max(xa, xb + 1)];
                const bool some = ua < ue;
#pragma unroll
                for (int k = NQ - 1 - iq; k > 0; --k) rq[k] = some ? rq[k - 1] : rq[k];
                rq[0] = some ? ua | ue << 16 : rq[0];
            }
            // candidates four at a time, the next four (of this row or the
            // next) loaded while these are tested; those past the row's end
            // (read from the padding or the next row) are infinitely far
            uint32_t u = rq[0] & 0xffffu, ue = rq[0] >> 16;
            float4 c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = Pf[u + q];
#pragma unroll 1
            while (u < ue) {
                float r2[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float dx = pf.x - c[q].x, ddy = pf.y - c[q].y, ddz = pf.z - c[q].z;
                    r2[q] = dx * dx + ddy * ddy + ddz * ddz;
                }
                uint32_t un = u + 4, uen = ue;
                if constexpr (NQ > 1) {
                    const bool ends = un >= ue;
                    un = ends ? rq[1] & 0xffffu : un;
                    uen = ends ? rq[1] >> 16 : ue;
#pragma unroll
                    for (int k = 1; k < NQ; ++k)
                        rq[k] = ends ? (k + 1 < NQ ? rq[k + 1] : 0u) : rq[k];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) c[q] = Pf[un + q];
                const uint32_t lim = ue - u;  // candidates left in the row
                uint32_t acc[4];
                bool band[4];
                bool anyband = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float x = (uint32_t)q < lim ? r2[q] : __builtin_huge_valf();
                    acc[q] = x < C.R2_lo ? 1u : 0u;
                    band[q] = fabsf(x - C.R2_mid) < C.R2_w;
                    anyband |= band[q];
                }
                if (__builtin_amdgcn_ballot_w64(anyband)) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (band[q]) acc[q] = exact(u + q) ? 1u : 0u;
                }
                const uint32_t before = cnt;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    my[cnt & (RING - 1)] = (Half)(u + q);
                    cnt += acc[q];
                }
                group(before, cnt);
                u = un;
                ue = uen;
            }
        }
    }
    return cnt;
}

// Neighbour lists of the tile's targets: ncnt[i] = |N(i)|, entries while the
// count is within cap; targets with more are left to the fallback, as are all
// targets of a tile whose union exceeds cap_union.  count_pairs: the
// interactions of the counted targets go to the tile's counter.  Only the
// float copy of the union is staged (so that several workgroups share a CU);
// the exact predicate inside the band reads the candidate's record from global
// memory.  A completed octet is stored at once.
template <int S, typename T>
__global__ __launch_bounds__(TileCfgOf<T>::type::kThreads) void k_tile_build(
    int n, Grid G, PairConst<T> C, Tiles TL, int cap_union,
    const typename Rec<T>::type* __restrict__ pos, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, uint4* __restrict__ list,
    uint32_t* __restrict__ ncnt, int count_pairs, unsigned long long* __restrict__ pairs,
    uint32_t epoch, uint32_t* __restrict__ fallback, TileTest test) {
    using R = typename Rec<T>::type;
    using CFG = typename TileCfgOf<T>::type;
    constexpr int NT = CFG::kThreads;
    __shared__ TileMeta<CFG> M;
    // float copy of the union (w: the particle's union cell), + the
    // candidates read past a row's end
    __shared__ float4 Pf[CFG::kCap + 8];
    // each thread's ring of 16 list entries (two octets), 40 bytes apart so
    // that the lanes' appends spread over the LDS banks; the staging's cell
    // table before that
    constexpr int kRingStride = 5;  // uint2 per thread
    __shared__ uint2 ringbuf[NT * kRingStride];
    static_assert(sizeof(ringbuf) >= CFG::kCap * sizeof(uint16_t), "cell table");
    const int blk = xcd_block();
    int c0[3];
    tile_origin(TL, blk, c0);
    // the cell-range loads go out before the empty-box probe, so that the
    // two round trips overlap
    const SetupLoads sl = tile_setup_loads(G, TL, c0, cstart, cend, (int)threadIdx.x);
    if (sizeof(T) == 8 && test.found && tiles_off(test)) return;
    if (tile_empty(G, TL, c0, cstart, cend)) {
        if (count_pairs) tile_count<NT>(0u, pairs, blk);
        return;
    }
    const uint32_t total = tile_setup_finish(G, TL, c0, n, sl, M, (int)threadIdx.x);
    bool overflow = total > (uint32_t)cap_union;
    if (!overflow) {
        bool far = false;
        tile_stage(TL, M, (uint16_t*)ringbuf, [&](uint32_t j) { return pos[j]; },
                   [&](uint32_t u, const R& r, int ux, int uy, int uz) {
                       const int uc[3] = {ux, uy, uz};
                       float4 f = filt_copy(r, uc, c0, G, TL, C, &far);
                       f.w = __int_as_float(ux + TL.uw * (uy + TL.uh * uz));
                       Pf[u] = f;
                   });
        if constexpr (sizeof(T) == 8)
            overflow = __syncthreads_or(far);
        else
            __syncthreads();
    }
    if (overflow) {
        tile_mark_overflow(M, ncnt, list, cap);
        if (threadIdx.x == 0 && M.ntargets) *fallback = epoch;
        // the counter is still touched: tile 0 raises the number of counters
        // the reader sums
        if (count_pairs) tile_count<NT>(0u, pairs, blk);
        return;
    }
    uint2* const myring = &ringbuf[threadIdx.x * kRingStride];
    uint32_t counted = 0;
    bool need_fb = false;
    for (uint32_t t = threadIdx.x; t < M.ntargets; t += NT) {
        uint32_t ui, i;
        int uc[3];
        tile_target(TL, M, t, &ui, &i, uc);
        const float4 pf = Pf[ui];
        const R ri = pos[i];
        // rows are clipped only for a target inside its cell (a particle
        // clamped into an edge cell from outside a non-periodic box walks
        // whole rows, as walk_pairs does)
        const bool clip = tile_inside(ri, pf, uc, TL);
        // exact predicate on the records (the candidate's from global memory)
        auto exact = [&](uint32_t u) {
            const int c = __float_as_int(Pf[u].w);
            int cu[3];
            union_coords(TL, c, cu);
            return tile_exact(ri, uc, pos[M.gs[c] + (u - M.off[c])], cu, c0, G, TL, C);
        };
        const uint32_t cnt = tile_candidates<S, 16>(
            TL, M, Pf, C, pf, uc, clip, myring, exact,
            [&](uint32_t before, uint32_t now) {
                // an octet completed (at most one per group of four)
                const uint32_t k8 = before >> 3;
                if (((before ^ now) & ~7u) && k8 < (cap >> 3))
                    list[tile_octet(i, cap, k8)] = ring_octet<16>(myring, k8);
            });
        // the last, partial octet is filled up with the target itself
        if (cnt <= cap && (cnt & 7)) {
            const uint32_t r = cnt & 7;
            auto fill = [&](uint32_t w, uint32_t k) {  // the word of entries k, k + 1
                const uint32_t lo = k < r ? w & 0xffffu : ui;
                return lo | (k + 1 < r ? w & 0xffff0000u : ui << 16);
            };
            const uint4 v = ring_octet<16>(myring, cnt >> 3);
            list[tile_octet(i, cap, cnt >> 3)] =
                make_uint4(fill(v.x, 0), fill(v.y, 2), fill(v.z, 4), fill(v.w, 6));
        }
        ncnt[i] = cnt;
        counted += cnt;
        need_fb |= cnt > cap;
    }
    if (__syncthreads_or(need_fb) && threadIdx.x == 0) *fallback = epoch;
    if (count_pairs) tile_count<NT>(counted, pairs, blk);
}

// Neighbour lists in the global format (k_nlist_walk's, entry for entry):
// candidates from the union staged in LDS instead of a walk of each
// particle's cells through L1 and L2.  Each staged particle has its list word
// for a target in union cell 0, to which a target adds a constant: the
// mixed-precision code of a stencil offset is linear in the two cells, the
// FP64 code is the neighbour's image alone.  Completed octets of union indices
// are turned into words and stored, 256 bytes apart (rows of 64 slots), after
// a group of candidates that leaves some lane with kFlush of them or more, by
// the lanes of a wave together: at every completed octet some lane or other
// would take the whole wave through the stores.  The targets of a tile whose
// union does not fit (or, in FP64, holds a particle far outside its cell) walk
// the cells.  Workgroup b takes every gridDim-th tile and adds the
// interactions it counted to pairs[b].
// Boxes of 4 x 4 x 4 half-size cells and 256 threads, two workgroups per CU.
template <int S, typename T>
__global__ __launch_bounds__(CfgD::kThreads, 2) void k_tile_nlist(
    int n, Grid G, PairConst<T> C, Tiles TL, const uint32_t* __restrict__ skey,
    const typename Rec<T>::type* __restrict__ pos, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, uint32_t* __restrict__ list,
    uint32_t* __restrict__ ncnt, int count_pairs,
    unsigned long long* __restrict__ pairs, TileTest test) {
    if (tiles_off(test)) return;  // k_nlist_walk's
    using R = typename Rec<T>::type;
    using CFG = CfgD;
    using Code = NbrCode<3, S, T>;
    constexpr int NT = CFG::kThreads, NR = 2 * S + 1;
    // each thread's ring of 64 list entries, 136 bytes apart
    constexpr int kRing = 64, kRingStride = kRing / 4 + 1;  // uint2 per thread
    constexpr uint32_t kFlush = 24;
    __shared__ TileMeta<CFG> M;
    __shared__ float4 Pf[CFG::kCap + 8];
    __shared__ uint32_t word[CFG::kCap];
    __shared__ uint2 ringbuf[NT * kRingStride];
    static_assert(sizeof(ringbuf) >= CFG::kCap * sizeof(uint16_t), "cell table");
    uint2* const myring = &ringbuf[threadIdx.x * kRingStride];
    const int blk = xcd_block();
    uint32_t counted = 0;
    for (int tile = blk; tile < TL.ntiles; tile += (int)gridDim.x) {
        int c0[3];
        tile_origin(TL, tile, c0);
        const uint32_t total = tile_setup(G, TL, c0, cstart, cend, n, M, (int)threadIdx.x);
        if (M.ntargets == 0) {
            __syncthreads();  // M is free
            continue;
        }
        bool overflow = total > (uint32_t)TL.cap;
        if (!overflow) {
            bool far = false;
            tile_cellof(TL, M, (uint16_t*)ringbuf);
            const uint16_t* cellof = (const uint16_t*)ringbuf;
            struct Rj {
                R r;
                uint32_t j;
            };
            StageRegs<CFG, Rj> regs;
            tile_stage_loads(M, cellof, [&](uint32_t j) { return Rj{pos[j], j}; }, regs,
                             (int)threadIdx.x);
            tile_stage_store(
                TL, M, cellof, regs,
                [&](uint32_t u, const Rj& r, int ux, int uy, int uz) {
                    const int uc[3] = {ux, uy, uz};
                    float4 f = filt_copy(r.r, uc, c0, G, TL, C, &far);
                    f.w = __int_as_float(ux + TL.uw * (uy + TL.uh * uz));
                    Pf[u] = f;
                    const int code =
                        sizeof(T) == 8
                            ? Code::row_base(0, 0, tile_wrap(G, 0, c0[0], ux, S),
                                             tile_wrap(G, 1, c0[1], uy, S),
                                             tile_wrap(G, 2, c0[2], uz, S))
                            : ux + NR * (uy + NR * uz);
                    word[u] = (r.j << Code::kBits) + (uint32_t)code;
                },
                (int)threadIdx.x);
            overflow = __syncthreads_or(sizeof(T) == 8 && far);
        }
        for (uint32_t t = threadIdx.x; t < M.ntargets; t += NT) {
            uint32_t ui, i;
            int uc[3];
            tile_target(TL, M, t, &ui, &i, uc);
            uint32_t* __restrict__ col = list + list_column(i, cap);
            const R ri = pos[i];
            uint32_t cnt = 0;
            if (overflow) {
                walk_pairs<3, S, T>(G, C, skey[i], ri, pos, skey, cstart, cend, (uint32_t)n,
                                    NoPayload(),
                                    [&](uint32_t j, const R&, int, const Geom<T>&, uint32_t code) {
                                        if (cnt < cap)
                                            col[cnt * kListTile] = (j << Code::kBits) | code;
                                        ++cnt;
                                    });
            } else {
                const float4 pf = Pf[ui];
                const bool clip = tile_inside(ri, pf, uc, TL);
                // word of a neighbour in union cell u, less that of cell uc
                const uint32_t base =
                    sizeof(T) == 8 ? 0u
                                   : (uint32_t)(S * (1 + NR + NR * NR) -
                                                (uc[0] + NR * (uc[1] + NR * uc[2])));
                auto exact = [&](uint32_t u) {
                    const int c = __float_as_int(Pf[u].w);
                    int cu[3];
                    union_coords(TL, c, cu);
                    return tile_exact(ri, uc, pos[(word[u] + base) >> Code::kBits], cu, c0, G, TL, C);
                };
                auto put = [&](uint32_t k8, uint32_t m) {  // m entries of octet k8
                    const uint4 v = ring_octet<kRing>(myring, k8);
                    uint32_t* __restrict__ c = col + (size_t)(8 * k8) * kListTile;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if ((uint32_t)e < m) c[e * (int)kListTile] = word[half_of(v, e)] + base;
                };
                uint32_t done = 0;  // entries stored (or beyond cap)
                auto flush = [&](uint32_t now) {
                    while (done + 8 <= now) {
                        if (done < cap) put(done >> 3, min(cap - done, 8u));
                        done += 8;
                    }
                };
                cnt = tile_candidates<S, kRing>(
                    TL, M, Pf, C, pf, uc, clip, myring, exact,
                    [&](uint32_t, uint32_t now) {
                        if (__builtin_amdgcn_ballot_w64(now - done >= kFlush)) flush(now);
                    });
                flush(cnt);
                if (done < cap && done < cnt) put(done >> 3, min(cap, cnt) - done);
            }
            ncnt[i] = cnt;
            counted += cnt;
        }
        __syncthreads();  // the tile's LDS is free
    }
    if (count_pairs) tile_count<NT>(counted, pairs, (int)blockIdx.x);
}

// The CSR lists (sph_neighbors) of the tile's targets with complete lists.  A
// wave takes 16 targets: it reads their octets as rows of 16 (adjacent slots
// are adjacent there) into LDS, 16 octets a target at a time, and writes each
// list as a run, a lane an entry, whose global slot comes from a table of the
// union in LDS.  off[i]: the first entry of slot i.  (100^3 cube, whole cells,
// 113M entries: 0.19 ms; a lane reading its entry's half word from memory
// fetched each octet row four times, 0.46 ms; a second cell walk 1.28 ms.)
template <typename CFG>
__global__ __launch_bounds__(CFG::kThreads) void k_tile_expand(
    int n, Grid G, Tiles TL, int cap_union, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, const uint4* __restrict__ list,
    const uint32_t* __restrict__ ncnt, const int64_t* __restrict__ off,
    int32_t* __restrict__ nbr) {
    constexpr uint32_t kT = 16, kO = 16;  // targets and octets at a time
    __shared__ TileMeta<CFG> M;
    __shared__ uint32_t slot[CFG::kCap];
    __shared__ uint4 buf_[CFG::kThreads / 64][kT][kO + 1];
    const int blk = xcd_block();
    int c0[3];
    tile_origin(TL, blk, c0);
    const SetupLoads sl = tile_setup_loads(G, TL, c0, cstart, cend, (int)threadIdx.x);
    if (tile_empty(G, TL, c0, cstart, cend)) return;
    const uint32_t total = tile_setup_finish(G, TL, c0, n, sl, M, (int)threadIdx.x);
    if (total > (uint32_t)cap_union) return;  // every target is the fallback's
    const int ncu = TL.uw * TL.uh * TL.ud;
    for (int c = threadIdx.x; c < ncu; c += CFG::kThreads)
        for (uint32_t u = M.off[c]; u < M.off[c + 1]; ++u) slot[u] = M.gs[c] + (u - M.off[c]);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t nt = M.ntargets;
    typedef uint16_t __attribute__((may_alias)) Half;
    for (uint32_t t0 = w * kT; t0 < nt; t0 += CFG::kThreads / 64 * kT) {
        // lane l: target t0 + l % 16
        uint32_t ui, i;
        int uc[3];
        const uint32_t tt = t0 + lane % kT;
        tile_target(TL, M, min(tt, nt - 1), &ui, &i, uc);
        uint32_t cnt = ncnt[i];
        const int64_t at = off[i];
        const uint4* __restrict__ base = list + tile_octet(i, cap, 0);
        // (left to the fallback: above the capacity or in a marked tile)
        if (tt >= nt || cnt > cap || half_of(base[0], 0) == kNoIndex) cnt = 0;
        uint32_t most = cnt;
#pragma unroll
        for (int d = kT / 2; d >= 1; d >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, d, 64));
        for (uint32_t k0 = 0; k0 < most; k0 += 8 * kO) {
#pragma unroll
            for (uint32_t q = 0; q < kO * kT / 64; ++q) {
                const uint32_t o = q * (64 / kT) + lane / kT;
                if (k0 + 8 * o < cnt) buf_[w][lane % kT][o] = base[(size_t)(k0 / 8 + o) * 64];
            }
            wave_sync();
#pragma unroll 4
            for (uint32_t t = 0; t < kT; ++t) {
                const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)cnt, (int)t);
                const int64_t a =
                    ((int64_t)__builtin_amdgcn_readlane((int)(at >> 32), (int)t) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)at, (int)t);
                const Half* e = (const Half*)&buf_[w][t][0];
#pragma unroll
                for (uint32_t h = 0; h < 8 * kO / 64; ++h) {
                    const uint32_t k = lane + 64 * h;
                    if (k0 + k < c) nbr[a + k0 + k] = (int32_t)slot[e[k]];
                }
            }
            wave_sync();
        }
    }
}

// What the tile build left of the CSR lists: counts of the targets of tiles
// that did not fit (before the scan), and the entries of those and of targets
// with more neighbours than the list capacity, by the cell walk.
template <int S, typename T>
__global__ __launch_bounds__(kBlock) void k_tile_fallback_count(
    int n, Grid G, PairConst<T> C, const uint32_t* __restrict__ skey,
    const typename Rec<T>::type* __restrict__ pos, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t* __restrict__ ncnt, uint32_t epoch,
    const uint32_t* __restrict__ fallback) {
    if (*fallback != epoch) return;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        if (ncnt[i] != kTileOverflow) continue;
        uint32_t c = 0;
        walk_pairs<3, S, T>(G, C, skey[i], pos[i], pos, skey, cstart, cend, (uint32_t)n, NoPayload(),
                            [&](uint32_t, const typename Rec<T>::type&, int, const Geom<T>&,
                                uint32_t) { ++c; });
        ncnt[i] = c;
    }
}
template <int S, typename T>
__global__ __launch_bounds__(kBlock) void k_tile_fallback_fill(
    int n, Grid G, PairConst<T> C, const uint32_t* __restrict__ skey,
    const typename Rec<T>::type* __restrict__ pos, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, const uint4* __restrict__ list,
    const uint32_t* __restrict__ ncnt, const int64_t* __restrict__ off, int32_t* __restrict__ nbr,
    uint32_t epoch, const uint32_t* __restrict__ fallback) {
    if (*fallback != epoch) return;
    const uint16_t* __restrict__ half = reinterpret_cast<const uint16_t*>(list);
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        if (ncnt[i] <= cap && half[8 * tile_octet((uint32_t)i, cap, 0)] != kNoIndex) continue;
        int64_t at = off[i];
        const int64_t end = off[i + 1];
        walk_pairs<3, S, T>(G, C, skey[i], pos[i], pos, skey, cstart, cend, (uint32_t)n, NoPayload(),
                            [&](uint32_t j, const typename Rec<T>::type&, int, const Geom<T>&,
                                uint32_t) {
                                if (at < end) nbr[at++] = (int32_t)j;
                            });
    }
}

// Summation density (eq. 2), and with_eos the Tait EOS (eq. eos), of the
// tile's targets with complete lists (as k_density), over the union's
// position records staged in LDS.
template <int S, int KERNEL>
__global__ __launch_bounds__(CfgF::kThreads) void k_tile_density(
    int n, Grid G, PairConst<float> C, Tiles TL, int cap_union, const int4* __restrict__ pos,
    const uint32_t* __restrict__ cstart, const uint32_t* __restrict__ cend, uint32_t cap,
    const uint4* __restrict__ list, const uint32_t* __restrict__ ncnt,
    float* __restrict__ rho_out, float* __restrict__ p_out, float4* __restrict__ vel,
    float2* __restrict__ rp, int with_eos) {
    __shared__ TileMeta<CfgF> M;
    __shared__ int4 Pi[CfgF::kCap];
    __shared__ uint16_t cellof[CfgF::kCap];
    const int blk = xcd_block();
    int c0[3];
    tile_origin(TL, blk, c0);
    const SetupLoads sl = tile_setup_loads(G, TL, c0, cstart, cend, (int)threadIdx.x);
    if (tile_empty(G, TL, c0, cstart, cend)) return;
    const uint32_t total = tile_setup_finish(G, TL, c0, n, sl, M, (int)threadIdx.x);
    if (total > (uint32_t)cap_union) return;  // every target is the fallback's
    tile_stage(TL, M, cellof, [&](uint32_t j) { return pos[j]; },
               [&](uint32_t u, const int4& r, int ux, int uy, int uz) {
                   Pi[u] = tile_rec(r, ux, uy, uz);
               });
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < M.ntargets; t += CfgF::kThreads) {
        uint32_t ui, i;
        int uc[3];
        tile_target(TL, M, t, &ui, &i, uc);
        const uint32_t cnt = ncnt[i];
        const ListHead head = tile_list_head(list, i, cap);
        if (cnt > cap) continue;  // the fallback's
        const int4 pi = Pi[ui];
        double acc = 0.0;
        tile_list_loop(list, i, cap, cnt, head, [&](uint32_t u) { return Pi[u]; },
                       [&](const int4& pj) {
                           const Geom<float> g = pair_geom<3>(pi, pj, 0, 0, 0, 0, 0, 0, C);
                           density_add<KERNEL, float>(acc, g, (double)rec_mass(pj), C);
                       });
        finish_density<3, float>((int)i, acc, C, rho_out, 0, p_out, vel, rp, with_eos);
    }
}

// Momentum equation (as k_momentum) of the tile's targets whose lists are
// complete, over the union's position, velocity and (rho, P) records staged
// in LDS, with momentum_close as the epilogue; per-tile partial sums of the
// diagnostics into diag_part[q * stride + tile].
//
// The staging takes most of the LDS, so one workgroup runs per CU and
// nothing else covers its global round trips (a tile's cell ranges, then
// its records, then its targets' counts and list heads: about 45% of the
// pass measured without the pair loops).  Each workgroup therefore takes
// every P-th tile (P workgroups, one per CU, so that the tiles in flight
// are P consecutive ones).  Its sixteen waves divide the work: eight, two per
// SIMD, take the tile's targets (about 490 in a box of 6 x 6 x 4 cells), the
// other eight meanwhile hold the next tile's records (10 registers each, six
// per thread) and the cell ranges of the one after, and store them to the LDS
// when tile t no longer needs it; two tile metas and two cell tables
// alternate.  The loads wait in waves of their own since a wave's loads
// return in order: held by the target waves they stood before the pair loops'
// first wait, and their 60 registers beside the pair loops'.  The pair loops
// take half octets at a time; the VALU is busy 83% of the time, the LDS 61%.
// (256^3 cube: 3.83 ms with the loads in the target waves, 3.64 with the loader
// waves; 75^3 quintic lattice 0.213 and 0.204.  Padded lists without the
// entry-by-entry tail, as in FP64: 3.55 and 0.209, not taken.)
constexpr int kMomThreads = 2 * CfgF::kThreads;
template <int S, int KERNEL>
__global__ __launch_bounds__(kMomThreads) void k_tile_momentum(
    int n, Grid G, PairConst<float> C, Tiles TL, int cap_union, const int4* __restrict__ pos,
    const float4* __restrict__ vel, const float2* __restrict__ rp,
    const uint8_t* __restrict__ type, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, const uint4* __restrict__ list,
    const uint32_t* __restrict__ ncnt, State St, int kick, int drift, double hdt, double dt,
    CellList cl, uint32_t* __restrict__ flags,
    double* __restrict__ diag_part, int stride) {
    __shared__ TileMeta<CfgF> MM[2];
    __shared__ uint16_t cellofs[2][CfgF::kCap];
    __shared__ int4 Pi[CfgF::kCap];
    __shared__ float4 V[CfgF::kCap];
    __shared__ float2 RP[CfgF::kCap];
    // set-up and staging thread: 0 .. 511 in the loader waves, the others take
    // part in the set-up's barriers
    const int tid = (int)(threadIdx.x ^ (unsigned)CfgF::kThreads);
    // uniform over a wave, and known to be
    const bool loader = __builtin_amdgcn_readfirstlane(tid) < CfgF::kThreads;
    const int NP = (int)gridDim.x;
    const int t0 = xcd_block();
    const int t1 = TL.ntiles;
    if (t0 >= t1) return;  // the whole workgroup
    struct Rc {
        int4 p;
        float4 v;
        float2 rp;
    };
    auto load_rc = [&](uint32_t j) { return Rc{pos[j], vel[j], rp[j]}; };
    auto store_rc = [&](uint32_t u, const Rc& r, int ux, int uy, int uz) {
        Pi[u] = tile_rec(r.p, ux, uy, uz);
        V[u] = r.v;
        RP[u] = r.rp;
    };
    auto fits = [&](const TileMeta<CfgF>& M) { return M.total <= (uint32_t)cap_union; };
    // prologue (t = t0 - NP): tile t0 set up; the loop's first round stages it
    int c0[3];
    tile_origin(TL, t0, c0);
    tile_setup(G, TL, c0, cstart, cend, n, MM[0], tid);
    tile_cellof<CfgF, kMomThreads>(TL, MM[0], cellofs[0]);
    // set-up of the tile after the next one into the meta that tile t leaves,
    // by all waves (the loaders hold its cell ranges); publishes the staging
    auto set_up = [&](int t, int cur, const SetupLoads& sl) {
        if (t + 2 * NP < t1) {
            int c2[3];
            tile_origin(TL, t + 2 * NP, c2);
            tile_setup_finish(G, TL, c2, n, sl, MM[cur], tid);
            tile_cellof<CfgF, kMomThreads>(TL, MM[cur], cellofs[cur]);
        } else {
            __syncthreads();
        }
    };
    // the two roles meet at the same barriers: one for the diagnostics' sums,
    // one when tile t's records, meta and cell table are free, and set_up's
    if (loader) {
        int cur = 1;
        for (int t = t0 - NP; t < t1; t += NP, cur ^= 1) {
            const TileMeta<CfgF>& MN = MM[cur ^ 1];
            const bool stage_next = t + NP < t1 && fits(MN);
            SetupLoads sl{};
            if (t + 2 * NP < t1) {
                int c2[3];
                tile_origin(TL, t + 2 * NP, c2);
                sl = tile_setup_loads(G, TL, c2, cstart, cend, tid);
            }
            StageRegs<CfgF, Rc> R;
            if (stage_next) tile_stage_loads(MN, cellofs[cur ^ 1], load_rc, R, tid);
            if (diag_part && t >= 0) __syncthreads();
            __syncthreads();
            if (stage_next) tile_stage_store(TL, MN, cellofs[cur ^ 1], R, store_rc, tid);
            set_up(t, cur, sl);
        }
        return;
    }
    int cur = 1;
    for (int t = t0 - NP; t < t1; t += NP, cur ^= 1) {
        const TileMeta<CfgF>& M = MM[cur];
        double dsum[4] = {0.0, 0.0, 0.0, 0.0};
        if (t >= 0 && fits(M)) {
            for (uint32_t tt = (uint32_t)(tid - CfgF::kThreads); tt < M.ntargets;
                 tt += CfgF::kThreads) {
                // every global load of a target up front (count, type, the
                // list's first octets, the epilogue's state)
                uint32_t ui, i;
                int uc[3];
                tile_target(TL, M, tt, &ui, &i, uc);
                const uint32_t cnt = ncnt[i];
                const bool fluid = type[i] == 0;
                const ListHead head = tile_list_head(list, i, cap);
                const CloseIn ci = close_load<3>((int)i, St, drift, diag_part != nullptr);
                if (cnt > cap) continue;  // the fallback's
                float acc[3] = {0.f, 0.f, 0.f};
                if (fluid) {
                    const int4 pi = Pi[ui];
                    const float4 vi = V[ui];
                    const float2 rpi = RP[ui];
                    float ax = C.g[0], ay = C.g[1], az = C.g[2];
                    struct Nb {
                        int4 p;
                        float4 v;
                        float2 rp;
                    };
                    tile_list_loop<4>(list, i, cap, cnt, head,
                                   [&](uint32_t u) { return Nb{Pi[u], V[u], RP[u]}; },
                                   [&](const Nb& b) {
                                       const Geom<float> g =
                                           pair_geom<3>(pi, b.p, 0, 0, 0, 0, 0, 0, C);
                                       momentum_add<3, KERNEL, float>(ax, ay, az, g,
                                                                      rec_mass(b.p), vi, rpi,
                                                                      b.v, b.rp, C);
                                   });
                    acc[0] = ax;
                    acc[1] = ay;
                    acc[2] = az;
                }
                double dv[4] = {0.0, 0.0, 0.0, 0.0};
                momentum_close<3, float>((int)i, acc, fluid, St, G, kick, drift, hdt, dt, cl,
                                         flags, diag_part != nullptr, dv, &ci);
                for (int q = 0; q < 4; ++q) dsum[q] += dv[q];
            }
        }
        if (diag_part && t >= 0) tile_block_sum<4, CfgF::kThreads>(dsum, diag_part, t, stride);
        __syncthreads();
        set_up(t, cur, SetupLoads{});
    }
}

// ---------------------------------------------------------------------------
// FP64 passes over the tiles: the lists of k_tile_build<S, double>, the
// union's records staged in LDS as they are (absolute positions), and the pair
// terms of the global passes in the same order, so the results are bitwise
// theirs.  A separation across a periodic face needs the neighbour's image
// (pair_geom's w): a byte per staged particle, read only in tiles whose
// union reaches over a face.
// (160^3 cube, h = 1.5 dx, half-size cells, against the walk build and the
// passes over global lists: build 1.63 against 4.62 ms, density 0.88 against
// 1.93, momentum 1.77 against 3.90; those gather 80 bytes a neighbour through
// L1 and L2 at 9 TB/s.  Boxes of 4 x 4 x 4 cells are what 72 bytes a staged
// particle leaves room for.)
struct RecD {
    double4 p;
    uint32_t w;
};
// Staged position records in two arrays of 16 bytes an entry: a 16-byte read
// at a random entry then starts at any of the LDS's 16 groups of four banks
// (at every other one with 32-byte entries).
struct PosD {
    double2 xy[CfgD::kCap], zm[CfgD::kCap];
    __device__ __forceinline__ void put(uint32_t u, const double4& r) {
        xy[u] = make_double2(r.x, r.y);
        zm[u] = make_double2(r.z, r.w);
    }
    __device__ __forceinline__ double4 get(uint32_t u) const {
        const double2 a = xy[u], b = zm[u];
        double4 r;
        r.x = a.x;
        r.y = a.y;
        r.z = b.x;
        r.w = b.y;
        return r;
    }
};
__device__ __forceinline__ uint32_t tile_image(const Grid& G, const Tiles& TL, const int c0[3],
                                               int ux, int uy, int uz) {
    return (uint32_t)(tile_wrap(G, 0, c0[0], ux, TL.S) + 1) |
           ((uint32_t)(tile_wrap(G, 1, c0[1], uy, TL.S) + 1) << 2) |
           ((uint32_t)(tile_wrap(G, 2, c0[2], uz, TL.S) + 1) << 4);
}
// Whether some union cell of the tile lies over a periodic face.
__device__ __forceinline__ bool tile_wraps(const Grid& G, const Tiles& TL, const int c0[3]) {
    const int hi[3] = {TL.tw, TL.th, TL.td};
    bool w = false;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        w |= G.periodic[k] && (c0[k] < TL.S || c0[k] + hi[k] + TL.S > G.nc[k]);
    return w;
}
template <bool WRAP>
__device__ __forceinline__ Geom<double> tile_geom(const double4& ri, const double4& rj, uint32_t w,
                                                  const PairConst<double>& C) {
    if (!WRAP) return pair_geom<3>(ri, rj, 0, 0, 0, 0, 0, 0, C);
    return pair_geom<3>(ri, rj, 0, 0, 0, (int)(w & 3u) - 1, (int)((w >> 2) & 3u) - 1,
                        (int)(w >> 4) - 1, C);
}

// Summation density (eq. 2), and with_eos the Tait EOS, of the tile's targets
// with complete lists, FP64 (as k_density).
template <int S, int KERNEL>
__global__ __launch_bounds__(CfgD::kThreads) void k_tile_density64(
    int n, Grid G, PairConst<double> C, Tiles TL, int cap_union, const double4* __restrict__ pos,
    const uint32_t* __restrict__ cstart, const uint32_t* __restrict__ cend, uint32_t cap,
    const uint4* __restrict__ list, const uint32_t* __restrict__ ncnt,
    double* __restrict__ rho_out, double* __restrict__ p_out, double4* __restrict__ vel,
    double2* __restrict__ rp, int with_eos, TileTest test) {
    __shared__ TileMeta<CfgD> M;
    __shared__ PosD P;
    __shared__ uint8_t W[CfgD::kCap];
    __shared__ uint16_t cellof[CfgD::kCap];
    const int blk = xcd_block();
    int c0[3];
    tile_origin(TL, blk, c0);
    const SetupLoads sl = tile_setup_loads(G, TL, c0, cstart, cend, (int)threadIdx.x);
    if (tiles_off(test)) return;
    if (tile_empty(G, TL, c0, cstart, cend)) return;
    const uint32_t total = tile_setup_finish(G, TL, c0, n, sl, M, (int)threadIdx.x);
    if (total > (uint32_t)cap_union) return;  // every target is the fallback's
    tile_stage(TL, M, cellof, [&](uint32_t j) { return pos[j]; },
               [&](uint32_t u, const double4& r, int ux, int uy, int uz) {
                   P.put(u, r);
                   W[u] = (uint8_t)tile_image(G, TL, c0, ux, uy, uz);
               });
    __syncthreads();
    const bool wraps = tile_wraps(G, TL, c0);
    for (uint32_t t = threadIdx.x; t < M.ntargets; t += CfgD::kThreads) {
        uint32_t ui, i;
        int uc[3];
        tile_target(TL, M, t, &ui, &i, uc);
        const uint32_t cnt = ncnt[i];
        const ListHead head = tile_list_head(list, i, cap);
        if (cnt > cap) continue;  // the fallback's
        const double4 pi = P.get(ui);
        double acc = 0.0;
        auto sum = [&](auto wrap) {
            constexpr bool kWrap = decltype(wrap)::value;
            tile_list_whole(list, i, cap, cnt, head,
                            [&](uint32_t u) { return RecD{P.get(u), kWrap ? (uint32_t)W[u] : 0u}; },
                            [&](const RecD& b, uint32_t k) {
                                const Geom<double> g = tile_geom<kWrap>(pi, b.p, b.w, C);
                                density_add<KERNEL, double>(acc, g, k < cnt ? rec_mass(b.p) : 0.0,
                                                            C);
                            });
        };
        if (wraps)
            sum(BoolC<true>());
        else
            sum(BoolC<false>());
        finish_density<3, double>((int)i, acc, C, rho_out, 0, p_out, vel, rp, with_eos);
    }
}

// Momentum equation of the tile's targets with complete lists, FP64 (as
// k_momentum), with momentum_close as the epilogue; per-tile partial sums of
// the diagnostics into diag_part[q * stride + tile].  A staged particle takes
// 73 bytes, so that one workgroup fills a CU's LDS and takes every P-th tile
// (P workgroups, one per CU).  Its eight waves divide the work: four, one per
// SIMD, take the tile's targets, the other four meanwhile hold the next tile's
// records (18 registers each, eight per thread) and the cell ranges of the one
// after in registers and store them when the four are done.  The loads wait in
// waves of their own, since a wave's loads return in order and the pair loops
// would wait for them.
constexpr int kMom64Threads = 2 * CfgD::kThreads;
template <int S, int KERNEL>
__global__ __launch_bounds__(kMom64Threads) void k_tile_momentum64(
    int n, Grid G, PairConst<double> C, Tiles TL, int cap_union, const double4* __restrict__ pos,
    const double4* __restrict__ vel, const double2* __restrict__ rp,
    const uint8_t* __restrict__ type, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t cap, const uint4* __restrict__ list,
    const uint32_t* __restrict__ ncnt, State St, int kick, int drift, double hdt, double dt,
    CellList cl, uint32_t* __restrict__ flags,
    double* __restrict__ diag_part, int stride, TileTest test) {
    __shared__ TileMeta<CfgD> MM[2];
    __shared__ uint16_t cellofs[2][CfgD::kCap];
    __shared__ PosD P;
    __shared__ double2 Vxy[CfgD::kCap];
    __shared__ double2 RP[CfgD::kCap];
    __shared__ double Vz[CfgD::kCap];
    __shared__ uint8_t W[CfgD::kCap];
    // set-up and staging thread: 0 .. 255 in the loader waves, the others take
    // part in the set-up's barriers
    const int tid = (int)(threadIdx.x ^ (unsigned)CfgD::kThreads);
    // uniform over a wave, and known to be
    const bool loader = __builtin_amdgcn_readfirstlane(tid) < CfgD::kThreads;
    const int NP = (int)gridDim.x;
    const int t0 = xcd_block();
    const int t1 = TL.ntiles;
    if (t0 >= t1) return;  // the whole workgroup
    struct Rc {
        double4 p;
        double2 vxy;
        double vz;
        double2 rp;
    };
    auto load_rc = [&](uint32_t j) {
        const double4 v = vel[j];
        return Rc{pos[j], make_double2(v.x, v.y), v.z, rp[j]};
    };
    int cs[3] = {0, 0, 0};  // origin of the tile being stored
    auto store_rc = [&](uint32_t u, const Rc& r, int ux, int uy, int uz) {
        P.put(u, r.p);
        Vxy[u] = r.vxy;
        Vz[u] = r.vz;
        RP[u] = r.rp;
        W[u] = (uint8_t)tile_image(G, TL, cs, ux, uy, uz);
    };
    auto fits = [&](const TileMeta<CfgD>& M) { return M.total <= (uint32_t)cap_union; };
    // prologue (t = t0 - NP): tile t0 set up; the loop's first round stages it
    tile_origin(TL, t0, cs);
    tile_setup(G, TL, cs, cstart, cend, n, MM[0], tid);
    if (tiles_off(test)) {  // the fallback's, all of them
        if (diag_part)
            for (int k = (int)threadIdx.x; t0 + (k >> 2) * NP < t1; k += kMom64Threads)
                diag_part[(int64_t)(k & 3) * stride + t0 + (k >> 2) * NP] = 0.0;
        return;
    }
    tile_cellof<CfgD, kMom64Threads>(TL, MM[0], cellofs[0]);
    // set-up of the tile after the next one into the meta that tile t leaves,
    // by all waves (the loaders hold its cell ranges); publishes the staging
    auto set_up = [&](int t, int cur, const SetupLoads& sl) {
        if (t + 2 * NP < t1) {
            int c2[3];
            tile_origin(TL, t + 2 * NP, c2);
            tile_setup_finish(G, TL, c2, n, sl, MM[cur], tid);
            tile_cellof<CfgD, kMom64Threads>(TL, MM[cur], cellofs[cur]);
        } else {
            __syncthreads();
        }
    };
    // the two roles meet at the same barriers: one for the diagnostics' sums,
    // one when tile t's records, meta and cell table are free, and set_up's
    if (loader) {
        int cur = 1;
        for (int t = t0 - NP; t < t1; t += NP, cur ^= 1) {
            const TileMeta<CfgD>& MN = MM[cur ^ 1];
            const bool stage_next = t + NP < t1 && fits(MN);
            SetupLoads sl{};
            if (t + 2 * NP < t1) {
                int c2[3];
                tile_origin(TL, t + 2 * NP, c2);
                sl = tile_setup_loads(G, TL, c2, cstart, cend, tid);
            }
            StageRegs<CfgD, Rc> R;
            if (stage_next) tile_stage_loads(MN, cellofs[cur ^ 1], load_rc, R, tid);
            if (diag_part && t >= 0) __syncthreads();
            __syncthreads();
            if (stage_next) {
                tile_origin(TL, t + NP, cs);
                tile_stage_store(TL, MN, cellofs[cur ^ 1], R, store_rc, tid);
            }
            set_up(t, cur, sl);
        }
        return;
    }
    int cur = 1;
    for (int t = t0 - NP; t < t1; t += NP, cur ^= 1) {
        const TileMeta<CfgD>& M = MM[cur];
        double dsum[4] = {0.0, 0.0, 0.0, 0.0};
        if (t >= 0 && fits(M)) {
            int c0[3];
            tile_origin(TL, t, c0);
            const bool wraps = tile_wraps(G, TL, c0);
            for (uint32_t tt = (uint32_t)(tid - CfgD::kThreads); tt < M.ntargets;
                 tt += CfgD::kThreads) {
                uint32_t ui, i;
                int uc[3];
                tile_target(TL, M, tt, &ui, &i, uc);
                const uint32_t cnt = ncnt[i];
                const bool fluid = type[i] == 0;
                const ListHead head = tile_list_head(list, i, cap);
                const CloseIn ci = close_load<3>((int)i, St, drift, diag_part != nullptr);
                if (cnt > cap) continue;  // the fallback's
                double acc[3] = {0.0, 0.0, 0.0};
                if (fluid) {
                    const double4 pi = P.get(ui);
                    double4 vi;
                    vi.x = Vxy[ui].x;
                    vi.y = Vxy[ui].y;
                    vi.z = Vz[ui];
                    vi.w = 0.0;
                    const double2 rpi = RP[ui];
                    double ax = C.g[0], ay = C.g[1], az = C.g[2];
                    struct Nb {
                        double4 p;
                        double2 vxy;
                        double vz;
                        double2 rp;
                        uint32_t w;
                    };
                    auto sum = [&](auto wrap) {
                        constexpr bool kWrap = decltype(wrap)::value;
                        // (the target itself adds exact zeros, see momentum_add)
                        tile_list_whole(
                            list, i, cap, cnt, head,
                            [&](uint32_t u) {
                                return Nb{P.get(u), Vxy[u], Vz[u], RP[u], kWrap ? (uint32_t)W[u] : 0u};
                            },
                            [&](const Nb& b, uint32_t) {
                                const Geom<double> g = tile_geom<kWrap>(pi, b.p, b.w, C);
                                double4 vj;
                                vj.x = b.vxy.x;
                                vj.y = b.vxy.y;
                                vj.z = b.vz;
                                vj.w = 0.0;
                                momentum_add<3, KERNEL, double>(ax, ay, az, g, rec_mass(b.p), vi, rpi,
                                                                vj, b.rp, C);
                            });
                    };
                    if (wraps)
                        sum(BoolC<true>());
                    else
                        sum(BoolC<false>());
                    acc[0] = ax;
                    acc[1] = ay;
                    acc[2] = az;
                }
                double dv[4] = {0.0, 0.0, 0.0, 0.0};
                momentum_close<3, double>((int)i, acc, fluid, St, G, kick, drift, hdt, dt, cl,
                                          flags, diag_part != nullptr, dv, &ci);
                for (int q = 0; q < 4; ++q) dsum[q] += dv[q];
            }
        }
        if (diag_part && t >= 0) tile_block_sum<4, CfgD::kThreads>(dsum, diag_part, t, stride);
        __syncthreads();
        set_up(t, cur, SetupLoads{});
    }
}

// Fallback density: the targets the tile build left (count above cap, or
// kTileOverflow), by the cell walk in global memory (density_one); only the
// kTileOverflow ones are counted (the build counted the others).  With the
// tiles off (FP64, tiles_off), every target, whose global-format list (list_cap entries
// at most) and count are written on the way.
template <int S, int KERNEL, typename T>
__global__ __launch_bounds__(kBlock) void k_tile_fallback_density(
    int n, Grid G, PairConst<T> C, const uint32_t* __restrict__ skey,
    const typename Rec<T>::type* __restrict__ pos, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, uint32_t* __restrict__ ncnt, uint32_t cap,
    uint32_t* __restrict__ list, uint32_t list_cap,
    T* __restrict__ rho_out, T* __restrict__ p_out, typename Vec4<T>::type* __restrict__ vel,
    typename Vec2<T>::type* __restrict__ rp, int with_eos, int count_pairs, unsigned long long* __restrict__ pairs,
    uint32_t epoch, const uint32_t* __restrict__ fallback, TileTest test) {
    const bool all = sizeof(T) == 8 && tiles_off(test);
    if (!all && *fallback != epoch) return;
    uint32_t counted = 0;
    if (all) {
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
            const typename Rec<T>::type ri = pos[i];
            uint32_t* __restrict__ col = list + list_column((uint32_t)i, list_cap);
            uint32_t cnt = 0;
            double acc = 0.0;
            walk_pairs<3, S, T>(G, C, skey[i], ri, pos, skey, cstart, cend, (uint32_t)n, NoPayload(),
                                [&](uint32_t j, const typename Rec<T>::type& rj, int,
                                    const Geom<T>& g, uint32_t code) {
                                    if (cnt < list_cap)
                                        col[cnt * kListTile] = (j << NbrCode<3, S, T>::kBits) | code;
                                    density_add<KERNEL, T>(acc, g, (double)rec_mass(rj), C);
                                    ++cnt;
                                });
            finish_density<3, T>(i, acc, C, rho_out, 0, p_out, vel, rp, with_eos);
            counted += cnt;
            ncnt[i] = cnt;
        }
        if (count_pairs) block_count(counted, pairs, blockIdx.x);
        return;
    }
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const uint32_t c = ncnt[i];
        if (c <= cap) continue;
        // a null list makes density_one walk the cells
        const uint32_t k = density_one<3, S, KERNEL, T>(i, G, C, skey, pos, cstart, cend, n,
                                                        nullptr, ncnt, cap, rho_out, 0, p_out,
                                                        vel, rp, with_eos);
        if (c == kTileOverflow) counted += k;
    }
    if (count_pairs) block_count(counted, pairs, blockIdx.x);
}

// Fallback momentum, as k_tile_fallback_density (list: the lists that it wrote
// if the tiles are off, null: no density pass went before); diagnostics partials
// of its blocks at diag_part[q * stride + b] (zeros when there is nothing to
// do).
template <int S, int KERNEL, typename T>
__global__ __launch_bounds__(kBlock, sizeof(T) == 8 && S == 1 ? 3 : 1) void k_tile_fallback_momentum(
    int n, Grid G, PairConst<T> C, const uint32_t* __restrict__ skey,
    const typename Rec<T>::type* __restrict__ pos, const typename Vec4<T>::type* __restrict__ vel,
    const typename Vec2<T>::type* __restrict__ rp, const uint8_t* __restrict__ type, const uint32_t* __restrict__ cstart,
    const uint32_t* __restrict__ cend, const uint32_t* __restrict__ ncnt, uint32_t cap,
    const uint32_t* __restrict__ list, uint32_t list_cap, State St,
    int kick, int drift, double hdt, double dt, CellList cl, uint32_t* __restrict__ flags, double* __restrict__ diag_part,
    int stride, uint32_t epoch, const uint32_t* __restrict__ fallback,
    TileTest test) {
    double dsum[4] = {0.0, 0.0, 0.0, 0.0};
    const bool all = sizeof(T) == 8 && tiles_off(test);
    if (all || *fallback == epoch) {
        if (!all) list = nullptr;
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
            if (!all && ncnt[i] <= cap) continue;
            double dv[4] = {0.0, 0.0, 0.0, 0.0};
            momentum_one<3, S, KERNEL, T>(i, G, C, skey, pos, vel, rp, type, cstart, cend, n,
                                          list, ncnt, list_cap, St, kick, drift, hdt, dt, cl, flags,
                                          diag_part != nullptr, dv);
            for (int q = 0; q < 4; ++q) dsum[q] += dv[q];
        }
    }
    if (diag_part) block_sum4<4>(dsum, diag_part, blockIdx.x, stride);
}

}  // namespace sph
