// near_tile.h -- staging of a group's near-field sources through LDS.
//
// The sources of a group are the particles of the cells on its union near
// list (ascending labels; within a cell, tree order). A wave takes the list
// 64 entries at a time: lane j reads entry j, and an exclusive scan of the
// cell sizes gives each entry's first source in the chunk. The entries that
// have sources stand in LDS by their rank among them. Sources are then staged
// 64 at a time: lane j of a tile finds its entry by counting the entries that
// start at or before it (a mark at each start inside the tile, read back as a
// ballot), and the caller takes them from its lane or puts them into LDS in the
// order it needs. Entries that the caller does not need (for example cells with no candidate bit, for the
// neighbour search) are given zero sources.
// The staging is a good part of a tile's instructions where cells are small
// (cells of 8: 64 sources are 8 rows of a dozen instructions). A binary search
// of the prefix for each source and centres of mass read and converted per
// source, not per entry, made it 140 instructions of 316.
#pragma once

#include "rcb_internal.h"

namespace rcb {

__device__ __forceinline__ void tile_sync() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// One lane's entry of a chunk
struct ChunkEntry {
    int32_t label, first;   // the cell and its first particle
    int32_t pos;            // its first source in the chunk (INT32_MAX: no sources)
    int rank;               // among the entries with sources
    int tot;                // sources of the chunk (the same on every lane)
    __device__ __forceinline__ bool has() const { return pos != INT32_MAX; }
    // particle of source q of this entry: q + off()
    __device__ __forceinline__ int32_t off() const { return first - pos; }
};
// Entries from cell sizes (0: not wanted)
__device__ __forceinline__ ChunkEntry chunk_entry(int32_t label, int32_t first, int32_t count) {
    ChunkEntry ce;
    const int incl = wave_incl_scan(count);
    ce.label = label;
    ce.first = first;
    ce.pos = count > 0 ? incl - count : INT32_MAX;
    ce.rank = rank_below(ballot(count > 0));
    ce.tot = __builtin_amdgcn_readlane(incl, kWave - 1);
    return ce;
}
// Entries [e0, min(e0 + 64, n1)) of a near list; those whose (near|cand) mask
// has no bit of keep_mask count as empty.
__device__ __forceinline__ ChunkEntry load_chunk(const uint64_t *__restrict__ gnear,
                                                 const int32_t *__restrict__ nfirst,
                                                 const int32_t *__restrict__ ncount, int64_t e0, int64_t n1,
                                                 uint32_t keep_mask) {
    const int64_t e = e0 + lane_id();
    const uint64_t ent = gnear[e < n1 ? e : n1 - 1];
    const int32_t lab = (int32_t)((uint32_t)ent & 0x7fffffffu);
    const bool want = e < n1 && ((uint32_t)(ent >> 32) & 0xffffu & keep_mask);
    int32_t f = 0, c = 0;
    if (want) {
        f = nfirst[lab];
        c = ncount[lab];
    }
    return chunk_entry(lab, f, c);
}
// The entry (by rank) of this lane's source of the tile of sources
// [t, t + 64). mark: 64 words of the wave's LDS, zero before the first tile;
// gen: counts the wave's tiles.
__device__ __forceinline__ int tile_entry(const ChunkEntry &ce, int t, uint32_t *mark, uint32_t &gen) {
    ++gen;
    const uint32_t o = (uint32_t)ce.pos - (uint32_t)t;
    if (o < (uint32_t)kWave) mark[o] = gen;
    tile_sync();
    const bool start = mark[lane_id()] == gen;
    tile_sync();
    return __popcll(ballot(ce.pos < t)) + rank_below(ballot(start)) + (start ? 1 : 0) - 1;
}

// a staged source, and what a chunk's entry adds to its particles: in the mixed
// form the FP32 shift from the entry's centre of mass to the leaf's
struct alignas(16) SrcF {
    float x, y, z, m;
};
struct alignas(16) SrcD {
    double x, y, z, m;
};
struct alignas(16) EntF {
    float x, y, z;
    int32_t off;
};
struct EntD {
    int32_t off;
};

// Lanes of a wave over the sinks of one leaf of c > 0 particles: S = min(c, 64)
// sinks per pass, J = 64 / S slices per sink, lane = sslot * J + slice. Lanes
// with sslot >= S hold no sink. Slice j of a sink takes tile sources
// j, j + J, j + 2J, ...
struct LeafLanes {
    int S, J, sslot, slice;
    uint32_t inv;   // of J, for rows(): exact for n < 65536 / J
    __device__ __forceinline__ int rows(int n) const { return (int)(((uint32_t)n * inv) >> 16); }   // n / J
};
__device__ __forceinline__ LeafLanes leaf_lanes(int c) {
    LeafLanes L;
    L.S = c < kWave ? c : kWave;
    L.J = __builtin_amdgcn_readfirstlane(kWave / L.S);
    L.inv = __builtin_amdgcn_readfirstlane(65536 / L.J + 1);
    L.sslot = lane_id() / L.J;
    L.slice = lane_id() - L.sslot * L.J;
    return L;
}

// Sum over the J consecutive lanes of each segment; the total lands on the
// segment's first lane (slice 0). After the step with offset o, lane i holds
// the sum of its segment's lanes [i, min(i + 2o, end)).
template <typename T>
__device__ __forceinline__ T seg_sum(T v, int slice, int J) {
    for (int o = 1; o < J; o <<= 1) {
        const T w = __shfl_down(v, o, kWave);
        if (slice + o < J) v += w;
    }
    return v;
}

// How far a leaf's sinks (this lane's: x, y, z from the leaf's centre of mass,
// its smoothing length h) reach from that centre: a source b farther from it
// than reach + h_b is farther than h_a + h_b from every sink a (the callers add
// 0.1%, far above the rounding). In the form's own type: squares of offsets of
// 1e-22 and below are nothing in FP32, and sources within the support would
// count as outside it.
__device__ __forceinline__ float sink_reach(float x, float y, float z, float h) {
    float reach = sqrtf((x * x + y * y) + z * z) + h;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) reach = fmaxf(reach, __shfl_xor(reach, o, kWave));
    return reach;
}
__device__ __forceinline__ double sink_reach(double x, double y, double z, double h) {
    return uniform_f64(wave_max(sqrt((x * x + y * y) + z * z) + h));
}

}  // namespace rcb
