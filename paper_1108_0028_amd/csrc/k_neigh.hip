// k_neigh.hip -- neighbour search from the walk's candidate cells
// (Sec. 2.3: "Neighbour walk" culled to the true neighbours, and the
// one-dimensional "Neighbour list").
//
// One or more waves per leaf (a workgroup), each with every H-th of the leaf's
// sinks. Lanes are sources: the candidate cells of the leaf (cells of its group's
// near list, ascending labels, whose candidate mask has the leaf) are staged 64
// particles at a time (near_tile.h), those inside the leaf's sphere wait in LDS
// until 64 are there, and then every sink is tested against them in a row of its
// own. A pair is a neighbour iff b != a and |r_a - r_b|^2 < (2 h_a)^2 in FP64 on
// the tree's copy of the inputs (the same predicate for every precision mode). A
// row's hits take the list's next slots by their rank in its ballot, the sinks'
// counts are kept one a lane, so the lists need no atomics.
// The sphere (centre g_A, radius h_node(A) padded by 2^-32, Sec. 2.3.1): a
// neighbour b of a sink a has |r_b - g_A| <= |r_b - r_a| + |r_a - g_A| < 2 h_a +
// |r_a - g_A| <= h_node(A), so no neighbour is dropped.
// Bound by its chains: loads and stores of a wave wait in order, a row is some
// 20 dependent instructions, seven waves a SIMD. With lanes as (sink, slice of the
// sources) and a slot from an LDS atomic for each hit, rows of many hits of few sinks
// serialised: rcb_neighbours_count of 37,000 particles (lists of up to 875) 192, now
// 110 us; 300,000 clumpy 560 and 380; 500,000 in cells of 61 800 and 715; 16M clumpy 8760 and
// 8190; 4M and 500,000 of even lists 1905 and 1930, 402 and 422.
// A leaf's work varies tenfold, so wider units of work leave the chip waiting
// for the longest: one wave per group of 8 leaves took 690 us for the 37,000 (512
// groups).
//
// The count call writes each particle's count into the caller's offsets
// array (scanned in place afterwards) and its first kNbCap ids into a slab
// row indexed by caller id (by tree position for very large N, see
// tree_rows), the next ones into a chain of chunks of a shared pool. The fill
// call streams the slab in caller order,
// sorts each list ascending (a 64-input sorting network held by 8 lanes) and
// stores it into the CSR; longer lists follow wave by wave. Lowest-level
// cells holding a particle for which the pool had no chunk left (queued by
// the count call) are searched again, one wave each, writing only those
// particles' lists at their offsets; each such list is then sorted by one
// workgroup.
#include <algorithm>

#include "near_tile.h"
#include "rcb_internal.h"

namespace rcb {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
constexpr int kNbCap = 64;        // slab slots per particle (~50 neighbours expected)
constexpr int kNbChunk = 64;      // slots of an overflow chunk
constexpr int kNbWaveMax = 256;   // lists of up to 256 ids are sorted by one wave in registers
constexpr int kLongLds = 4096;    // lists searched again: sorted in LDS up to this length
constexpr int kSinks = 32;        // sinks of a pass over the candidates

struct NeighArgs {
    int64_t nleaf;
    int gk;
    const double4 *rec;       // walk records: rec[2 label] = (box centre, h_node_int)
    const double *hnode;
    const int32_t *nfirst, *ncount;
    const int64_t *gnear_beg, *gnear_end;
    const uint64_t *gnear;
    const double *px, *py, *pz, *ph;
    const int32_t *pid;
    int64_t *counts;          // slab mode: per-particle counts (caller order)
    const int64_t *offsets;   // fill mode: list starts (caller order)
    int32_t *ids;             // fill mode: final lists; slab mode: kNbCap slots per caller index
    int32_t *pool;            // slab mode: overflow chunks of kNbChunk slots
    int32_t *next;            // slab mode: the chunk after each chunk of a list
    int64_t sub_cap;          // chunks of each sub-pool
    int32_t sub_mask;         // sub-pools - 1 (a power of two of them)
    int32_t *head;            // per caller index: its first chunk, or -1 for a list searched again
    int32_t *ctl;             // [0] lists searched again, [1] leaves queued, [2] kept lists of more than
                              // kNbWaveMax ids (slab mode); [kSubCtl (1 + i)] chunks taken from sub-pool
                              // i; fill mode: [0] lists appended to longq
    int32_t *queue;           // leaves (index from 0) holding a list searched again: appended in
                              // slab mode, searched again (wave i: queue[i]) otherwise
    int32_t *longq;           // fill mode: the caller indices of the lists written here
    int64_t first;            // slab mode: this launch's first leaf (one per workgroup)
    bool tree_rows;           // slab mode: rows by tree position (else by caller index)
};

struct alignas(16) SrcN {
    double x, y, z;
    int32_t pb;   // tree position
    int32_t id;   // caller index
};
struct alignas(16) SinkN {
    double x, y, z;
    double lim;   // (2 h)^2, or -1: takes no neighbours
};

// wait: the kept sources that no pass has taken yet (at most 63, and a tile
// joins them). chunk: per sink, its list's last two chunks, by parity (the slots
// that one row hands out are at most 64 consecutive ones and touch at most two).
struct NeighShared {
    int32_t off[kWave];     // of the chunk's entries with sources
    uint32_t mark[kWave];
    SrcN wait[2 * kWave];
    SinkN sink[kSinks];
    int32_t chunk[kSinks][2];
};

// Chunk counters: one per sub-pool, 64 bytes apart, and neighbouring groups
// take different sub-pools. With one counter every list past its row (nearly
// all of them at 105 neighbours) waited for the same address: 500,000 such
// lists cost 5.0 of the search's 5.7 ms, about 10 ns each.
constexpr int kSubMax = 64;
constexpr int kSubCtl = 16;
inline size_t ctl_bytes(int subs) { return sizeof(int32_t) * kSubCtl * (1 + subs); }

// SLAB: ids go to slab row (caller index) while it has room, then to a chain
// of chunks, each taken by the hit of its first slot; lists whose chunk could
// not be had are only counted from there on, and their leaf is queued.
// Otherwise only the sinks queued that way are searched, their ids going to
// offsets[pid] + slot.
template <bool SLAB, int H>
__global__ __launch_bounds__(H * kWave) void k_neigh(NeighArgs a) {
    __shared__ NeighShared sh_all[H];
    __shared__ int over_any;
    const int lane = lane_id();
    const int wv = H > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) : 0;
    NeighShared &sh = sh_all[wv];
    const int G = 1 << a.gk;
    int64_t l;   // the workgroup's leaf, from 0
    if constexpr (SLAB) {
        l = a.first + xcd_block<kXcdLeaves>();
    } else {
        l = __builtin_amdgcn_readfirstlane(a.queue[blockIdx.x]);
    }
    const int64_t gi = l >> a.gk, A = a.nleaf + l;
    const int li = (int)(l & (G - 1));
    const int32_t sA = a.nfirst[A], c = a.ncount[A];
    if (c == 0) return;
    const int64_t n0 = a.gnear_beg[gi], n1 = a.gnear_end[gi];
    bool leaf_over = false;   // slab mode: a list of this leaf is searched again
    const double4 gA = a.rec[2 * A];
    const double rA = a.hnode[A] * kReachPad;
    const double rA2 = rA * rA;
    sh.mark[lane] = 0;
    uint32_t gen = 0;
    for (int g0 = 0; g0 < c; g0 += kSinks) {
        const int cs = c - g0 < kSinks ? c - g0 : kSinks;
        // lane i: sink i, if it is one of this wave's
        const int32_t p0 = sA + g0;
        const int32_t pa = p0 + (lane < cs ? lane : 0);
        const int32_t oa = a.pid[pa];
        bool has_sink = lane < cs && (H == 1 || lane % H == wv);
        int64_t o0 = 0;
        if constexpr (!SLAB) {   // the lists the count call could not keep
            o0 = has_sink ? a.offsets[oa] : 0;
            has_sink = has_sink && a.offsets[oa + 1] - o0 > kNbCap && a.head[oa] < 0;
        }
        if (ballot(has_sink) == 0ull) continue;
        if (lane < cs) {
            const double two_h = 2.0 * a.ph[pa];
            sh.sink[lane] = SinkN{a.px[pa], a.py[pa], a.pz[pa], has_sink ? two_h * two_h : -1.0};
        }
        const int32_t row_of = a.tree_rows ? pa : oa;   // slab mode
        int count = 0;                                  // lane i: neighbours of sink i so far
        tile_sync();
        // slab mode, slots past the row: hit lanes with slot r of sink i, in one of
        // the list's chunks, each taken by the hit of its first slot
        auto put_far = [&](int i, bool hit, uint32_t r, int32_t id) {
            const bool far = hit && r >= (uint32_t)kNbCap;
            const uint32_t q = (r - kNbCap) / kNbChunk, o = (r - kNbCap) % kNbChunk;
            if (far && o == 0) {
                const int32_t prev = q ? sh.chunk[i][(q - 1) & 1] : 0;
                int32_t ch = -1;
                if (prev >= 0) {
                    const int32_t sub = (int32_t)gi & a.sub_mask;
                    const int32_t k = atomicAdd(a.ctl + kSubCtl * (1 + sub), 1);
                    if (k < a.sub_cap) {
                        ch = (int32_t)(sub * a.sub_cap) + k;
                        if (q) a.next[prev] = ch;
                        else a.head[a.pid[p0 + i]] = ch;
                    }
                }
                sh.chunk[i][q & 1] = ch;
            }
            tile_sync();
            if (far) {
                const int32_t ch = sh.chunk[i][q & 1];
                if (ch >= 0) a.pool[(int64_t)ch * kNbChunk + o] = id;
            }
            tile_sync();
        };
        // one pass: the waiting sources [at, at + n), one a lane, against every sink
        auto pass = [&](int at, int n) {
            const SrcN s = sh.wait[at + (lane < n ? lane : 0)];
            const double sx = lane < n ? s.x : __builtin_inf();   // (never within lim)
            auto put = [&](int i, bool hit) {
                const uint64_t m = ballot(hit);
                if (m == 0) return;
                const int have = __builtin_amdgcn_readlane(count, i);
                const int r = have + rank_below(m), now = have + __popcll(m);
                count = lane == i ? now : count;
                if constexpr (SLAB) {
                    int32_t *const row = a.ids + (int64_t)__builtin_amdgcn_readlane(row_of, i) * kNbCap;
                    if (hit && r < kNbCap) row[r] = s.id;
                    if (now > kNbCap) put_far(i, hit, (uint32_t)r, s.id);
                } else {
                    const int64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)o0, i);
                    const int64_t hi = __builtin_amdgcn_readlane((int)(o0 >> 32), i);
                    int32_t *const row = a.ids + (lo | hi << 32);
                    if (hit) row[r] = s.id;
                }
            };
            auto test = [&](int i) {
                const SinkN k = sh.sink[i];
                return (dist2(k.x, k.y, k.z, sx, s.y, s.z) < k.lim) & (s.pb != p0 + i);
            };
            int i = wv;
            for (; i + H < cs; i += 2 * H) {   // (two rows per step: their LDS reads overlap)
                const bool h0 = test(i), h1 = test(i + H);
                put(i, h0);
                put(i + H, h1);
            }
            if (i < cs) put(i, test(i));
        };
        int fill = 0;   // kept sources waiting
        for (int64_t e0 = n0; e0 < n1; e0 += kWave) {
            const ChunkEntry ce = load_chunk(a.gnear, a.nfirst, a.ncount, e0, n1, 1u << (8 + li));
            const int tot = ce.tot;
            if (ce.has()) sh.off[ce.rank] = ce.off();
            for (int t = 0; t < tot; t += kWave) {
                const int nt = tot - t < kWave ? tot - t : kWave;
                // (lanes past the end read the last source again)
                const int32_t spb = sh.off[tile_entry(ce, t, sh.mark, gen)] + (t + (lane < nt ? lane : nt - 1));
                const double sx = a.px[spb], sy = a.py[spb], sz = a.pz[spb];
                const int32_t sid = a.pid[spb];
                const bool keep = lane < nt && dist2(gA.x, gA.y, gA.z, sx, sy, sz) < rA2;
                const uint64_t kb = ballot(keep);
                if (keep) sh.wait[fill + rank_below(kb)] = SrcN{sx, sy, sz, spb, sid};
                fill += __popcll(kb);
                tile_sync();
                if (fill >= kWave) {
                    fill -= kWave;
                    pass(fill, kWave);
                    tile_sync();
                }
            }
        }
        if (fill > 0) pass(0, fill);
        if (SLAB && has_sink) {
            a.counts[oa] = count;
            if (count > kNbCap) {
                const int last = (count - kNbCap - 1) / kNbChunk;   // its last chunk
                if (sh.chunk[lane][last & 1] >= 0) {
                    if (count > kNbWaveMax) atomicAdd(a.ctl + 2, 1);
                } else {
                    a.head[oa] = -1;
                    atomicAdd(a.ctl, 1);
                    leaf_over = true;
                }
            }
        }
        if (!SLAB && has_sink) a.longq[atomicAdd(a.ctl, 1)] = oa;
        tile_sync();   // sink / chunk are reset by the next pass
    }
    if constexpr (SLAB) {   // the leaf is queued once
        bool any = ballot(leaf_over) != 0ull;
        if constexpr (H > 1) {
            if (threadIdx.x == 0) over_any = 0;
            __syncthreads();
            if (any && lane == 0) atomicOr(&over_any, 1);
            __syncthreads();
            any = over_any != 0;
        }
        if (any && threadIdx.x == 0) a.queue[atomicAdd(a.ctl + 1, 1)] = (int32_t)l;
    }
}

// caller index -> tree position (slab rows by tree position)
__global__ __launch_bounds__(kBlock) void k_inv(int64_t n, const int32_t *__restrict__ pid,
                                                int32_t *__restrict__ inv) {
    const int64_t p = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (p < n) inv[pid[p]] = (int32_t)p;
}

// Sorting network on 8 U keys, all comparators ascending: for k = 2, 4, ...,
// 8 U the first stage pairs i with i ^ (k - 1), the following ones i with
// i ^ d (d = k/4, ..., 1); the smaller key goes to the lower index. Key i sits
// in register i % U of lane i / U of an aligned group of 8 lanes, so strides
// below U are exchanges between registers and the others between lanes.
__device__ __forceinline__ void cex(uint32_t &lo, uint32_t &hi) {
    const uint32_t a = lo, b = hi;
    lo = a < b ? a : b;
    hi = a < b ? b : a;
}

// v of lane (lane ^ M) for M < 8, by DPP moves within rows (no LDS path):
// quad permutations give xor 1, 2 and 3, the half-row mirror xor 7, and the
// mirror followed by the quad reversal xor 4.
template <int M>
__device__ __forceinline__ uint32_t xor_lanes(uint32_t v) {
    constexpr int kQuadXor1 = 0xb1, kQuadXor2 = 0x4e, kQuadXor3 = 0x1b, kHalfMirror = 0x141;
    const int x = (int)v;
    if constexpr (M == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(x, kQuadXor1, 0xf, 0xf, true);
    if constexpr (M == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(x, kQuadXor2, 0xf, 0xf, true);
    if constexpr (M == 3) return (uint32_t)__builtin_amdgcn_mov_dpp(x, kQuadXor3, 0xf, 0xf, true);
    if constexpr (M == 7) return (uint32_t)__builtin_amdgcn_mov_dpp(x, kHalfMirror, 0xf, 0xf, true);
    if constexpr (M == 4)
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, kHalfMirror, 0xf, 0xf, true),
                                                  kQuadXor3, 0xf, 0xf, true);
    static_assert(M == 1 || M == 2 || M == 3 || M == 4 || M == 7, "lane xor not provided");
    return v;
}

template <int U, int K>
__device__ __forceinline__ void net_flip(uint32_t (&v)[U], int j0) {
    if constexpr (K <= U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < (u ^ (K - 1))) cex(v[u], v[u ^ (K - 1)]);
    } else {
        // partner: lane j0 ^ (K / U - 1), register U - 1 - u
        const bool lower = (j0 & (K / (2 * U))) == 0;
        uint32_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = xor_lanes<K / U - 1>(v[U - 1 - u]);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = lower ? (v[u] < w[u] ? v[u] : w[u]) : (v[u] < w[u] ? w[u] : v[u]);
    }
}

template <int U, int D>
__device__ __forceinline__ void net_strides(uint32_t (&v)[U], int j0) {   // D, D / 2, ..., 1
    if constexpr (D >= 1) {
        if constexpr (D < U) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((u & D) == 0) cex(v[u], v[u | D]);
        } else {
            const bool lower = (j0 & (D / U)) == 0;   // partner: lane j0 ^ (D / U)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t w = xor_lanes<D / U>(v[u]);
                v[u] = lower ? (v[u] < w ? v[u] : w) : (v[u] < w ? w : v[u]);
            }
        }
        net_strides<U, D / 2>(v, j0);
    }
}

template <int U, int K = 2>
__device__ __forceinline__ void net_sort(uint32_t (&v)[U], int j0) {
    if constexpr (K <= 8 * U) {
        net_flip<U, K>(v, j0);
        net_strides<U, K / 4>(v, j0);
        net_sort<U, 2 * K>(v, j0);
    }
}

// One wave's 8 lists of at most 8 U ids (8 lanes each, this lane's with c ids,
// 0: none here): the row and the chunks ch[] loaded 8 slots a lane at a time
// (keys past the count are 2^32 - 1, i.e. last), sorted, and stored 64 keys of
// each list at a time through LDS, each list by consecutive lanes.
template <int U>
__device__ __forceinline__ void compact_lists(int c, int64_t o, const int32_t *__restrict__ row,
                                              const int32_t (&ch)[3], const int32_t *__restrict__ pool,
                                              uint32_t *st, int32_t *__restrict__ ids) {
    const int lane = lane_id(), j0 = lane % 8, p = lane / 8;
    uint32_t v[U];
#pragma unroll
    for (int b = 0; b < U / 8; ++b) {
        const int i0 = kNbCap * b + 8 * j0;
        if (i0 < c) {
            const int4 *src = reinterpret_cast<const int4 *>((b ? pool + (int64_t)ch[b ? b - 1 : 0] * kNbChunk : row) + 8 * j0);
            const int4 x = src[0], y = src[1];
            const int32_t k[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int u = 0; u < 8; ++u) v[8 * b + u] = i0 + u < c ? (uint32_t)k[u] : 0xffffffffu;
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) v[8 * b + u] = 0xffffffffu;
        }
    }
    net_sort<U>(v, j0);
    constexpr int kLanes = kWave / U;   // lanes of a list that hold 64 of its keys
#pragma unroll
    for (int r = 0; r < U / 8; ++r) {
        if (j0 / kLanes == r) {
#pragma unroll
            for (int u = 0; u < U; ++u) st[p * kNbCap + (j0 % kLanes) * U + u] = v[u];
        }
        tile_sync();
#pragma unroll
        for (int q = 0; q < 8; ++q) {   // list q of the wave
            const int64_t oq = ((int64_t)__builtin_amdgcn_readlane((int)(o >> 32), 8 * q) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)o, 8 * q);
            const int cq = __builtin_amdgcn_readlane(c, 8 * q);
            if (kNbCap * r + lane < cq) ids[oq + kNbCap * r + lane] = (int32_t)st[q * kNbCap + lane];
        }
        tile_sync();
    }
}

// slab rows and chunks -> the caller's CSR, in caller order: 8 lanes per
// particle, 8, 16 or 32 keys per lane by the wave's longest list (of up to
// kNbWaveMax ids); longer lists are copied and queued for k_nb_sort_long.
// Lists searched again (head -1) are skipped.
// 500,000 particles with 102 neighbours each: 76 us; one list after the other,
// 4 keys on each of the wave's lanes and shuffles between them, took 460.
__global__ __launch_bounds__(kBlock) void k_nb_compact(int64_t n, const int32_t *__restrict__ inv,
                                                       const int64_t *__restrict__ offsets,
                                                       const int32_t *__restrict__ slab,
                                                       const int32_t *__restrict__ head,
                                                       const int32_t *__restrict__ next,
                                                       const int32_t *__restrict__ pool,
                                                       int32_t *__restrict__ ids, int32_t *__restrict__ nlong,
                                                       int32_t *__restrict__ longq) {
    __shared__ uint32_t stage[kWaves][8 * kNbCap];
    uint32_t *st = stage[threadIdx.x / kWave];
    const int lane = lane_id();
    const int64_t a = (blockIdx.x * (int64_t)kBlock + threadIdx.x) / 8;
    int64_t o = 0;
    int call = 0;   // < n <= 2^31 - 1
    if (a < n) {
        o = offsets[a];
        call = (int)(offsets[a + 1] - o);
    }
    const int32_t *row = slab;
    if (call > 0) row += (inv ? (int64_t)inv[a] : a) * kNbCap;
    int32_t ch[3] = {-1, -1, -1};
    if (ballot(call > kNbCap) == 0ull) {
        compact_lists<8>(call, o, row, ch, pool, st, ids);
        return;
    }
    if (call > kNbCap) {
        ch[0] = head[a];
        if (call <= kNbWaveMax && ch[0] >= 0) {
            if (call > kNbCap + kNbChunk) ch[1] = next[ch[0]];
            if (call > kNbCap + 2 * kNbChunk) ch[2] = next[ch[1]];
        }
    }
    const int c = call > kNbCap && (call > kNbWaveMax || ch[0] < 0) ? 0 : call;
    if (ballot(c > 2 * kNbCap) != 0ull) compact_lists<32>(c, o, row, ch, pool, st, ids);
    else if (ballot(c > kNbCap) != 0ull) compact_lists<16>(c, o, row, ch, pool, st, ids);
    else compact_lists<8>(c, o, row, ch, pool, st, ids);
    uint64_t lm = ballot(lane % 8 == 0 && call > kNbWaveMax && ch[0] >= 0);
    const int64_t a0 = a - lane / 8;
    while (lm) {
        const int l = __ffsll((long long)lm) - 1;
        lm &= lm - 1;
        const int64_t al = a0 + l / 8;
        const int64_t ol = ((int64_t)__builtin_amdgcn_readlane((int)(o >> 32), l) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)o, l);
        const int cl = __builtin_amdgcn_readlane(call, l);
        int32_t cq = __builtin_amdgcn_readlane(ch[0], l);
        ids[ol + lane] = slab[(inv ? (int64_t)inv[al] : al) * kNbCap + lane];
        for (int i = kNbCap;; i += kNbChunk) {
            if (i + lane < cl) ids[ol + i + lane] = pool[(int64_t)cq * kNbChunk + lane];
            if (i + kNbChunk >= cl) break;
            cq = next[cq];
        }
        if (lane == 0) longq[atomicAdd(nlong, 1)] = (int32_t)al;
    }
}

// Network of the same kind over P = 2^logP keys in LDS (P <= kLongLds),
// comparators split over the nt threads of the caller (tid < nt); sync() is
// called after each stage.
template <typename Sync>
__device__ __forceinline__ void lds_network(uint32_t *key, int logP, int tid, int nt, Sync sync) {
    const int P = 1 << logP;
    for (int lk = 1; lk <= logP; ++lk) {
        for (int ld = lk - 1; ld >= 0; --ld) {
            const int d = 1 << ld;
            for (int t = tid; t < P / 2; t += nt) {
                const int i = ((t >> ld) << (ld + 1)) | (t & (d - 1));   // bit d of i is clear
                const int j = ld == lk - 1 ? (i ^ ((1 << lk) - 1)) : (i + d);
                const uint32_t x = key[i], y = key[j];
                if (y < x) {
                    key[i] = y;
                    key[j] = x;
                }
            }
            sync();
        }
    }
}

// One workgroup per list of more than kNbWaveMax ids or searched again by the
// fill call: the same network
// over the list's length rounded up to a power of two P, in LDS (padded with
// 2^32 - 1) when P <= kLongLds, else in place in the CSR with the comparators
// that reach past the end left out (with every comparator ascending, keys of
// 2^32 - 1 past the end would never move).
__device__ __forceinline__ void sort_long_list(uint32_t *sm, int32_t a, const int64_t *__restrict__ offsets,
                                               int32_t *__restrict__ ids) {
    const int64_t o = offsets[a], L = offsets[a + 1] - o;
    int logP = 0;
    while (((int64_t)1 << logP) < L) ++logP;
    const int64_t P = (int64_t)1 << logP;
    const int tid = threadIdx.x;
    if (P <= kLongLds) {
        for (int i = tid; i < P; i += kBlock) sm[i] = i < L ? (uint32_t)ids[o + i] : 0xffffffffu;
        __syncthreads();
        lds_network(sm, logP, tid, kBlock, [] { __syncthreads(); });
        for (int i = tid; i < L; i += kBlock) ids[o + i] = (int32_t)sm[i];
        return;
    }
    uint32_t *key = reinterpret_cast<uint32_t *>(ids + o);
    for (int lk = 1; lk <= logP; ++lk) {
        for (int ld = lk - 1; ld >= 0; --ld) {
            const int64_t d = (int64_t)1 << ld;
            for (int64_t t = tid; t < P / 2; t += kBlock) {
                const int64_t i = ((t >> ld) << (ld + 1)) | (t & (d - 1));
                const int64_t j = ld == lk - 1 ? (i ^ (((int64_t)1 << lk) - 1)) : (i + d);
                if (j < L) {
                    const uint32_t x = key[i], y = key[j];
                    if (y < x) {
                        key[i] = y;
                        key[j] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_nb_sort_long(int64_t nsort, const int32_t *__restrict__ longq,
                                                         const int64_t *__restrict__ offsets,
                                                         int32_t *__restrict__ ids) {
    __shared__ uint32_t sm[kLongLds];
    for (int64_t i = blockIdx.x; i < nsort; i += gridDim.x) {
        sort_long_list(sm, longq[i], offsets, ids);
        __syncthreads();
    }
}

// The same for clouds of at most kBitsMax particles: the ids of a list, all
// different, are set in a bitmap of the caller's indices in LDS, and an id's
// place is the number of bits below it -- the sum before its group of 8 words,
// kept from one scan, and the bits of the group. A network is a chain of some 60
// stages with a barrier each.
// rcb_neighbours_fill in us, network and bitmap: 2000 particles, 134 lists of up
// to 1999 ids 91 and 58; 37,000, 2600 lists of up to 875 95 and 69; 300,000, 7200 of
// up to 1476 219 and 221 (the bitmap's words are cleared and scanned for every
// list), hence the limit.
constexpr int kBitsMax = 1 << 18;
constexpr int kBitsOwn = 16;   // ids a thread keeps; of longer lists they are read from the bitmap
__global__ __launch_bounds__(kBlock) void k_nb_sort_bits(int64_t nsort, const int32_t *__restrict__ longq,
                                                         const int64_t *__restrict__ offsets,
                                                         int32_t *__restrict__ ids, int n) {
    extern __shared__ uint32_t bits[];
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const int ng = (n + 255) / 256;          // groups of 8 words
    uint32_t *const before = bits + 8 * ng;   // set bits before each group
    uint32_t *const wsum = before + ng;       // per wave
    const int per = (ng + kBlock - 1) / kBlock;
    const int gb = tid * per < ng ? tid * per : ng, ge = gb + per < ng ? gb + per : ng;   // this thread's groups
    auto group_bits = [&](int g, int words) {
        int c = 0;
        for (int w = 0; w < words; ++w) c += __popc(bits[8 * g + w]);
        return c;
    };
    for (int64_t i = blockIdx.x; i < nsort; i += gridDim.x) {
        const int32_t q = longq[i];
        const int64_t b = offsets[q];
        const int len = (int)(offsets[q + 1] - b);
        int32_t *const list = ids + b;
        for (int w = tid; w < 8 * ng; w += kBlock) bits[w] = 0;
        const bool own = len <= kBitsOwn * kBlock;
        int32_t v[kBitsOwn];
        __syncthreads();
        if (own) {
#pragma unroll
            for (int u = 0; u < kBitsOwn; ++u) {
                v[u] = tid + u * kBlock < len ? list[tid + u * kBlock] : -1;
                if (v[u] >= 0) atomicOr(&bits[v[u] >> 5], 1u << (v[u] & 31));
            }
        } else {
            for (int j = tid; j < len; j += kBlock) {
                const int32_t x = list[j];
                atomicOr(&bits[x >> 5], 1u << (x & 31));
            }
        }
        __syncthreads();
        int c = 0;
        for (int g = gb; g < ge; ++g) c += group_bits(g, 8);
        const int incl = wave_incl_scan(c);
        if (lane == kWave - 1) wsum[wv] = incl;
        __syncthreads();
        int at = incl - c;
        for (int w = 0; w < wv; ++w) at += wsum[w];
        for (int g = gb; g < ge; ++g) {
            before[g] = at;
            if (own) {
                at += group_bits(g, 8);
            } else {
                for (int w = 0; w < 8; ++w)
                    for (uint32_t m = bits[8 * g + w]; m; m &= m - 1) list[at++] = 256 * g + 32 * w + __ffs(m) - 1;
            }
        }
        __syncthreads();
        if (own) {
#pragma unroll
            for (int u = 0; u < kBitsOwn; ++u) {
                if (v[u] >= 0) {
                    const int g = v[u] >> 8, w = (v[u] >> 5) & 7;
                    list[before[g] + group_bits(g, w) + __popc(bits[v[u] >> 5] & ((1u << (v[u] & 31)) - 1u))] = v[u];
                }
            }
        }
        __syncthreads();
    }
}
inline size_t bits_lds(int64_t n) { return sizeof(uint32_t) * (9 * ((n + 255) / 256) + kWaves); }

// Slab rows go by caller index, so that the fill call streams them in the
// CSR's order; past 4 GiB of slab (16.7M particles) by tree position instead,
// where a wave's rows are contiguous: the search's scattered stores into a
// slab of tens of GB otherwise cost more than reading the rows back through
// the inverse permutation (1e8 particles: 83 -> 73 ms).
bool tree_rows(const rcb_tree *t) { return t->n * kNbCap * (int64_t)sizeof(int32_t) > ((int64_t)4 << 30); }

// The count call's scratch with `subs` sub-pools of `cap` chunks each: all of it,
// or nothing.
bool take_scratch(rcb_tree *t, int32_t subs, int64_t cap, hipStream_t s) {
    Scratch tmp(t, s);
    bool all = true;
    auto A = [&](size_t bytes) -> int32_t * {
        void *p = all ? dalloc(t, bytes, s, tmp) : nullptr;
        all = all && p;
        return (int32_t *)p;
    };
    int32_t *slab = A(sizeof(int32_t) * t->n * kNbCap), *pool = A(sizeof(int32_t) * cap * subs * kNbChunk);
    int32_t *next = A(sizeof(int32_t) * cap * subs), *head = A(sizeof(int32_t) * t->n);
    int32_t *queue = A(sizeof(int32_t) * t->nleaf), *ctl = A(ctl_bytes(subs));
    if (!all) return false;
    t->list_allocs.insert(t->list_allocs.end(), tmp.begin(), tmp.end());
    tmp.clear();
    t->nb_slab = slab;
    t->nb_pool = pool;
    t->nb_next = next;
    t->nb_head = head;
    t->nb_queue = queue;
    t->nb_ctl = ctl;
    t->nb_subs = subs;
    t->nb_sub_cap = cap;
    return true;
}

// chunk ids of sub-pools of `cap` chunks -> of `to` (-1 stays; heads that were not
// written are not read)
__device__ __forceinline__ int32_t moved_chunk(int32_t ch, int64_t cap, int64_t to) {
    return ch < 0 ? ch : (int32_t)(ch / cap * to + ch % cap);
}
__global__ __launch_bounds__(kBlock) void k_nb_move_heads(int64_t n, int64_t cap, int64_t to,
                                                          int32_t *__restrict__ head) {
    const int64_t a = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (a < n) head[a] = moved_chunk(head[a], cap, to);
}
// one wave per chunk of the new pool
__global__ __launch_bounds__(kBlock) void k_nb_move_chunks(int64_t chunks, int64_t cap, int64_t to,
                                                           const int32_t *__restrict__ pool,
                                                           const int32_t *__restrict__ next,
                                                           int32_t *__restrict__ npool, int32_t *__restrict__ nnext) {
    const int64_t w = wave_index();
    if (w >= chunks) return;
    const int64_t from = w / to * cap + w % to;
    npool[w * kNbChunk + lane_id()] = pool[from * kNbChunk + lane_id()];
    if (lane_id() == 0) nnext[w] = moved_chunk(next[from], cap, to);
}

}  // namespace

// Count: one search that writes every particle's count into offsets (then
// scanned in place) and its ids into the slab row (and a chunk of the pool
// past the row); fill then compacts and sorts those, and searches again only
// the cells holding a list that did not fit.
rcb_status neighbours_count(rcb_tree *t, int64_t *offsets, int64_t *total, hipStream_t s) {
    if (t->lists_kept) {
        set_error("rcb_neighbours_count: the interaction lists were kept across rcb_refresh "
                  "(keep_lists = 1) and may miss neighbours of the new inputs; call rcb_walk first");
        return RCB_ESTATE;
    }
    rcb_status st = ensure_walk(t, s);
    if (st != RCB_OK) return st;
    if (!t->nb_slab) {
        // overflow chunks: one for every 8th particle (lists past 64 ids are 3%
        // (Plummer) to 8% (clumps) at ~50 neighbours on average), and the number
        // that the walk's estimate of each cell's neighbour count asks for (at
        // most 4 per particle; at 105 neighbours, one for nearly each), and for
        // small clouds what the longest lists possible take, up to 16 MiB: a few
        // lists of thousands searched again cost 2000 particles 38 of 380 us
        // (the N/8 chunks alone, in one sub-pool, where that cannot be had)
        int32_t subs = 1;
        while (subs < kSubMax && subs * 8 < t->ngroup) subs *= 2;
        const int64_t all = t->n > kNbCap ? t->n * ((t->n - kNbCap + kNbChunk - 1) / kNbChunk) : 0;
        const int64_t small = std::min<int64_t>(all, (int64_t)1 << 16);
        const int64_t base = t->n / 8 + 1;
        const int64_t more = std::max<int64_t>(
            small, std::min<int64_t>({t->nb_est, 4 * t->n, ((int64_t)1 << 30) - base}));   // (int32 chunk ids)
        if (!take_scratch(t, subs, (base + more + subs - 1) / subs + 8, s) && !take_scratch(t, 1, base, s))
            return RCB_ENOMEM;
    }
    RCB_ZERO(t->nb_ctl, ctl_bytes(t->nb_subs), s);
    NeighArgs a{t->nleaf, t->gk, t->wrec, t->nhnode, t->nfirst, t->ncount, t->gnear_beg,
                t->gnear_end, t->gnear, t->px, t->py, t->pz, t->ph, t->pid, offsets, nullptr, t->nb_slab,
                t->nb_pool, t->nb_next, t->nb_sub_cap, t->nb_subs - 1, t->nb_head, t->nb_ctl, t->nb_queue, nullptr,
                0, tree_rows(t)};
    for (; a.first < t->nleaf; a.first += kMaxGrid) {
        const unsigned g = (unsigned)std::min(kMaxGrid, t->nleaf - a.first);
        // waves per leaf while leaves are few; each stages the sources again (in
        // us with 1, 2, 4, 8: 256 leaves 119, 93, 78, 73; 1024 leaves 80, 60, 57, 64, of 58
        // particles 216, 159, 141, 182; 4096 leaves 113, 107, 109, 131; 8192 leaves 163,
        // 147, 168, 237, of 61 particles 724, 737, 911, 1310; 32,768 377, 427, 576, 887)
        if (t->nleaf <= 2048) k_neigh<true, 4><<<g, 4 * kWave, 0, s>>>(a);
        else if (t->nleaf <= 4096) k_neigh<true, 2><<<g, 2 * kWave, 0, s>>>(a);
        else k_neigh<true, 1><<<g, kWave, 0, s>>>(a);
        RCB_LAUNCH_CHECK("k_neigh<slab>");
    }
    st = scan_i64(t, offsets, offsets, t->n, s);   // in place
    if (st != RCB_OK) return st;
    int32_t ctl[4] = {0, 0, 0, 0};
    const HostRead r[2] = {{offsets + t->n, total, (int)sizeof(int64_t)}, {t->nb_ctl, ctl, (int)sizeof(ctl)}};
    st = read_small(s, r, 2, "rcb_neighbours_count");
    if (st != RCB_OK) return st;
    t->nb_total = *total;
    t->nb_over = ctl[0];
    t->nb_nq = ctl[1];
    t->nb_long = ctl[2];
    return RCB_OK;
}

bool shrink_neigh_pool(rcb_tree *t, hipStream_t s) {
    if (!t->nb_slab) return false;
    if (t->nb_total < 0) {   // no count to fill from
        for (int32_t **p : {&t->nb_slab, &t->nb_pool, &t->nb_next, &t->nb_head, &t->nb_queue, &t->nb_ctl}) {
            free_list_block(t, *p, s);
            *p = nullptr;
        }
        return true;
    }
    int32_t ctl[kSubCtl * (1 + kSubMax)];
    if (hipMemcpyAsync(ctl, t->nb_ctl, ctl_bytes(t->nb_subs), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return false;
    int64_t used = 1;   // chunks of the fullest sub-pool
    for (int i = 0; i < t->nb_subs; ++i) used = std::max<int64_t>(used, ctl[kSubCtl * (1 + i)]);
    if (used >= t->nb_sub_cap) return false;
    const int64_t chunks = used * t->nb_subs;
    Scratch tmp(t, s);
    int32_t *pool = (int32_t *)dalloc(t, sizeof(int32_t) * chunks * kNbChunk, s, tmp);
    int32_t *next = (int32_t *)dalloc(t, sizeof(int32_t) * chunks, s, tmp);
    if (!pool || !next) return false;
    k_nb_move_heads<<<(unsigned)((t->n + kBlock - 1) / kBlock), kBlock, 0, s>>>(t->n, t->nb_sub_cap, used, t->nb_head);
    k_nb_move_chunks<<<(unsigned)((chunks + kWaves - 1) / kWaves), kBlock, 0, s>>>(chunks, t->nb_sub_cap, used,
                                                                                   t->nb_pool, t->nb_next, pool, next);
    for (int32_t **p : {&t->nb_pool, &t->nb_next}) free_list_block(t, *p, s);
    for (void *p : {(void *)pool, (void *)next}) {
        tmp.keep(p);
        t->list_allocs.push_back(p);
    }
    t->nb_pool = pool;
    t->nb_next = next;
    t->nb_sub_cap = used;
    return true;
}

rcb_status neighbours_fill(rcb_tree *t, const int64_t *offsets, int32_t *ids, int64_t cap,
                           hipStream_t s) {
    if (t->nb_total < 0) {
        set_error("rcb_neighbours_fill: call rcb_neighbours_count on this tree first");
        return RCB_ESTATE;
    }
    if (t->nb_total > cap) {
        set_error("rcb_neighbours_fill: capacity " + std::to_string(cap) + " < total " +
                  std::to_string(t->nb_total));
        return RCB_ECAPACITY;
    }
    Scratch tmp(t, s);
    int32_t *inv = nullptr;   // caller index -> slab row, when rows go by tree position
    if (tree_rows(t)) {
        inv = (int32_t *)dalloc(t, sizeof(int32_t) * t->n, s, tmp);
        if (!inv) return RCB_ENOMEM;
        k_inv<<<(unsigned)((t->n + kBlock - 1) / kBlock), kBlock, 0, s>>>(t->n, t->pid, inv);
        RCB_LAUNCH_CHECK("k_inv");
    }
    // the lists that one workgroup each sorts: those of more than kNbWaveMax
    // ids (copied by the compaction) and those searched again
    int32_t *longq = nullptr, *nlong = nullptr;
    const int64_t sorts = (int64_t)t->nb_long + t->nb_over;
    if (sorts > 0) {
        longq = (int32_t *)dalloc(t, sizeof(int32_t) * (sorts + 1), s, tmp);
        if (!longq) return RCB_ENOMEM;
        nlong = longq + sorts;
        RCB_ZERO(nlong, sizeof(int32_t), s);
    }
    const unsigned gridc = (unsigned)((t->n * 8 + kBlock - 1) / kBlock);
    k_nb_compact<<<gridc, kBlock, 0, s>>>(t->n, inv, offsets, t->nb_slab, t->nb_head, t->nb_next, t->nb_pool, ids,
                                          nlong, longq);
    RCB_LAUNCH_CHECK("k_nb_compact");
    if (t->nb_nq > 0) {
        NeighArgs a{t->nleaf, t->gk, t->wrec, t->nhnode, t->nfirst, t->ncount, t->gnear_beg,
                    t->gnear_end, t->gnear, t->px, t->py, t->pz, t->ph, t->pid, nullptr, offsets, ids,
                    nullptr, nullptr, 0, 0, t->nb_head, nlong, t->nb_queue, longq, 0, false};
        k_neigh<false, 1><<<(unsigned)t->nb_nq, kWave, 0, s>>>(a);
        RCB_LAUNCH_CHECK("k_neigh<fill>");
    }
    if (sorts > 0) {   // exactly this many lists appended themselves
        const unsigned g = (unsigned)std::min(kMaxGrid, sorts);
        if (t->n <= kBitsMax) {
            k_nb_sort_bits<<<g, kBlock, bits_lds(t->n), s>>>(sorts, longq, offsets, ids, (int)t->n);
            RCB_LAUNCH_CHECK("k_nb_sort_bits");
        } else {
            k_nb_sort_long<<<g, kBlock, 0, s>>>(sorts, longq, offsets, ids);
            RCB_LAUNCH_CHECK("k_nb_sort_long");
        }
    }
    return RCB_OK;
}

}  // namespace rcb
