// k_grav.hip -- gravitational accelerations from the interaction lists
// (Sec. 2.4: near field by kernel-softened direct summation, far field by
// quadrupole cell-cell interaction, Taylor-expanded about the sink leaf's
// centre of mass).
//
// k_far: a workgroup per group of up to 8 sibling leaves (k_walk.hip). Lanes
//        are (entry slot e = lane/8, leaf slot i = lane%8); the lane evaluates
//        node B at R = com_A(i) - com_B in FP64 for leaf i, accumulating f_i,
//        J_il, H_ilm of Eq. 5's field (far_math.h). Windows of the group's far
//        list go to the waves in turn; lanes and waves of the same leaf are
//        summed at the end, and the coefficients are written (they are kept
//        for the VJP).
// k_near: one or more waves per leaf. Lanes are (sink slot, slice) over the
//        leaf's particles (near_tile.h: S = min(c, 64) sinks, J = 64 / S
//        slices; c: the sinks still to do). The cells of the group's near list
//        whose mask has the leaf are staged 64 sources at a time in LDS;
//        slice j of a sink takes tile entries j, j + J, ...:
//        a_a -= m_b F(r, h_ab) (r_a - r_b), F = S(q)/r (Sec. 2.4.3); the
//        slices are summed at the end. Sources outside the support of every
//        sink of the pass stand behind the others in the tile, and their rows
//        take F = r^-3 with no test.
// Both are bound by VALU issue (k_far at 90% of it at the clock the card holds
// under FP64, ~1.85 GHz). One kernel for both, a wave per group of 8 leaves,
// left the chip idle where groups are few and waiting for the longest: 2,000
// particles 478 us, now 47; 500,000 in cells of 61 8.1 ms, now 0.82; 300,000
// clumpy 2.19 ms, now 0.48. At 4M in cells of 8 k_near's staging was nearly half of
// its instructions: 3.0 ms with a search of the entries for every source, five
// arrays of particles and a division per tile, now 2.5.
//        L2P: a_a += f + J d + H[d, d] / 2,  d = r_a - com_A  (Eq. 6).
// FP64 form: everything in FP64. Mixed form: the sink leaf's frame. Sinks
// are their FP32 offsets from the leaf centre of mass; a source of cell B is
// its FP32 offset plus the FP64 difference com_B - com_A rounded to FP32;
// pairs, accumulation and L2P in FP32; M2L in FP64.
#include <algorithm>
#include <type_traits>

#include "far_math.h"
#include "near_tile.h"
#include "rcb_internal.h"
#include "soft.h"

namespace rcb {
namespace {

using rcbfar::hidx;
using rcbfar::jidx;
using rcbfar::m2l_accumulate;

struct GravArgs {
    int64_t nleaf;
    int gk;
    const int32_t *nfirst, *ncount;
    const double *ncom, *nM, *nQ;
    const int64_t *gnear_beg, *gnear_end, *gfar_beg, *gfar_end;
    const uint64_t *gnear, *gfar;
    const double *px, *py, *pz, *pm, *ph;
    const float4 *fd;
    const float *fh;
    const int32_t *pid;
    void *ax, *ay, *az;
    double *farc;   // if given: each leaf's far coefficients at farc[leaf * kLeafC]
    int64_t first;  // this launch's first group (one per workgroup)
};

// Far-field coefficients of the group's leaves into coef[8][19] (LDS).
// The union far list is taken in windows of kFarWin entries, whose node data
// (centre of mass, mass, quadrupole) are staged in LDS by one coalesced pass.
// For each window every leaf gets the list of the window positions whose mask
// has it (ballot ranks, in list order); then lane (s, i) evaluates entries
// s, s + 8, ... of leaf i's list, so a leaf's lanes only idle at the end of
// the window rather than on every entry the leaf did not accept.
constexpr int kFarWin = kWave;
struct FarWindow {
    uint8_t idx[8][kFarWin];
    double nd[kFarWin][10];
};

// One wave's share of the group's far field: windows first, first + step, ...
// of kFarWin entries; on return c holds, on lane li of every slot, the sum of
// leaf li's terms over these windows.
template <bool RB>
__device__ __forceinline__ void far_windows(const GravArgs &g, int64_t gi, int first, int step, FarWindow &fw,
                                            double (&c)[rcbfar::kAcc]) {
    const int lane = lane_id();
    const int slot = lane >> 3, li = lane & 7;
    const int G = 1 << g.gk;
    const int64_t A = g.nleaf + gi * G + (li < G ? li : 0);
    const double cA[3] = {g.ncom[3 * A], g.ncom[3 * A + 1], g.ncom[3 * A + 2]};
#pragma unroll
    for (int q = 0; q < rcbfar::kAcc; ++q) c[q] = 0.0;
    const int64_t f0 = g.gfar_beg[gi], f1 = g.gfar_end[gi];
    int64_t w0 = f0 + (int64_t)first * kFarWin;
    uint64_t next = w0 + lane < f1 ? g.gfar[w0 + lane] : 0ull;   // this lane's entry of the next window
    for (; w0 < f1; w0 += (int64_t)step * kFarWin) {
        const uint64_t ent = next;
        const uint32_t m = (uint32_t)(ent >> 32) & 0xffu;   // 0 past the end
        int base[8];
        if (m) {
            const int64_t Bn = (uint32_t)ent & 0x7fffffffu;
            fw.nd[lane][0] = g.ncom[3 * Bn];
            fw.nd[lane][1] = g.ncom[3 * Bn + 1];
            fw.nd[lane][2] = g.ncom[3 * Bn + 2];
            fw.nd[lane][3] = g.nM[Bn];
#pragma unroll
            for (int q = 0; q < 6; ++q) fw.nd[lane][4 + q] = g.nQ[6 * Bn + q];
        }
        const int64_t w1 = w0 + (int64_t)step * kFarWin + lane;
        next = w1 < f1 ? g.gfar[w1] : 0ull;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            const bool has = (m >> l) & 1u;
            const uint64_t bl = ballot(has);
            if (has) fw.idx[l][rank_below(bl)] = (uint8_t)lane;
            base[l] = __popcll(bl);
        }
        int most = 0, mine = 0;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            most = base[l] > most ? base[l] : most;
            mine = li == l ? base[l] : mine;
        }
        tile_sync();
        const int rounds = (most + 7) >> 3;
        for (int r = 0; r < rounds; ++r) {
            const int k = 8 * r + slot;
            if (k < mine) {
                const double *nd = fw.nd[fw.idx[li][k]];
                double qq[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) qq[q] = nd[4 + q];
                m2l_accumulate<RB>(cA[0] - nd[0], cA[1] - nd[1], cA[2] - nd[2], nd[3], qq, c);
            }
        }
        tile_sync();
    }
#pragma unroll
    for (int q = 0; q < rcbfar::kAcc; ++q) {
        double v = c[q];
        v += __shfl_xor(v, 8, kWave);
        v += __shfl_xor(v, 16, kWave);
        v += __shfl_xor(v, 32, kWave);
        c[q] = v;
    }
}

// partial sums of a wave that takes part of a group's windows
struct FarPart {
    double acc[8][rcbfar::kAcc];
};

// Far-field coefficients of the group's leaves, one workgroup of W waves per
// group: the windows go to the waves in turn, the waves' sums are added in
// order, and the 19 coefficients of each leaf are written to farc.
template <bool RB, int W>
__global__ __launch_bounds__(W * kWave) void k_far(GravArgs g) {
    __shared__ union {
        FarWindow fw;
        FarPart part;   // (after its windows)
    } sh[W];
    const int64_t gi = g.first + xcd_block<kXcdGroups>();
    const int G = 1 << g.gk;
    if (g.ncount[(g.nleaf >> g.gk) + gi] == 0) return;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int slot = lane_id() >> 3, li = lane_id() & 7;
    double c[rcbfar::kAcc];
    far_windows<RB>(g, gi, wv, W, sh[wv].fw, c);
    if (slot == 0 && wv > 0) {
#pragma unroll
        for (int q = 0; q < rcbfar::kAcc; ++q) sh[wv].part.acc[li][q] = c[q];
    }
    __syncthreads();
    if (wv == 0 && slot == 0 && li < G) {
        for (int w = 1; w < W; ++w)
#pragma unroll
            for (int q = 0; q < rcbfar::kAcc; ++q) c[q] += sh[w].part.acc[li][q];
        double full[19];
        rcbfar::m2l_finish(c, full);
        double *const o = g.farc + (gi * G + li) * kLeafC;
#pragma unroll
        for (int q = 0; q < 19; ++q) o[q] = full[q];
    }
}

// tile: 64 staged sources, then 64 zero-mass sources that pad the last
// partial row of slices, so the pair loop needs no bounds test
template <bool MIXED>
struct NearStage {
    using T = typename std::conditional<MIXED, float, double>::type;
    typename std::conditional<MIXED, EntF, EntD>::type ent[kWave];
    typename std::conditional<MIXED, SrcF, SrcD>::type tile[2 * kWave];
    T h[2 * kWave];
    uint32_t mark[kWave];
};
constexpr int kFew = 2;
__device__ __forceinline__ double lane_sum(double v) { return wave_sum(v); }
__device__ __forceinline__ float lane_sum(float v) { return wave_sumf(v); }
template <typename T>
__device__ __forceinline__ T lane_value(T v, int lane) {
    union {
        T t;
        int w[sizeof(T) / 4];
    } u;
    u.t = v;
#pragma unroll
    for (int i = 0; i < (int)sizeof(T) / 4; ++i) u.w[i] = __builtin_amdgcn_readlane(u.w[i], lane);
    return u.t;
}
// Near field and L2P, a workgroup of H waves per leaf: the tiles go to the
// waves in turn and the waves' sums are added in order.
// FEW: for trees of small leaves. Those of one or two sinks take lanes as sources,
// straight from their loads, and each sink's sums over all lanes: a row or two of a
// tile cost less than the tile's order and the reach it needs (FP64, 500,000 particles
// in cells of one 2.79 ms, now 2.68). (A branch in every instance made cells of 8
// to 61 particles 1 to 2% slower.) Gravity without and with it, 131,072 leaves of 0.95,
// 1.9, 2.3, 2.8 and 3.9 particles: FP64 587 and 561, 668 and 651, 700 and 689, 738 and
// 735, 839 and 858 us; mixed 517 and 492, 569 and 547, 587 and 570, 601 and 591, 642 and
// 646; 524,288 leaves of 2.8 FP64 3446 and 3508: up to 2.5 on average.
template <bool MIXED, int H, bool FEW = false>
__global__ __launch_bounds__(H * kWave, MIXED ? 6 : 5) void k_near(GravArgs g) {
    using T = typename std::conditional<MIXED, float, double>::type;
    __shared__ NearStage<MIXED> sh_all[H];
    __shared__ T red[H > 1 ? H : 1][3][kWave];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    NearStage<MIXED> &np = sh_all[wv];
    const int64_t leaf = g.first + xcd_block<kXcdLeaves>();
    const int64_t gi = leaf >> g.gk, A = g.nleaf + leaf;
    const int li = (int)(leaf & ((1 << g.gk) - 1));
    const int lane = lane_id();
    const int32_t sA = g.nfirst[A], c = g.ncount[A];
    if (c == 0) return;
    using Src = typename std::conditional<MIXED, SrcF, SrcD>::type;
    np.tile[kWave + lane] = Src{0, 0, 0, 0};
    np.h[kWave + lane] = 1;
    np.mark[lane] = 0;
    uint32_t gen = 0;
    const int64_t n0 = g.gnear_beg[gi], n1 = g.gnear_end[gi];
    const double cA[3] = {g.ncom[3 * A], g.ncom[3 * A + 1], g.ncom[3 * A + 2]};
    for (int g0 = 0; g0 < c; g0 += kWave) {
        const LeafLanes L = leaf_lanes(c - g0);
        const int si = g0 + L.sslot;
        const bool has_sink = L.sslot < L.S && si < c;
        const int32_t pa = sA + (has_sink ? si : 0);
        T xa, ya, za, ha;
        if constexpr (MIXED) {   // leaf frame
            const float4 f = g.fd[pa];
            xa = f.x;
            ya = f.y;
            za = f.z;
            ha = g.fh[pa];
        } else {
            xa = g.px[pa];
            ya = g.py[pa];
            za = g.pz[pa];
            ha = g.ph[pa];
        }
        const bool few = FEW && c <= kFew;
        T sx[kFew], sy[kFew], sz[kFew], ss[kFew];
        if constexpr (FEW) {
#pragma unroll
            for (int q = 0; q < kFew; ++q) {   // (of one sink every lane has it)
                sx[q] = lane_value(xa, q * (kWave / kFew));
                sy[q] = lane_value(ya, q * (kWave / kFew));
                sz[q] = lane_value(za, q * (kWave / kFew));
                ss[q] = lane_value(ha, q * (kWave / kFew));
            }
        }
        T reach = 0;
        if (!few)
            reach = MIXED ? sink_reach(xa, ya, za, ha)
                          : sink_reach(T(xa - cA[0]), T(ya - cA[1]), T(za - cA[2]), ha);
        T ax = 0, ay = 0, az = 0;
        T ex = 0, ey = 0, ez = 0;   // few: the second sink's
        int turn = 0;   // H > 1: the wave that takes the next tile
        for (int64_t e0 = n0; e0 < n1; e0 += kWave) {
            const ChunkEntry ce = load_chunk(g.gnear, g.nfirst, g.ncount, e0, n1, 1u << li);
            const int tot = ce.tot;
            if (ce.has()) {
                if constexpr (MIXED) {
                    const double *cB = g.ncom + 3 * (int64_t)ce.label;
                    np.ent[ce.rank] = EntF{(float)(cB[0] - cA[0]), (float)(cB[1] - cA[1]), (float)(cB[2] - cA[2]),
                                           ce.off()};
                } else {
                    np.ent[ce.rank].off = ce.off();
                }
            }
            for (int t = 0; t < tot; t += kWave) {
                if constexpr (H > 1) {
                    const bool mine = turn == wv;
                    turn = turn + 1 < H ? turn + 1 : 0;
                    if (!mine) continue;
                }
                const int nt = tot - t < kWave ? tot - t : kWave;
                const uint64_t valid = ~0ull >> (kWave - nt);
                const auto en = np.ent[tile_entry(ce, t, np.mark, gen)];
                // (lanes past the end take the last source with no mass)
                const int64_t pb = (int64_t)en.off + (t + (lane < nt ? lane : nt - 1));
                Src s;
                T sh, bx, by, bz;   // b: from the leaf's centre of mass
                if constexpr (MIXED) {
                    const float4 f = g.fd[pb];
                    sh = g.fh[pb];
                    s.x = bx = en.x + f.x;
                    s.y = by = en.y + f.y;
                    s.z = bz = en.z + f.z;
                    s.m = f.w;
                } else {
                    s.x = g.px[pb];
                    s.y = g.py[pb];
                    s.z = g.pz[pb];
                    s.m = g.pm[pb];
                    sh = g.ph[pb];
                    bx = s.x - cA[0];
                    by = s.y - cA[1];
                    bz = s.z - cA[2];
                }
                s.m = lane < nt ? s.m : (T)0;
                if constexpr (FEW) {
                    if (few) {
                        auto pair = [&](int q, T &px, T &py, T &pz) {
                            const T vx = sx[q] - s.x, vy = sy[q] - s.y, vz = sz[q] - s.z;
                            const T r2 = (vx * vx + vy * vy) + vz * vz;
                            const T hsum = ss[q] + sh;
                            const T ri = rsq_t(r2);
                            const T r3 = ri * ri * ri;
                            T F = r3;
                            if (!soft_outside<T>(r2, hsum)) F = soft_F<T>(r2, ri, r3, hsum);
                            F *= s.m;
                            px -= F * vx;
                            py -= F * vy;
                            pz -= F * vz;
                        };
                        pair(0, ax, ay, az);
                        if (c > 1) pair(1, ex, ey, ez);
                        continue;
                    }
                }
                // sources outside the support of every sink go behind the others
                // (those past the end last)
                const T lim = (reach + sh) * (T)1.001;
                const bool out = (bx * bx + by * by) + bz * bz > lim * lim;
                const uint64_t cb = ~ballot(out) & valid;
                const int nc = __popcll(cb), before = rank_below(cb);
                const int at = (cb >> lane) & 1 ? before : nc + lane - before;
                np.tile[at] = s;
                np.h[at] = sh;
                tile_sync();
                const int full = L.rows(nt), soft = L.rows(nc + L.J - 1);
                auto row = [&](int r) {
                    const int i = r * L.J + L.slice;
                    const Src s = np.tile[i];
                    const T vx = xa - s.x, vy = ya - s.y, vz = za - s.z;
                    const T r2 = (vx * vx + vy * vy) + vz * vz;
                    const T hsum = ha + np.h[i];
                    const T ri = rsq_t(r2);
                    const T r3 = ri * ri * ri;
                    T F = r3;
                    if (!soft_outside<T>(r2, hsum)) F = soft_F<T>(r2, ri, r3, hsum);
                    F *= s.m;
                    ax -= F * vx;
                    ay -= F * vy;
                    az -= F * vz;
                };
                auto plain = [&](const Src &s) {
                    const T vx = xa - s.x, vy = ya - s.y, vz = za - s.z;
                    const T r2 = (vx * vx + vy * vy) + vz * vz;
                    const T ri = rsq_t(r2);
                    const T F = (ri * ri * ri) * s.m;
                    ax -= F * vx;
                    ay -= F * vy;
                    az -= F * vz;
                };
                for (int r = 0; r < soft; ++r) row(r);
                int r = soft;
                for (; r + 1 < full; r += 2) {   // (two rows per step: their LDS reads overlap)
                    const Src *p = np.tile + (r * L.J + L.slice);
                    const Src s0 = p[0], s1 = p[L.J];
                    plain(s0);
                    plain(s1);
                }
                if (r < full) plain(np.tile[r * L.J + L.slice]);
                if (soft <= full && full * L.J < nt) row(full);   // the last, padded row
                tile_sync();
            }
            if constexpr (H > 1) tile_sync();   // (a wave may have taken none of the chunk's tiles)
        }
        if (FEW && few) {
            // (over all lanes, before a lane takes its sink's)
            const T sum[3] = {lane_sum(ax), lane_sum(ay), lane_sum(az)};
            T sum2[3] = {0, 0, 0};
            if (c > 1) {
                sum2[0] = lane_sum(ex);
                sum2[1] = lane_sum(ey);
                sum2[2] = lane_sum(ez);
            }
            ax = L.sslot > 0 ? sum2[0] : sum[0];
            ay = L.sslot > 0 ? sum2[1] : sum[1];
            az = L.sslot > 0 ? sum2[2] : sum[2];
        } else {
            ax = seg_sum(ax, L.slice, L.J);
            ay = seg_sum(ay, L.slice, L.J);
            az = seg_sum(az, L.slice, L.J);
        }
        if constexpr (H > 1) {
            if (L.slice == 0) {
                red[wv][0][L.sslot] = ax;
                red[wv][1][L.sslot] = ay;
                red[wv][2][L.sslot] = az;
            }
            __syncthreads();
            if (wv == 0 && L.slice == 0) {
                for (int w = 1; w < H; ++w) {
                    ax += red[w][0][L.sslot];
                    ay += red[w][1][L.sslot];
                    az += red[w][2][L.sslot];
                }
            }
            __syncthreads();
        }
        if (wv == 0 && has_sink && L.slice == 0) {
            const double *lc = g.farc + leaf * kLeafC;
            double c19[19];
#pragma unroll
            for (int q = 0; q < 19; ++q) c19[q] = lc[q];
            T d[3], out[3];
            if constexpr (MIXED) {
                d[0] = xa;
                d[1] = ya;
                d[2] = za;
            } else {
                d[0] = xa - cA[0];
                d[1] = ya - cA[1];
                d[2] = za - cA[2];
            }
            rcbfar::l2p<T>(c19, d, out);
            const int32_t o = g.pid[pa];
            ((T *)g.ax)[o] = ax + out[0];
            ((T *)g.ay)[o] = ay + out[1];
            ((T *)g.az)[o] = az + out[2];
        }
    }
}

GravArgs grav_args(const rcb_tree *t, void *ax, void *ay, void *az, double *farc) {
    return GravArgs{t->nleaf, t->gk, t->nfirst, t->ncount, t->ncom, t->nM, t->nQ,
                    t->gnear_beg, t->gnear_end, t->gfar_beg, t->gfar_end, t->gnear, t->gfar, t->px, t->py, t->pz, t->pm, t->ph,
                    t->fd, t->fh, t->pid, ax, ay, az, farc, 0};
}

// Waves per group: 4 where groups are few (SIMDs to fill) or their lists long
// (the waves of a group end together), else 2, as each wave's last sums cost
// what about two windows do (gravity in us with 1, 2, 4: 8192 groups of ~560
// entries 1051, 986, 1073; 8192 of ~1700 entries 1021, 1040, 945; 16384 of ~3000
// 3240, 3100, 3032; 65,536 of ~2100 entries 7160, 6862, 6907).
template <bool RB>
rcb_status launch_far(const rcb_tree *t, GravArgs g, int64_t g0, int64_t g1, hipStream_t s) {   // groups [g0, g1)
    const bool four = t->ngroup <= 2048 || (t->ngroup < 65536 && t->far_entries >= 1024 * t->ngroup);
    for (g.first = g0; g.first < g1; g.first += kMaxGrid) {
        const unsigned n = (unsigned)std::min(kMaxGrid, g1 - g.first);
        if (four) k_far<RB, 4><<<n, 4 * kWave, 0, s>>>(g);
        else k_far<RB, 2><<<n, 2 * kWave, 0, s>>>(g);
        RCB_LAUNCH_CHECK("k_far");
    }
    return RCB_OK;
}

// Waves per leaf: as many as fill the SIMDs (gravity in us with 1, 2, 4, 8 waves:
// 256 leaves 120, 76, 51, 40; 4096 leaves 193, 120, 94, 90; 8192 leaves of 61
// particles 1362, 1102, 988, 1000; 32,768 clumpy 629, 574, 570, 712; 131,072
// 1887, 2000, 2072, 2607). Each wave reads the whole list, and of leaves of fewer than
// five particles on average that is most of the work: they take one wave where
// there are enough of them and none is large (256 leaves of 2.5 particles 26, 24, 23, 22; 4096 of 5
// particles 57, 57, 62, 80, of 1.5 40, 43, 49, 65; 32,768 of 5 262, 278, 344, 530).
template <bool MIXED>
rcb_status launch_near(const rcb_tree *t, GravArgs g, int64_t g0, int64_t g1, hipStream_t s) {   // of groups [g0, g1)
    const int64_t end = g1 << t->gk;
    for (g.first = g0 << t->gk; g.first < end; g.first += kMaxGrid) {
        const unsigned n = (unsigned)std::min(kMaxGrid, end - g.first);
        const bool one = t->nleaf > 1024 && t->n < 5 * t->nleaf && !t->large_leaf;
        if (one && 2 * t->n < 5 * t->nleaf) k_near<MIXED, 1, true><<<n, kWave, 0, s>>>(g);
        else if (one) k_near<MIXED, 1><<<n, kWave, 0, s>>>(g);
        else if (t->nleaf <= 4096) k_near<MIXED, 8><<<n, 8 * kWave, 0, s>>>(g);
        else if (t->nleaf <= 16384) k_near<MIXED, 4><<<n, 4 * kWave, 0, s>>>(g);
        else if (t->nleaf <= 32768) k_near<MIXED, 2><<<n, 2 * kWave, 0, s>>>(g);
        else k_near<MIXED, 1><<<n, kWave, 0, s>>>(g);
        RCB_LAUNCH_CHECK("k_near");
    }
    return RCB_OK;
}

}  // namespace

rcb_status far_coefficients(rcb_tree *t, double *out, hipStream_t s) {
    rcb_status st = ensure_walk(t, s);
    if (st != RCB_OK) return st;
    return launch_far<false>(t, grav_args(t, nullptr, nullptr, nullptr, out), 0, t->ngroup, s);
}

rcb_status gravity(rcb_tree *t, void *ax, void *ay, void *az, hipStream_t s) {
    rcb_status st = ensure_walk(t, s);
    if (st != RCB_OK) return st;
    const bool rb = t->p.taylor_reading == RCB_READING_B;
    const int64_t per_group = (int64_t)kLeafC << t->gk;   // doubles
    // the far coefficients of all leaves, kept for a VJP on the same moments (there
    // is none for reading B); if they cannot be had, of ranges of groups in turn
    Scratch tmp(t, s);
    double *buf = rb ? nullptr : t->farc;
    if (!buf) buf = (double *)dalloc(t, sizeof(double) * per_group * t->ngroup, s, rb ? tmp : t->list_allocs);
    if (!rb) t->farc = buf;
    int64_t range = t->ngroup;
    while (!buf && range > 1) {
        range = (range + 7) / 8;
        buf = (double *)dalloc(t, sizeof(double) * per_group * range, s, tmp);
    }
    if (!buf) return RCB_ENOMEM;
    for (int64_t g0 = 0; g0 < t->ngroup; g0 += range) {
        const int64_t g1 = std::min(g0 + range, t->ngroup);
        const GravArgs g = grav_args(t, ax, ay, az, buf - per_group * g0);
        st = rb ? launch_far<true>(t, g, g0, g1, s) : launch_far<false>(t, g, g0, g1, s);
        if (st != RCB_OK) return st;
        st = t->p.precision == RCB_MIXED ? launch_near<true>(t, g, g0, g1, s) : launch_near<false>(t, g, g0, g1, s);
        if (st != RCB_OK) return st;
    }
    t->farc_valid = !rb && t->farc;
    return RCB_OK;
}

}  // namespace rcb
