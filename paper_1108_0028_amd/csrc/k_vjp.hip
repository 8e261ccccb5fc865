// k_vjp.hip -- vector-Jacobian product of the accelerations with the tree
// held fixed (topology, particle-to-leaf map and interaction lists frozen;
// M, COM and Q of every node are functions of the inputs). For
// L = sum_a g_a . a_a it returns dL/dx, dL/dy, dL/dz, dL/dm.
//
// Near field (Sec. 2.4.3), pair (a, b), v = r_a - r_b:
//   K = F I + (dF/dr / r) v v^T;  dr_a -= m_b K g_a;  dr_b += m_b K g_a;
//   dm_b -= F (v . g_a).
// Pairs are recomputed from the lists, not stored. The source-side terms
// are summed over the wave's sinks and added with FP64 atomics.
// Far field (Sec. 2.4.2, Eq. 6): per sink leaf the cotangent moments G0, G1,
// G2, stored symmetrised and traceless (far_math.h: only those parts reach Psi),
// then
//   dr_a += J g_a + H[g_a, d_a]                       (d_a = r_a - com_A)
//   com_A receives cot = sum_B d(G2:H/2)/dR  ->  dr_a += m_a/M_A cot,
//                                              dm_a += cot . d_a / M_A
//   node B receives dM, -dPsi/dR, dQ: summed over the group's leaves that
//   accepted B, then added with FP64 atomics.
// Push: every node's adjoint reaches its particles b through
//   M = sum m, COM = sum m r / M, Q = sum m (3 d d^T - |d|^2 I), d = r - COM:
//   dr_b += aR m_b / M + m_b (6 aQ d - 2 tr(aQ) d)
//   dm_b += aM + aR . d / M + 3 d.aQ.d - |d|^2 tr(aQ)
// (dQ/dCOM = 0 because sum m d = 0).
// Kernels: moments (per group) -> far (per group) -> near (per leaf) -> push.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "far_math.h"
#include "near_rows.h"
#include "rcb_internal.h"
#include "soft.h"

namespace rcb {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
// M, R(3) and the traceless part of the Q adjoint, (xx, xy, xz, yy, yz) with
// zz = -(xx + yy): Q is traceless, so the push (the only reader) sees the
// adjoint's traceless part alone (6 aQ d - 2 tr(aQ) d = 6 (aQ - tr/3 I) d, and
// likewise for dm), and one atomic per entry fewer goes out
constexpr int kAdj = 9;
// Nodes of the levels above kMidLevel sit in the far lists of many groups at
// once: their adjoints are added to several copies, in their own array of
// kAdj * 2^kMidLevel per copy, which k_adj_reduce adds in FP64. FP64 form: 8 copies
// (with 64, and 8 of the deeper nodes, the VJP of 300,000 particles took 2.88 ms, so
// 2.74). Mixed form: 64 of FP32, which keep each FP32 sum short. The deeper nodes
// are added to in FP64 in both forms: a node that all 16,384 groups of a cloud
// accept has its mass adjoint to 2.7e-8 so, to 2.4e-7 from 8 FP32 copies and to
// 1.9e-6 from one (mixed VJP of 1M particles 5.74, 5.81 and 5.70 ms, of 4M 21.83,
// 22.18 and 21.91).
constexpr int kMidLevel = 16;
template <typename AT>
constexpr int kAdjMidCopies = sizeof(AT) == 4 ? 64 : 8;
constexpr int kAcc = 30;    // G0(3), G1(9), G2(18) while accumulating
constexpr int kMom = 19;    // S1(3), S2(6), S3(10): far_math.h SymMoments

using rcbfar::hidx;
using rcbfar::jidx;

struct VjpArgs {
    int64_t nleaf;
    int gk;
    int64_t ngroup;
    const int32_t *nfirst, *ncount;
    const double *ncom, *nM, *nQ;
    const int64_t *gnear_beg, *gnear_end, *gfar_beg, *gfar_end;
    const uint64_t *gnear, *gfar;
    const double *px, *py, *pz, *pm, *ph;
    const float4 *fd;
    const float *fh;
    const int32_t *pid;
    const void *gx, *gy, *gz;
    double *mom;    // kMom per leaf: symmetrised cotangent moments
    double *leafc;  // kLeafC per leaf
    double *sink;   // 4 n, tree order: dx dy dz dm
    double *src;    // 4 per particle, tree order, atomics (FP64 form)
    float *srcf;    // the same in the mixed form (FP32 atomics, its contract's accumulation)
    int64_t nmid;   // labels below nmid have kAdjMidCopies adjoint copies
    int64_t n;
    int64_t nlab;
    // deterministic form: each far entry's node adjoint (kAdj FP64) at row
    // cbase[group] + (entry - the group's first entry)
    double *contrib;
    const int64_t *cbase;
    // deterministic form: the cotangents in tree order, 3 n values of the
    // output type (component c of tree position p at c * n + p)
    void *gtree;
    // deterministic form: source-side near terms, 4 per (chunk of the cell's
    // sink groups, particle of the cell) from row srcp[cell], chunk by chunk;
    // the cell's chunks are srcc[cell] .. srcc[cell + 1]
    double *srcpart;
    const int64_t *srcc, *srcp;
    int64_t srcchunk;   // sink groups of a chunk
    int64_t first;   // this launch's first leaf, where a workgroup takes one
};

template <bool MIXED>
__device__ __forceinline__ double load_g(const void *p, int32_t i) {
    if constexpr (MIXED) return (double)((const float *)p)[i];
    else return ((const double *)p)[i];
}

// leaf slot (within the group) of tree position pa
__device__ __forceinline__ int leaf_slot(const int32_t (&lf)[8], int32_t pa) {
    int la = 0;
#pragma unroll
    for (int i = 1; i < 8; ++i)
        if (lf[i] <= pa) la = i;
    return la;
}

// cotangent moments G0, G1, G2 of every leaf of the group, stored symmetrised
template <bool MIXED>
__global__ __launch_bounds__(kBlock) void k_vjp_moments(VjpArgs a) {
    __shared__ double acc_all[kWaves][8][kAcc];
    double(*acc)[kAcc] = acc_all[threadIdx.x / kWave];
    const int64_t gi = wave_index();
    if (gi >= a.ngroup) return;
    const int lane = lane_id();
    const int G = 1 << a.gk;
    const int64_t GL = (a.nleaf >> a.gk) + gi;
    const int32_t sG = a.nfirst[GL], nG = a.ncount[GL];
    for (int i = lane; i < 8 * kAcc; i += kWave) acc[i / kAcc][i % kAcc] = 0.0;
    __builtin_amdgcn_wave_barrier();
    int32_t lf[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) lf[i] = i < G ? a.nfirst[a.nleaf + gi * G + i] : 0x7fffffff;
    for (int s0 = 0; s0 < nG; s0 += kWave) {
        const int si = s0 + lane;
        if (si < nG) {
            const int32_t p = sG + si;
            const int la = leaf_slot(lf, p);
            const int64_t A = a.nleaf + gi * G + la;
            const int32_t o = a.pid[p];
            const double g[3] = {load_g<MIXED>(a.gx, o), load_g<MIXED>(a.gy, o), load_g<MIXED>(a.gz, o)};
            const double d[3] = {a.px[p] - a.ncom[3 * A], a.py[p] - a.ncom[3 * A + 1],
                                 a.pz[p] - a.ncom[3 * A + 2]};
            double *m = acc[la];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                atomicAdd(&m[u], g[u]);
#pragma unroll
                for (int l = 0; l < 3; ++l) atomicAdd(&m[3 + 3 * u + l], g[u] * d[l]);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const int l = k < 3 ? 0 : (k < 5 ? 1 : 2);
                    const int mm = k < 3 ? k : (k < 5 ? k - 2 : 2);
                    atomicAdd(&m[12 + 6 * u + k], g[u] * d[l] * d[mm]);
                }
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (lane < G) {
        const double *m = acc[lane];
        rcbfar::SymMoments S;
        rcbfar::sym_moments(m, m + 3, m + 12, S);
        double *o = a.mom + (gi * G + lane) * kMom;
#pragma unroll
        for (int q = 0; q < 3; ++q) o[q] = S.S1[q];
#pragma unroll
        for (int q = 0; q < 6; ++q) o[3 + q] = S.S2[q];
#pragma unroll
        for (int q = 0; q < 10; ++q) o[9 + q] = S.S3[q];
    }
}

// far field: a workgroup of kFarWaves waves per group, lanes = far entries (64
// per window, the windows going to the waves in turn); the group's leaves are taken in
// turn with their centre of mass and cotangent moments held uniform (scalar
// registers), so each lane sums its entry's node adjoint over the leaves that
// accepted it. The sink-centre term is kept per four lanes and leaf in LDS and
// summed over lanes and waves once per group. A window's adjoints are turned
// round in LDS, so that consecutive lanes hold the kAdj components of one
// entry and its atomics fall into one or two lines. Device-scope atomics run
// past L2, so their number of lines is what they cost: component by component,
// every lane's in a line of its own, this kernel took 5.5 ms for 1M particles
// (mixed, 36M entries), now 3.2; one wave per group of a 64-group cloud 87 us,
// four 23.
constexpr int kFarWaves = 4;
template <typename AT>
struct VjpFarShared {
    double cot[8][3][kWave / 4];   // per four lanes and leaf
    AT rows[kWave * kAdj];         // the window's node adjoints
    int32_t lab[kWave];            // and its labels (-1: past the end)
};

// AT: the type of the node-adjoint copies (FP64; FP32 in the mixed form, whose
// contract allows FP32 accumulation), summed in FP64 by k_adj_reduce; adj takes the
// nodes that have none
// MODE kFarAtomic: node adjoints added atomically to the copies. The
// deterministic form: kFarStore writes each entry's node adjoint (its sum over
// the group's leaves, in leaf order) to a.contrib, summed per node later;
// kFarCot computes the sink-centre sums only (k_vjp_far_node then computes
// the node adjoints itself).
constexpr int kFarAtomic = 0, kFarCot = 1, kFarStore = 2;
template <typename AT, int MODE>
__global__ __launch_bounds__(kFarWaves * kWave, sizeof(AT) == 4 ? 4 : 3) void k_vjp_far(VjpArgs a, double *__restrict__ adj,
                                                               AT *__restrict__ adjmc) {
    __shared__ VjpFarShared<AT> sh_all[kFarWaves];
    __shared__ double mom[8][kMom];   // the group's leaves: symmetrised moments
    __shared__ double com[8][3];      // and centres of mass
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    VjpFarShared<AT> &sh = sh_all[wv];
    const int64_t gi = a.first + blockIdx.x;
    const int lane = lane_id();
    const int G = 1 << a.gk;
    for (int i = lane; i < 8 * 3 * (kWave / 4); i += kWave) (&sh.cot[0][0][0])[i] = 0.0;
    for (int i = threadIdx.x; i < G * kMom; i += kFarWaves * kWave) mom[i / kMom][i % kMom] = a.mom[gi * G * kMom + i];
    if ((int)threadIdx.x < 3 * G) com[threadIdx.x / 3][threadIdx.x % 3] = a.ncom[3 * (a.nleaf + gi * G) + threadIdx.x];
    __syncthreads();
    const int64_t f0 = a.gfar_beg[gi], f1 = a.gfar_end[gi];
    for (int64_t e0 = f0 + wv * kWave; e0 < f1; e0 += kFarWaves * kWave) {
        const int64_t e = e0 + lane;
        const uint64_t ent = e < f1 ? a.gfar[e] : 0ull;
        const uint32_t emask = (uint32_t)(ent >> 32) & 0xffu;
        const int64_t B = (uint32_t)ent & 0x7fffffffu;
        double qq[6], cB[3], MB = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) qq[q] = 0.0;
        cB[0] = cB[1] = cB[2] = 0.0;
        if (emask) {
#pragma unroll
            for (int q = 0; q < 6; ++q) qq[q] = a.nQ[6 * B + q];
            cB[0] = a.ncom[3 * B];
            cB[1] = a.ncom[3 * B + 1];
            cB[2] = a.ncom[3 * B + 2];
            MB = a.nM[B];
        }
        double ad[kAdj];
#pragma unroll
        for (int q = 0; q < kAdj; ++q) ad[q] = 0.0;
        for (int i = 0; i < G; ++i) {
            const bool mine = (emask >> i) & 1u;
            if (ballot(mine) == 0) continue;
            // the leaf's moments and centre are the same on every lane
            const double *mo = mom[i];
            rcbfar::SymMoments Sm;
#pragma unroll
            for (int q = 0; q < 3; ++q) Sm.S1[q] = uniform_f64(mo[q]);
#pragma unroll
            for (int q = 0; q < 6; ++q) Sm.S2[q] = uniform_f64(mo[3 + q]);
#pragma unroll
            for (int q = 0; q < 10; ++q) Sm.S3[q] = uniform_f64(mo[9 + q]);
            const double cA[3] = {uniform_f64(com[i][0]), uniform_f64(com[i][1]), uniform_f64(com[i][2])};
            double ct[3] = {0.0, 0.0, 0.0};
            if (mine) {
                double rho[3], aM, aQ[6];
                rcbfar::far_pair_adjoint_sym(cA[0] - cB[0], cA[1] - cB[1], cA[2] - cB[2], MB, qq, Sm,
                                             rho, ct, aM, aQ);
                ad[0] += aM;
#pragma unroll
                for (int u = 0; u < 3; ++u) ad[1 + u] -= rho[u];
                const double tq = (aQ[0] + aQ[3] + aQ[5]) * (1.0 / 3.0);
                ad[4] += aQ[0] - tq;
                ad[5] += aQ[1];
                ad[6] += aQ[2];
                ad[7] += aQ[3] - tq;
                ad[8] += aQ[4];
            }
            // four lanes add their terms, the first of them keeps the sum
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                double t = ct[u] + swap_adjacent_lanes(ct[u]);
                t += swap_lane_pairs(t);
                if (!(lane & 3)) sh.cot[i][u][lane >> 2] += t;
            }
        }
        if constexpr (MODE != kFarCot) {
#pragma unroll
            for (int q = 0; q < kAdj; ++q) sh.rows[lane * kAdj + q] = (AT)ad[q];
            sh.lab[lane] = emask ? (int32_t)B : -1;
            tile_sync();
            const int nw = (int)(f1 - e0 < kWave ? f1 - e0 : kWave);
            AT *const out = MODE == kFarStore ? (AT *)a.contrib + (a.cbase[gi] + (e0 - f0)) * kAdj : nullptr;
            // each copy takes the groups of one residue mod the number of
            // copies, i.e. of one XCD under round-robin dispatch (8 | copies)
            AT *const mid = adjmc + (int64_t)(blockIdx.x % kAdjMidCopies<AT>) * kAdj * a.nmid;
#pragma unroll 1
            for (int f = lane; f < nw * kAdj; f += kWave) {
                const int r = f / kAdj;
                if constexpr (MODE == kFarStore) {
                    out[f] = sh.rows[f];
                } else {
                    const int32_t L = sh.lab[r];
                    if (L < 0) continue;
                    auto add = [&](auto *p, int64_t row) {
                        using V = typename std::remove_pointer<decltype(p)>::type;
                        __hip_atomic_fetch_add(p + row * kAdj + (f - r * kAdj), (V)sh.rows[f], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    };
                    if constexpr (std::is_same<AT, double>::value) add(L < a.nmid ? mid : adj, L);
                    else if (L < a.nmid) add(mid, L);
                    else add(adj, L);
                }
            }
            tile_sync();
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < 3 * G) {
        const int i = threadIdx.x / 3, u = threadIdx.x % 3;
        double v = 0.0;
        for (int w = 0; w < kFarWaves; ++w)
            for (int l = 0; l < kWave / 4; ++l) v += sh_all[w].cot[i][u][l];
        a.leafc[(gi * G + i) * kLeafC + 19 + u] = v;
    }
}

// near field and the sink-side far terms, per leaf, by rows (near_rows.h). A
// pass's source-side sums go out with one set of atomics per source, four
// consecutive lanes to a source's four and 16 sources at a time: atomics are
// bound by the cache lines they touch. 1M particles, mixed: 0.68 ms for them
// with a particle's four in four arrays, now 0.45.
constexpr int kRowSinks = 8;   // 48 registers of sink sums (12: 250,000 particles deterministic 3117 us, with 8 3000)
template <bool MIXED>
struct VjpShared : RowLds<MIXED, kRowSinks> {
    using T = typename std::conditional<MIXED, float, double>::type;
    T g[kWave][4];         // the sinks' cotangents
    int32_t pa[kWave];     // and tree positions
};

// The source-side sums of n <= 64 staged sources (value(j, c): component c of
// source j; pos(j): its tree position) added to the sources' four (dx dy dz
// dm), four lanes to a source; in the mixed form those sums are FP32 (its
// contract's accumulation).
template <bool MIXED, typename V, typename P>
__device__ __forceinline__ void source_atomics(const VjpArgs &a, int n, V value, P pos) {
    using T = typename std::conditional<MIXED, float, double>::type;
    T *const out = MIXED ? (T *)(void *)a.srcf : (T *)(void *)a.src;
    const int c = lane_id() & 3;
    for (int j = lane_id() >> 2; j < n; j += kWave / 4) {
        const T x = (T)value(j, c);
        if (x != (T)0)
            __hip_atomic_fetch_add(out + 4 * (int64_t)pos(j) + c, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// A pair's term m_b K g_a, K = F I + (dF/dr / r) v v^T, which the sink loses and
// the source gains, and F (v . g_a): one form for k_vjp_near and k_vjp_near_src,
// so that the two sides of a pair are the same bits and cancel in a sum.
template <typename T>
__device__ __forceinline__ void pair_term(const T (&v)[3], const T (&ga)[3], T F, T dFr, T mb, T (&K)[3], T &Fvg) {
    const T vg = v[0] * ga[0] + v[1] * ga[1] + v[2] * ga[2];
    const T Fm = F * mb, vm = dFr * vg * mb;
#pragma unroll
    for (int c = 0; c < 3; ++c) K[c] = Fm * ga[c] + vm * v[c];
    Fvg = F * vg;
}

// SRC = false (the deterministic form): sink-side terms only; the source-side
// terms are summed per source cell by k_vjp_near_src instead.
// A workgroup of H waves per cell, whose sink sums are added in order.
// (One wave per group of 8 cells: 491 us for 4096 particles, now 73.)
template <bool MIXED, bool SRC, int H>
__global__ __launch_bounds__(H * kWave, MIXED ? 4 : 3) void k_vjp_near(VjpArgs a) {
    using T = typename std::conditional<MIXED, float, double>::type;
    using Src = typename std::conditional<MIXED, SrcF, SrcD>::type;
    constexpr int SB = kRowSinks;
    __shared__ VjpShared<MIXED> sh_all[H];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    auto &sh = sh_all[wv];
    const int64_t leaf = a.first + xcd_block<kXcdLeaves>();
    const int64_t gi = leaf >> a.gk, A = a.nleaf + leaf;
    const int li = (int)(leaf & ((1 << a.gk) - 1));
    const int lane = lane_id();
    const int32_t sA = a.nfirst[A], c = a.ncount[A];
    if (c == 0) return;
    const int64_t n0 = a.gnear_beg[gi], n1 = a.gnear_end[gi];
    const double cA[3] = {a.ncom[3 * A], a.ncom[3 * A + 1], a.ncom[3 * A + 2]};
    sh.mark[lane] = 0;
    uint32_t gen = 0;
    // the sink-side terms of the particle at pa from its near-field sums
    auto finish = [&](int32_t pa, const double (&acc)[3]) {
        const int32_t oa = a.pid[pa];
        const double gd[3] = {load_g<MIXED>(a.gx, oa), load_g<MIXED>(a.gy, oa), load_g<MIXED>(a.gz, oa)};
        const double *lc = a.leafc + leaf * kLeafC;
        const double d[3] = {a.px[pa] - cA[0], a.py[pa] - cA[1], a.pz[pa] - cA[2]};
        const double ma = a.pm[pa];
        const double MA = a.nM[A];
        const double cot[3] = {lc[19], lc[20], lc[21]};
        double out[3];
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            double v = acc[l] + ma / MA * cot[l];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                v += gd[i] * lc[3 + jidx(i, l)];
#pragma unroll
                for (int m = 0; m < 3; ++m) v += gd[i] * lc[9 + hidx(i, l, m)] * d[m];
            }
            out[l] = v;
        }
        a.sink[pa] = out[0];
        a.sink[a.n + pa] = out[1];
        a.sink[2 * a.n + pa] = out[2];
        a.sink[3 * a.n + pa] = (cot[0] * d[0] + cot[1] * d[1] + cot[2] * d[2]) / MA;
    };
    for (int g0 = 0; g0 < c; g0 += kWave) {
        const int cs = c - g0 < kWave ? c - g0 : kWave;
        const RowShape rs = row_shape<SB>(cs);
        const bool real = lane < cs;
        const int32_t pa = sA + g0 + (real ? lane : 0);
        // (slots past the sinks: the first one, with no cotangent)
        Src me;
        if constexpr (MIXED) {   // leaf frame
            const float4 f = a.fd[pa];
            me = Src{f.x, f.y, f.z, a.fh[pa]};
        } else {
            me = Src{a.px[pa], a.py[pa], a.pz[pa], a.ph[pa]};
        }
        const int32_t oa = a.pid[pa];
        sh.sink[lane] = me;
        sh.g[lane][0] = real ? (T)load_g<MIXED>(a.gx, oa) : (T)0;
        sh.g[lane][1] = real ? (T)load_g<MIXED>(a.gy, oa) : (T)0;
        sh.g[lane][2] = real ? (T)load_g<MIXED>(a.gz, oa) : (T)0;
        sh.pa[lane] = real ? pa : -1;
        const T reach = MIXED ? sink_reach(me.x, me.y, me.z, me.m)
                              : sink_reach(T(me.x - cA[0]), T(me.y - cA[1]), T(me.z - cA[2]), me.m);
        double acc[SB][3];
#pragma unroll
        for (int i = 0; i < SB; ++i) acc[i][0] = acc[i][1] = acc[i][2] = 0.0;
        // a pass; the sources' slots then hold their sums
        auto pass = [&](auto soft, int n, auto slot) {
            const int at = slot(rs.in_seg < n ? rs.in_seg : 0);
            Src s = sh.src[at];
            const T hb = soft ? sh.h[at] : (T)0;
            const int32_t pb = sh.pb[at];
            s.m = rs.in_seg < n ? s.m : (T)0;
            double src[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                if (i < rs.per) {
                    const Src k = sh.sink[rs.sink0 + i];
                    const T *gp = sh.g[rs.sink0 + i];
                    const T ga[3] = {gp[0], gp[1], gp[2]};
                    const T v[3] = {k.x - s.x, k.y - s.y, k.z - s.z};
                    const T r2 = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
                    const T ri = rsq_t(r2);
                    const T ri2 = ri * ri;
                    const T r3 = ri2 * ri;
                    const T r5 = r3 * ri2;
                    T F = r3, dFr = (T)-3 * r5;
                    if constexpr (soft) {
                        const T hsum = k.m + hb;
                        if (!soft_outside<T>(r2, hsum)) soft_FdF<T>(r2, ri, r3, r5, hsum, F, dFr);
                    }
                    // the deterministic form leaves out the self pair, whose sink and
                    // source terms cancel exactly (v = 0) but would be computed in two
                    // kernels there
                    const T mb = !SRC && soft && pb == sh.pa[rs.sink0 + i] ? (T)0 : s.m;
                    T Kg[3], Fvg;
                    pair_term<T>(v, ga, F, dFr, mb, Kg, Fvg);
#pragma unroll
                    for (int cc = 0; cc < 3; ++cc) {
                        acc[i][cc] -= (double)Kg[cc];
                        if (SRC) src[cc] += (double)Kg[cc];
                    }
                    if (SRC) src[3] -= (double)Fvg;
                }
            }
            if constexpr (SRC) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {   // the segments' sums of the same source
                    if (rs.kk > 0) src[q] = pair_sum<32>(src[q]);
                    if (rs.kk > 1) src[q] = pair_sum<16>(src[q]);
                    if (rs.kk > 2) src[q] += row_rotate<8>(src[q]);
                }
                if (lane < n) sh.src[at] = Src{(T)src[0], (T)src[1], (T)src[2], (T)src[3]};
                tile_sync();
                source_atomics<MIXED>(
                    a, n, [&](int j, int q) { return ((const T *)&sh.src[slot(j)])[q]; },
                    [&](int j) { return sh.pb[slot(j)]; });
                tile_sync();
            }
        };
        tile_sync();
        list_rows<MIXED, H>(
            a, sh, wv, li, n0, n1, cA, reach, rs.P, gen,
            [&](int n, auto slot) { pass(std::true_type{}, n, slot); },
            [&](int n, auto slot) { pass(std::false_type{}, n, slot); });
        sum_rows<SB>(rs, acc, sh.out);
        if constexpr (H > 1) __syncthreads();
        if (wv == 0 && real) {
            double sum[3] = {0.0, 0.0, 0.0};
            for (int w = 0; w < H; ++w) row_total<SB>(rs, lane, sh_all[w].out, sum);
            finish(pa, sum);
        }
        if constexpr (H > 1) __syncthreads();
        else tile_sync();
    }
}

// One node's adjoint (aM, aR, aQ) pushed to a particle at r of mass mb
// through M, COM and Q of the node.
__device__ __forceinline__ void push_node(const double (&ad)[kAdj], double MB, const double (&cB)[3],
                                          const double (&r)[3], double mb, double (&dr)[3],
                                          double &dmb) {
    const double Q[3][3] = {{ad[4], ad[5], ad[6]}, {ad[5], ad[7], ad[8]}, {ad[6], ad[8], -(ad[4] + ad[7])}};
    const double d[3] = {r[0] - cB[0], r[1] - cB[1], r[2] - cB[2]};
    double Qd[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) Qd[l] = Q[l][0] * d[0] + Q[l][1] * d[1] + Q[l][2] * d[2];
#pragma unroll
    for (int l = 0; l < 3; ++l) dr[l] += ad[1 + l] * mb / MB + mb * (6.0 * Qd[l]);
    dmb += ad[0] + (ad[1] * d[0] + ad[2] * d[1] + ad[3] * d[2]) / MB +
           3.0 * (d[0] * Qd[0] + d[1] * Qd[1] + d[2] * Qd[2]);
}

// node adjoints -> particles along each particle's ancestor chain; then the
// three parts are summed and written in caller order. One wave per group,
// lanes over the group's particles: the chain below the group node differs
// per lane, the chain from the group node up is the same for every lane.
template <bool MIXED>
__global__ __launch_bounds__(kBlock) void k_vjp_push(VjpArgs a, const double *__restrict__ adj,
                                                     const double *__restrict__ ncom,
                                                     const double *__restrict__ nM, void *dx, void *dy,
                                                     void *dz, void *dm) {
    const int64_t gi = wave_index();
    if (gi >= a.ngroup) return;
    const int G = 1 << a.gk;
    const int64_t GL = (a.nleaf >> a.gk) + gi;
    const int32_t sG = a.nfirst[GL], nG = a.ncount[GL];
    int32_t lf[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) lf[i] = i < G ? a.nfirst[a.nleaf + gi * G + i] : 0x7fffffff;
    for (int s0 = 0; s0 < nG; s0 += kWave) {
        const int si = s0 + lane_id();
        if (si >= nG) continue;
        const int64_t p = (int64_t)sG + si;
        const double r[3] = {a.px[p], a.py[p], a.pz[p]};
        const double mb = a.pm[p];
        double sr[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) sr[c] = 0.0;
        const int64_t A = a.nleaf + gi * G + leaf_slot(lf, (int32_t)p);
        if (a.srcpart) {   // the chunks' terms in order
            const int64_t bl = A - a.nleaf, c1 = a.srcc[bl + 1] - a.srcc[bl];
            const double *row = a.srcpart + 4 * (a.srcp[bl] + (p - a.nfirst[A]));
            for (int64_t q = 0; q < c1; ++q, row += 4 * (int64_t)a.ncount[A])
#pragma unroll
                for (int c = 0; c < 4; ++c) sr[c] += row[c];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) sr[c] = MIXED ? (double)a.srcf[4 * p + c] : a.src[4 * p + c];
        }
        double dr[3] = {a.sink[p] + sr[0], a.sink[a.n + p] + sr[1], a.sink[2 * a.n + p] + sr[2]};
        double dmb = a.sink[3 * a.n + p] + sr[3];
        for (int64_t B = A; B > GL; B >>= 1) {
            double ad[kAdj];
#pragma unroll
            for (int q = 0; q < kAdj; ++q) ad[q] = adj[B * kAdj + q];
            const double cB[3] = {ncom[3 * B], ncom[3 * B + 1], ncom[3 * B + 2]};
            push_node(ad, nM[B], cB, r, mb, dr, dmb);
        }
        for (int64_t B = GL; B >= 1; B >>= 1) {   // wave-uniform
            double ad[kAdj];
#pragma unroll
            for (int q = 0; q < kAdj; ++q) ad[q] = adj[B * kAdj + q];
            const double cB[3] = {ncom[3 * B], ncom[3 * B + 1], ncom[3 * B + 2]};
            push_node(ad, nM[B], cB, r, mb, dr, dmb);
        }
        const int32_t o = a.pid[p];
        if constexpr (MIXED) {
            ((float *)dx)[o] = (float)dr[0];
            ((float *)dy)[o] = (float)dr[1];
            ((float *)dz)[o] = (float)dr[2];
            ((float *)dm)[o] = (float)dmb;
        } else {
            ((double *)dx)[o] = dr[0];
            ((double *)dy)[o] = dr[1];
            ((double *)dz)[o] = dr[2];
            ((double *)dm)[o] = dmb;
        }
    }
}

// adjoints of the nodes below nmid into out: the sum of their copies in order
template <typename A>
__global__ void k_adj_reduce(double *__restrict__ out, const A *__restrict__ adjmc, int64_t nmid) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= kAdj * nmid) return;
    double v = (double)adjmc[i];
#pragma unroll 8
    for (int c = 1; c < kAdjMidCopies<A>; ++c) v += (double)adjmc[(int64_t)c * kAdj * nmid + i];
    out[i] = v;
}

// ---------------------------------------------------------------------------
// Deterministic form: no atomics. The per-group lists are turned into lists
// of the groups that hold each node (far) or each lowest-level cell (near),
// ascending by group (k_sort.hip), and every sum runs in a fixed order.
// ---------------------------------------------------------------------------
constexpr int kDetChunk = 512;   // far entries per wave of k_vjp_far_node

// cotangent moments without atomics: the group's leaves in turn, 64 particles
// at a time, each of the 30 sums a canonical wave sum (wave_sum)
template <bool MIXED>
__global__ __launch_bounds__(kBlock) void k_vjp_moments_det(VjpArgs a) {
    const int64_t gi = wave_index();
    if (gi >= a.ngroup) return;
    const int lane = lane_id();
    const int G = 1 << a.gk;
    for (int li = 0; li < G; ++li) {
        const int64_t A = a.nleaf + gi * G + li;
        const int32_t sA = a.nfirst[A], c = a.ncount[A];
        double m[kAcc];
#pragma unroll
        for (int q = 0; q < kAcc; ++q) m[q] = 0.0;
        for (int s0 = 0; s0 < c; s0 += kWave) {
            const int si = s0 + lane;
            double g[3] = {0.0, 0.0, 0.0}, d[3] = {0.0, 0.0, 0.0};
            if (si < c) {
                const int32_t p = sA + si;
                const int32_t o = a.pid[p];
                g[0] = load_g<MIXED>(a.gx, o);
                g[1] = load_g<MIXED>(a.gy, o);
                g[2] = load_g<MIXED>(a.gz, o);
                d[0] = a.px[p] - a.ncom[3 * A];
                d[1] = a.py[p] - a.ncom[3 * A + 1];
                d[2] = a.pz[p] - a.ncom[3 * A + 2];
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                m[u] += wave_sum(g[u]);
#pragma unroll
                for (int l = 0; l < 3; ++l) m[3 + 3 * u + l] += wave_sum(g[u] * d[l]);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const int l = k < 3 ? 0 : (k < 5 ? 1 : 2);
                    const int mm = k < 3 ? k : (k < 5 ? k - 2 : 2);
                    m[12 + 6 * u + k] += wave_sum(g[u] * d[l] * d[mm]);
                }
            }
        }
        if (lane == 0) {
            rcbfar::SymMoments S;
            rcbfar::sym_moments(m, m + 3, m + 12, S);
            double *o = a.mom + (gi * G + li) * kMom;
#pragma unroll
            for (int q = 0; q < 3; ++q) o[q] = S.S1[q];
#pragma unroll
            for (int q = 0; q < 6; ++q) o[3 + q] = S.S2[q];
#pragma unroll
            for (int q = 0; q < 10; ++q) o[9 + q] = S.S3[q];
        }
    }
}

// the cotangents in tree order (contiguous per cell for the source-side pass)
template <bool MIXED>
__global__ void k_det_gather_g(VjpArgs a) {
    using T = typename std::conditional<MIXED, float, double>::type;
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= a.n) return;
    const int32_t o = a.pid[p];
    T *gt = (T *)a.gtree;
    gt[p] = (T)load_g<MIXED>(a.gx, o);
    gt[a.n + p] = (T)load_g<MIXED>(a.gy, o);
    gt[2 * a.n + p] = (T)load_g<MIXED>(a.gz, o);
}

// entries per group
__global__ void k_det_count(const int64_t *__restrict__ beg, const int64_t *__restrict__ end,
                            int64_t ngroup, int64_t *__restrict__ cnt) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g < ngroup) cnt[g] = end[g] - beg[g];
}

// item = label << 32 | group << 8 | mask (bits 32-39 of the list entry: the far
// mask, or the near mask), or with compact = true label << 32 | the item's own
// index; written in group order at the group's offset
__global__ __launch_bounds__(kBlock) void k_det_items(const int64_t *__restrict__ beg,
                                                      const int64_t *__restrict__ end,
                                                      const uint64_t *__restrict__ list, int64_t ngroup,
                                                      const int64_t *__restrict__ base, bool compact,
                                                      uint64_t *__restrict__ items) {
    const int64_t gi = wave_index();
    if (gi >= ngroup) return;
    const int64_t e0 = beg[gi], ne = end[gi] - e0, o = base[gi];
    for (int64_t j = lane_id(); j < ne; j += kWave) {
        const uint64_t ent = list[e0 + j];
        const uint64_t lab = (uint32_t)ent & 0x7fffffffu;
        const uint64_t mask = (ent >> 32) & 0xffu;
        items[o + j] = (lab << 32) | (compact ? (uint64_t)(o + j) : (((uint64_t)gi << 8) | mask));
    }
}

// each label's range [lb, le) in the sorted items (lb = le = 0 if absent)
__global__ void k_det_bounds(const uint64_t *__restrict__ it, int64_t n, int64_t *__restrict__ lb,
                             int64_t *__restrict__ le) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t B = (uint32_t)(it[i] >> 32);
    if (i == 0 || (uint32_t)(it[i - 1] >> 32) != B) lb[B] = i;
    if (i == n - 1 || (uint32_t)(it[i + 1] >> 32) != B) le[B] = i + 1;
}

// chunks of kDetChunk entries per label
__global__ void k_det_nchunk(const int64_t *__restrict__ lb, const int64_t *__restrict__ le,
                             int64_t nlab, int64_t *__restrict__ nc) {
    const int64_t B = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (B < nlab) nc[B] = (le[B] - lb[B] + kDetChunk - 1) / kDetChunk;
}

__global__ void k_det_owner(const int64_t *__restrict__ cb, int64_t nlab, int32_t *__restrict__ owner) {
    const int64_t B = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (B >= nlab) return;
    for (int64_t c = cb[B]; c < cb[B + 1]; ++c) owner[c] = (int32_t)B;
}

// node adjoints, one wave per chunk of one node's entries: lanes over the
// entries, each taking the entry's adjoint stored by k_vjp_far (STORED) or
// summing it over the leaves of the entry's far mask in order; the chunk's
// sum is a canonical wave sum
template <bool STORED>
__global__ __launch_bounds__(kBlock) void k_vjp_far_node(VjpArgs a, const uint64_t *__restrict__ items,
                                                         const int64_t *__restrict__ lb,
                                                         const int64_t *__restrict__ le,
                                                         const int64_t *__restrict__ cb,
                                                         const int32_t *__restrict__ owner, int64_t nchunk,
                                                         double *__restrict__ part) {
    const int64_t c = wave_index();
    if (c >= nchunk) return;
    const int lane = lane_id();
    const int G = 1 << a.gk;
    const int64_t B = __builtin_amdgcn_readfirstlane(owner[c]);
    const int64_t e_beg = lb[B] + (c - cb[B]) * kDetChunk;
    const int64_t e_end = e_beg + kDetChunk < le[B] ? e_beg + kDetChunk : le[B];
    double qq[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) qq[q] = a.nQ[6 * B + q];
    const double cB[3] = {a.ncom[3 * B], a.ncom[3 * B + 1], a.ncom[3 * B + 2]};
    const double MB = a.nM[B];
    double ad[kAdj];
#pragma unroll
    for (int q = 0; q < kAdj; ++q) ad[q] = 0.0;
    for (int64_t e0 = e_beg; e0 < e_end; e0 += kWave) {
        const int64_t e = e0 + lane;
        if (e >= e_end) continue;
        const uint64_t it = items[e];
        if constexpr (STORED) {
            const double *row = a.contrib + (int64_t)(uint32_t)it * kAdj;
#pragma unroll
            for (int q = 0; q < kAdj; ++q) ad[q] += row[q];
            continue;
        }
        const int64_t gi = (uint32_t)it >> 8;
        const uint32_t mask = (uint32_t)it & 0xffu;
        for (int i = 0; i < G; ++i) {
            if (!((mask >> i) & 1u)) continue;
            const int64_t leaf = gi * G + i;
            const int64_t A = a.nleaf + leaf;
            const double *mo = a.mom + leaf * kMom;
            rcbfar::SymMoments Sm;
#pragma unroll
            for (int q = 0; q < 3; ++q) Sm.S1[q] = mo[q];
#pragma unroll
            for (int q = 0; q < 6; ++q) Sm.S2[q] = mo[3 + q];
#pragma unroll
            for (int q = 0; q < 10; ++q) Sm.S3[q] = mo[9 + q];
            double rho[3], ct[3] = {0.0, 0.0, 0.0}, aM, aQ[6];
            rcbfar::far_pair_adjoint_sym(a.ncom[3 * A] - cB[0], a.ncom[3 * A + 1] - cB[1],
                                         a.ncom[3 * A + 2] - cB[2], MB, qq, Sm, rho, ct, aM, aQ);
            ad[0] += aM;
#pragma unroll
            for (int u = 0; u < 3; ++u) ad[1 + u] -= rho[u];
            const double tq = (aQ[0] + aQ[3] + aQ[5]) * (1.0 / 3.0);
            ad[4] += aQ[0] - tq;
            ad[5] += aQ[1];
            ad[6] += aQ[2];
            ad[7] += aQ[3] - tq;
            ad[8] += aQ[4];
        }
    }
#pragma unroll
    for (int q = 0; q < kAdj; ++q) {
        const double v = wave_sum(ad[q]);
        if (lane == 0) part[c * kAdj + q] = v;
    }
}

// adj[B * kAdj + q] = sum of the node's chunk sums in chunk order (0 if none)
__global__ void k_det_adj_sum(const double *__restrict__ part, const int64_t *__restrict__ cb, int64_t nlab,
                              double *__restrict__ adj) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= kAdj * nlab) return;
    const int64_t B = i / kAdj, q = i % kAdj;
    double v = 0.0;
    for (int64_t c = cb[B]; c < cb[B + 1]; ++c) v += part[c * kAdj + q];
    adj[i] = v;
}

// chunks of `chunk` sink groups per lowest-level cell, and their rows of
// source terms (one per particle of the cell): kSrcChunk, or all of a cell's in one
// (32 bytes a particle in all) where the rows of more cannot be had
constexpr int64_t kSrcChunk = 64, kSrcAll = (int64_t)1 << 40;
__global__ void k_src_count(const int64_t *__restrict__ lb, const int64_t *__restrict__ le,
                            const int32_t *__restrict__ ncount, int64_t chunk, int64_t nleaf, int64_t *__restrict__ nc,
                            int64_t *__restrict__ nrow) {
    const int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (l >= nleaf) return;
    const int64_t c = ncount[nleaf + l] > 0 ? (le[nleaf + l] - lb[nleaf + l] + chunk - 1) / chunk : 0;
    nc[l] = c;
    nrow[l] = c * ncount[nleaf + l];
}

// source-side near terms, one wave per chunk of a.srcchunk sink groups of a
// lowest-level cell B: lanes (source
// slot, slice) over B's particles as in leaf_lanes. The sink cells A whose
// near list holds B (the groups ascending, then the cells of each group's
// near mask) are taken 8 groups (64 cells) at a time; an exclusive scan of
// their sizes gives each cell's first sink, and the sinks are staged 64 at a
// time in LDS (near_tile.h's chunk layout), each slice taking every J-th.
// In the mixed form a staged sink carries the FP32 shift from its cell's
// centre of mass to B's, so the pair arithmetic is exactly that of
// k_vjp_near. The slices' sums are combined by seg_sum and written to the
// chunk's rows, which k_vjp_push adds in order.
// A cell of a cloud's halo is near to thousands of cells: with one wave per
// cell the longest of 250,000 Plummer particles held the launch for 5.2 ms.
template <typename T>
struct SinkTile {
    T x[kWave], y[kWave], z[kWave], h[kWave], g[3][kWave];
    float sx[kWave], sy[kWave], sz[kWave];   // mixed form: (float)(com_B - com_A)
    int32_t pa[kWave];                       // tree position (the self pair is left out)
};
template <bool MIXED>
struct SrcShared {
    typename std::conditional<MIXED, EntF, EntD>::type ent[kWave];
    SinkTile<typename std::conditional<MIXED, float, double>::type> t;
    uint32_t mark[kWave];
};

template <bool MIXED>
__global__ __launch_bounds__(kWave) void k_vjp_near_src(VjpArgs a, const uint64_t *__restrict__ items,
                                                        const int64_t *__restrict__ lb,
                                                        const int64_t *__restrict__ le,
                                                        const int32_t *__restrict__ owner) {
    using T = typename std::conditional<MIXED, float, double>::type;
    __shared__ SrcShared<MIXED> sh;
    const int64_t ci = a.first + xcd_block<kXcdLeaves>();
    const int lane = lane_id();
    const int G = 1 << a.gk;
    const int64_t bl = __builtin_amdgcn_readfirstlane(owner[ci]);
    const int64_t B = a.nleaf + bl;
    const int32_t sB = a.nfirst[B], c = a.ncount[B];
    const int64_t part = ci - a.srcc[bl];
    double *const rows = a.srcpart + 4 * (a.srcp[bl] + part * c);
    const int64_t e_beg = lb[B] + part * a.srcchunk;
    const int64_t e_end = e_beg + a.srcchunk < le[B] ? e_beg + a.srcchunk : le[B];
    const double cB[3] = {a.ncom[3 * B], a.ncom[3 * B + 1], a.ncom[3 * B + 2]};
    sh.mark[lane] = 0;
    uint32_t gen = 0;
    for (int g0 = 0; g0 < c; g0 += kWave) {
        const LeafLanes L = leaf_lanes(c - g0);
        const int si = g0 + L.sslot;
        const bool has_src = L.sslot < L.S && si < c;
        const int32_t pb = sB + (has_src ? si : 0);
        T mb, hb, bx, by, bz;   // bx..: FP64 position, or the FP32 offset from com_B
        if constexpr (MIXED) {
            const float4 f = a.fd[pb];
            mb = f.w;
            hb = a.fh[pb];
            bx = f.x;
            by = f.y;
            bz = f.z;
        } else {
            mb = a.pm[pb];
            hb = a.ph[pb];
            bx = a.px[pb];
            by = a.py[pb];
            bz = a.pz[pb];
        }
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t e0 = e_beg; e0 < e_end; e0 += kWave / 8) {
            // lane = (group entry e0 + lane / 8, cell lane % 8 of its mask)
            const int64_t e = e0 + (lane >> 3);
            const int li = lane & 7;
            int32_t fA = 0, cA = 0, A = 0;
            if (e < e_end && li < G) {
                const uint64_t it = items[e];
                if (((uint32_t)it >> li) & 1u) {
                    A = (int32_t)(a.nleaf + (int64_t)((uint32_t)it >> 8) * G + li);
                    fA = a.nfirst[A];
                    cA = a.ncount[A];
                }
            }
            const ChunkEntry ce = chunk_entry(A, fA, cA);
            const int tot = ce.tot;
            if (ce.has()) {
                if constexpr (MIXED) {
                    const double *cK = a.ncom + 3 * (int64_t)ce.label;
                    sh.ent[ce.rank] = EntF{(float)(cB[0] - cK[0]), (float)(cB[1] - cK[1]), (float)(cB[2] - cK[2]),
                                           ce.off()};
                } else {
                    sh.ent[ce.rank].off = ce.off();
                }
            }
            for (int t = 0; t < tot; t += kWave) {
                const int nt = tot - t < kWave ? tot - t : kWave;
                const auto en = sh.ent[tile_entry(ce, t, sh.mark, gen)];
                {   // (lanes past the end stage the last sink again: no source reads it)
                    const int32_t pa = en.off + (t + (lane < nt ? lane : nt - 1));
                    sh.t.pa[lane] = pa;
                    if constexpr (MIXED) {
                        const float4 f = a.fd[pa];
                        sh.t.x[lane] = f.x;
                        sh.t.y[lane] = f.y;
                        sh.t.z[lane] = f.z;
                        sh.t.h[lane] = a.fh[pa];
                        sh.t.sx[lane] = en.x;
                        sh.t.sy[lane] = en.y;
                        sh.t.sz[lane] = en.z;
                    } else {
                        sh.t.x[lane] = a.px[pa];
                        sh.t.y[lane] = a.py[pa];
                        sh.t.z[lane] = a.pz[pa];
                        sh.t.h[lane] = a.ph[pa];
                    }
                    const T *gt = (const T *)a.gtree;
                    sh.t.g[0][lane] = gt[pa];
                    sh.t.g[1][lane] = gt[a.n + pa];
                    sh.t.g[2][lane] = gt[2 * a.n + pa];
                }
                tile_sync();
                if (has_src) {
                    for (int j = L.slice; j < nt; j += L.J) {
                        if (sh.t.pa[j] == pb) continue;   // the self pair: v = 0, no term
                        T v[3];
                        if constexpr (MIXED) {   // the source in the sink cell's frame, as in k_vjp_near
                            v[0] = sh.t.x[j] - (sh.t.sx[j] + bx);
                            v[1] = sh.t.y[j] - (sh.t.sy[j] + by);
                            v[2] = sh.t.z[j] - (sh.t.sz[j] + bz);
                        } else {
                            v[0] = sh.t.x[j] - bx;
                            v[1] = sh.t.y[j] - by;
                            v[2] = sh.t.z[j] - bz;
                        }
                        const T r2 = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
                        const T hsum = sh.t.h[j] + hb;
                        const T ri = rsq_t(r2);
                        const T ri2 = ri * ri;
                        const T r3 = ri2 * ri;
                        const T r5 = r3 * ri2;
                        T F = r3, dFr = (T)-3 * r5;
                        if (!soft_outside<T>(r2, hsum)) soft_FdF<T>(r2, ri, r3, r5, hsum, F, dFr);
                        const T ga[3] = {sh.t.g[0][j], sh.t.g[1][j], sh.t.g[2][j]};
                        T Kg[3], Fvg;
                        pair_term<T>(v, ga, F, dFr, mb, Kg, Fvg);
#pragma unroll
                        for (int cc = 0; cc < 3; ++cc) acc[cc] += (double)Kg[cc];
                        acc[3] -= (double)Fvg;
                    }
                }
                tile_sync();
            }
        }
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) acc[cc] = seg_sum(acc[cc], L.slice, L.J);
        if (has_src && L.slice == 0) {
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) rows[4 * (int64_t)si + cc] = acc[cc];
        }
    }
}

// per-node lists of one list kind: the items sorted by label and each
// label's range in them
struct DetLists {
    int64_t *base = nullptr;   // each group's first item (exclusive scan of the list sizes)
    int64_t total = 0;
    uint64_t *items = nullptr;
    int64_t *lb = nullptr, *le = nullptr;
};

rcb_status det_count(rcb_tree *t, const int64_t *beg, const int64_t *end, Scratch &tmp, hipStream_t s,
                     DetLists &out) {
    const int64_t NG = t->ngroup;
    int64_t *cnt = (int64_t *)dalloc(t, sizeof(int64_t) * (NG + 1), s, tmp);
    if (!cnt) return RCB_ENOMEM;
    k_det_count<<<(unsigned)((NG + 255) / 256), 256, 0, s>>>(beg, end, NG, cnt);
    RCB_LAUNCH_CHECK("k_det_count");
    rcb_status st = scan_i64(t, cnt, cnt, NG, s);
    if (st != RCB_OK) return st;
    HostRead rd{cnt + NG, &out.total, (int)sizeof(int64_t)};
    st = read_small(s, &rd, 1, "deterministic VJP: list size");
    if (st != RCB_OK) return st;
    out.base = cnt;
    return RCB_OK;
}

rcb_status det_sort(rcb_tree *t, const int64_t *beg, const int64_t *end, const uint64_t *list, bool compact,
                    Scratch &tmp, hipStream_t s, DetLists &out) {
    const int64_t NG = t->ngroup, total = out.total;
    const int64_t cap = total > 0 ? total : 1;
    uint64_t *ia = (uint64_t *)dalloc(t, sizeof(uint64_t) * cap, s, tmp);
    uint64_t *ib = (uint64_t *)dalloc(t, sizeof(uint64_t) * cap, s, tmp);
    int64_t *lbe = (int64_t *)dalloc(t, sizeof(int64_t) * 2 * t->nlab, s, tmp);
    if (!ia || !ib || !lbe) return RCB_ENOMEM;
    k_det_items<<<(unsigned)((NG + kWaves - 1) / kWaves), kBlock, 0, s>>>(beg, end, list, NG, out.base, compact,
                                                                          ia);
    RCB_LAUNCH_CHECK("k_det_items");
    rcb_status st = sort_by_label(t, ia, ib, total, t->k + 1, s, &out.items);
    if (st != RCB_OK) return st;
    RCB_ZERO(lbe, sizeof(int64_t) * 2 * t->nlab, s);
    out.lb = lbe;
    out.le = lbe + t->nlab;
    if (total > 0) {
        k_det_bounds<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(out.items, total, out.lb, out.le);
        RCB_LAUNCH_CHECK("k_det_bounds");
    }
    return RCB_OK;
}

// The deterministic form after the cotangent moments and far coefficients:
// sink-centre sums and node adjoints (FP64, B * kAdj + q) of the far field,
// and the source-side near terms. Each far entry's node adjoint is stored by
// k_vjp_far and summed per node (72 B per entry); if that array cannot be had
// (or store is false) k_vjp_far_node recomputes it per node.
rcb_status vjp_det(rcb_tree *t, VjpArgs &a, double *adj, bool mixed, bool store, Scratch &tmp, hipStream_t s) {
    const int64_t nlab = t->nlab;
    DetLists far, near;
    rcb_status st = det_count(t, t->gfar_beg, t->gfar_end, tmp, s, far);
    if (st != RCB_OK) return st;
    double *contrib = nullptr;
    if (far.total > 0 && far.total < (int64_t(1) << 32) && store)
        contrib = (double *)dalloc(t, sizeof(double) * kAdj * far.total, s, tmp);
    a.contrib = contrib;
    a.cbase = far.base;
    for (a.first = 0; a.first < t->ngroup; a.first += kMaxGrid) {
        const unsigned gf = (unsigned)std::min(kMaxGrid, t->ngroup - a.first);
        if (contrib) k_vjp_far<double, kFarStore><<<gf, kFarWaves * kWave, 0, s>>>(a, nullptr, nullptr);
        else k_vjp_far<double, kFarCot><<<gf, kFarWaves * kWave, 0, s>>>(a, nullptr, nullptr);
        RCB_LAUNCH_CHECK("k_vjp_far");
    }
    st = det_sort(t, t->gfar_beg, t->gfar_end, t->gfar, contrib != nullptr, tmp, s, far);
    if (st != RCB_OK) return st;
    int64_t *cb = (int64_t *)dalloc(t, sizeof(int64_t) * (nlab + 1), s, tmp);
    if (!cb) return RCB_ENOMEM;
    const unsigned gl = (unsigned)((nlab + 255) / 256);
    k_det_nchunk<<<gl, 256, 0, s>>>(far.lb, far.le, nlab, cb);
    RCB_LAUNCH_CHECK("k_det_nchunk");
    st = scan_i64(t, cb, cb, nlab, s);
    if (st != RCB_OK) return st;
    int64_t nchunk = 0;
    HostRead rd{cb + nlab, &nchunk, (int)sizeof(int64_t)};
    st = read_small(s, &rd, 1, "deterministic VJP: chunk count");
    if (st != RCB_OK) return st;
    const int64_t ncap = nchunk > 0 ? nchunk : 1;
    int32_t *owner = (int32_t *)dalloc(t, sizeof(int32_t) * ncap, s, tmp);
    double *part = (double *)dalloc(t, sizeof(double) * kAdj * ncap, s, tmp);
    if (!owner || !part) return RCB_ENOMEM;
    if (nchunk > 0) {
        k_det_owner<<<gl, 256, 0, s>>>(cb, nlab, owner);
        RCB_LAUNCH_CHECK("k_det_owner");
        const unsigned gc = (unsigned)((nchunk + kWaves - 1) / kWaves);
        if (contrib) k_vjp_far_node<true><<<gc, kBlock, 0, s>>>(a, far.items, far.lb, far.le, cb, owner, nchunk, part);
        else k_vjp_far_node<false><<<gc, kBlock, 0, s>>>(a, far.items, far.lb, far.le, cb, owner, nchunk, part);
        RCB_LAUNCH_CHECK("k_vjp_far_node");
    }
    k_det_adj_sum<<<(unsigned)((kAdj * nlab + 255) / 256), 256, 0, s>>>(part, cb, nlab, adj);
    RCB_LAUNCH_CHECK("k_det_adj_sum");
    st = det_count(t, t->gnear_beg, t->gnear_end, tmp, s, near);
    if (st != RCB_OK) return st;
    st = det_sort(t, t->gnear_beg, t->gnear_end, t->gnear, false, tmp, s, near);
    if (st != RCB_OK) return st;
    a.gtree = dalloc(t, (mixed ? sizeof(float) : sizeof(double)) * 3 * t->n, s, tmp);
    if (!a.gtree) return RCB_ENOMEM;
    const unsigned gp = (unsigned)((t->n + 255) / 256);
    if (mixed) k_det_gather_g<true><<<gp, 256, 0, s>>>(a);
    else k_det_gather_g<false><<<gp, 256, 0, s>>>(a);
    RCB_LAUNCH_CHECK("k_det_gather_g");
    const int64_t NL = t->nleaf;
    int64_t *sc = (int64_t *)dalloc(t, sizeof(int64_t) * 2 * (NL + 1), s, tmp), *sp = sc + NL + 1;
    if (!sc) return RCB_ENOMEM;
    const unsigned gs = (unsigned)((NL + 255) / 256);
    int64_t tot[2] = {0, 0};   // chunks, rows
    int32_t *sown = nullptr;
    for (int64_t chunk : {kSrcChunk, kSrcAll}) {
        a.srcchunk = chunk;
        k_src_count<<<gs, 256, 0, s>>>(near.lb, near.le, t->ncount, chunk, NL, sc, sp);
        RCB_LAUNCH_CHECK("k_src_count");
        st = scan_i64(t, sc, sc, NL, s);
        if (st != RCB_OK) return st;
        st = scan_i64(t, sp, sp, NL, s);
        if (st != RCB_OK) return st;
        const HostRead rs[2] = {{sc + NL, &tot[0], (int)sizeof(int64_t)}, {sp + NL, &tot[1], (int)sizeof(int64_t)}};
        st = read_small(s, rs, 2, "deterministic VJP: source chunks");
        if (st != RCB_OK) return st;
        Scratch rows(t, s);
        a.srcpart = (double *)dalloc(t, sizeof(double) * 4 * (tot[1] + 1), s, rows);
        sown = (int32_t *)dalloc(t, sizeof(int32_t) * (tot[0] + 1), s, rows);
        if (sown && a.srcpart) {
            tmp.insert(tmp.end(), rows.begin(), rows.end());
            rows.clear();
            break;
        }
        a.srcpart = nullptr;
    }
    if (!a.srcpart) return RCB_ENOMEM;
    a.srcc = sc;
    a.srcp = sp;
    k_det_owner<<<gs, 256, 0, s>>>(sc, NL, sown);
    RCB_LAUNCH_CHECK("k_det_owner");
    for (a.first = 0; a.first < tot[0]; a.first += kMaxGrid) {
        const unsigned gn = (unsigned)std::min(kMaxGrid, tot[0] - a.first);
        if (mixed) k_vjp_near_src<true><<<gn, kWave, 0, s>>>(a, near.items, near.lb, near.le, sown);
        else k_vjp_near_src<false><<<gn, kWave, 0, s>>>(a, near.items, near.lb, near.le, sown);
    }
    RCB_LAUNCH_CHECK("k_vjp_near_src");
    return RCB_OK;
}

}  // namespace

rcb_status gravity_vjp(rcb_tree *t, const void *gx, const void *gy, const void *gz, void *dx,
                       void *dy, void *dz, void *dm, hipStream_t s) {
    rcb_status st = ensure_walk(t, s);
    if (st != RCB_OK) return st;
    Scratch tmp(t, s), lists(t, s);   // lists: of the deterministic form
    const int64_t n = t->n;
    double *sink = (double *)dalloc(t, sizeof(double) * 4 * n, s, tmp);
    const bool mixed = t->p.precision == RCB_MIXED;
    const bool det = t->p.deterministic != 0;
    void *srcv = det ? (void *)sink : dalloc(t, (mixed ? sizeof(float) : sizeof(double)) * 4 * n, s, tmp);
    if (det && t->ngroup > (int64_t(1) << 24)) {
        set_error("rcb_gravity_vjp: the deterministic form takes at most 2^24 groups of 8 cells (k <= 27)");
        return RCB_ECAPACITY;
    }
    const int64_t nmid = std::min<int64_t>(t->nlab, int64_t(1) << kMidLevel);
    // the copies of the upper nodes' adjoints; the others go into adj itself, as all
    // do in the deterministic form
    const size_t adjm_bytes = det ? 0
                                  : (mixed ? sizeof(float) * kAdjMidCopies<float> : sizeof(double) * kAdjMidCopies<double>) *
                                        kAdj * (size_t)nmid;
    double *adj = (double *)dalloc(t, sizeof(double) * kAdj * t->nlab, s, tmp);
    void *adjmc = det ? (void *)adj : dalloc(t, adjm_bytes, s, tmp);
    double *mom = (double *)dalloc(t, sizeof(double) * kMom * t->nleaf, s, tmp);
    if (!t->farc) {
        t->farc = (double *)dalloc(t, sizeof(double) * kLeafC * t->nleaf, s, t->list_allocs);
        t->farc_valid = false;
    }
    double *leafc = t->farc;   // 19 far coefficients + the leaf's cotangent sum per leaf
    if (!sink || !srcv || !adj || !adjmc || !mom || !leafc) return RCB_ENOMEM;
    if (!det) {
        RCB_ZERO(srcv, (mixed ? sizeof(float) : sizeof(double)) * 4 * n, s);
        RCB_ZERO(adj + kAdj * nmid, sizeof(double) * kAdj * (t->nlab - nmid), s);
        RCB_ZERO(adjmc, adjm_bytes, s);
    }
    VjpArgs a{t->nleaf, t->gk, t->ngroup, t->nfirst, t->ncount, t->ncom, t->nM, t->nQ,
              t->gnear_beg, t->gnear_end, t->gfar_beg, t->gfar_end, t->gnear, t->gfar, t->px, t->py, t->pz, t->pm, t->ph,
              t->fd, t->fh, t->pid, gx, gy, gz, mom, leafc, sink, mixed ? nullptr : (double *)srcv,
              mixed ? (float *)srcv : nullptr, nmid, n, t->nlab, nullptr, nullptr, nullptr, nullptr, nullptr,
              nullptr, kSrcChunk, 0};
    const unsigned gridg = (unsigned)((t->ngroup + kWaves - 1) / kWaves);
    if (det && mixed) k_vjp_moments_det<true><<<gridg, kBlock, 0, s>>>(a);
    else if (det) k_vjp_moments_det<false><<<gridg, kBlock, 0, s>>>(a);
    else if (mixed) k_vjp_moments<true><<<gridg, kBlock, 0, s>>>(a);
    else k_vjp_moments<false><<<gridg, kBlock, 0, s>>>(a);
    RCB_LAUNCH_CHECK("k_vjp_moments");
    if (!t->farc_valid) {   // else kept by the last rcb_gravity on these moments
        st = far_coefficients(t, leafc, s);
        if (st != RCB_OK) return st;
        t->farc_valid = true;
    }

    // two waves per cell while the cells leave SIMDs idle (4096 particles, 512
    // cells: 241 us the VJP with one, 199 with 2, 191 with 8; 32,768 cells 3.64
    // and 3.56 ms), one from there on (131,072 cells: 8.65 and 8.80 ms)
    auto near = [&](auto src) {
        constexpr bool S = decltype(src)::value;
        auto launch = [&](auto mixed_c, auto waves) {
            constexpr bool M = decltype(mixed_c)::value;
            constexpr int H = decltype(waves)::value;
            k_vjp_near<M, S, H><<<(unsigned)std::min(kMaxGrid, t->nleaf - a.first), H * kWave, 0, s>>>(a);
        };
        auto sized = [&](auto mixed_c) {
            if (t->nleaf <= 32768) launch(mixed_c, std::integral_constant<int, 2>{});
            else launch(mixed_c, std::integral_constant<int, 1>{});
        };
        for (a.first = 0; a.first < t->nleaf; a.first += kMaxGrid) {
            if (mixed) sized(std::true_type{});
            else sized(std::false_type{});
        }
    };
    const unsigned gridr = (unsigned)((kAdj * nmid + 255) / 256);
    if (det) {
        // far field, then node adjoints and source-side terms from the
        // per-node lists
        st = vjp_det(t, a, adj, mixed, getenv("RCB_VJP_DET_RECOMPUTE") == nullptr, lists, s);
        if (st == RCB_ENOMEM && a.contrib) {   // the stored adjoints left too little for the rest
            for (void *p : lists) dfree(t, p, s);
            lists.clear();
            st = vjp_det(t, a, adj, mixed, false, lists, s);
        }
        if (st != RCB_OK) return st;
        near(std::false_type{});
        RCB_LAUNCH_CHECK("k_vjp_near");
    } else {
        for (a.first = 0; a.first < t->ngroup; a.first += kMaxGrid) {
            const unsigned gf = (unsigned)std::min(kMaxGrid, t->ngroup - a.first);
            if (mixed) k_vjp_far<float, kFarAtomic><<<gf, kFarWaves * kWave, 0, s>>>(a, adj, (float *)adjmc);
            else k_vjp_far<double, kFarAtomic><<<gf, kFarWaves * kWave, 0, s>>>(a, adj, (double *)adjmc);
            RCB_LAUNCH_CHECK("k_vjp_far");
        }
        if (mixed) k_adj_reduce<float><<<gridr, 256, 0, s>>>(adj, (const float *)adjmc, nmid);
        else k_adj_reduce<double><<<gridr, 256, 0, s>>>(adj, (const double *)adjmc, nmid);
        RCB_LAUNCH_CHECK("k_adj_reduce");
        near(std::true_type{});
        RCB_LAUNCH_CHECK("k_vjp_near");
    }
    if (mixed) k_vjp_push<true><<<gridg, kBlock, 0, s>>>(a, adj, t->ncom, t->nM, dx, dy, dz, dm);
    else k_vjp_push<false><<<gridg, kBlock, 0, s>>>(a, adj, t->ncom, t->nM, dx, dy, dz, dm);
    RCB_LAUNCH_CHECK("k_vjp_push");
    return RCB_OK;
}

}  // namespace rcb
