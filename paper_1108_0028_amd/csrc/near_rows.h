// near_rows.h -- near field by rows: lanes are sources. The staged sources wait
// in two stacks in LDS, those that may lie in the support of a sink and those
// that cannot, until one holds a pass of 64 >> kk. The lanes are 1 << kk
// segments; segment s takes a pass's sources against the sinks s per ..
// s per + per - 1, one sink a row, per <= SB. The sinks' sums stay in the lanes'
// registers, SB rows of three, until the list is done, and a source's in its
// lane for the whole pass; no lane idles but in a wave's last two passes.
//
// Lanes as (sink, slice), the other way, read every source back from LDS and
// add its four terms there by LDS atomics, for every pair. Both are bound by
// VALU issue. VJP with slices and with rows: 250,000 particles deterministic FP64
// 3349 and 3000 us; 300,000 in cells of up to 24 FP64 3215 and 2160, of up to 64
// 2434 and 2090, of up to 40 mixed 3488 and 2590; 1M in cells of 8 mixed 5557 and
// 5560. The forward sums, with no terms of the sources, lose a little by it (16M
// 17.0 and 17.6 ms) and keep their slices.
#pragma once

#include "near_tile.h"

namespace rcb {

constexpr int kRowWait = 190;   // at most 63 wait in either stack, and a tile joins them
struct RowShape {
    int kk, per, P;      // P: sources of a pass
    int seg, in_seg;     // of this lane
    int sink0;           // its segment's first sink
};
template <int SB>
__device__ __forceinline__ RowShape row_shape(int c) {   // c <= 64 <= 8 SB sinks
    RowShape r;
    r.kk = c <= SB ? 0 : c <= 2 * SB ? 1 : c <= 4 * SB ? 2 : 3;
    r.per = (c + (1 << r.kk) - 1) >> r.kk;
    r.P = kWave >> r.kk;
    r.seg = lane_id() >> (6 - r.kk);
    r.in_seg = lane_id() & (r.P - 1);
    r.sink0 = r.seg * r.per;
    return r;
}
template <bool MIXED, int SB>
struct RowLds {
    using T = typename std::conditional<MIXED, float, double>::type;
    using Src = typename std::conditional<MIXED, SrcF, SrcD>::type;
    typename std::conditional<MIXED, EntF, EntD>::type ent[kWave];
    uint32_t mark[kWave];
    union {
        struct {
            // sources that may be in reach from the front, others from the back
            Src src[kRowWait];
            T h[kRowWait];
            int32_t pb[kRowWait];   // their tree positions
            Src sink[kWave];        // position, h
        };
        double out[8][SB][3];       // after the passes: partial sums (sum_rows)
    };
};

// Takes the near list [n0, n1) of the leaf with mask bit li and centre of mass
// cA through the stacks; tiles go to the H waves in turn. near(n, slot) and
// far(n, slot) take a pass of n <= P sources, number j at sh.src[slot(j)]
// (far: none in the support of a sink). sh.mark: as tile_entry.
template <bool MIXED, int H, typename A, typename Lds, typename Near, typename Far>
__device__ __forceinline__ void list_rows(const A &a, Lds &sh, int wv, int li, int64_t n0, int64_t n1,
                                          const double (&cA)[3], typename Lds::T reach, int P, uint32_t &gen, Near near,
                                          Far far) {
    using T = typename Lds::T;
    using Src = typename Lds::Src;
    const int lane = lane_id();
    int64_t e0 = n0;
    ChunkEntry ce{};
    int t = 0, nc = 0, no = 0;   // nc, no: waiting in the stacks
    int turn = 0;                // the wave that takes the next tile
    for (;;) {
        while (t >= ce.tot && e0 < n1) {
            ce = load_chunk(a.gnear, a.nfirst, a.ncount, e0, n1, 1u << li);
            if (ce.has()) {
                if constexpr (MIXED) {
                    const double *cB = a.ncom + 3 * (int64_t)ce.label;
                    sh.ent[ce.rank] = EntF{(float)(cB[0] - cA[0]), (float)(cB[1] - cA[1]), (float)(cB[2] - cA[2]),
                                           ce.off()};
                } else {
                    sh.ent[ce.rank].off = ce.off();
                }
            }
            tile_sync();
            t = kWave * (wv >= turn ? wv - turn : wv - turn + H);
            turn = (turn + (ce.tot + kWave - 1) / kWave) % H;
            e0 += kWave;
        }
        const bool more = t < ce.tot;
        if (more) {
            const int nt = ce.tot - t < kWave ? ce.tot - t : kWave;
            const uint64_t valid = ~0ull >> (kWave - nt);
            const auto en = sh.ent[tile_entry(ce, t, sh.mark, gen)];
            // (lanes past the end read the last source again)
            const int32_t pb = en.off + (t + (lane < nt ? lane : nt - 1));
            Src s;
            T h, bx, by, bz;   // b: from the leaf's centre of mass
            if constexpr (MIXED) {
                const float4 f = a.fd[pb];
                h = a.fh[pb];
                s = Src{en.x + f.x, en.y + f.y, en.z + f.z, f.w};
                bx = s.x;
                by = s.y;
                bz = s.z;
            } else {
                s = Src{a.px[pb], a.py[pb], a.pz[pb], a.pm[pb]};
                h = a.ph[pb];
                bx = s.x - cA[0];
                by = s.y - cA[1];
                bz = s.z - cA[2];
            }
            const T lim = (reach + h) * (T)1.001;
            const bool out = (bx * bx + by * by) + bz * bz > lim * lim;
            const uint64_t ob = ballot(out) & valid, cb = ~ballot(out) & valid;
            const int at = out ? kRowWait - 1 - (no + rank_below(ob)) : nc + rank_below(cb);
            if (lane < nt) {
                sh.src[at] = s;
                sh.h[at] = h;
                sh.pb[at] = pb;
            }
            nc += __popcll(cb);
            no += __popcll(ob);
            t += H * kWave;
            tile_sync();
        }
        const int need = more ? P : 1;
        while (nc >= need) {
            const int cnt = nc < P ? nc : P;
            nc -= cnt;
            // at the end the others join the last pass if they fit
            const int join = !more && nc == 0 && no > 0 && cnt + no <= P ? no : 0;
            no -= join;
            near(cnt + join, [&](int i) { return i < cnt ? nc + i : kRowWait - 1 - (i - cnt); });
        }
        while (no >= need) {
            const int cnt = no < P ? no : P;
            no -= cnt;
            far(cnt, [&](int i) { return kRowWait - 1 - (no + i); });
        }
        if (!more) break;
        tile_sync();
    }
    tile_sync();
}

// The rows' sums over the lanes of each segment: the rows are halved twice
// between the lanes of a quad, then the quads of 16 lanes (8 for segments of
// 8) are added into out[lane / 16 (8)]; row_total adds those of a sink.
template <int SB>
__device__ __forceinline__ void sum_rows(const RowShape &rs, const double (&acc)[SB][3], double (&out)[8][SB][3]) {
    constexpr int R = SB / 4;
    const int lane = lane_id();
    const bool odd = lane & 1, pair = lane & 2;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            double v[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const double lo = acc[i + R * j][cc], hi = acc[i + R * j + 2 * R][cc];
                v[j] = (odd ? hi : lo) + quad_perm<0xB1>(odd ? lo : hi);
            }
            double w = (pair ? v[1] : v[0]) + quad_perm<0x4E>(pair ? v[0] : v[1]);
            const int row = 2 * R * (lane & 1) + R * ((lane >> 1) & 1) + i;
            if (rs.P >= 16) {
                w += row_rotate<4>(w);
                w += row_rotate<8>(w);
                if ((lane & 15) < 4) out[lane >> 4][row][cc] = w;
            } else {
                w += __shfl_xor(w, 4, kWave);
                if ((lane & 7) < 4) out[lane >> 3][row][cc] = w;
            }
        }
    tile_sync();
}
template <int SB>
__device__ __forceinline__ void row_total(const RowShape &rs, int sink, const double (&out)[8][SB][3],
                                          double (&sum)[3]) {
    const int seg = sink / rs.per, i = sink - seg * rs.per;
    const int n = rs.P >= 16 ? rs.P >> 4 : 1;   // partial sums of a segment
    for (int r = seg * n; r < seg * n + n; ++r)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) sum[cc] += out[r][i][cc];
}

}  // namespace rcb
