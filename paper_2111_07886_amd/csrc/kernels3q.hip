// kernels3q.hip -- fully-3D projectors on quads of mirror-image rays (volumes
// of at most 64 slices).
//
// Four LORs share every piece of one walk.  Bin p and its mirror bin p' =
// Nr - 1 - p see the image through transaxial lines that are point reflections
// of each other (s_p' = -s_p), and a LOR of ring difference d and one of -d
// climb in opposite directions at the same rate.  If the LOR (bin p, +d) whose
// first ring is r1 crosses column c in slice r1 + o over length l, then, with
// c' the point reflection of c,
//     (p , -d)  crosses c  in slice r1 - o,
//     (p', +d)  crosses c' in slice r1 + d - o,
//     (p', -d)  crosses c' in slice r1 - d + o,     each over the length l
// (tau -> 1 - tau under the reflection).  Counted from the opposite end of the
// axial range where the sign is negative, all four run over slice k + o for
// k = 0 .. nz - 1 - |d|:
//     x: (p , +d), r1 = k          on f_c [s],          s = k + o
//     y: (p , -d), r1 = nz-1-k     on f_c [nz-1-s]
//     z: (p', +d), r1 = nz-1-d-k   on f_c'[nz-1-s]
//     w: (p', -d), r1 = k + d      on f_c'[s]
// so a quad is a float4 everywhere: one 16-byte LDS read and four FMAs per
// piece, and a quarter of the walks.  Axis-parallel rays (Q == 0) keep the
// half-open cell rule, which a reflection does not preserve on cell edges:
// their mirror ray takes its own cells.
//
//   k_fp3q  one block per (angle, bin pair, 16 ring-difference magnitudes); the
//           lanes are k.  Per stretch of 32 major cells the columns the ray can
//           enter are staged in LDS as quads.
//   k_bp3q  one block per 4 x 4 tile of the upper half image and, with it, the
//           mirror tile; a wave owns four column pairs, the lanes are k, and
//           the quads of w are staged in LDS by ring-difference magnitude.
//
// The subset sinogram between them holds quads, wq[angle][d][p][k] (zeros for
// k > nz - 1 - d; y and w zero for d = 0, where they repeat x and z), and the
// back-projection is left with z fastest.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "devutil.h"
#include "internal.h"
#include "pen3.h"

namespace petos {

// ------------------------------------------------------------------ layout

static int q_pairs(int n_radial) { return (n_radial + 1) / 2; }

size_t quad_floats(const pet_os_geom* G, int n_al) {
    return 4 * (size_t)n_al * (G->d.max_ring_diff + 1) * q_pairs(G->d.n_radial) * G->d.nz;
}

// memory ordering of LDS traffic between the lanes of one wave
__device__ __forceinline__ void q_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ forward projection

struct FP3QArgs {
    const float* fz;        // image with z fastest: fz[(iy * nx + ix) * nz + iz]
    const float* y;
    const float* r;
    const float2* yr;       // null, or (y, r) bin-major, read instead of y and r
    float* out;             // weights: quads, or compact [angle][plane][bin]; FP_PLAIN: natural layout
    int quad;               // weights as quads
    const int* angles;
    int n_al;
    int mode;
    Reduction red;
};

constexpr int FQ_CELLS = 32;                  // major cells per stretch
constexpr int FQ_COLS = 2 * FQ_CELLS + 1;     // staged columns: a cell adds one, a crossing one
constexpr int FQ_LIST = 3 * FQ_CELLS;         // pieces of a stretch, filled up to eights by pieces of no length
constexpr int FQ_W = 8;                       // waves per block

// float4 of the staged columns; the parts' sums take their place at the end.
// (A lane past the last ring reads up to 63 + 31 entries past the column it is
// at, at most into the lists behind, and its rays are not used.)
__host__ __device__ inline int fq_col_quads(int nz) { return max(FQ_COLS * nz, FQ_W * 128); }

static size_t fq_lds(int nz) {
    return (size_t)fq_col_quads(nz) * sizeof(float4) + FQ_W * (2 * FQ_LIST * sizeof(int2) + (FQ_COLS + 3) * sizeof(int));
}

// A wave takes two ring-difference magnitudes; where there are fewer than 16,
// 2, 4 or 8 waves take the pieces of the same two in turn (parts).
__host__ __device__ inline int fq_parts(int max_rd) {
    const int pairs = (max_rd + 2) / 2;
    return pairs > 4 ? 1 : pairs > 2 ? 2 : pairs > 1 ? 4 : 8;
}
// blocks per (angle, bin pair): 16 magnitudes each
__host__ __device__ inline int fq_chunks(int max_rd) { return (max_rd + 16) / 16; }

static int fq_grid(const pet_os_geom* G, int n_al) {
    return n_al * q_pairs(G->d.n_radial) * fq_chunks(G->d.max_ring_diff);
}

// The transaxial part of a lane's major cell in a stretch: the cell and its
// columns' slots, whether and at what fraction the ray leaves it sideways.
struct FQCell {
    int m, slot, nsl;
    float tX;
    bool xc, own0, own1, live;
};

// Bound by LDS reads (16 bytes per lane and piece, 256 B/clk per CU) where
// many ring differences share a staged column, by the latency of a stretch
// (walk, loads, two barriers) where few do.  So the next stretch's columns are
// on their way in registers while this one's pieces are applied, the loads have
// scalar bases and no branches, and where the magnitudes leave waves idle
// several share the pieces.  Stretches of 32 cells keep two blocks on a CU at
// 64 slices (81 KB); 16 cells (four blocks, as many waves) walk twice as often
// and measured 97.6 against 89.5 us.  One subset's weights of a 200x200x64
// image (281 bins, 8 angles, ring differences to 15): 126.8 us with a block per
// bin that staged its columns for all its LORs singly, 89.5 us here; to 1 at
// 170x169x64 26.1 and 34.7 us (weights for the quad back-projector, which gives
// that back, 57.4 and 43.9 us; the rest of the few-difference calls go to
// k_fp3), to 5 44.4 and 42.0 us.
//
// KL lanes per k-range: 64, or 32 where the volume has at most 32 slices (the
// half-waves then take the wave's two ring-difference magnitudes side by side).
template <int KL>
__device__ __forceinline__ void fp3q_body(const GeoK& g, const FP3QArgs& A, int vblock, char* smem) {
    constexpr int G = 64 / KL;
    constexpr int NT_ACC = 2 / G;
    constexpr int PF = 2 * FQ_CELLS / (FQ_W * G);     // columns a lane group stages ahead
    __shared__ double s_red[FQ_W];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int D = g.max_rd, ND = 2 * D + 1, Nr = g.n_radial, nz = g.nz, NP = (Nr + 1) / 2;
    float4* s_col = reinterpret_cast<float4*>(smem);
    int2* s_pc = reinterpret_cast<int2*>(s_col + fq_col_quads(nz)) + wave * 2 * FQ_LIST;    // LDS byte offset, length
    int* s_tab = reinterpret_cast<int*>(reinterpret_cast<int2*>(s_col + fq_col_quads(nz)) + FQ_W * 2 * FQ_LIST) +
                 wave * (FQ_COLS + 3);

    // groups of eight angles (an XCD each, blocks being dealt round-robin),
    // within them the longest rays, at the centre, first
    const int chunks = fq_chunks(D), parts = fq_parts(D);
    const int ch = vblock % chunks, v = vblock / chunks;
    const int ag = v / (8 * NP), rem = v - ag * 8 * NP, na = min(8, A.n_al - 8 * ag);
    const int p = NP - 1 - rem / na, al = 8 * ag + rem % na;
    const int pm = Nr - 1 - p;
    const int part = wave / (FQ_W / parts), pair = wave % (FQ_W / parts);
    const int a = A.angles[al];
    const AngleK& AK = g.ang[a];
    const TxRay tx = tx_ray(g, AK, p);
    const ZBin zb = z_bin(g, AK, p);
    const int n_major = tx.row_major ? g.ny : g.nx;
    const int n_minor = tx.row_major ? g.nx : g.ny;
    const int ncol = g.nx * g.ny;
    const int qstep = (tx.Q >= 0.0) ? 1 : -1;
    const float invQf = (float)tx.invQ;
    // column of (minor cell c, major cell m): m ms + c cs
    const int cs = tx.row_major ? 1 : g.nx, ms = tx.row_major ? g.nx : 1;
    int m0, m1;
    major_range(tx, n_major, n_minor, m0, m1);
    // axis-parallel: the mirror ray's own cell, and the cells of either ray
    const bool axis = tx.Q == 0.0;
    int cm = 0;
    bool cm_in = false;
    if (axis) {
        const double cf = floor(tx_ray(g, AK, pm).P);
        cm_in = cf >= 0.0 && cf < (double)n_minor;
        cm = cm_in ? (int)cf : 0;
        if (cm_in) {
            m0 = 0;
            m1 = n_major - 1;
        }
    }

    // the lane's walk: major cell i of the stretch, magnitude t of the wave's two
    const int i = lane & 31, t = lane >> 5;
    const int dd0 = 16 * ch + 2 * pair;
    const int dd = dd0 + t;
    const double zeta0 = __fma_rn((double)dd, zb.tau0, 0.5);
    const double Qz = (double)dd * zb.tauQ;
    const bool zup = Qz >= 0.0;
    const int ddc = min(dd, D);
    const float Lkf = (float)(tx.L * g.kappa[(long long)p * ND + D + ddc]);
    const float invQzf = (float)((dd == 0) ? 0.0 : g.inv_d[D + ddc] * zb.inv_tauQ);
    // the lane's ring
    const int grp = lane / KL, k = lane % KL;

    float acc[NT_ACC][4];
#pragma unroll
    for (int u = 0; u < NT_ACC; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[u][q] = 0.0f;
    // slots no cell names keep a column that can be staged
    for (int e = lane; e < FQ_COLS; e += 64) s_tab[e] = -1;
    // A piece of no length reads the wave's own lists, 16 bytes per lane, which
    // never hold anything but finite numbers (offsets, as denormals, and
    // lengths): a column of the image could hold an infinity.
    const int pad = (int)(reinterpret_cast<char*>(s_pc) - smem);
    static_assert(2 * FQ_LIST * sizeof(int2) >= 64 * sizeof(float4), "the lists hold a quad per lane");
    for (int e = lane; e < 2 * FQ_LIST; e += 64) s_pc[e] = make_int2(0, 0);

    // (1) the transaxial part of a stretch, as in the per-wave projector
    // (lanes past the last cell repeat it and keep no piece), and its columns'
    // slots: a cell takes the next slot, a crossing one more
    auto walk = [&](int mb) {
        FQCell c;
        c.live = mb + i <= m1;
        c.m = min(mb + i, m1);
        const double gm = __fma_rn(tx.Q, (double)c.m, tx.P);
        const double cf = floor(gm);
        const int c0 = (int)cf, c1 = c0 + qstep;
        const double ce = (tx.Q >= 0.0) ? cf + 1.0 : cf;
        const double ge = gm + tx.Q;
        c.xc = (tx.Q >= 0.0) ? (ge > ce) : (ge < ce);
        c.tX = c.xc ? (float)(ce - gm) * invQf : 1.0f;
        c.own0 = (unsigned)c0 < (unsigned)n_minor;
        c.own1 = (unsigned)c1 < (unsigned)n_minor;
        const int cfirst = __builtin_amdgcn_readfirstlane(c0);
        c.slot = min(c.m - mb + (c0 - cfirst) * qstep, FQ_COLS - 2);
        c.nsl = __builtin_amdgcn_readlane(c.slot, 31) + 2;
        s_tab[c.slot + 1] = c.own1 ? c.m * ms + c1 * cs : -1;
        q_wave_sync();
        s_tab[c.slot] = c.own0 ? c.m * ms + c0 * cs : -1;
        q_wave_sync();
        return c;
    };
    // A staged column and its mirror at the lane's slice and the opposite one,
    // whole volume columns whatever the slot holds (a slot no cell names
    // repeats one, lanes past the last slice repeat that).
    const int kb = min(k, nz - 1), kt = nz - 1 - kb;
    auto column = [&](int mb, int s, int j) {
        const int jj = max(j, 0), mm = min(mb + s, m1);
        const int c = jj * nz, c2 = (axis ? (n_major - 1 - mm) * ms + cm * cs : ncol - 1 - jj) * nz;
        const float* fc = A.fz + c;
        const float* f2 = A.fz + c2;
        return make_float4(img_at(fc, kb), img_at(fc, kt), img_at(f2, kt), img_at(f2, kb));
    };
    // the stretch's columns into registers, a share per wave
    float4 f4[PF];
    unsigned none = 0;      // slots without a column
    auto load = [&](int mb) {
        const int jt = s_tab[min(lane, FQ_COLS - 1)];
        none = 0;
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int s0 = (u * FQ_W + wave) * G;
            int j = __builtin_amdgcn_readlane(jt, s0);
            if (G == 2) j = grp ? __builtin_amdgcn_readlane(jt, s0 + G - 1) : j;
            if (j < 0) none |= 1u << u;
            f4[u] = column(mb, s0 + grp, j);
        }
    };
    // axis-parallel rays: nothing where one of the two is outside
    auto inside = [&](float4 x, bool no) {
        if (axis) {
            if (no) x.x = x.y = 0.0f;
            if (!cm_in) x.z = x.w = 0.0f;
        }
        return x;
    };

    FQCell c{};
    if (m0 <= m1) {
        c = walk(m0);
        load(m0);
    }
    for (int mb = m0; mb <= m1; mb += FQ_CELLS) {
        // (2) the axial part and the pieces of the lane's cell and magnitude
        const double zm = __fma_rn(Qz, (double)c.m, zeta0);
        const double of = floor(zm);
        const int o0 = (int)of, o1 = o0 + (zup ? 1 : -1);
        const double oe = zup ? of + 1.0 : of;
        const double ze = zm + Qz;
        const bool zc = zup ? (ze > oe) : (ze < oe);
        const float tZ = zc ? (float)(oe - zm) * invQzf : 1.0f;
        const bool x_first = c.tX <= tZ;
        const float t1 = fminf(c.tX, tZ), t2 = fmaxf(c.tX, tZ);
        const int po1 = x_first ? o0 : o1;
        const bool in0 = c.own0 || (axis && cm_in), in1 = c.own1;
        const bool pin1 = x_first ? in1 : in0;
        const float fr0 = t1, fr1 = t2 - t1, fr2 = 1.0f - t2;
        const bool v0 = fr0 > 0.0f && in0 && o0 >= 0 && o0 <= dd;
        const bool v1 = (c.xc || zc) && fr1 > 0.0f && pin1 && po1 >= 0 && po1 <= dd;
        const bool v2 = c.xc && zc && fr2 > 0.0f && in1 && o1 >= 0 && o1 <= dd;
        const int e0 = c.slot * nz, e1 = e0 + nz;
        const int off[3] = {e0 + o0, (x_first ? e1 : e0) + po1, e1 + o1};
        const float len[3] = {Lkf * fr0, Lkf * fr1, Lkf * fr2};
        const int present = (c.live && dd <= D) ? (v0 ? 1 : 0) | (v1 ? 2 : 0) | (v2 ? 4 : 0) : 0;
        // (3) the two lists of the wave, in cell order, filled up to eights by
        // pieces of no length
        const int cnt = __popc(present);
        const unsigned long long b0 = __ballot(cnt & 1), b1 = __ballot(cnt & 2);
        const unsigned lo0 = (unsigned)b0, lo1 = (unsigned)b1, hi0 = (unsigned)(b0 >> 32), hi1 = (unsigned)(b1 >> 32);
        int pos = t ? __builtin_amdgcn_mbcnt_hi(hi0, 0u) + 2 * __builtin_amdgcn_mbcnt_hi(hi1, 0u)
                    : __builtin_amdgcn_mbcnt_lo(lo0, 0u) + 2 * __builtin_amdgcn_mbcnt_lo(lo1, 0u);
        const int tot0 = __popc(lo0) + 2 * __popc(lo1), tot1 = __popc(hi0) + 2 * __popc(hi1);
        const int tot = t ? tot1 : tot0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (present & (1 << q)) {
                s_pc[t * FQ_LIST + pos] = make_int2(off[q] * 16, __float_as_int(len[q]));
                ++pos;
            }
        }
        if (i < ((8 - tot) & 7)) s_pc[t * FQ_LIST + tot + i] = make_int2(pad, 0);
        __syncthreads();    // the previous stretch's columns are read no more
        // (4) the columns into LDS, and the next stretch's on their way
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int sl = (u * FQ_W + wave) * G + grp;
            if (sl < c.nsl && k < nz) s_col[sl * nz + k] = inside(f4[u], (none >> u) & 1u);
        }
        if (c.nsl == FQ_COLS && wave == 0 && grp == 0 && k < nz) {
            // (a crossing in every cell: one column more)
            const int j = s_tab[FQ_COLS - 1];
            s_col[(FQ_COLS - 1) * nz + k] = inside(column(mb, FQ_COLS - 1, j), j < 0);
        }
        __syncthreads();    // every wave's columns (and this wave's lists) are in LDS
        if (mb + FQ_CELLS <= m1) {
            c = walk(mb + FQ_CELLS);
            load(mb + FQ_CELLS);
        }

        // (5) every lane k applies every piece (of its part) to its four rays
#pragma unroll
        for (int u = 0; u < NT_ACC; ++u) {
            const int tl = G == 1 ? u : grp;
            const int n = G == 1 ? (u ? tot1 : tot0) : (grp ? tot1 : tot0);
            const int2* pc = s_pc + tl * FQ_LIST;
            const char* col = reinterpret_cast<const char*>(s_col + k);
            for (int e = 8 * part; e < n; e += 8 * parts) {
                int4 q[4];
                float4 x[8];
#pragma unroll
                for (int h = 0; h < 4; ++h) q[h] = *reinterpret_cast<const int4*>(pc + e + 2 * h);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    x[2 * h] = *reinterpret_cast<const float4*>(col + q[h].x);
                    x[2 * h + 1] = *reinterpret_cast<const float4*>(col + q[h].z);
                }
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    const float l = __int_as_float((h & 1) ? q[h >> 1].w : q[h >> 1].y);
                    acc[u][0] = fmaf(l, x[h].x, acc[u][0]);
                    acc[u][1] = fmaf(l, x[h].y, acc[u][1]);
                    acc[u][2] = fmaf(l, x[h].z, acc[u][2]);
                    acc[u][3] = fmaf(l, x[h].w, acc[u][3]);
                }
            }
        }
    }
    // the parts of a pair of magnitudes added in order, into the first
    if (parts > 1) {
        __syncthreads();    // the columns are read no more
#pragma unroll
        for (int u = 0; u < NT_ACC; ++u)
            s_col[(wave * NT_ACC + u) * 64 + lane] = make_float4(acc[u][0], acc[u][1], acc[u][2], acc[u][3]);
        __syncthreads();
        for (int q = 1; q < parts; ++q) {
#pragma unroll
            for (int u = 0; u < NT_ACC; ++u) {
                const float4 x = s_col[((q * (FQ_W / parts) + pair) * NT_ACC + u) * 64 + lane];
                acc[u][0] += x.x;
                acc[u][1] += x.y;
                acc[u][2] += x.z;
                acc[u][3] += x.w;
            }
        }
    }

    // (6) the rays' outputs
    double term = 0.0;
#pragma unroll 1
    for (int u = 0; u < NT_ACC; ++u) {
        float mine[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) mine[q] = u ? acc[NT_ACC - 1][q] : acc[0][q];
        const int od = dd0 + (G == 1 ? u : grp);
        if (od > D || k >= nz || part > 0) continue;
        const bool ok = k <= nz - 1 - od;
        const int pp = g.plane_base[D + od], pn = g.plane_base[D - od], kr = nz - 1 - od - k;
        const int plane[4] = {pp + k, pn + kr, pp + kr, pn + k};
        const int bin[4] = {p, p, pm, pm};
        // rays counted once: d = 0 has no negative side, the centre bin no mirror
        const bool twin[4] = {false, od == 0, p == pm, od == 0 || p == pm};
        if (A.mode == FP_RATIO || A.mode == FP_EM) {
            float o4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                o4[q] = 0.0f;
                if (!ok || (od == 0 && (q & 1))) continue;
                float yv, rv;
                if (A.yr != nullptr) {
                    const float2 d2 = A.yr[((long long)a * Nr + bin[q]) * g.n_planes + plane[q]];
                    yv = d2.x;
                    rv = d2.y;
                } else {
                    const long long nat = ((long long)plane[q] * g.n_angles + a) * Nr + bin[q];
                    yv = A.y[nat];
                    rv = A.r[nat];
                }
                o4[q] = A.mode == FP_RATIO ? 1.0f - yv / (mine[q] + rv) : yv / (mine[q] + rv);
            }
            if (A.quad) {
                const long long e = (((long long)al * (D + 1) + od) * NP + p) * nz + k;
                reinterpret_cast<float4*>(A.out)[e] = make_float4(o4[0], o4[1], o4[2], o4[3]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (ok && !twin[q]) A.out[((long long)al * g.n_planes + plane[q]) * Nr + bin[q]] = o4[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (!ok || twin[q]) continue;
                const long long nat = ((long long)plane[q] * g.n_angles + a) * Nr + bin[q];
                if (A.mode == FP_PLAIN) {
                    A.out[nat] = mine[q];
                } else {
                    const double qv = (double)mine[q];
                    term += qv - (double)A.y[nat] * log(qv + (double)A.r[nat]);
                }
            }
        }
    }
    if (A.mode == FP_OBJECTIVE) write_partial(term, A.red, s_red, vblock);
}

extern __shared__ __attribute__((aligned(16))) char q_smem[];

template <int KL>
__global__ __launch_bounds__(FQ_W * 64, 4) void k_fp3q(GeoK g, FP3QArgs A) {
    fp3q_body<KL>(g, A, blockIdx.x, q_smem);
}

// ------------------------------------------------------------------ back projection

struct BP3QArgs {
    const float4* wq;        // quads [angle of the list][d][p][k]
    const int* angles;
    int n_al;
    float* out;              // A_i^T w, z fastest
    int nr;                  // staged bin pairs per angle at most
    int buf;                 // float4 of one staging buffer
    int add;                 // add to what out holds
    Pen3Args pen;            // the penalty blocks' arguments (gradR set) when n_pen > 0
    int n_pen;
};

constexpr int BQ_X = 4, BQ_Y = 4;      // column pairs of a tile: a row of four per wave
constexpr int BQ_C = BQ_X * BQ_Y;      // column pairs of a tile
constexpr int BQ_W = 4;                // column pairs of a wave
// ring-difference magnitudes staged together, by the lanes per k-range
__host__ __device__ constexpr int bq_dg(int kl) { return kl == 32 ? 4 : 2; }
constexpr int BQ_PAD = 64;             // zeros before the first staged row (k - o < 0, and pieces that are none)
constexpr int BQ_AMAX = 16;            // angles per chunk (axis-parallel ones, two at most, count twice)
constexpr int BQ_E = 4;                // angles whose hits are found together
constexpr int BQ_DC = 8;               // magnitudes whose pieces are held at once
constexpr size_t BQ_LDS_MAX = 65536;   // bytes of dynamic LDS at most

// One (column, bin) hit of an angle: tau at the low end of the column's cell
// on the ray, its extent, the transaxial length and the axial slope per
// magnitude; the staged row, with BQ_UPPER where the bin lies past the centre
// (it is then taken as its mirror bin seen by the mirror column), or -1.
constexpr int BQ_UPPER = 1 << 16;

__host__ __device__ inline int bq_tiles_x(int nx);

struct BP3QShared {
    float4 hit[BQ_E][BQ_C][2];
    int row[BQ_E][BQ_C][2];
    int2 piece[NT / 64][BQ_W][2][BQ_DC];    // of a wave's columns: byte offset in the staged rows, length
    // the chunk's angles, axis-parallel ones last and twice (for the columns,
    // then for their mirrors): angle, place in the chunk, the tile's bin pairs
    int ang[BQ_AMAX + 2], al[BQ_AMAX + 2], plo[BQ_AMAX + 2], nrow[BQ_AMAX + 2];
    int n_oblique;
    double red[NT / 64];
};

// ballots over a wave's lanes (column, hit, magnitude): the hit is there; it is
// past the centre; the piece reaches into the next slice, over length next
struct BQMasks {
    unsigned long long valid, upper, split;
    float next;
};
constexpr unsigned long long BQ_SECOND = 0xff00ff00ff00ff00ull;    // lanes of second hits

// Copy the rows of magnitudes d .. d + ng - 1 (largest first: a row's zeros
// past k = nz - 1 - d then serve the next row's k - o < 0) of n4 / nz bin
// pairs to dst, a quad per thread at a time.  s: the pairs' row of magnitude
// d, dstep bytes to the next (wave-uniform, so that a copy's address is a
// scalar base and the thread's offset).  Returns without waiting.
template <int DG>
__device__ __forceinline__ void bq_stage(float4* dst, const char* s, long long dstep, int ng, int n4, int wave) {
    typedef __attribute__((address_space(3))) void* Lds;
    for (int e0 = 0; e0 < n4; e0 += NT) {
        if (e0 + (int)threadIdx.x < n4) {
#pragma unroll
            for (int e = 0; e < DG; ++e)
                if (e < ng)
                    __builtin_amdgcn_global_load_lds(
                        reinterpret_cast<const float*>(s + e * dstep + (size_t)e0 * 16 + threadIdx.x * 16u),
                        (Lds)(dst + (ng - 1 - e) * n4 + e0 + wave * 64), 16, 0, 0);
        }
    }
}

// The hits of the tile's columns for entries e0 .. e0 + BQ_E - 1 of the chunk's
// angles: two entries per wave, lane = (entry, column, candidate bin).  A
// column meets two bins of an angle at most (quad_ok).
__device__ __forceinline__ void bq_hits(const GeoK& g, BP3QShared& sh, int e0, int ne, int tx0, int ty0) {
    static_assert(BQ_E <= 2 * (NT / 64) && BQ_E % 2 == 0 && BQ_C == 16, "a wave takes two entries of 16 columns by two bins");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave >= BQ_E / 2) return;
    const int el = 2 * wave + (lane >> 5), c = (lane >> 1) & 15, cand = lane & 1;
    const int ncol = g.nx * g.ny, Nr = g.n_radial;
    const int e = min(e0 + el, ne - 1);
    const AngleK& AK = g.ang[sh.ang[e]];
    const int plo = sh.plo[e], nrow = sh.nrow[e];
    const bool mir = e > sh.n_oblique && ((e - sh.n_oblique) & 1);
    const int ix = tx0 + c % BQ_X, iy = ty0 + c / BQ_X;
    const bool live = ix < g.nx && 2 * (iy * g.nx + ix) <= ncol - 1;
    const int cx = mir ? g.nx - 1 - ix : ix, cy = mir ? g.ny - 1 - iy : iy;
    const int m = AK.row_major ? cy : cx, mc = AK.row_major ? cx : cy;
    // candidates: g(m) in [mc - max(Q,0), mc + 1 - min(Q,0)]
    const double base = __fma_rn(AK.Q, (double)m, AK.wC);
    const double bA = ((double)mc - fmax(AK.Q, 0.0) - 1e-7 - base) * AK.inv_wslope;
    const double bB = ((double)mc + 1.0 - fmin(AK.Q, 0.0) + 1e-7 - base) * AK.inv_wslope;
    const int b = (int)fmax(ceil(fmin(bA, bB) - 1e-6), 0.0) + cand;
    const int bc = min(b, Nr - 1);
    const BinK& B = g.bin[bc];
    const double P = AK.Q == 0.0 ? (AK.row_major ? B.axis_pos_x : B.axis_pos_y) : __fma_rn(B.sb, AK.icv, AK.K);
    // the psi-interval of the column's cell on the bin's ray, kept as tau
    // (FP64 differences)
    double ax, bx;
    cell_interval(__fma_rn(AK.Q, (double)m, P), AK.Q, AK.invQ, mc, ax, bx);
    const bool upper = 2 * bc > Nr - 1;
    const int row = (upper ? Nr - 1 - bc : bc) - plo;
    const bool hit = live && b < Nr && bx > ax && (unsigned)row < (unsigned)nrow;
    const double tau0 = (__fma_rn(B.sb, AK.Au, AK.Bu) + B.h) * B.inv2h, tauQ = AK.du * B.inv2h;
    const double tA = __fma_rn(tauQ, (double)m + ax, tau0), tB = __fma_rn(tauQ, (double)m + bx, tau0);
    // a bin past the centre: tau -> 1 - tau
    const float t0 = (float)(upper ? 1.0 - fmax(tA, tB) : fmin(tA, tB));
    // the first hit in slot 0
    const bool other = __builtin_amdgcn_update_dpp(0, (int)hit, DPP_XOR1, 0xF, 0xF, false);
    const int slot = cand ? (hit && !other ? 0 : 1) : (!hit && other ? 1 : 0);
    sh.hit[el][c][slot] =
        make_float4(t0, (float)fabs(tB - tA), (float)(AK.L * (bx - ax)), (float)g.vz * (float)B.inv2h);
    sh.row[el][c][slot] = hit ? row | (upper ? BQ_UPPER : 0) : -1;
}

// The pieces of the wave's columns for magnitudes ddc .. ddc + BQ_DC - 1: lane =
// (column, hit, magnitude).
template <int DG>
__device__ __forceinline__ void bq_pieces(const GeoK& g, BP3QShared& sh, int el, int ddc, int nrow, int wave, int lane,
                                          BQMasks& M) {
    static_assert(BQ_W * 2 * BQ_DC == 64, "a lane per column, hit and magnitude");
    const int c = lane >> 4, h = (lane >> 3) & 1, dd = ddc + (lane & 7);
    const int ds = min(DG, g.max_rd + 1 - (dd - dd % DG)) - 1 - dd % DG;   // largest first
    const float4 H = sh.hit[el][wave * BQ_W + c][h];
    const int rf = sh.row[el][wave * BQ_W + c][h];
    // the piece's axial range in slice units (FP32: at most 1/2 + D, its
    // rounding far below a slice); it spans less than a slice
    const float fd = (float)dd;
    const float zlo = fmaf(fd, H.x, 0.5f), span = fd * H.y, zhi = zlo + span;
    const float flo = floorf(zlo), fhi = floorf(zhi);
    const int o1 = (int)flo, o2 = (int)fhi;
    // 3D length per transaxial length of this (bin, d)
    const float x = fd * H.w;
    const float LK = H.z * __builtin_amdgcn_sqrtf(fmaf(x, x, 1.0f));
    const float frac = fminf(1.0f, fmaxf(0.0f, (fhi - zlo) * __builtin_amdgcn_rcpf(span)));
    const float l1 = o2 != o1 ? LK * frac : LK;
    // (what is no piece reads the zeros before the rows)
    const bool ok = rf >= 0 && dd <= g.max_rd && o1 >= 0 && o2 <= dd && o2 <= o1 + 1;
    const int entry = BQ_PAD + (ds * nrow + (rf & (BQ_UPPER - 1))) * g.nz - o1;
    sh.piece[wave][c][h][lane & 7] = ok ? make_int2(entry * 16, __float_as_int(l1)) : make_int2(0, 0);
    M.next = ok ? LK - l1 : 0.0f;
    M.valid = __ballot(rf >= 0);
    M.upper = __ballot(rf >= 0 && (rf & BQ_UPPER));
    M.split = __ballot(M.next > 0.0f);
    q_wave_sync();
}

// x, y of the quad to acc[0], acc[1], z, w to acc[2], acc[3]; axis-parallel
// angles take the half that holds the column's bin only (up: z, w)
template <bool AXIS>
__device__ __forceinline__ void bq_fma(float (&acc)[4], int l, bool up, const float4& x) {
    const float len = __int_as_float(l);
    const float s0 = fmaf(len, x.x, acc[0]), s1 = fmaf(len, x.y, acc[1]);
    const float s2 = fmaf(len, x.z, acc[2]), s3 = fmaf(len, x.w, acc[3]);
    acc[0] = AXIS && up ? acc[0] : s0;
    acc[1] = AXIS && up ? acc[1] : s1;
    acc[2] = AXIS && !up ? acc[2] : s2;
    acc[3] = AXIS && !up ? acc[3] : s3;
}

// exchange the parts of c and c'
__device__ __forceinline__ void bq_swap(float (&acc)[4], bool on) {
    if (on) {
        const float a0 = acc[0], a1 = acc[1];
        acc[0] = acc[3];
        acc[1] = acc[2];
        acc[2] = a1;
        acc[3] = a0;
    }
}

// of a mask over (column, hit, magnitude): the bit of column slot J's first
// hit (of the calling lane's group, for KL = 32); whether any group has it
template <int KL>
__device__ __forceinline__ bool bq_bit(unsigned long long m, int J, int grp) {
    return (m >> (KL == 64 ? 16 * J : 32 * grp + 16 * J)) & 1ull;
}
template <int KL>
__device__ __forceinline__ bool bq_any(unsigned long long m, int J) {
    return KL == 64 ? (m >> (16 * J)) & 1ull : ((m >> (16 * J)) | (m >> (32 + 16 * J))) & 1ull;
}

// acc holds c from the low end, c from the high end, c' from the high end and
// c' from the low end, or with c and c' exchanged (sw): whichever the first
// hits need
template <int KL, int... J>
__device__ __forceinline__ void bq_orient(float (&acc)[sizeof...(J)][4], unsigned long long& sw, const BQMasks& M,
                                          bool mir, int grp, std::integer_sequence<int, J...>) {
    const unsigned long long turn = ((mir ? ~M.upper : M.upper) ^ sw) & M.valid & ~BQ_SECOND;
    if (turn == 0) return;
    ((bq_any<KL>(turn, J) ? bq_swap(acc[J], bq_bit<KL>(turn, J, grp)) : (void)0), ...);
    sw ^= turn;
}

// the parts, in their next slice, of hit h's pieces of column slot J
template <int KL, bool AXIS, int J>
__device__ __forceinline__ void bq_next(float (&acc)[4], const BQMasks& M, const int2* pl, const char* __restrict__ lb,
                                        int h, int src0, unsigned long long turn, int grp) {
    constexpr int DG = bq_dg(KL);
    const int src = 16 * J + 8 * h + src0;
    unsigned m = (unsigned)(M.split >> src);
    if (KL == 32) m |= (unsigned)(M.split >> (32 + src));
    m &= (1u << DG) - 1;
    if (m == 0) return;
    const bool any = h == 1 && bq_any<KL>(turn, J), on = any && bq_bit<KL>(turn, J, grp);
    const bool up = bq_bit<KL>(h ? M.upper >> 8 : M.upper, J, grp);
    if (any) bq_swap(acc, on);
#pragma unroll 1
    do {
        const int e = __builtin_ctz(m);
        m &= m - 1;
        const int l0 = __builtin_amdgcn_readlane(__float_as_int(M.next), src + e);
        const int l1 = KL == 32 ? __builtin_amdgcn_readlane(__float_as_int(M.next), 32 + src + e) : l0;
        const int l = KL == 32 && grp ? l1 : l0;
        if (KL == 64 || l != 0)
            bq_fma<AXIS>(acc, l, up, *reinterpret_cast<const float4*>(lb + pl[(J * 2 + h) * BQ_DC + e].x - 16));
    } while (m);
    if (any) bq_swap(acc, on);
}

// apply hit h's pieces of column slots J0 .. J0 + N - 1, DG magnitudes each,
// from the staged rows: their reads in flight together
template <int KL, bool AXIS, int J0, int N, int CPG>
__device__ __forceinline__ void bq_apply(float (&acc)[CPG][4], const int2* pl, int h, const char* __restrict__ lb,
                                         unsigned long long upper, int grp) {
    constexpr int DG = bq_dg(KL);
    int4 q[N][DG / 2];
    float4 x[N][DG];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int e = 0; e < DG / 2; ++e)
            q[j][e] = *reinterpret_cast<const int4*>(pl + ((J0 + j) * 2 + h) * BQ_DC + 2 * e);
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int e = 0; e < DG / 2; ++e) {
            x[j][2 * e] = *reinterpret_cast<const float4*>(lb + q[j][e].x);
            x[j][2 * e + 1] = *reinterpret_cast<const float4*>(lb + q[j][e].z);
        }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const bool up = bq_bit<KL>(upper, J0 + j, grp);
#pragma unroll
        for (int e = 0; e < DG / 2; ++e) {
            bq_fma<AXIS>(acc[J0 + j], q[j][e].y, up, x[j][2 * e]);
            bq_fma<AXIS>(acc[J0 + j], q[j][e].w, up, x[j][2 * e + 1]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);    // (bounds the registers of the reads in flight)
}

// second hits of column slot J
template <int KL, bool AXIS, int J, int CPG>
__device__ __forceinline__ void bq_column(float (&acc)[CPG][4], const BQMasks& M, const int2* pl,
                                          const char* __restrict__ lb, int grp) {
    if (bq_any<KL>(M.valid >> 8, J)) bq_apply<KL, AXIS, J, 1>(acc, pl, 1, lb, M.upper >> 8, grp);
}

// apply the pieces of magnitudes dd0 .. dd0 + DG - 1 (src0: the first
// one's place among those held): the first hits of the wave's columns, the
// second hits that there are, and the few second slices
template <int KL, bool AXIS, int... J>
__device__ __forceinline__ void bq_gather(float (&acc)[sizeof...(J)][4], const BQMasks& M, const int2* pl,
                                          const char* __restrict__ lb, int src0, int grp,
                                          std::integer_sequence<int, J...>) {
    constexpr int DG = bq_dg(KL), CPG = sizeof...(J), N = std::min(CPG, 4 / DG);
    static_assert(DG % 2 == 0 && CPG <= 2 * N, "pairs of magnitudes, at most two batches of columns");
    bq_apply<KL, AXIS, 0, N>(acc, pl, 0, lb, M.upper, grp);
    if constexpr (N < CPG) bq_apply<KL, AXIS, N, CPG - N>(acc, pl, 0, lb, M.upper, grp);
    // columns whose second hit lies on the other side of the centre
    const unsigned long long turn = (M.upper ^ (M.upper >> 8)) & (M.valid >> 8) & ~BQ_SECOND;
    if (M.valid & BQ_SECOND) {
        if (turn) (bq_swap(acc[J], bq_bit<KL>(turn, J, grp)), ...);
        (bq_column<KL, AXIS, J, CPG>(acc, M, pl, lb, grp), ...);
        if (turn) (bq_swap(acc[J], bq_bit<KL>(turn, J, grp)), ...);
    }
    constexpr unsigned long long LANES = ((1ull << DG) - 1) * 0x0101010101010101ull;
    if (M.split & (LANES << src0))
        ((bq_next<KL, AXIS, J>(acc[J], M, pl, lb, 0, src0, turn, grp),
          bq_next<KL, AXIS, J>(acc[J], M, pl, lb, 1, src0, turn, grp)), ...);
}

// The (angle, magnitude group) steps of entries [e0, e1) of the chunk's ne,
// whose hits are in sh, double buffered: the copies of step s + 1 run while
// step s is gathered (the first step's are under way).  cur: the buffer
// gathered next.
template <int KL, bool AXIS, int CPG>
__device__ __forceinline__ void bq_angles(const GeoK& g, const BP3QArgs& A, BP3QShared& sh, int e0, int e1, int ne, int c0,
                                          float (&acc)[CPG][4], unsigned long long& sw, int& cur, float4* s_w, int wave,
                                          int lane) {
    constexpr int DG = bq_dg(KL);
    constexpr auto COLS = std::make_integer_sequence<int, CPG>{};
    const int D = g.max_rd, nz = g.nz, NP = (g.n_radial + 1) / 2, grp = lane / KL;
    const long long dstep = (long long)NP * nz * 16;  // bytes of one magnitude
    const int2* pl = &sh.piece[wave][KL == 64 ? 0 : 2 * grp][0][0];
#pragma unroll 1
    for (int e = e0; e < e1; ++e) {
        const int plo = __builtin_amdgcn_readfirstlane(sh.plo[e]), nrow = __builtin_amdgcn_readfirstlane(sh.nrow[e]);
        const int al = __builtin_amdgcn_readfirstlane(sh.al[e]);
        const int en = min(e + 1, ne - 1);
        const int plon = __builtin_amdgcn_readfirstlane(sh.plo[en]), nrown = __builtin_amdgcn_readfirstlane(sh.nrow[en]);
        const int aln = __builtin_amdgcn_readfirstlane(sh.al[en]);
        const char* src = reinterpret_cast<const char*>(A.wq + ((long long)(c0 + al) * (D + 1) * NP + plo) * nz);
        const char* srcn = reinterpret_cast<const char*>(A.wq + ((long long)(c0 + aln) * (D + 1) * NP + plon) * nz);
        BQMasks M;
#pragma unroll 1
        for (int dd0 = 0; dd0 <= D; dd0 += DG) {
            const int src0 = dd0 % BQ_DC;
            if (src0 == 0) {
                bq_pieces<DG>(g, sh, e % BQ_E, dd0, nrow, wave, lane, M);
                bq_orient<KL>(acc, sw, M, AXIS && ((e - sh.n_oblique) & 1), grp, COLS);
            }
            const int ddn = dd0 + DG <= D ? dd0 + DG : 0;
            const bool more = ddn > 0 || e + 1 < ne;
            float4* nxt = s_w + (cur ? 0 : A.buf) + BQ_PAD;
            const char* lb = reinterpret_cast<const char*>(s_w + (cur ? A.buf : 0) + lane % KL);
            cur ^= 1;
            __builtin_amdgcn_s_waitcnt(0);      // this wave's copies have landed
            __syncthreads();                    // and every wave's; the other buffer is read no more
            if (more)
                bq_stage<DG>(nxt, ddn ? src + ddn * dstep : srcn, dstep, min(DG, D + 1 - ddn), (ddn ? nrow : nrown) * nz,
                         wave);
            bq_gather<KL, AXIS>(acc, M, pl + src0, lb, src0, grp, COLS);
        }
    }
}

template <int KL>
__device__ __forceinline__ void bp3q_body(const GeoK& g, const BP3QArgs& A, int vblock, BP3QShared& sh, float4* s_w) {
    constexpr int G = 64 / KL, CPG = BQ_W / G;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, grp = lane / KL;
    const int tiles_x = bq_tiles_x(g.nx);
    const int tx0 = (vblock % tiles_x) * BQ_X, ty0 = (vblock / tiles_x) * BQ_Y;
    const int Nr = g.n_radial, nz = g.nz, ncol = g.nx * g.ny;
    float acc[CPG][4], tot[CPG][2];
#pragma unroll
    for (int j = 0; j < CPG; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[j][q] = 0.0f;
        tot[j][0] = tot[j][1] = 0.0f;
    }
    const int kk = lane % KL, rev = grp * KL + max(0, nz - 1 - kk);    // the slice, the lane of the opposite one
    unsigned long long sw = 0;
    __syncthreads();    // (batched blocks: the staging area is read no more)
    if ((int)threadIdx.x < 2 * BQ_PAD)
        s_w[((int)threadIdx.x < BQ_PAD ? 0 : A.buf - BQ_PAD) + threadIdx.x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

#pragma unroll 1
    for (int c0 = 0; c0 < A.n_al; c0 += BQ_AMAX) {
        const int na = min(BQ_AMAX, A.n_al - c0);
        __syncthreads();    // the previous chunk's windows are read no more
        // (1) per angle of the chunk (one thread each): the bin pairs whose
        // rays meet the tile (the mirror tile meets the same pairs)
        if ((int)threadIdx.x < na) {
            const int q = threadIdx.x, a = A.angles[c0 + q];
            const AngleK& AK = g.ang[a];
            // (the tile's corner made anew per chunk: held across the steps, it
            // and what follows from it would cost registers)
            const int tx = __builtin_amdgcn_readfirstlane(tx0), ty = __builtin_amdgcn_readfirstlane(ty0);
            const double X0 = ((double)tx - 0.5 * g.nx) * g.vx, X1 = X0 + BQ_X * g.vx;
            const double Y0 = ((double)ty - 0.5 * g.ny) * g.vy, Y1 = Y0 + BQ_Y * g.vy;
            const double xa = X0 * AK.c, xb = X1 * AK.c, ya = Y0 * AK.s, yb = Y1 * AK.s;
            const double umin = fmin(xa, xb) + fmin(ya, yb), umax = fmax(xa, xb) + fmax(ya, yb);
            const int blo = (int)fmax(ceil(umin / g.ds + g.h0 - 1e-6), 0.0);
            const int bhi = (int)fmin(floor(umax / g.ds + g.h0 + 1e-6), (double)(Nr - 1));
            int plo = 0, n = 0;
            if (bhi >= blo) {
                const int mlo = Nr - 1 - bhi, mhi = Nr - 1 - blo;
                plo = min(blo, mlo);
                // both ends on one side of the centre, or the pairs up to it
                const int phi = bhi <= mlo ? bhi : (blo >= mhi ? mhi : (Nr - 1) / 2);
                n = min(phi - plo + 1, A.nr);
            }
            const bool axis = AK.Q == 0.0;
            const unsigned long long ax = __ballot(axis), ob = __ballot(!axis), below = (1ull << q) - 1;
            const int at = axis ? __popcll(ob) + 2 * __popcll(ax & below) : __popcll(ob & below);
            for (int u = 0; u < (axis ? 2 : 1); ++u) {
                sh.ang[at + u] = a;
                sh.al[at + u] = q;
                sh.plo[at + u] = plo;
                sh.nrow[at + u] = n;
            }
            if (q == 0) sh.n_oblique = __popcll(ob);
        }
        __syncthreads();
        // (2) the steps of its entries, the hits of four entries at a time
        const int nob = __builtin_amdgcn_readfirstlane(sh.n_oblique), ne = nob + 2 * (na - nob);
        int cur = 0;
        {
            const int plo = __builtin_amdgcn_readfirstlane(sh.plo[0]), nrow = __builtin_amdgcn_readfirstlane(sh.nrow[0]);
            const int al = __builtin_amdgcn_readfirstlane(sh.al[0]), D = g.max_rd, NP = (Nr + 1) / 2;
            bq_stage<bq_dg(KL)>(s_w + BQ_PAD,
                     reinterpret_cast<const char*>(A.wq + ((long long)(c0 + al) * (D + 1) * NP + plo) * nz),
                     (long long)NP * nz * 16, min(bq_dg(KL), D + 1), nrow * nz, wave);
        }
#pragma unroll 1
        for (int e0 = 0; e0 < ne; e0 += BQ_E) {
            if (e0 > 0) __syncthreads();    // the last entries' hits are read no more
            bq_hits(g, sh, e0, ne, tx0, ty0);
            __syncthreads();
            const int e1 = min(e0 + BQ_E, ne), em = min(max(nob, e0), e1);
            bq_angles<KL, false, CPG>(g, A, sh, e0, em, ne, c0, acc, sw, cur, s_w, wave, lane);
            bq_angles<KL, true, CPG>(g, A, sh, em, e1, ne, c0, acc, sw, cur, s_w, wave, lane);
            // (3) their sums: the two ends of each column added, to the
            // chunk's.  (In one chain through all of 10 angles with 10
            // magnitudes each the image was 1.34e-7 from 64-bit sums, 0.86e-7
            // so; k_bp3's four sums per column 0.89e-7.)
#pragma unroll
            for (int j = 0; j < CPG; ++j) {
                bq_swap(acc[j], bq_bit<KL>(sw, j, grp));
                tot[j][0] += acc[j][0] + __shfl(acc[j][1], rev);
                tot[j][1] += acc[j][3] + __shfl(acc[j][2], rev);
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[j][q] = 0.0f;
            }
            sw = 0;
        }
        // (4) the chunk's columns (later chunks add to what is there)
#pragma unroll
        for (int j = 0; j < CPG; ++j) {
            const int ix = tx0 + grp * CPG + j, col = (ty0 + wave) * g.nx + ix;
            if (ix < g.nx && 2 * col <= ncol - 1 && kk < nz) {
                float* o = A.out + (long long)col * nz + kk;
                float* om = A.out + (long long)(ncol - 1 - col) * nz + kk;
                if (c0 > 0 || A.add) {
                    tot[j][0] += *o;
                    tot[j][1] += *om;
                }
                *o = tot[j][0];
                if (2 * col != ncol - 1) *om = tot[j][1];
            }
            tot[j][0] = tot[j][1] = 0.0f;
        }
    }
}

// Tile of a block.  Blocks are dealt to the 8 XCDs round-robin; an XCD takes a
// run of the tiles as ordered here, in four strips of columns, row by row: a
// patch of about half a strip, whose tiles meet few bins of each angle, and as
// many tiles as the other XCDs.  False for the blocks past the last tile.
__host__ __device__ inline int bq_tiles_x(int nx) { return (nx + BQ_X - 1) / BQ_X; }
__host__ __device__ inline int bq_tiles_y(int ny) { return ((ny + 1) / 2 + BQ_Y - 1) / BQ_Y; }
__device__ __forceinline__ bool bq_tile(const GeoK& g, int block, int& tile) {
    const int tx = bq_tiles_x(g.nx), ty = bq_tiles_y(g.ny), n = tx * ty;
    const int i = (block % 8) * ((n + 7) / 8) + block / 8;
    const int w = (tx + 3) / 4, s = i / (w * ty), ws = min(w, tx - s * w), r = i - s * w * ty;
    tile = (r / max(ws, 1)) * tx + s * w + r % max(ws, 1);
    return block / 8 < (n + 7) / 8 && i < n;
}

// Bound by instruction issue: a piece costs one 16-byte LDS read and four FMAs,
// and about as many scalar and address instructions to choose it; HBM (the
// subset sinogram, once per tile row) and LDS stay below half their rates.
// Tiles of 4 x 4 column pairs with two magnitudes double buffered stay below
// 32 KB of LDS, so that five blocks of a CU hide each other's waits: four
// magnitudes at a time (three blocks) measured 171 us, this 117 (200x200x64,
// 281 bins, 8 angles, ring differences to 15, with the penalty blocks); the
// column tiles of k_bp3, which take every LOR by itself, 180.9.  With at most
// 32 slices four magnitudes fit, and half the barriers and copies in flight
// per piece: 41.0 -> 33.9 us (128x128x32, 185 bins, 9 angles, to 7).
//
// The first bp_blocks blocks back-project; A.n_pen more compute the penalty
// gradient and mu of the entering iterate (pen3_body, halo tile in the
// staging area).
//
// OCC blocks per CU: five, or four, whose registers hold the chunk's sums that
// five keep in scratch memory (with which a kernel starts 1 us later).
template <int KL, int OCC>
__global__ __launch_bounds__(NT, OCC) void k_bp3q(GeoK g, BP3QArgs A, int bp_blocks) {
    __shared__ BP3QShared sh;
    if ((int)blockIdx.x >= bp_blocks) {
        pen3_body(g, A.pen, (int)blockIdx.x - bp_blocks, reinterpret_cast<float*>(q_smem), sh.red);
        return;
    }
    int tile;
    if (!bq_tile(g, (int)blockIdx.x, tile)) return;
    bp3q_body<KL>(g, A, tile, sh, reinterpret_cast<float4*>(q_smem));
}

// ------------------------------------------------------------------ host side

// bin pairs of a tile's window at most: the whole bins in an interval of the
// tile's extent on the detector axis
static int bq_rows(const pet_os_geom* G) {
    const auto& d = G->d;
    const double ex = BQ_X * d.vx, ey = BQ_Y * d.vy;
    return std::min(q_pairs(d.n_radial), (int)std::floor(std::sqrt(ex * ex + ey * ey) / d.ds + 1e-5) + 1);
}

// (a lane past the last slice reads up to 63 - nz past a row)
static int bq_buf(const pet_os_geom* G) {
    return BQ_PAD + bq_dg(G->d.nz > 32 ? 64 : 32) * bq_rows(G) * G->d.nz + 64 - std::min(G->d.nz, 64);
}

size_t bp3q_lds(const pet_os_geom* G) {
    return std::max<size_t>(2 * (size_t)bq_buf(G) * sizeof(float4), PEN3_HALO * sizeof(float));
}

int bp3q_rows(const pet_os_geom* G) { return bq_rows(G); }
int bp3q_buf(const pet_os_geom* G) { return bq_buf(G); }

// The quad forward projector takes volumes of at most 64 slices (a lane per
// ring), unless k_fp3 is faster (fp3s_better); deeper ones keep the per-wave one.
bool fp3q_ok(const pet_os_geom* G) { return G->d.dim == 3 && G->d.nz <= 64; }

// The quad back-projector, and with it the quad layout of the weights, also
// asks that a column meets two bins of an angle at most (the bins of a window
// narrower than two: bins finer than 0.71 of a square voxel do not qualify),
// that the staged rows fit LDS, and that the layout's zeros (few unless nearly
// every ring pair is measured) keep the subset sinogram below 2.2 times its
// bins, and that its tiles and the image's make a launch (2^32 threads; an image
// of 2^28 columns takes half of them); other geometries keep the column tiles of
// k_bp3.  Where it qualifies it
// is the faster at every size and ring difference tried: 15.6 against 23.9 us
// at 60x59x12 to difference 1, 61.6 against 91.2 at 170x169x64 to 8.
bool quad_ok(const pet_os_geom* G) {
    const auto& d = G->d;
    return fp3q_ok(G) && std::sqrt(d.vx * d.vx + d.vy * d.vy) < 1.999 * d.ds &&
           2 * (size_t)bq_buf(G) * sizeof(float4) <= BQ_LDS_MAX &&
           5 * quad_floats(G, 1) <= 11 * (size_t)G->n_planes * d.n_radial && (int64_t)d.nx * d.ny <= (int64_t)1 << 28;
}

int fp3q_grid(const pet_os_geom* G, int n_al) { return fq_grid(G, n_al); }

int bp3q_grid(const pet_os_geom* G) { return 8 * ((bq_tiles_x(G->d.nx) * bq_tiles_y(G->d.ny) + 7) / 8); }

int launch_fp3q(const pet_os_geom* G, const FPLaunch& L, hipStream_t s) {
    FP3QArgs a;
    a.fz = L.fz;
    a.y = L.y;
    a.r = L.r;
    a.yr = L.yr;
    a.out = L.out;
    a.quad = L.quad;
    a.angles = L.angles;
    a.n_al = L.n_al;
    a.mode = L.mode;
    a.red = L.red;
    const int grid = fp3q_grid(G, L.n_al);
    if (L.mode == FP_OBJECTIVE && grid > L.red.cap) return fail(PET_OS_ERR_DEVICE, "objective partials too small");
    const size_t lds = fq_lds(G->d.nz);
    if (G->d.nz > 32) petos_launch(k_fp3q<64>, dim3(grid), dim3(FQ_W * 64), lds, s, G->k, a);
    else petos_launch(k_fp3q<32>, dim3(grid), dim3(FQ_W * 64), lds, s, G->k, a);
    PETOS_HIP(hipGetLastError());
    return PET_OS_OK;
}

// the back-projection's blocks and those of the penalty
static int bq_launch(const pet_os_geom* G, const BP3QArgs& a, hipStream_t s) {
    const int n = bp3q_grid(G);
    const dim3 blocks(n + a.n_pen), threads(NT);
    const size_t lds = bp3q_lds(G);
    if (G->d.nz > 32) petos_launch(k_bp3q<64, 5>, blocks, threads, lds, s, G->k, a, n);
    // Five blocks per CU where the tiles are more than four each and the LDS of
    // five is there (handed out by 1280 bytes of 160 KB): 10 angles of a
    // 200x199x24 image to difference 9 (1250 tiles) 81.2 and 103 us with five
    // and four, of 32 slices (four fit) 107.5 and 106.4, of a 127x125x29 image
    // (512 tiles) 61.3 and 60.4.
    else if (n > 4 * 256 && 5 * ((lds + sizeof(BP3QShared) + 1279) / 1280) <= 128)
        petos_launch(k_bp3q<32, 5>, blocks, threads, lds, s, G->k, a, n);
    else petos_launch(k_bp3q<32, 4>, blocks, threads, lds, s, G->k, a, n);
    PETOS_HIP(hipGetLastError());
    return PET_OS_OK;
}

int launch_bp3q(const pet_os_geom* G, const BPLaunch& L, hipStream_t s) {
    if ((L.f != nullptr) != (L.gradR != nullptr))
        return fail(PET_OS_ERR_DEVICE, "3D back-projection: the penalty blocks need both f and gradR");
    BP3QArgs a{};
    a.wq = reinterpret_cast<const float4*>(L.w);
    a.angles = L.angles;
    a.n_al = L.n_al;
    a.out = L.out;
    a.nr = bq_rows(G);
    a.buf = bq_buf(G);
    if (L.gradR != nullptr) {
        fill_pen3(L, a.pen);
        a.pen.gradR = L.gradR;
        a.n_pen = pen3_grid(G);
        if (L.want_mu && a.n_pen > L.red_mu.cap) return fail(PET_OS_ERR_DEVICE, "mu partials too small");
    }
    return bq_launch(G, a, s);
}

// ------------------------------------------------------------------ natural weights

// Back-projection of weights in the natural layout: the listed angles' weights
// are laid out as quads (k_pack3q), back-projected, and the image turned to its
// natural layout (k_turn3).  Both copies are bound by memory and take a few
// microseconds; k_bp3, which stages natural rows and takes every LOR by itself,
// took 102 us for 10 of 175 angles of a 127x125x29 image (181 bins, ring
// differences to 9), the three kernels 59 us (7 + 48 + 4).  Angles go in runs of at most
// BACK_QUADS bytes of quads, a multiple of the 16 whose sums are added together.
constexpr size_t BACK_QUADS = (size_t)64 << 20;

static int back3q_run(const pet_os_geom* G) {
    const size_t one = quad_floats(G, 1) * sizeof(float);
    return (int)std::max<size_t>(1, std::min<size_t>(4096, BACK_QUADS / one / BQ_AMAX)) * BQ_AMAX;
}

static size_t back3q_image(const pet_os_geom* G) { return ((size_t)G->n_vox * sizeof(float) + 255) & ~(size_t)255; }

size_t back3q_bytes(const pet_os_geom* G, int n_al) {
    return back3q_image(G) + quad_floats(G, std::min(n_al, back3q_run(G))) * sizeof(float);
}

constexpr int PQ_P = 32;        // bin pairs per block

__global__ __launch_bounds__(NT) void k_pack3q(GeoK g, const float* __restrict__ w, float4* __restrict__ wq,
                                               const int* __restrict__ angles) {
    float4* s_q = reinterpret_cast<float4*>(q_smem);        // [PQ_P][nz + 1]
    const int D = g.max_rd, Nr = g.n_radial, nz = g.nz, NP = (Nr + 1) / 2;
    const int p0 = blockIdx.x * PQ_P, d = blockIdx.y, al = blockIdx.z;
    const long long ab = (long long)angles[al] * Nr, plane = (long long)g.n_angles * Nr;
    const int pp = g.plane_base[D + d], pn = g.plane_base[D - d], c = threadIdx.x % PQ_P, p = p0 + c;
    if (p < NP) {
        const float* lo = w + ab + p;
        const float* hi = w + ab + (Nr - 1 - p);
        for (int k = threadIdx.x / PQ_P; k < nz; k += NT / PQ_P) {
            float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            const int kr = nz - 1 - d - k;
            if (kr >= 0) {
                q.x = lo[(pp + k) * plane];
                q.z = hi[(pp + kr) * plane];
                if (d > 0) {
                    q.y = lo[(pn + kr) * plane];
                    q.w = hi[(pn + k) * plane];
                }
            }
            s_q[c * (nz + 1) + k] = q;
        }
    }
    __syncthreads();
    float4* out = wq + (((long long)al * (D + 1) + d) * NP + p0) * nz;
    const int n = min(PQ_P, NP - p0) * nz;
    for (int e = threadIdx.x; e < n; e += NT) out[e] = s_q[e + e / nz];
}

// out (natural) from z (z fastest), or z + beta out, tiles of 32 x 32 (a block
// per row y, TURN_Y of them along the grid's y, which holds 65535)
constexpr int TURN_Y = 32768;
__global__ __launch_bounds__(NT) void k_turn3(const float* __restrict__ z, float* __restrict__ out, int nx, int ny,
                                              int nz, int add, float beta) {
    __shared__ float s_t[32][33];
    const int tz = (nz + 31) / 32, z0 = (blockIdx.z % tz) * 32, y = (blockIdx.z / tz) * TURN_Y + blockIdx.y;
    const int x0 = blockIdx.x * 32, l = threadIdx.x % 32;
    if (y >= ny) return;
    for (int k = threadIdx.x / 32; k < 32; k += NT / 32)
        if (x0 + k < nx && z0 + l < nz) s_t[k][l] = z[((long long)y * nx + x0 + k) * nz + z0 + l];
    __syncthreads();
    for (int k = threadIdx.x / 32; k < 32; k += NT / 32)
        if (x0 + l < nx && z0 + k < nz) {
            float* o = out + ((long long)(z0 + k) * ny + y) * nx + x0 + l;
            *o = add ? fmaf(beta, *o, s_t[l][k]) : s_t[l][k];
        }
}

int launch_turn3(const pet_os_geom* G, const float* z, float* out, const float* beta, hipStream_t s) {
    const auto& d = G->d;
    const int rows = std::min(d.ny, TURN_Y), turns = (d.ny + TURN_Y - 1) / TURN_Y;
    hipLaunchKernelGGL(k_turn3, dim3((d.nx + 31) / 32, rows, (d.nz + 31) / 32 * turns), dim3(NT), 0, s, z, out, d.nx, d.ny, d.nz,
                       beta != nullptr, beta != nullptr ? *beta : 0.0f);
    PETOS_HIP(hipGetLastError());
    return PET_OS_OK;
}

int launch_back3q(const pet_os_geom* G, const BPLaunch& L, void* scratch, hipStream_t s) {
    const auto& d = G->d;
    float* img = reinterpret_cast<float*>(scratch);
    float4* wq = reinterpret_cast<float4*>((char*)scratch + back3q_image(G));
    const int run = back3q_run(G);
    for (int a0 = 0; a0 < L.n_al; a0 += run) {
        BP3QArgs a{};
        a.wq = wq;
        a.angles = L.angles + a0;
        a.n_al = std::min(run, L.n_al - a0);
        a.out = img;
        a.nr = bq_rows(G);
        a.buf = bq_buf(G);
        a.add = a0 > 0;
        // (a grid's z holds 65535 blocks, a run at most 65536 angles: by halves)
        for (int h = 0; h < a.n_al; h += 32768) {
            const int na = std::min(32768, a.n_al - h);
            hipLaunchKernelGGL(k_pack3q, dim3((q_pairs(d.n_radial) + PQ_P - 1) / PQ_P, d.max_ring_diff + 1, na), dim3(NT),
                               (size_t)PQ_P * (d.nz + 1) * sizeof(float4), s, G->k, L.w,
                               wq + quad_floats(G, h) / 4, a.angles + h);
        }
        const int rc = bq_launch(G, a, s);
        if (rc) return rc;
    }
    return launch_turn3(G, img, L.out, nullptr, s);
}

// ------------------------------------------------------------------ batched (persistent) kernels

template <int KL>
__global__ __launch_bounds__(FQ_W * 64, 4) void k_fp3q_batch(const SlotDev* __restrict__ S,
                                                                const Item* __restrict__ items,
                                                                const int* __restrict__ count, int step) {
    const int n = *count;
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const Item I = items[it];
        const SlotDev& d = S[I.slot];
        const int J = d.J + step;
        if (!(d.active && J <= d.J_end)) continue;
        const int i = (J - 1) % d.g.n_subsets;
        FP3QArgs A{};
        A.fz = d.fz;
        A.y = d.y;
        A.r = d.r;
        A.out = d.w;
        A.quad = d.quad;
        A.angles = d.subset_lists + (long long)i * d.max_sub;
        A.n_al = d.subset_count[i];
        A.mode = FP_RATIO;
        // (the list is made for the largest subset)
        const int per_angle = ((d.g.n_radial + 1) / 2) * fq_chunks(d.g.max_rd);
        if (I.block < A.n_al * per_angle) fp3q_body<KL>(d.g, A, I.block, q_smem);
        __syncthreads();
    }
}

template <int KL>
__global__ __launch_bounds__(NT, 5) void k_bp3q_batch(const SlotDev* __restrict__ S, const Item* __restrict__ items,
                                                      const int* __restrict__ count, int step) {
    __shared__ BP3QShared sh;
    const int n = *count;
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const Item I = items[it];
        const SlotDev& d = S[I.slot];
        int tile;
        const int J = d.J + step;
        if (!(d.active && J <= d.J_end) || !bq_tile(d.g, I.block, tile)) continue;
        const int i = (J - 1) % d.g.n_subsets;
        BP3QArgs A{};
        A.wq = reinterpret_cast<const float4*>(d.w);
        A.angles = d.subset_lists + (long long)i * d.max_sub;
        A.n_al = d.subset_count[i];
        A.out = d.G;
        A.nr = d.rows_max;
        A.buf = d.chunk;
        bp3q_body<KL>(d.g, A, tile, sh, reinterpret_cast<float4*>(q_smem));
        __syncthreads();
    }
}

void launch_batch3q_fp(const SlotDev* d_slots, const Item* list, const int* cnt, int grid, int step, int kl,
                       hipStream_t s) {
    if (kl == 64)
        hipLaunchKernelGGL((k_fp3q_batch<64>), dim3(grid), dim3(FQ_W * 64), fq_lds(64), s, d_slots, list, cnt, step);
    else
        hipLaunchKernelGGL((k_fp3q_batch<32>), dim3(grid), dim3(FQ_W * 64), fq_lds(32), s, d_slots, list, cnt, step);
}

void launch_batch3q_bp(const SlotDev* d_slots, const Item* list, const int* cnt, int grid, int step, int kl, size_t lds,
                       hipStream_t s) {
    if (kl == 64) hipLaunchKernelGGL((k_bp3q_batch<64>), dim3(grid), dim3(NT), lds, s, d_slots, list, cnt, step);
    else hipLaunchKernelGGL((k_bp3q_batch<32>), dim3(grid), dim3(NT), lds, s, d_slots, list, cnt, step);
}

}  // namespace petos
