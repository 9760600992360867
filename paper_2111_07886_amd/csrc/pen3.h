// pen3.h -- the image-space part of a 3D subiteration (penalty gradient and
// smoothness measure), shared by the back-projectors' launches and k_pen3.
#pragma once
#include "devutil.h"
#include "internal.h"

namespace petos {

// The image-space part of a 3D subiteration: grad R(f) (eqn:gradRD, 26
// in-image neighbours), either added after the back-projection b = A_i^T w
// as G = b + (beta/M) grad R(f) in place over b, or (gradR given) stored on
// its own for the update to add, so that it can run in the back-projector's
// launch; with want_mu the smoothness measure mu = max(0.01, |grad f| /
// mean f) (Sec. III-B) with the block's FP64 partial of sum mu.  One block
// per 32 (x) x 8 (y) x 8 (z) voxels (a thread per (x, y), eight slices
// each); f with a one-voxel halo in LDS.
constexpr int PEN3_X = 32, PEN3_Y = 8, PEN3_Z = 8;
constexpr int PEN3_HALO = (PEN3_X + 2) * (PEN3_Y + 2) * (PEN3_Z + 2);   // floats of the halo tile

struct Pen3Args {
    const float* f;
    float* G;                // in: b, out: G (gradR null)
    int g_zfast;             // G is z-fastest
    float* gradR;            // non-null: grad R(f) goes here and G is left alone
    float* mu;
    int want_mu;
    float beta_over_M, gamma_R, eps;
    const double* part_f;    // partials of sum f of the entering iterate (mean f)
    int n_part_f;
    Reduction red_mu;
};

__host__ __device__ inline int pen3_tiles(int n, int t) { return (n + t - 1) / t; }

// s_f: PEN3_HALO floats of LDS, s_red: NT / 64 doubles
__device__ inline void pen3_body(const GeoK& g, const Pen3Args& A, int vblock, float* s_f, double* s_red) {
    constexpr int HX = PEN3_X + 2, HY = PEN3_Y + 2, HZ = PEN3_Z + 2;
    const int tx = pen3_tiles(g.nx, PEN3_X), ty = pen3_tiles(g.ny, PEN3_Y);
    const int x0 = (vblock % tx) * PEN3_X, y0 = ((vblock / tx) % ty) * PEN3_Y, z0 = (vblock / (tx * ty)) * PEN3_Z;
    for (int e = threadIdx.x; e < HX * HY * HZ; e += NT) {
        const int hx = e % HX, hy = (e / HX) % HY, hz = e / (HX * HY);
        const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
        float v = 0.0f;
        if (gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny && gz >= 0 && gz < g.nz)
            v = A.f[((long long)gz * g.ny + gy) * g.nx + gx];
        s_f[e] = v;
    }
    float meanf = 1.0f;
    if (A.want_mu) meanf = (float)(sum_partials(A.part_f, A.n_part_f, s_red) / (double)g.nvox);
    __syncthreads();
    const int lx = threadIdx.x % PEN3_X, ly = threadIdx.x / PEN3_X;
    const int ix = x0 + lx, iy = y0 + ly;
    double mu_part = 0.0;
    if (ix < g.nx && iy < g.ny) {
        // The thread's column, slice by slice, with the 3x3 neighbourhood of
        // three slices in registers (one new slice read from LDS per step)
        // and the out-of-image neighbours masked instead of branched around
        // (the 26 in-image neighbours of eqn:gradRD, in stencil_at's order).
        const bool okx[3] = {ix > 0, true, ix < g.nx - 1};
        const bool oky[3] = {iy > 0, true, iy < g.ny - 1};
        const float gR = A.gamma_R, eps = A.eps;
        float pl[3][9];     // slices lz - 1, lz, lz + 1 of the halo tile (hz = lz .. lz + 2)
        auto load = [&](float (&p)[9], int hz) {
#pragma unroll
            for (int q = 0; q < 9; ++q) p[q] = s_f[(hz * HY + ly + q / 3) * HX + lx + q % 3];
        };
        load(pl[0], 0);
        load(pl[1], 1);
        const long long colz = ((long long)iy * g.nx + ix) * g.nz;
#pragma unroll
        for (int lz = 0; lz < PEN3_Z; ++lz) {
            const int iz = z0 + lz;
            if (iz >= g.nz) break;
            float (&pm)[9] = pl[lz % 3];
            float (&pc)[9] = pl[(lz + 1) % 3];
            float (&pp)[9] = pl[(lz + 2) % 3];
            load(pp, lz + 2);
            const bool okz[3] = {iz > 0, true, iz < g.nz - 1};
            const float fj = pc[4], fje = fj + eps, fj2e = fj + 2.0f * eps;
            float acc = 0.0f;
#pragma unroll
            for (int dz = 0; dz < 3; ++dz) {
                const float* p = dz == 0 ? pm : (dz == 1 ? pc : pp);
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    if (dz == 1 && q == 4) continue;
                    const RdpPair t = rdp_pair(fj, fje, fj2e, p[q], gR);
                    // an out-of-image neighbour adds 0
                    acc = fmaf(t.num, (okz[dz] && oky[q / 3] && okx[q % 3]) ? t.rden : 0.0f, acc);
                }
            }
            const float gradR = 2.0f * acc;
            const float gx = mat_der(ix, g.nx, pc[5], fj, pc[3]);
            const float gy = mat_der(iy, g.ny, pc[7], fj, pc[1]);
            const float gz = mat_der(iz, g.nz, pp[4], fj, pm[4]);
            const float gmag = sqrtf(gx * gx + gy * gy + gz * gz);
            const long long j = ((long long)iz * g.ny + iy) * g.nx + ix;
            if (A.gradR != nullptr) A.gradR[j] = gradR;
            else {
                float* G = A.G + (A.g_zfast ? colz + iz : j);
                *G = fmaf(A.beta_over_M, gradR, *G);
            }
            if (A.want_mu) {
                const float mu = fmaxf(0.01f, gmag / meanf);
                A.mu[j] = mu;
                mu_part += (double)mu;
            }
        }
    }
    if (A.want_mu) write_partial(mu_part, A.red_mu, s_red, vblock);
}

// the launch's penalty inputs (G, gradR and the layouts are the caller's)
inline void fill_pen3(const BPLaunch& L, Pen3Args& a) {
    a = Pen3Args{};
    a.f = L.f;
    a.mu = L.mu;
    a.want_mu = L.want_mu;
    a.beta_over_M = L.beta_over_M;
    a.gamma_R = L.gamma_R;
    a.eps = L.eps;
    a.part_f = L.part_f;
    a.n_part_f = L.n_part_f;
    a.red_mu = L.red_mu;
}

}  // namespace petos
