// HIP kernels and C ABI of the spectral-element right-hand-side library
// (gfx950).  See include/sem.h for the contract of every entry point.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <algorithm>
#include <array>
#include <cstring>
#include <memory>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "adapt.h"
#include "handle.h"
#include "nodeval.h"
#include "rows.h"

namespace sem {
std::string& last_error() {
    thread_local std::string msg;
    return msg;
}
}  // namespace sem

namespace {

using sem::fail;
constexpr int NF = SEM_NFIELDS;

}  // namespace

using sem::DevMesh;

// ====================================================================== kernels
namespace sem {

__global__ void k_nc_scatter(DevMesh m, const double* __restrict__ src, double* __restrict__ dst) {
    const int64_t n = int64_t(m.n_hh) * m.nzn;
    const int64_t fs = int64_t(m.n_h) * m.ldz, fsh = int64_t(m.n_hh) * m.ldz;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int hh = int(t / m.nzn), kz = int(t % m.nzn);
        double s[NF] = {0, 0, 0, 0, 0};
        for (int r = m.hang_ptr[hh]; r < m.hang_ptr[hh + 1]; ++r) {
            const double w = m.hang_w[r];
            const int64_t base = int64_t(m.hang_src[r]) * m.ldz + kz;
#pragma unroll
            for (int f = 0; f < NF; ++f) s[f] += w * src[f * fs + base];
        }
        const int64_t o = int64_t(hh) * m.ldz + kz;
#pragma unroll
        for (int f = 0; f < NF; ++f) dst[f * fsh + o] = s[f];
    }
}

__global__ void k_nc_gather(DevMesh m, const double* __restrict__ src, double* __restrict__ dst) {
    const int64_t n = int64_t(m.n_hT) * m.nzn;
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    const int64_t fsh = int64_t(m.n_hh) * m.ldz;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int li = int(t / m.nzn), kz = int(t % m.nzn);
        const int h = m.hT_list[li];
        double s[NF] = {0, 0, 0, 0, 0};
        for (int r = m.hT_ptr[li]; r < m.hT_ptr[li + 1]; ++r) {
            const double w = m.hT_w[r];
            const int64_t base = int64_t(m.hT_hh[r]) * m.ldz + kz;
#pragma unroll
            for (int f = 0; f < NF; ++f) s[f] += w * src[f * fsh + base];
        }
        const int64_t o = int64_t(h) * m.ldz + kz;
#pragma unroll
        for (int f = 0; f < NF; ++f) dst[f * fs + o] += s[f];
    }
}

// Element right-hand side: a workgroup takes up to LZ stacked elements of a
// column, a thread per local node.  Their rows are loaded once, kz fastest, into
// tiles shared by the elements; (u, v), (w, theta') and (rho, p') are read in
// pairs by the six sums of each direction.
// Two-level mesh over 64 x 64 x 8 elements at N = 4: 132 us, 0.35 GB read and
// written (145 with two layers per workgroup, 179 with one); 208 with a
// workgroup per element, rows of 40 bytes and eight tiles read one by one.  The
// rest is LDS reads (45 of 16 bytes per node) and latency at 4 waves per SIMD.
template <int NP>
constexpr int rhs_layers() {
    return NP == 2 ? 16 : NP <= 5 ? 4 : 1;
}
// The instance (LZ = 1, 2, 4, 8, 16, at most rhs_layers) for n_z layers.  Threads
// of empty layers hold their registers, and a chunk costs the same however full
// it is: N = 3 and 4 take the largest LZ that divides n_z, two for odd numbers of
// five and more.  us with 8, 4, 2 and 1 layers per workgroup at N = 3, 107 x 137 x
// 2 elements and two levels 127, 75, 57, 81, 64 x 64 x 9 74, 49, 48, 57, 64 x 64 x
// 16 84, 76, 79, 105; with 4, 2 and 1 at N = 4, 128 x 128 x 1 96, 66, 59, 100 x
// 100 x 3 99, 92, 87, 64 x 64 x 5 83, 59, 68, x 9 130, 109, 115; with 2 and 1 at N
// = 5, 64 x 64 x 8 290, 202.  Where a layer is 8 or 27 threads a chunk costs about
// four layers (N = 1) or half a one (N = 2) more than its own: N = 1, 128 x 128 x
// 16 with 16, 8 and 4 33, 38, 53, x 20 67, 51, 75, 160 x 160 x 5 32, 25, 43; N = 2,
// 160 x 160 x 3 with 8, 4, 2 and 1 77, 52, 62, 77, 128 x 128 x 5 61, 67, 55, 78.
template <int NP>
int rhs_pick(int n_z) {
    if constexpr (NP > 3) return std::min(rhs_layers<NP>(), n_z % 2 == 0 ? n_z & -n_z : n_z < 5 ? 1 : 2);
    auto cost = [&](int lz) { return (n_z + lz - 1) / lz * (2 * lz + (NP == 2 ? 8 : 1)); };
    int best = rhs_layers<NP>();
    for (int lz = best; lz >= 1; lz /= 2)
        if (cost(lz) < cost(best)) best = lz;
    return best;
}
template <int NP, int LZ>
constexpr int rhs_threads() {
    return (LZ * NP * NP * NP + 63) / 64 * 64;
}
template <int NP, int LZ, typename T>
__global__ void __launch_bounds__((rhs_threads<NP, LZ>()))
k_rhs(DevMesh m, const double* __restrict__ q, const double* __restrict__ hv,
      double* __restrict__ rE) {
    using T2 = std::conditional_t<sizeof(T) == 8, double2, float2>;
    constexpr int NP2 = NP * NP, NP3 = NP2 * NP, N = NP - 1;
    constexpr int RT = rhs_threads<NP, LZ>(), ST = (LZ * N + 1) | 1;
    __shared__ T2 t_uv[NP2 * ST], t_wt[NP2 * ST], t_rp[NP2 * ST];
    __shared__ T t_r[NP2 * ST];           // rho'
    __shared__ T sD[NP2];
    __shared__ double s_zs[NP2];          // terrain: surface height per position
    const int nc = (m.n_z + LZ - 1) / LZ, c = int(blockIdx.x) / nc;
    const int l0 = (int(blockIdx.x) - c * nc) * LZ, nl = min(LZ, m.n_z - l0), nk = nl * N + 1, z0 = l0 * N;
    const int tid = threadIdx.x;
    const int64_t fs = int64_t(m.n_h) * m.ldz, fsh = int64_t(m.n_hh) * m.ldz;
    const int64_t fsr = int64_t(m.n_h + m.n_hh) * m.ldz;   // terrain reference rows
    const bool ter = m.zs != nullptr;
    for (int x = tid; x < NP2; x += RT) {
        sD[x] = T(m.D[x]);
        if (ter) {
            const int gz = m.gmap[c * NP2 + x];
            s_zs[x] = m.zs[gz >= 0 ? gz : m.n_h - gz - 1];
        }
    }
    for (int n = tid; n < NP2 * nk; n += RT) {
        const int pos = n / nk, kl = n - pos * nk, kz = z0 + kl;
        const int g = m.gmap[c * NP2 + pos];
        const double* src = g >= 0 ? q + int64_t(g) * m.ldz + kz : hv + int64_t(-g - 1) * m.ldz + kz;
        const int64_t st = g >= 0 ? fs : fsh;
        double x[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) x[f] = src[f * st];
        // reference state: per vertical node, or per node with terrain (the
        // hanging rows hold the coarse face's interpolant)
        double r0, ir0, ith0, p0;
        if (ter) {
            const int64_t o = int64_t(g >= 0 ? g : m.n_h - g - 1) * m.ldz + kz;
            r0 = m.ref_n[o];
            ir0 = m.ref_n[fsr + o];
            ith0 = m.ref_n[2 * fsr + o];
            p0 = m.ref_n[3 * fsr + o];
        } else {
            r0 = m.rho0[kz];
            ir0 = m.inv_rho0[kz];
            ith0 = m.inv_theta0[kz];
            p0 = m.p0[kz];
        }
        // p' = p0 ((1 + rho'/rho0)(1 + theta'/theta0))^gamma - p0: the
        // ideal-gas pressure minus the reference pressure, free of
        // cancellation; in FP64 for both precisions, rounded once (the
        // hydrostatic balance in the w tendency cancels most of dp'/dz)
        const double ra = x[0] * ir0, tb = x[4] * ith0;
        double pp;
        if constexpr (sizeof(T) == 8) pp = p0 * pow1p_minus1(m, ra + tb + ra * tb);
        else pp = p0 * expm1(m.gamma * (log1p(ra) + log1p(tb)));
        const int o = pos * ST + kl;
        t_uv[o] = T2{T(x[1]), T(x[2])};
        t_wt[o] = T2{T(x[3]), T(x[4])};
        t_rp[o] = T2{T(r0) + T(x[0]), T(pp)};
        t_r[o] = T(x[0]);
    }
    __syncthreads();
    const int lay = tid / NP3, t = tid - lay * NP3;
    if (lay >= nl) return;
    const int layer = l0 + lay;
    const int i = t % NP, j = (t / NP) % NP, k = t / NP2;
    const int kl = lay * N + k, kz = z0 + kl, o = (i + NP * j) * ST + kl;
    const T sx = T(2.0 / m.col_dx[c]), sy = T(2.0 / m.col_dy[c]), sz = T(2.0 / m.dz[layer]);
    // derivatives along each direction: of the momentum of its own velocity
    // (over terrain of every velocity along z), u, v, w, p', theta'
    T ru[3] = {0, 0, 0}, d[5][3];
    T rz[2] = {0, 0};                     // d(rho u)/dz, d(rho v)/dz, for terrain
#pragma unroll
    for (int a = 0; a < 5; ++a) d[a][0] = d[a][1] = d[a][2] = 0;
#pragma unroll
    for (int mm = 0; mm < NP; ++mm) {
        const int oo[3] = {(mm + NP * j) * ST + kl, (i + NP * mm) * ST + kl, (i + NP * j) * ST + lay * N + mm};
        const T dm[3] = {sD[i * NP + mm], sD[j * NP + mm], sD[k * NP + mm]};
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
            const T2 uv = t_uv[oo[dir]], wt = t_wt[oo[dir]], rp = t_rp[oo[dir]];
            ru[dir] += dm[dir] * (rp.x * (dir == 0 ? uv.x : dir == 1 ? uv.y : wt.x));
            d[0][dir] += dm[dir] * uv.x;
            d[1][dir] += dm[dir] * uv.y;
            d[2][dir] += dm[dir] * wt.x;
            d[3][dir] += dm[dir] * rp.y;
            d[4][dir] += dm[dir] * wt.y;
        }
    }
    const T s3[3] = {sx, sy, sz};
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
        ru[dir] *= s3[dir];
#pragma unroll
        for (int a = 0; a < 5; ++a) d[a][dir] *= s3[dir];
    }
    // terrain-following mapping: d/dx = box d/dx + a_x d/dzf, d/dy likewise,
    // d/dz = g_s d/dzf (g_s = 1/(1 - zs/(H - z0)), a_x = -g_s (H - zf)/(H - z0) dzs/dx)
    double mfac = 1.0;
    if (ter) {
        double zx = 0.0, zy = 0.0;
        for (int mm = 0; mm < NP; ++mm) {
            zx += m.D[i * NP + mm] * s_zs[mm + NP * j];
            zy += m.D[j * NP + mm] * s_zs[i + NP * mm];
            const int oz = (i + NP * j) * ST + lay * N + mm;
            rz[0] += sD[k * NP + mm] * (t_rp[oz].x * t_uv[oz].x);
            rz[1] += sD[k * NP + mm] * (t_rp[oz].x * t_uv[oz].y);
        }
        mfac = 1.0 - s_zs[i + NP * j] * m.inv_depth;
        const double gs = 1.0 / mfac, tg = m.tfac[kz] * gs;
        const T ax = T(-tg * zx * m.col_sx[c]), ay = T(-tg * zy * m.col_sy[c]);
        ru[0] += ax * (rz[0] * sz);
        ru[1] += ay * (rz[1] * sz);
        ru[2] *= T(gs);
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            d[a][0] += ax * d[a][2];
            d[a][1] += ay * d[a][2];
            d[a][2] *= T(gs);
        }
    }
    const T2 uv = t_uv[o];
    const T u = uv.x, v = uv.y, w = t_wt[o].x, rho = t_rp[o].x, rho_p = t_r[o];
    const T f = T(m.f), g = T(m.g);
    const T inv_rho = T(1) / rho;
    double dth0 = ter ? 0.0 : m.dth0[kz];
    if (ter) {
        const int gn = m.gmap[c * NP2 + i + NP * j];
        dth0 = m.ref_n[4 * fsr + int64_t(gn >= 0 ? gn : m.n_h - gn - 1) * m.ldz + kz];
    }
    T R[NF];
    R[0] = -(ru[0] + ru[1] + ru[2]);
    R[1] = -(u * d[0][0] + v * d[0][1] + w * d[0][2]) - d[3][0] * inv_rho + f * v;
    R[2] = -(u * d[1][0] + v * d[1][1] + w * d[1][2]) - d[3][1] * inv_rho - f * u;
    R[3] = -(u * d[2][0] + v * d[2][1] + w * d[2][2]) - d[3][2] * inv_rho - rho_p * inv_rho * g;
    R[4] = -(u * d[4][0] + v * d[4][1] + w * d[4][2]) - w * T(dth0);
    const double mass = m.w[i] * m.w[j] * m.w[k] * 0.125 * m.col_dx[c] * m.col_dy[c] * m.dz[layer] * mfac;
    const int64_t es = int64_t(m.n_col) * m.n_z * NP3;
    const int64_t e = int64_t(c) * m.n_z + layer;
#pragma unroll
    for (int fld = 0; fld < NF; ++fld) rE[fld * es + e * NP3 + t] = mass * double(R[fld]);
}

// Sub-grid and absorbing-layer tendencies of one element, times the lumped
// mass (the paper's model setup, Section 5): horizontal Smagorinsky-Lilly,
//   R_u += d/dx(2 nu S_xx) + d/dy(2 nu S_xy), and likewise for v (S_yx, S_yy)
//   and w (S_zx, S_zy), nu = (C_s Delta)^2 sqrt(2 S:S), Delta = (dx+dy)/(2N),
// with S from the element-local velocity derivatives; and the Rayleigh layer,
// R_f -= R(kz) q'_f for every field.  accumulate = true adds to rE (the
// unfused element right-hand side), false overwrites it; col selects the
// column-row layout of rE (see sum_local).
// stacked elements of one column per workgroup (about 500 threads)
template <int NP>
constexpr int dissip_layers() { return NP * NP * NP <= 125 ? 4 : (NP * NP * NP <= 343 ? 2 : 1); }

template <int NP>
__global__ void __launch_bounds__(((dissip_layers<NP>() * NP * NP * NP + 63) / 64) * 64)
k_dissip(DevMesh m, const double* __restrict__ q, const double* __restrict__ hv,
         double* __restrict__ rE, bool accumulate, bool col) {
    constexpr int NP2 = NP * NP, NP3 = NP2 * NP;
    constexpr int N = NP - 1;
    constexpr int L = dissip_layers<NP>(), NPL = L * NP3;
    __shared__ double sv[3][NPL];       // u, v, w of the L elements
    __shared__ double st[5][NPL];       // 2 nu (S_xx, S_xy, S_yy, S_xz, S_yz)
    __shared__ double sD[NP2];
    __shared__ double s_zs[NP2];        // terrain: surface height per position
    const int nzb = (m.n_z + L - 1) / L;
    const int c = blockIdx.x / nzb, layer0 = (blockIdx.x - c * nzb) * L;
    const int t = threadIdx.x;
    if (t < NP2) sD[t] = m.D[t];
    // node of this thread, k fastest, then the element of the stack (vertical
    // runs of the state and of the column-row output are contiguous); tl is
    // its index in the LDS tiles, el * NP3 + the element-local index
    const int k = t % NP, el = (t / NP) % L, i = (t / (NP * L)) % NP, j = t / (NP * L * NP);
    const int layer = layer0 + el;
    const bool active = t < NPL && layer < m.n_z;
    const int e = c * m.n_z + layer;
    const int eo = el * NP3;
    const int tl = eo + i + NP * (j + NP * k);
    const int kz = layer * N + k;
    const int64_t fs = int64_t(m.n_h) * m.ldz, fsh = int64_t(m.n_hh) * m.ldz;
    const bool ter = m.zs != nullptr;
    if (ter && t < NP2) {
        const int gz = m.gmap[c * NP2 + t];
        s_zs[t] = m.zs[gz >= 0 ? gz : m.n_h - gz - 1];
    }
    double x[NF] = {0, 0, 0, 0, 0};
    if (active) {
        const int g = m.gmap[c * NP2 + i + NP * j];
        if (g >= 0) {
#pragma unroll
            for (int f = 0; f < NF; ++f) x[f] = q[f * fs + int64_t(g) * m.ldz + kz];
        } else {
#pragma unroll
            for (int f = 0; f < NF; ++f) x[f] = hv[f * fsh + int64_t(-g - 1) * m.ldz + kz];
        }
        sv[0][tl] = x[1];
        sv[1][tl] = x[2];
        sv[2][tl] = x[3];
    }
    __syncthreads();
    const double sx = 2.0 / m.col_dx[c], sy = 2.0 / m.col_dy[c], sz = active ? 2.0 / m.dz[layer] : 0.0;
    // terrain-following mapping: d/dx = box d/dx + a_x d/dzf, d/dy likewise,
    // d/dz = g_s d/dzf (g_s = 1/(1 - zs/(H - z0)), a_x = -g_s (H - zf)/(H - z0) dzs/dx);
    // the lumped mass gains 1/g_s
    double ax = 0.0, ay = 0.0, gs = 1.0, mfac = 1.0;
    if (ter && active) {
        double zx = 0.0, zy = 0.0;
        for (int mm = 0; mm < NP; ++mm) {
            zx += sD[i * NP + mm] * s_zs[mm + NP * j];
            zy += sD[j * NP + mm] * s_zs[i + NP * mm];
        }
        mfac = 1.0 - s_zs[i + NP * j] * m.inv_depth;
        gs = 1.0 / mfac;
        const double tg = m.tfac[kz] * gs;
        ax = -tg * zx * sx;
        ay = -tg * zy * sy;
    }
    double R[NF] = {0, 0, 0, 0, 0};
    const bool sgs = m.cs > 0.0;
    if (sgs && active) {
        double g3[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};   // g3[a][b] = d(u_a)/d(x_b)
        for (int mm = 0; mm < NP; ++mm) {
            const double dxm = sD[i * NP + mm], dym = sD[j * NP + mm], dzm = sD[k * NP + mm];
            const int ox = eo + mm + NP * (j + NP * k), oy = eo + i + NP * (mm + NP * k),
                      oz = eo + i + NP * (j + NP * mm);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                g3[a][0] += dxm * sv[a][ox];
                g3[a][1] += dym * sv[a][oy];
                g3[a][2] += dzm * sv[a][oz];
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) { g3[a][0] *= sx; g3[a][1] *= sy; g3[a][2] *= sz; }
        if (ter) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                g3[a][0] += ax * g3[a][2];
                g3[a][1] += ay * g3[a][2];
                g3[a][2] *= gs;
            }
        }
        const double sxx = g3[0][0], syy = g3[1][1], szz = g3[2][2];
        const double sxy = 0.5 * (g3[0][1] + g3[1][0]);
        const double sxz = 0.5 * (g3[0][2] + g3[2][0]);
        const double syz = 0.5 * (g3[1][2] + g3[2][1]);
        const double ss = sxx * sxx + syy * syy + szz * szz + 2.0 * (sxy * sxy + sxz * sxz + syz * syz);
        const double delta = (m.col_dx[c] + m.col_dy[c]) / (2.0 * N);
        const double cd = m.cs * delta;
        const double two_nu = 2.0 * cd * cd * sqrt(2.0 * ss);
        st[0][tl] = two_nu * sxx;
        st[1][tl] = two_nu * sxy;
        st[2][tl] = two_nu * syy;
        st[3][tl] = two_nu * sxz;
        st[4][tl] = two_nu * syz;
    }
    __syncthreads();
    if (!active) return;
    if (sgs) {
        double dx_[5] = {0, 0, 0, 0, 0}, dy_[5] = {0, 0, 0, 0, 0}, dz_[5] = {0, 0, 0, 0, 0};
        for (int mm = 0; mm < NP; ++mm) {
            const double dxm = sD[i * NP + mm], dym = sD[j * NP + mm], dzm = sD[k * NP + mm];
            const int ox = eo + mm + NP * (j + NP * k), oy = eo + i + NP * (mm + NP * k),
                      oz = eo + i + NP * (j + NP * mm);
#pragma unroll
            for (int a = 0; a < 5; ++a) {
                dx_[a] += dxm * st[a][ox];
                dy_[a] += dym * st[a][oy];
                if (ter) dz_[a] += dzm * st[a][oz];
            }
        }
        // physical d/dx and d/dy of the stresses (box part plus the mapping's)
        double tx[5], ty[5];
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            tx[a] = dx_[a] * sx + ax * (dz_[a] * sz);
            ty[a] = dy_[a] * sy + ay * (dz_[a] * sz);
        }
        R[1] = tx[0] + ty[1];
        R[2] = tx[1] + ty[2];
        R[3] = tx[3] + ty[4];
    }
    if (m.sponge) {
        double rz = m.sponge[kz];
        if (ter) {
            // the layer at the node's physical height z = H - t_f (H - z0 - zs)
            const double zp = m.z_top - m.tfac[kz] * (m.depth - s_zs[i + NP * j]);
            rz = 0.0;
            if (zp >= m.z_top - m.sp_depth) {
                const double sn = sin(0.5 * M_PI * (1.0 - (m.z_top - zp) / m.sp_depth));
                rz = fmin(1.0, fmax(0.0, m.sp_gamma * sn * sn));
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) R[f] -= rz * x[f];
    }
    const double mass = m.w[i] * m.w[j] * m.w[k] * 0.125 * m.col_dx[c] * m.col_dy[c] * m.dz[layer] * mfac;
    const int64_t es = int64_t(m.n_col) * m.n_z * NP3;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int64_t o = f * es + (col ? (int64_t(c) * NP2 + i + NP * j) * (int64_t(m.n_z) * NP) + layer * NP + k
                                        : int64_t(e) * NP3 + (tl - eo));
        rE[o] = (accumulate ? rE[o] : 0.0) + mass * R[f];
    }
}

// sum of element contributions at the local copies of (slot-list, kz)
// rE layouts: element-local [F][elem][k][j][i] (col = false, the sem_rhs /
// sem_dss layout), or column rows [F][col][pos][layer][k] (col = true, the
// dissipation pre-pass's own buffer), where consecutive kz are contiguous.
__device__ __forceinline__ void sum_local(const DevMesh& m, const double* __restrict__ rE,
                                          const int* __restrict__ slots, int s0, int s1, int kz,
                                          double* out, bool col) {
    const int np1 = m.N + 1, np2 = np1 * np1, np3 = np2 * np1;
    const int64_t es = int64_t(m.n_col) * m.n_z * np3;
    int lay[2], kk[2], nv = 0;
    if (kz % m.N == 0 && kz > 0 && kz < m.nzn - 1) {
        lay[0] = kz / m.N - 1; kk[0] = m.N;
        lay[1] = kz / m.N;     kk[1] = 0;
        nv = 2;
    } else {
        lay[0] = (kz == m.nzn - 1) ? m.n_z - 1 : kz / m.N;
        kk[0] = kz - lay[0] * m.N;
        nv = 1;
    }
    for (int f = 0; f < NF; ++f) out[f] = 0.0;
    for (int s = s0; s < s1; ++s) {
        const int slot = slots[s];
        const int c = slot / np2, pos = slot - c * np2;
        for (int a = 0; a < nv; ++a) {
            const int64_t idx = col ? (int64_t(c) * np2 + pos) * (int64_t(m.n_z) * np1) + lay[a] * np1 + kk[a]
                                    : int64_t(c * m.n_z + lay[a]) * np3 + pos + np2 * kk[a];
#pragma unroll
            for (int f = 0; f < NF; ++f) out[f] += rE[f * es + idx];
        }
    }
}

// a thread per node and level: from column rows (the dissipation pre-pass), and
// at N = 1 from the element layout too, whose lanes' doubles are 64 bytes apart
// there (128 x 128 x 20 elements and a level 116 us, 177 by k_assemble_elem, whose
// levels are all between two elements; from N = 2 that one is ahead)
__global__ void k_assemble(DevMesh m, const double* __restrict__ rE, double* __restrict__ acc, bool col) {
    const int64_t n = int64_t(m.n_h) * m.nzn;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int h = int(t / m.nzn), kz = int(t % m.nzn);
        double s[NF];
        sum_local(m, rE, m.asm_slot, m.asm_ptr[h], m.asm_ptr[h + 1], kz, s, col);
        const int64_t o = int64_t(h) * m.ldz + kz, fs = int64_t(m.n_h) * m.ldz;
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f * fs + o] = s[f];
    }
}

__global__ void k_assemble_hang(DevMesh m, const double* __restrict__ rE, double* __restrict__ cH, bool col) {
    const int64_t n = int64_t(m.n_hh) * m.nzn;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int hh = int(t / m.nzn), kz = int(t % m.nzn);
        double s[NF];
        sum_local(m, rE, m.asmH_slot, m.asmH_ptr[hh], m.asmH_ptr[hh + 1], kz, s, col);
        const int64_t o = int64_t(hh) * m.ldz + kz, fsh = int64_t(m.n_hh) * m.ldz;
#pragma unroll
        for (int f = 0; f < NF; ++f) cH[f * fsh + o] = s[f];
    }
}

// Assembly from the element layout of rE (position fastest): a workgroup takes
// ASM_H horizontal nodes, a lane each, and ASM_K levels, a quarter per wave, so
// that consecutive lanes read the consecutive positions of an element's plane
// and a level's elements are the same for a whole wave (the quarter of what is
// left in rows shorter than that: 107 x 137 x 2 elements at N = 3 73 to 65 us, 160
// x 160 x 1 at N = 2 24 to 20); the sums (in
// sum_local's order) are turned through LDS into rows, one 128-byte line per
// node and field.
// Bound by memory and the latency of the chain node - slots - planes: two-level
// mesh over 64 x 64 x 8 elements at N = 4, 0.35 GB read and written, 132 us (149
// with the workgroups dealt to the XCDs in turn); 264 with a thread per node
// and level, kz fastest, whose lanes read one double of a 200-byte plane each.
constexpr int ASM_H = 64, ASM_K = 16;
__global__ void __launch_bounds__(256)
k_assemble_elem(DevMesh m, const double* __restrict__ rE, double* __restrict__ acc) {
    constexpr int Q = ASM_K / 4;
    __shared__ double tile[NF][ASM_H][ASM_K + 1];
    const int np1 = m.N + 1, np2 = np1 * np1, np3 = np2 * np1;
    const int64_t es = int64_t(m.n_col) * m.n_z * np3, fs = int64_t(m.n_h) * m.ldz;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the workgroups of one XCD take contiguous nodes, bottom to top
    const int n_kb = (m.nzn + ASM_K - 1) / ASM_K, G = gridDim.x, xcd = blockIdx.x & 7;
    const int b = xcd * (G >> 3) + min(xcd, G & 7) + (int(blockIdx.x) >> 3);
    const int h0 = b / n_kb * ASM_H, kz0 = b % n_kb * ASM_K;
    const int nq = (min(ASM_K, m.nzn - kz0) + 3) / 4;      // levels per wave
    const int h = h0 + lane;
    double s[Q][NF];
#pragma unroll
    for (int k = 0; k < Q; ++k)
#pragma unroll
        for (int f = 0; f < NF; ++f) s[k][f] = 0.0;
    if (h < m.n_h)
        for (int r = m.asm_ptr[h]; r < m.asm_ptr[h + 1]; ++r) {
            const int slot = m.asm_slot[r], c = slot / np2;
            const double* base = rE + int64_t(c) * m.n_z * np3 + (slot - c * np2);
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                const int kz = kz0 + wave * nq + k;
                if (k >= nq || kz >= m.nzn) break;
                const int el = kz / m.N, kk = kz - el * m.N;
                if (kk == 0 && el > 0)
#pragma unroll
                    for (int f = 0; f < NF; ++f) s[k][f] += base[f * es + int64_t(el - 1) * np3 + m.N * np2];
                if (el < m.n_z)
#pragma unroll
                    for (int f = 0; f < NF; ++f) s[k][f] += base[f * es + int64_t(el) * np3 + kk * np2];
            }
        }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int k = 0; k < Q; ++k)
            if (k < nq) tile[f][lane][wave * nq + k] = s[k][f];
    __syncthreads();
    const int kl = threadIdx.x % ASM_K, kz = kz0 + kl;
    if (kz < m.nzn)
        for (int r = threadIdx.x / ASM_K; r < ASM_H && h0 + r < m.n_h; r += 256 / ASM_K)
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f * fs + int64_t(h0 + r) * m.ldz + kz] = tile[f][r][kl];
}

// r = M_G^-1 acc at unique node (h, kz), then the boundary rules: rigid lids;
// with terrain the surface keeps only the tangential part of the momentum
// tendency
__device__ __forceinline__ void finalize_node(const DevMesh& m, int h, int kz, double* v) {
    const bool ter = m.zs != nullptr;
    const double minv = (ter ? m.minv_ht[h] : m.minv_h[h]) * m.minv_v[kz];
    const bool lid = ter ? (kz == m.nzn - 1) : (kz == 0 || kz == m.nzn - 1);
#pragma unroll
    for (int f = 0; f < NF; ++f) v[f] *= minv;
    if (ter && kz == 0) {
        const double n0 = m.nrm[h], n1 = m.nrm[m.n_h + h], n2 = m.nrm[2 * m.n_h + h];
        const double dn = v[1] * n0 + v[2] * n1 + v[3] * n2;
        v[1] -= dn * n0;
        v[2] -= dn * n1;
        v[3] -= dn * n2;
    }
    if (lid) v[3] = 0.0;
}

__global__ void k_finalize(DevMesh m, const double* __restrict__ acc, double* __restrict__ r) {
    const int64_t n = int64_t(m.n_h) * m.nzn;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int h = int(t / m.nzn), kz = int(t % m.nzn);
        const int64_t o = int64_t(h) * m.ldz + kz, fs = int64_t(m.n_h) * m.ldz;
        double v[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f] = acc[f * fs + o];
        finalize_node(m, h, kz, v);
#pragma unroll
        for (int f = 0; f < NF; ++f) r[f * fs + o] = v[f];
    }
}

// assemble and finalize in one pass, for meshes without hanging points (no
// Z^T contribution has to arrive between the two), from column rows
__global__ void k_assemble_finalize(DevMesh m, const double* __restrict__ rE, double* __restrict__ r) {
    const int64_t n = int64_t(m.n_h) * m.nzn;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int h = int(t / m.nzn), kz = int(t % m.nzn);
        double v[NF];
        sum_local(m, rE, m.asm_slot, m.asm_ptr[h], m.asm_ptr[h + 1], kz, v, true);
        finalize_node(m, h, kz, v);
        const int64_t o = int64_t(h) * m.ldz + kz, fs = int64_t(m.n_h) * m.ldz;
#pragma unroll
        for (int f = 0; f < NF; ++f) r[f * fs + o] = v[f];
    }
}

__global__ void k_update(int64_t n, double a, double b, double c, const double* qn,
                         const double* qs, const double* r, double* qout) {
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n;
         t += int64_t(gridDim.x) * blockDim.x)
        qout[t] = a * qn[t] + b * qs[t] + c * r[t];
}

struct Thr { double v[SEM_MAX_LEVEL]; };

// Refinement flag of every element (element pass of nodeval.h).  6,220 columns
// of 8 layers at N = 4: 40 us; 87 with a workgroup per element.
template <int NP>
__global__ void __launch_bounds__(pass_threads<NP>())
k_amr_elem(DevMesh m, const double* __restrict__ q, int criterion, Thr thr, int lvl_max,
           int8_t* __restrict__ adapt) {
    constexpr int NP2 = NP * NP, N = NP - 1;
    constexpr int PT = pass_threads<NP>(), ST = pass_stride<NP>();
    __shared__ double2 t_uv[NP2 * ST];
    __shared__ double t_w[NP2 * ST], red[PT];
    __shared__ double sD[NP2], s_zs[NP2];     // s_zs, terrain: surface height per position
    const PassItem it = pass_item<NP>(m);
    const int c = it.c, nk = it.layers * N + 1, z0 = it.layer0 * N, tid = threadIdx.x;
    const bool speed = criterion == SEM_CRIT_SPEED;
    for (int x = tid; x < NP2; x += PT) {
        sD[x] = m.D[x];
        if (m.zs) {
            const int gz = m.gmap[c * NP2 + x];
            s_zs[x] = m.zs[gz >= 0 ? gz : m.n_h - gz - 1];
        }
    }
    for (int x = tid; x < NP2 * nk; x += PT) {
        const int pos = x / nk, kl = x - pos * nk;
        const int g = m.gmap[c * NP2 + pos];
        double a[2];
        node_values<1, 2>(m, q, g, z0 + kl, a);
        t_uv[pos * ST + kl] = double2{a[0], a[1]};
        if (speed) t_w[pos * ST + kl] = node_value(m, q, g, 3, z0 + kl);
    }
    __syncthreads();
    // maximum of the criterion over a position's nodes (of its square for the
    // speed: the root keeps their order)
    double C = -INFINITY;
    const int lay = tid / NP2, p = tid - lay * NP2;
    if (lay < it.layers) {
        const int i = p % NP, j = p / NP;
        const double sx = 2.0 / m.col_dx[c], sy = 2.0 / m.col_dy[c], sz = 2.0 / m.dz[it.layer0 + lay];
        double zx = 0, zy = 0;
        if (m.zs)
            for (int mm = 0; mm < NP; ++mm) {
                zx += sD[i * NP + mm] * s_zs[mm + NP * j];
                zy += sD[j * NP + mm] * s_zs[i + NP * mm];
            }
#pragma unroll 1
        for (int k = 0; k < NP; ++k) {
            const int kl = lay * N + k, o = p * ST + kl;
            if (speed) {
                const double2 uv = t_uv[o];
                const double w = t_w[o];
                C = fmax(C, uv.x * uv.x + uv.y * uv.y + w * w);
                continue;
            }
            double vx = 0, uy = 0;
#pragma unroll
            for (int mm = 0; mm < NP; ++mm) {
                vx += sD[i * NP + mm] * t_uv[(mm + NP * j) * ST + kl].y;
                uy += sD[j * NP + mm] * t_uv[(i + NP * mm) * ST + kl].x;
            }
            double z = vx * sx - uy * sy;
            if (m.zs) {
                // terrain-following mapping: d/dx = box d/dx + a_x d/dzf, d/dy likewise
                double vz = 0, uz = 0;
                for (int mm = 0; mm < NP; ++mm) {
                    const double2 uv = t_uv[p * ST + lay * N + mm];
                    vz += m.D[k * NP + mm] * uv.y;
                    uz += m.D[k * NP + mm] * uv.x;
                }
                const double tg = m.tfac[z0 + kl] / (1.0 - s_zs[p] * m.inv_depth);
                const double ax = -tg * zx * sx, ay = -tg * zy * sy;
                z += ax * vz * sz - ay * uz * sz;
            }
            C = fmax(C, z);
        }
    }
    red[tid] = C;
    __syncthreads();
    if (tid < it.layers) {
        double cm = red[tid * NP2];
        for (int n = 1; n < NP2; ++n) cm = fmax(cm, red[tid * NP2 + n]);
        if (speed && cm >= 0.0) cm = sqrt(cm);
        const int lv = m.col_level[c];
        int8_t flag = 0;
        if (lv < lvl_max && cm > thr.v[lv]) flag = 1;
        else if (lv > 0 && cm <= thr.v[lv - 1]) flag = -1;
        adapt[c * m.n_z + it.layer0 + tid] = flag;
    }
}

__global__ void k_amr_col(DevMesh m, const int8_t* __restrict__ ae, int8_t* __restrict__ ac) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= m.n_col) return;
    ac[c] = column_rule(m, ae, c);
}

// Solution transfer between two meshes with the same vertical structure:
// every row (new horizontal node) is a weighted sum of old horizontal nodes,
// applied to the whole vertical row of each field.  A thread per row and pair
// of levels, kz fastest, takes all five fields: a row's table entries are read
// once, and five independent 16-byte loads are in flight per old node (the
// arrays need no more than their doubles' alignment).  The padding entries kz
// in [nzn, ldz) are written as zero.
// Most rows copy one node, but where columns split or merge a row sums 25 to
// several hundred: one thread's chain of loads over such a row sets the time
// of the whole pass.  The first n_long workgroups take one such row each (more
// than TRANSFER_SHORT nodes), its nodes divided among groups of threads whose
// sums are added in the groups' order.
// 100,344 rows of 33 levels at N = 4 (94 % copies, 3 % of 25 nodes, 1 % of 72 to
// 285): 93 us, of which 71 are the short rows at 4.6 TB/s; 187 with a thread
// per long row too; 236 with a wave per row and field.  Rows of 25 and fewer
// are cheaper in a thread's unrolled chain than in a workgroup (102 us with
// the line at 8, 93 at 30 and 48, 96 at 72).
constexpr int TRANSFER_SHORT = 32;
__global__ void __launch_bounds__(256)
k_transfer(const int32_t* __restrict__ ptr, const int32_t* __restrict__ src,
           const double* __restrict__ w, const int32_t* __restrict__ long_rows, int n_long, int64_t n_rows,
           int64_t n_h_from, int nzn, int ldz, const double* __restrict__ qa, double* __restrict__ qb) {
    using vec = double __attribute__((ext_vector_type(2), aligned(8)));
    __shared__ vec part[SEM_NFIELDS][256];
    const unsigned L = unsigned(ldz) / 2;             // threads of a row
    const int64_t fsa = n_h_from * ldz, fsb = n_rows * ldz;
    auto sum = [&](int r, int r1, int k, vec* acc) {
#pragma unroll
        for (int f = 0; f < SEM_NFIELDS; ++f) acc[f] = vec(0.0);
#pragma unroll 4
        for (; r < r1; ++r) {
            const double wr = w[r];
            const double* q = qa + int64_t(src[r]) * ldz + level_pair(k, nzn);
#pragma unroll
            for (int f = 0; f < SEM_NFIELDS; ++f) acc[f] += wr * *reinterpret_cast<const vec*>(q + f * fsa);
        }
    };
    auto put = [&](int64_t h, int k, int f, vec v) {
        if (k + 1 == nzn) v = vec{v[1], 0.0};             // (level_pair)
        *reinterpret_cast<vec*>(qb + f * fsb + h * ldz + k) = v;
    };
    if (int(blockIdx.x) < n_long) {
        const int h = long_rows[blockIdx.x];
        const int r0 = ptr[h], n = ptr[h + 1] - r0;
        // G groups of `lanes` threads; more than one pass over the levels
        // only in rows of more than 512 levels
        const int lanes = min(int(L), 256), G = 256 / lanes;
        const int g = int(threadIdx.x) / lanes, lane = int(threadIdx.x) - g * lanes;
        for (int k0 = 0; k0 < int(L); k0 += lanes) {
            const int k = (k0 + lane) * 2;
            const bool mine = g < G && k < ldz;
            vec acc[SEM_NFIELDS];
            const bool some = mine && k < nzn;
            sum(some ? r0 + int(int64_t(n) * g / G) : 0, some ? r0 + int(int64_t(n) * (g + 1) / G) : 0, k, acc);
#pragma unroll
            for (int f = 0; f < SEM_NFIELDS; ++f) part[f][threadIdx.x] = acc[f];
            __syncthreads();
            if (mine)
                for (int f = g; f < SEM_NFIELDS; f += G) {
                    vec s = part[f][lane];
                    for (int x = 1; x < G; ++x) s += part[f][x * lanes + lane];
                    put(h, k, f, s);
                }
            __syncthreads();
        }
        return;
    }
    const int64_t t0 = int64_t(blockIdx.x - n_long) * 256, first = t0 / L;
    const unsigned x = unsigned(t0 - first * L) + threadIdx.x, dh = x / L;
    const int64_t h = first + dh;
    if (h >= n_rows) return;
    const int k = int(x - dh * L) * 2, r0 = ptr[h], r1 = ptr[h + 1];
    if (r1 - r0 > TRANSFER_SHORT) return;
    vec acc[SEM_NFIELDS];
    sum(r0, k < nzn ? r1 : r0, k, acc);
#pragma unroll
    for (int f = 0; f < SEM_NFIELDS; ++f) put(h, k, f, acc[f]);
}

}  // namespace sem

// ====================================================================== helpers
namespace {

int grid_for(int64_t n, int block = 256) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return int(g);
}

template <int NP, typename T, int LZ = sem::rhs_layers<NP>()>
void launch_rhs_k(const DevMesh& d, int lz, const double* q, const double* hv, double* rE, hipStream_t s) {
    if constexpr (LZ > 1)
        if (lz < LZ) return launch_rhs_k<NP, T, LZ / 2>(d, lz, q, hv, rE, s);
    hipLaunchKernelGGL((sem::k_rhs<NP, LZ, T>), dim3(unsigned(d.n_col) * ((d.n_z + LZ - 1) / LZ)),
                       dim3(sem::rhs_threads<NP, LZ>()), 0, s, d, q, hv, rE);
}

template <typename T>
int launch_rhs_t(const sem_mesh* M, const double* q, const double* hv, double* rE, hipStream_t s) {
    const DevMesh& d = M->d;
    switch (d.N) {
#define CASE(NN)                                                                             \
    case NN:                                                                                 \
        launch_rhs_k<NN + 1, T>(d, sem::rhs_pick<NN + 1>(d.n_z), q, hv, rE, s);              \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
        default: return fail(SEM_ERR_N, "unsupported N");
    }
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int check_mesh(const sem_mesh* M) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!M->have_ref && !M->d.zs)
        return fail(SEM_ERR_STATE, "sem_mesh_set_reference has not been called");
    return SEM_OK;
}


}  // namespace

// m * (sub-grid + absorbing-layer tendency) of every element into rE
// (added to what is there when accumulate is true), in the element layout or
// in column rows (col)
int launch_dissip(const sem_mesh* M, const double* q, const double* hv, double* rE, bool accumulate,
                  bool col, hipStream_t s) {
    const DevMesh& d = M->d;
    switch (d.N) {
#define CASE(NN)                                                                                  \
    case NN: {                                                                                    \
        constexpr int L = sem::dissip_layers<NN + 1>();                                           \
        const int nb = d.n_col * ((d.n_z + L - 1) / L);                                           \
        hipLaunchKernelGGL((sem::k_dissip<NN + 1>), dim3(nb),                                     \
                           dim3(((L * (NN + 1) * (NN + 1) * (NN + 1) + 63) / 64) * 64), 0, s, d, q, \
                           hv, rE, accumulate, col);                                              \
        break;                                                                                    \
    }
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
        default: return fail(SEM_ERR_N, "unsupported N");
    }
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

bool dissipation_on(const sem_mesh* M) { return M->d.cs > 0.0 || M->d.sponge != nullptr; }

static int sem_launch_rhs(const sem_mesh* M, const double* q, const double* hv, double* rE, int prec,
                   hipStream_t s) {
    int rc;
    if (prec == SEM_FP64) rc = launch_rhs_t<double>(M, q, hv, rE, s);
    else if (prec == SEM_FP32) rc = launch_rhs_t<float>(M, q, hv, rE, s);
    else return fail(SEM_ERR_ARG, "precision must be SEM_FP64 or SEM_FP32");
    if (rc == SEM_OK && dissipation_on(M)) rc = launch_dissip(M, q, hv, rE, true, false, s);
    return rc;
}

// dissipation tendency of q per unique node (M^-1 Z^T m R_dissip, lid rule)
// into the handle's buffer, read by the fused stage
int dissip_prepass(const sem_mesh* M, const double* q, hipStream_t s) {
    const DevMesh& d = M->d;
    const double* hv = nullptr;
    if (d.n_hh > 0) {
        hipLaunchKernelGGL(sem::k_nc_scatter, dim3(grid_for(int64_t(d.n_hh) * d.nzn)), dim3(256), 0, s, d, q,
                           M->diss_c);
        hv = M->diss_c;
    }
    // the pre-pass's own element buffer in column rows: the assembly then
    // reads consecutive kz from consecutive addresses
    int rc = launch_dissip(M, q, hv, M->diss_rE, false, true, s);
    if (rc != SEM_OK) return rc;
    if (d.n_hh == 0) {
        hipLaunchKernelGGL(sem::k_assemble_finalize, dim3(grid_for(int64_t(d.n_h) * d.nzn)), dim3(256), 0, s, d,
                           M->diss_rE, M->diss_r);
        HIPCHK(hipGetLastError());
        return SEM_OK;
    }
    hipLaunchKernelGGL(sem::k_assemble, dim3(grid_for(int64_t(d.n_h) * d.nzn)), dim3(256), 0, s, d, M->diss_rE,
                       M->diss_acc, true);
    hipLaunchKernelGGL(sem::k_assemble_hang, dim3(grid_for(int64_t(d.n_hh) * d.nzn)), dim3(256), 0, s, d,
                       M->diss_rE, M->diss_c, true);
    hipLaunchKernelGGL(sem::k_nc_gather, dim3(grid_for(int64_t(d.n_hT) * d.nzn)), dim3(256), 0, s, d,
                       M->diss_c, M->diss_acc);
    hipLaunchKernelGGL(sem::k_finalize, dim3(grid_for(int64_t(d.n_h) * d.nzn)), dim3(256), 0, s, d, M->diss_acc,
                       M->diss_r);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

// ====================================================================== C ABI
extern "C" {

const char* sem_last_error(void) { return sem::last_error().c_str(); }

static int sem_mesh_create_impl(const sem_mesh_desc* desc, sem_mesh** out) {
    if (!desc || !out) return fail(SEM_ERR_ARG, "null argument");
    *out = nullptr;
    sem::MeshInput in{desc->N, desc->nx0, desc->ny0, desc->n_z, desc->n_col,
                      desc->h_col_level, desc->h_col_ix, desc->h_col_iy, desc->Lx, desc->Ly,
                      desc->h_z_edges, desc->periodic_x != 0, desc->periodic_y != 0,
                      desc->f, desc->g, desc->R_d, desc->c_p, desc->p00};
    std::unique_ptr<sem_mesh> M(new sem_mesh());
    std::string err;
    int rc = sem::build_host_mesh(in, M->host, err);
    if (rc != SEM_OK) return fail(rc, err);
    const sem::HostMesh& H = M->host;
    DevMesh& d = M->d;
    d.N = H.N; d.n_z = H.n_z; d.nzn = H.nzn; d.ldz = H.ldz; d.n_col = H.n_col;
    d.n_h = int(H.n_h); d.n_hh = int(H.n_hh); d.n_hT = int(H.hT_list.size());
    d.f = H.f; d.g = H.g;
    d.gamma = H.c_p / (H.c_p - H.R_d);
    {
        // C(gamma, n) by the product rule in extended precision
        long double cgam = (long double)H.c_p / ((long double)H.c_p - (long double)H.R_d);
        long double cn = 1.0L;
        d.binom[0] = 1.0;
        for (int n = 1; n <= 10; ++n) {
            cn *= (cgam - (long double)(n - 1)) / (long double)n;
            d.binom[n] = (double)cn;
        }
    }
#define UP(vec, field) if ((rc = M->upload(vec, &d.field)) != SEM_OK) return rc;
    UP(H.gmap, gmap) UP(H.col_dx, col_dx) UP(H.col_dy, col_dy) UP(H.dz, dz)
    UP(H.col_sx, col_sx) UP(H.col_sy, col_sy) UP(H.sz, sz)
    UP(H.hang_ptr, hang_ptr) UP(H.hang_src, hang_src) UP(H.hang_w, hang_w)
    UP(H.hT_list, hT_list) UP(H.hT_ptr, hT_ptr) UP(H.hT_hh, hT_hh) UP(H.hT_w, hT_w)
    UP(H.asm_ptr, asm_ptr) UP(H.asm_slot, asm_slot) UP(H.asmH_ptr, asmH_ptr)
    UP(H.asmH_slot, asmH_slot) UP(H.minv_h, minv_h) UP(H.minv_v, minv_v)
    UP(H.sib, sib) UP(H.col_level, col_level) UP(H.basis.D, D) UP(H.basis.w, w)
    UP(H.nbr_ptr, nbr_ptr) UP(H.nbr_col, nbr_col)
#undef UP
    if ((rc = M->upload(H.h_xy, &M->d_hxy)) != SEM_OK) return rc;
    HIPCHK(hipMalloc(&M->wind_part, sizeof(double) * 256));
    HIPCHK(hipMalloc(&M->feat_aux, sizeof(double) * 2 * size_t(std::max<int64_t>(1, int64_t(H.n_col) * H.n_z))));
    M->ws_bytes += int64_t(sizeof(double)) * 2 * int64_t(H.n_col) * H.n_z;
    if ((rc = sem::fused_plan_build(H, SEM_LAYOUT_COLUMNS, 0, M->fused, true)) != SEM_OK)
        return fail(rc, "could not build the fused-stage tables");
    *out = M.release();
    return SEM_OK;
}

int sem_mesh_create(const sem_mesh_desc* desc, sem_mesh** out) {
    return sem::guarded("sem_mesh_create", [&] { return sem_mesh_create_impl(desc, out); });
}

static int sem_mesh_plan_impl(const sem_mesh_desc* desc, sem_mesh_info* o, double* hxy, double* hhxy, double* z,
                  double* mass) {
    if (!desc || !o) return fail(SEM_ERR_ARG, "null argument");
    sem::MeshInput in{desc->N, desc->nx0, desc->ny0, desc->n_z, desc->n_col,
                      desc->h_col_level, desc->h_col_ix, desc->h_col_iy, desc->Lx, desc->Ly,
                      desc->h_z_edges, desc->periodic_x != 0, desc->periodic_y != 0,
                      desc->f, desc->g, desc->R_d, desc->c_p, desc->p00};
    sem::HostMesh H;
    std::string err;
    int rc = sem::build_host_mesh(in, H, err);
    if (rc != SEM_OK) return fail(rc, err);
    o->N = H.N; o->n_z = H.n_z; o->nzn = H.nzn; o->ldz = H.ldz; o->max_level = H.max_level;
    o->n_col = H.n_col; o->n_elem = int64_t(H.n_col) * H.n_z;
    o->n_h = H.n_h; o->n_hh = H.n_hh;
    o->n_dof = H.n_h * H.nzn; o->n_hang = H.n_hh * H.nzn;
    o->n_local = o->n_elem * H.np1 * H.np1 * H.np1;
    o->workspace_bytes = 0;
    if (hxy) std::memcpy(hxy, H.h_xy.data(), H.h_xy.size() * sizeof(double));
    if (hhxy) std::memcpy(hhxy, H.hh_xy.data(), H.hh_xy.size() * sizeof(double));
    if (z) std::memcpy(z, H.zn.data(), H.zn.size() * sizeof(double));
    if (mass)
        for (int64_t h = 0; h < H.n_h; ++h)
            for (int kz = 0; kz < H.nzn; ++kz)
                mass[h * H.nzn + kz] = 1.0 / (H.minv_h[h] * H.minv_v[kz]);
    return SEM_OK;
}

int sem_mesh_plan(const sem_mesh_desc* desc, sem_mesh_info* o, double* hxy, double* hhxy, double* z,
                  double* mass) {
    return sem::guarded("sem_mesh_plan", [&] { return sem_mesh_plan_impl(desc, o, hxy, hhxy, z, mass); });
}

int sem_mesh_destroy(sem_mesh* mesh) {
    if (!mesh) return fail(SEM_ERR_ARG, "null mesh");
    delete mesh;
    return SEM_OK;
}

int sem_mesh_get_info(const sem_mesh* M, sem_mesh_info* o) {
    if (!M || !o) return fail(SEM_ERR_ARG, "null argument");
    const sem::HostMesh& H = M->host;
    o->N = H.N; o->n_z = H.n_z; o->nzn = H.nzn; o->ldz = H.ldz; o->max_level = H.max_level;
    o->n_col = H.n_col; o->n_elem = int64_t(H.n_col) * H.n_z;
    o->n_h = H.n_h; o->n_hh = H.n_hh;
    o->n_dof = H.n_h * H.nzn; o->n_hang = H.n_hh * H.nzn;
    o->n_local = o->n_elem * H.np1 * H.np1 * H.np1;
    o->workspace_bytes = M->ws_bytes + M->fused.bytes;
    return SEM_OK;
}

static int sem_mesh_coords_impl(const sem_mesh* M, double* hxy, double* hhxy, double* z) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    const sem::HostMesh& H = M->host;
    if (hxy) std::memcpy(hxy, H.h_xy.data(), H.h_xy.size() * sizeof(double));
    if (hhxy) std::memcpy(hhxy, H.hh_xy.data(), H.hh_xy.size() * sizeof(double));
    if (z) std::memcpy(z, H.zn.data(), H.zn.size() * sizeof(double));
    return SEM_OK;
}

int sem_mesh_coords(const sem_mesh* M, double* hxy, double* hhxy, double* z) {
    return sem::guarded("sem_mesh_coords", [&] { return sem_mesh_coords_impl(M, hxy, hhxy, z); });
}

static int sem_mesh_set_reference_impl(sem_mesh* M, const double* rho0, const double* theta0,
                           const double* dth0) {
    if (!M || !rho0 || !theta0 || !dth0) return fail(SEM_ERR_ARG, "null argument");
    const sem::HostMesh& H = M->host;
    std::vector<double> r(rho0, rho0 + H.nzn), t(theta0, theta0 + H.nzn), dt(dth0, dth0 + H.nzn),
        p0(H.nzn), ir(H.nzn), it(H.nzn);
    const double gam = H.c_p / (H.c_p - H.R_d);
    for (int k = 0; k < H.nzn; ++k) {
        if (!(r[k] > 0) || !(t[k] > 0)) return fail(SEM_ERR_ARG, "reference state must be positive");
        p0[k] = H.p00 * std::pow(H.R_d * r[k] * t[k] / H.p00, gam);
        ir[k] = 1.0 / r[k];
        it[k] = 1.0 / t[k];
    }
    // the tables the owner kernel reads, row by row
    std::vector<double> lev;
    lev.reserve(size_t(7) * H.nzn);
    for (const auto* row : {&r, &ir, &it, &p0, &dt}) lev.insert(lev.end(), row->begin(), row->end());
    lev.resize(size_t(7) * H.nzn, 0.0);
    for (int el = 0; el < H.n_z; ++el) {
        if (el > 0) lev[size_t(5) * H.nzn + el * H.N] = H.dz[el - 1] / (H.dz[el - 1] + H.dz[el]);
        lev[size_t(6) * H.nzn + el] = H.sz[el];
    }
    const std::vector<double>* src[7] = {&r, &t, &dt, &p0, &ir, &it, &lev};
    const double** dst[7] = {&M->d.rho0, &M->d.theta0, &M->d.dth0, &M->d.p0, &M->d.inv_rho0,
                             &M->d.inv_theta0, &M->d.lev};
    for (int q = 0; q < 7; ++q) {
        if (M->have_ref) {
            HIPCHK(hipMemcpy((void*)*dst[q], src[q]->data(), src[q]->size() * 8, hipMemcpyHostToDevice));
        } else {
            int rc = M->upload(*src[q], dst[q]);
            if (rc != SEM_OK) return rc;
        }
    }
    M->have_ref = true;
    ++M->epoch;
    return SEM_OK;
}

int sem_mesh_set_reference(sem_mesh* M, const double* rho0, const double* theta0,
                           const double* dth0) {
    return sem::guarded("sem_mesh_set_reference", [&] { return sem_mesh_set_reference_impl(M, rho0, theta0, dth0); });
}

static int sem_mesh_set_terrain_impl(sem_mesh* M, const double* zs, const double* rho0, const double* theta0,
                         const double* dth0) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    const sem::HostMesh& H = M->host;
    DevMesh& d = M->d;
    HIPCHK(hipDeviceSynchronize());
    if (!zs) {
        d.zs = d.nrm = d.minv_ht = d.ref_n = d.tfac = nullptr;
        M->zs_host.clear();
        ++M->epoch;
        return SEM_OK;
    }
    if (!rho0 || !theta0 || !dth0) return fail(SEM_ERR_ARG, "null reference array");
    const double z0 = H.z_edges.front(), top = H.z_edges.back(), depth = top - z0;
    for (int64_t h = 0; h < H.n_h; ++h)
        if (!(zs[h] >= 0.0) || !(zs[h] < depth))
            return fail(SEM_ERR_ARG, "terrain heights must lie in [0, H - z0)");
    const int np1 = H.np1, np2 = np1 * np1, nzn = H.nzn, ldz = H.ldz;
    const int64_t nh = H.n_h, nhh = H.n_hh;
    for (int64_t h = 0; h < nh; ++h)
        for (int k = 0; k < nzn; ++k)
            if (!(rho0[h * nzn + k] > 0.0) || !(theta0[h * nzn + k] > 0.0))
                return fail(SEM_ERR_ARG, "reference state must be positive");
    // one buffer: zs[n_h + n_hh], nrm[3][n_h], minv_ht[n_h],
    // ref_n[5][n_h + n_hh][ldz] (hanging points after the unique nodes), tfac[nzn]
    const int64_t fs = (nh + nhh) * ldz;
    const int64_t total = nh + nhh + 3 * nh + nh + 5 * fs + nzn;
    std::vector<double> buf(size_t(total), 0.0);
    double* b_zs = buf.data();
    double* b_zh = b_zs + nh;
    double* b_n = b_zh + nhh;
    double* b_mi = b_n + 3 * nh;
    double* b_ref = b_mi + nh;
    double* b_tf = b_ref + 5 * fs;
    const double gam = H.c_p / (H.c_p - H.R_d);
    auto fill_ref = [&](double* dst, int64_t stride, int64_t o, double r, double t, double dt) {
        dst[o] = r;
        dst[stride + o] = 1.0 / r;
        dst[2 * stride + o] = 1.0 / t;
        dst[3 * stride + o] = H.p00 * std::pow(H.R_d * r * t / H.p00, gam);
        dst[4 * stride + o] = dt;
    };
    for (int64_t h = 0; h < nh; ++h) {
        b_zs[h] = zs[h];
        for (int k = 0; k < nzn; ++k) {
            const int64_t src = h * nzn + k;
            fill_ref(b_ref, fs, h * ldz + k, rho0[src], theta0[src], dth0[src]);
        }
    }
    // hanging points: the coarse face's interpolant of zs and of the reference
    for (int64_t hh = 0; hh < nhh; ++hh) {
        double z = 0.0;
        for (int32_t r = H.hang_ptr[hh]; r < H.hang_ptr[hh + 1]; ++r) z += H.hang_w[r] * zs[H.hang_src[r]];
        b_zh[hh] = z;
        for (int k = 0; k < nzn; ++k) {
            double ri = 0.0, ti = 0.0, di = 0.0;
            for (int32_t r = H.hang_ptr[hh]; r < H.hang_ptr[hh + 1]; ++r) {
                const int64_t src = int64_t(H.hang_src[r]) * nzn + k;
                ri += H.hang_w[r] * rho0[src];
                ti += H.hang_w[r] * theta0[src];
                di += H.hang_w[r] * dth0[src];
            }
            if (!(ri > 0.0) || !(ti > 0.0)) return fail(SEM_ERR_ARG, "reference state must be positive");
            fill_ref(b_ref, fs, (nh + hh) * ldz + k, ri, ti, di);
        }
    }
    // per column position: the element-local gradient of zs (LGL derivative
    // of its nodal values times 2/dx, 2/dy) and the horizontal lumped mass
    // with the terrain factor (1 - zs/(H - z0)); both are summed onto the
    // unique horizontal nodes, hanging positions through their rows (Z^T)
    std::vector<double> gx(size_t(nh), 0.0), gy(size_t(nh), 0.0), wt(size_t(nh), 0.0), mh(size_t(nh), 0.0);
    const std::vector<double>& Dm = H.basis.D;
    const std::vector<double>& w = H.basis.w;
    std::vector<double> zp(static_cast<size_t>(np2));
    for (int c = 0; c < H.n_col; ++c) {
        const int32_t* gm = &H.gmap[size_t(c) * np2];
        for (int p = 0; p < np2; ++p) zp[p] = gm[p] >= 0 ? zs[gm[p]] : b_zh[-gm[p] - 1];
        for (int j = 0; j < np1; ++j)
            for (int i = 0; i < np1; ++i) {
                double sx = 0.0, sy = 0.0;
                for (int m = 0; m < np1; ++m) {
                    sx += Dm[i * np1 + m] * zp[j * np1 + m];
                    sy += Dm[j * np1 + m] * zp[m * np1 + i];
                }
                sx *= H.col_sx[c];
                sy *= H.col_sy[c];
                const double wij = w[i] * w[j] * 0.25 * H.col_dx[c] * H.col_dy[c];
                const double mt = wij * (1.0 - zp[j * np1 + i] / depth);
                const int32_t g = gm[j * np1 + i];
                auto add = [&](int64_t h, double f) {
                    gx[h] += f * mt * sx;
                    gy[h] += f * mt * sy;
                    wt[h] += f * mt;
                    mh[h] += f * mt;
                };
                if (g >= 0) add(g, 1.0);
                else
                    for (int32_t r = H.hang_ptr[-g - 1]; r < H.hang_ptr[-g]; ++r) add(H.hang_src[r], H.hang_w[r]);
            }
    }
    for (int64_t h = 0; h < nh; ++h) {
        if (!(mh[h] > 0.0)) return fail(SEM_ERR_MESH, "non-positive assembled mass");
        const double nx = -gx[h] / wt[h], ny = -gy[h] / wt[h];
        const double inv = 1.0 / std::sqrt(1.0 + nx * nx + ny * ny);
        b_n[h] = nx * inv;
        b_n[nh + h] = ny * inv;
        b_n[2 * nh + h] = inv;
        b_mi[h] = 1.0 / mh[h];
    }
    for (int k = 0; k < nzn; ++k) b_tf[k] = (top - H.zn[k]) / depth;
    if (M->terrain_bytes != int64_t(sizeof(double)) * total) {
        if (M->terrain_buf) {
            (void)hipFree(M->terrain_buf);
            M->ws_bytes -= M->terrain_bytes;
            M->terrain_buf = nullptr;
            M->terrain_bytes = 0;
        }
        HIPCHK(hipMalloc(&M->terrain_buf, sizeof(double) * total));
        M->terrain_bytes = int64_t(sizeof(double)) * total;
        M->ws_bytes += M->terrain_bytes;
    }
    HIPCHK(hipMemcpy(M->terrain_buf, buf.data(), sizeof(double) * total, hipMemcpyHostToDevice));
    double* base = M->terrain_buf;
    d.zs = base;
    d.nrm = base + nh + nhh;
    d.minv_ht = d.nrm + 3 * nh;
    d.ref_n = d.minv_ht + nh;
    d.tfac = d.ref_n + 5 * fs;
    d.inv_depth = 1.0 / depth;
    d.z_top = top;
    d.depth = depth;
    M->zs_host.assign(zs, zs + nh);
    ++M->epoch;
    return SEM_OK;
}

int sem_mesh_set_terrain(sem_mesh* M, const double* zs, const double* rho0, const double* theta0,
                         const double* dth0) {
    return sem::guarded("sem_mesh_set_terrain", [&] { return sem_mesh_set_terrain_impl(M, zs, rho0, theta0, dth0); });
}

static int sem_mesh_heights_impl(const sem_mesh* M, const double* zs, double* z) {
    if (!M || !z) return fail(SEM_ERR_ARG, "null argument");
    const sem::HostMesh& H = M->host;
    const double z0 = H.z_edges.front(), top = H.z_edges.back(), depth = top - z0;
    const double* s = zs ? zs : (M->zs_host.empty() ? nullptr : M->zs_host.data());
    if (zs)
        for (int64_t h = 0; h < H.n_h; ++h)
            if (!(zs[h] >= 0.0) || !(zs[h] < depth))
                return fail(SEM_ERR_ARG, "terrain heights must lie in [0, H - z0)");
    for (int64_t h = 0; h < H.n_h; ++h)
        for (int k = 0; k < H.nzn; ++k) {
            const double zf = H.zn[k];
            z[h * H.nzn + k] = s ? zf + s[h] * (top - zf) / depth : zf;
        }
    return SEM_OK;
}

int sem_mesh_heights(const sem_mesh* M, const double* zs, double* z) {
    return sem::guarded("sem_mesh_heights", [&] { return sem_mesh_heights_impl(M, zs, z); });
}

static int sem_nc_project_impl(const sem_mesh* M, int dir, const double* src, double* dst, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (dir != SEM_SCATTER && dir != SEM_GATHER) return fail(SEM_ERR_ARG, "bad direction");
    const DevMesh& d = M->d;
    if (d.n_hh == 0) return SEM_OK;
    if (!src || !dst) return fail(SEM_ERR_ARG, "null array");
    hipStream_t s = (hipStream_t)stream;
    if (dir == SEM_SCATTER)
        hipLaunchKernelGGL(sem::k_nc_scatter, dim3(grid_for(int64_t(d.n_hh) * d.nzn)), dim3(256), 0, s, d, src, dst);
    else
        hipLaunchKernelGGL(sem::k_nc_gather, dim3(grid_for(int64_t(d.n_hT) * d.nzn)), dim3(256), 0, s, d, src, dst);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int sem_nc_project(const sem_mesh* M, int dir, const double* src, double* dst, void* stream) {
    return sem::guarded("sem_nc_project", [&] { return sem_nc_project_impl(M, dir, src, dst, stream); });
}

static int sem_rhs_impl(const sem_mesh* M, const double* q, const double* hv, double* rE, int prec, void* stream) {
    int rc = check_mesh(M);
    if (rc != SEM_OK) return rc;
    if (!q || !rE || (M->d.n_hh > 0 && !hv)) return fail(SEM_ERR_ARG, "null array");
    return sem_launch_rhs(M, q, hv, rE, prec, (hipStream_t)stream);
}

int sem_rhs(const sem_mesh* M, const double* q, const double* hv, double* rE, int prec, void* stream) {
    return sem::guarded("sem_rhs", [&] { return sem_rhs_impl(M, q, hv, rE, prec, stream); });
}

static int sem_dss_impl(const sem_mesh* M, int phase, const double* rE, double* acc, double* c, double* r,
            void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    const DevMesh& d = M->d;
    hipStream_t s = (hipStream_t)stream;
    if (phase == SEM_ASSEMBLE) {
        if (!rE || !acc || (d.n_hh > 0 && !c)) return fail(SEM_ERR_ARG, "null array");
        const int64_t grid = int64_t((d.n_h + sem::ASM_H - 1) / sem::ASM_H) * ((d.nzn + sem::ASM_K - 1) / sem::ASM_K);
        if (d.N == 1)
            hipLaunchKernelGGL(sem::k_assemble, dim3(grid_for(int64_t(d.n_h) * d.nzn)), dim3(256), 0, s, d, rE, acc,
                               false);
        else
            hipLaunchKernelGGL(sem::k_assemble_elem, dim3(unsigned(grid)), dim3(256), 0, s, d, rE, acc);
        if (d.n_hh > 0)
            hipLaunchKernelGGL(sem::k_assemble_hang, dim3(grid_for(int64_t(d.n_hh) * d.nzn)), dim3(256), 0, s, d, rE, c,
                               false);
    } else if (phase == SEM_FINALIZE) {
        if (!acc || !r) return fail(SEM_ERR_ARG, "null array");
        hipLaunchKernelGGL(sem::k_finalize, dim3(grid_for(int64_t(d.n_h) * d.nzn)), dim3(256), 0, s, d, acc, r);
    } else {
        return fail(SEM_ERR_ARG, "bad phase");
    }
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int sem_dss(const sem_mesh* M, int phase, const double* rE, double* acc, double* c, double* r,
            void* stream) {
    return sem::guarded("sem_dss", [&] { return sem_dss_impl(M, phase, rE, acc, c, r, stream); });
}

static int sem_stage_update_impl(const sem_mesh* M, double a, double b, double c, const double* qn,
                     const double* qs, const double* r, double* qout, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!qn || !qs || !r || !qout) return fail(SEM_ERR_ARG, "null array");
    const int64_t n = int64_t(NF) * M->d.n_h * M->d.ldz;
    hipLaunchKernelGGL(sem::k_update, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, n, a, b, c,
                       qn, qs, r, qout);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int sem_stage_update(const sem_mesh* M, double a, double b, double c, const double* qn,
                     const double* qs, const double* r, double* qout, void* stream) {
    return sem::guarded("sem_stage_update", [&] { return sem_stage_update_impl(M, a, b, c, qn, qs, r, qout, stream); });
}

static int sem_stage_impl(const sem_mesh* M, double a, double b, double c, const double* qn, const double* qs,
              double* qout, int prec, void* stream) {
    int rc = check_mesh(M);
    if (rc != SEM_OK) return rc;
    if (!qn || !qs || !qout) return fail(SEM_ERR_ARG, "null array");
    if (qout == qs || qout == qn) return fail(SEM_ERR_ARG, "qout must not alias qs or qn");
    if (prec != SEM_FP64 && prec != SEM_FP32) return fail(SEM_ERR_ARG, "bad precision");
    if (dissipation_on(M) && !sem::fused_dissipation_inline(M->d, M->fused, prec) &&
        (rc = dissip_prepass(M, qs, (hipStream_t)stream)) != SEM_OK)
        return rc;
    rc = sem::fused_stage_launch(M->d, M->fused, a, b, c, qn, qs, qout, prec, (hipStream_t)stream);
    if (rc != SEM_OK) return fail(rc, "fused stage launch failed");
    return SEM_OK;
}

int sem_stage(const sem_mesh* M, double a, double b, double c, const double* qn, const double* qs,
              double* qout, int prec, void* stream) {
    return sem::guarded("sem_stage", [&] { return sem_stage_impl(M, a, b, c, qn, qs, qout, prec, stream); });
}

static int sem_mesh_set_dissipation_impl(sem_mesh* M, double cs, double sponge_gamma, double sponge_depth) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!(cs >= 0.0) || !(sponge_gamma >= 0.0) || (sponge_gamma > 0.0 && !(sponge_depth > 0.0)))
        return fail(SEM_ERR_ARG, "need Cs >= 0, sponge_gamma >= 0 and sponge_depth > 0");
    const sem::HostMesh& H = M->host;
    DevMesh& d = M->d;
    HIPCHK(hipDeviceSynchronize());
    if (cs == 0.0 && sponge_gamma == 0.0) {
        d.cs = 0.0;
        d.sponge = nullptr;
        d.rx = nullptr;
        ++M->epoch;
        return SEM_OK;
    }
    const int64_t nloc = int64_t(H.n_col) * H.n_z * H.np1 * H.np1 * H.np1;
    const int64_t nst = int64_t(NF) * H.n_h * H.ldz, nhs = int64_t(NF) * H.n_hh * H.ldz;
    if (!M->diss_rE) {
        HIPCHK(hipMalloc(&M->diss_rE, sizeof(double) * NF * nloc));
        HIPCHK(hipMalloc(&M->diss_acc, sizeof(double) * nst));
        HIPCHK(hipMalloc(&M->diss_r, sizeof(double) * nst));
        HIPCHK(hipMalloc(&M->diss_c, sizeof(double) * std::max<int64_t>(nhs, 1)));
        HIPCHK(hipMalloc(&M->diss_sponge, sizeof(double) * H.nzn));
        // the row padding of the tendency stays zero (finalize writes kz < nzn only)
        HIPCHK(hipMemset(M->diss_r, 0, sizeof(double) * nst));
        M->ws_bytes += int64_t(sizeof(double)) * (NF * nloc + 2 * nst + std::max<int64_t>(nhs, 1) + H.nzn);
    }
    // absorbing layer per vertical node: min(1, max(0, gamma sin^2(pi/2 (1 - (z_top - z)/depth))))
    // inside z >= z_top - depth, zero below
    std::vector<double> sp(H.nzn, 0.0);
    const double ztop = H.z_edges.back();
    for (int kz = 0; kz < H.nzn; ++kz) {
        const double z = H.zn[kz];
        if (sponge_gamma > 0.0 && z >= ztop - sponge_depth) {
            const double sn = std::sin(0.5 * M_PI * (1.0 - (ztop - z) / sponge_depth));
            sp[kz] = std::min(1.0, std::max(0.0, sponge_gamma * sn * sn));
        }
    }
    HIPCHK(hipMemcpy(M->diss_sponge, sp.data(), sizeof(double) * H.nzn, hipMemcpyHostToDevice));
    d.cs = cs;
    d.sponge = sponge_gamma > 0.0 ? M->diss_sponge : nullptr;
    d.sp_gamma = sponge_gamma;
    d.sp_depth = sponge_depth;
    d.rx = M->diss_r;
    ++M->epoch;
    return SEM_OK;
}

int sem_mesh_set_dissipation(sem_mesh* M, double cs, double sponge_gamma, double sponge_depth) {
    return sem::guarded("sem_mesh_set_dissipation", [&] { return sem_mesh_set_dissipation_impl(M, cs, sponge_gamma, sponge_depth); });
}

static int sem_stage_set_layout_impl(sem_mesh* M, int layout, int param) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    const bool columns = layout == SEM_LAYOUT_COLUMNS || layout == SEM_LAYOUT_COLUMNS_KZ ||
                         layout == SEM_LAYOUT_COLUMNS_SPLIT;
    if (!columns && layout != SEM_LAYOUT_BLOCKS)
        return fail(SEM_ERR_ARG, "unknown layout");
    if (param < 0) return fail(SEM_ERR_ARG, "negative layout parameter");
    if (columns && param > 0 && !sem::fused_lpc_supported(M->host.N, param))
        return fail(SEM_ERR_ARG, "unsupported layers_per_chunk for this order");
    if (layout == SEM_LAYOUT_COLUMNS_SPLIT && param > 0 && !sem::fused_split_supported(M->host.N, param))
        return fail(SEM_ERR_ARG, "the split-element order needs two or more layers per chunk");
    if (layout == SEM_LAYOUT_BLOCKS && !sem::fused_blocks_supported(M->host))
        return fail(SEM_ERR_ARG, "no block layout for this mesh (order 3 to 5 with 2 x 2 column blocks)");
    sem::FusedPlan P;
    int rc = sem::fused_plan_build(M->host, layout, param, P, sem::fused_plan_owner(layout, param));
    if (rc != SEM_OK) { sem::fused_plan_free(P); return fail(rc, "could not build the fused-stage tables"); }
    HIPCHK(hipDeviceSynchronize());
    sem::fused_plan_free(M->fused);
    M->fused = P;
    ++M->epoch;
    return SEM_OK;
}

int sem_stage_set_layout(sem_mesh* M, int layout, int param) {
    return sem::guarded("sem_stage_set_layout", [&] { return sem_stage_set_layout_impl(M, layout, param); });
}

int sem_stage_get_layout(const sem_mesh* M, int* layout, int* param) {
    if (!M || !layout || !param) return fail(SEM_ERR_ARG, "null argument");
    *layout = M->fused.layout;
    *param = M->fused.layout == SEM_LAYOUT_BLOCKS ? M->fused.bt.n_seg
             : M->fused.own && M->fused.by_default ? 0 : M->fused.t.layers_per_chunk;
    return SEM_OK;
}

static int sem_stage_tune_impl(sem_mesh* M, int layers_per_chunk) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (layers_per_chunk < 0 ||
        (layers_per_chunk > 0 && !sem::fused_lpc_supported(M->host.N, layers_per_chunk)))
        return fail(SEM_ERR_ARG, "unsupported layers_per_chunk for this order");
    return sem_stage_set_layout(M, SEM_LAYOUT_COLUMNS, layers_per_chunk);
}

int sem_stage_tune(sem_mesh* M, int layers_per_chunk) {
    return sem::guarded("sem_stage_tune", [&] { return sem_stage_tune_impl(M, layers_per_chunk); });
}

static int sem_stage_autotune_impl(sem_mesh* M, const double* qn, const double* qs, double* qout, int prec,
                       int reps, int* best_lpc, float* best_ms, void* stream) {
    int rc = check_mesh(M);
    if (rc != SEM_OK) return rc;
    if (!qn || !qs || !qout) return fail(SEM_ERR_ARG, "null array");
    if (qout == qs || qout == qn) return fail(SEM_ERR_ARG, "qout must not alias qs or qn");
    if (prec != SEM_FP64 && prec != SEM_FP32) return fail(SEM_ERR_ARG, "bad precision");
    if (reps < 1) reps = 5;
    hipStream_t s = (hipStream_t)stream;
    // the tables of all column candidates and of all block ones (built by the
    // first of them)
    struct Tables : sem::FusedPlan {
        ~Tables() { sem::fused_plan_free(*this); }
    } cols, blks;
    if ((rc = sem::fused_plan_build(M->host, SEM_LAYOUT_COLUMNS, 0, cols, true)) != SEM_OK)
        return fail(rc, "could not build the fused-stage tables");
    hipEvent_t e0, e1;
    HIPCHK(hipEventCreate(&e0));
    HIPCHK(hipEventCreate(&e1));
    // candidates: where the owner kernel runs, the default layout; single
    // columns in chunks of 1, 2, 4, 8 layers, in FP64 in each thread order
    // (float runs the natural order in any); column blocks in 1, 2, 4, ...
    // vertical segments (distinct segment lengths)
    std::vector<std::pair<int, int>> cand;
    const bool own = cols.own && sem::own_used(M->d, prec);
    if (own) cand.push_back({SEM_LAYOUT_COLUMNS, 0});
    for (int lpc = 1; lpc <= 16; lpc *= 2)
        if (sem::fused_lpc_supported(M->host.N, lpc) && lpc <= 2 * M->host.n_z) {
            cand.push_back({SEM_LAYOUT_COLUMNS, lpc});
            if (prec == SEM_FP64) {
                cand.push_back({SEM_LAYOUT_COLUMNS_KZ, lpc});
                if (sem::fused_split_supported(M->host.N, lpc))
                    cand.push_back({SEM_LAYOUT_COLUMNS_SPLIT, lpc});
            }
        }
    if (sem::fused_blocks_supported(M->host) && !M->d.zs && !sem::fused_blocks_wrap(M->host)) {
        int last_ls = -1;
        for (int S = 1; S <= M->host.n_z; S *= 2) {
            const int ls = (M->host.n_z + S - 1) / S;
            if (ls == last_ls) continue;
            last_ls = ls;
            cand.push_back({SEM_LAYOUT_BLOCKS, S});
        }
    }
    int best = -1, best_named = -1;                        // (of the column candidates that name a chunk)
    float best_t = 0.0f, best_named_t = 0.0f;
    bool blocks = true;
    for (size_t ci = 0; ci < cand.size(); ++ci) {
        const auto [layout, param] = cand[ci];
        const bool blk = layout == SEM_LAYOUT_BLOCKS, named = !blk && param > 0;
        if (blk && blks.allocs.empty() && blocks)
            blocks = sem::fused_plan_build(M->host, layout, param, blks, false) == SEM_OK;
        if (blk && !blocks) continue;
        sem::FusedPlan P = blk ? blks : cols;              // (the tables stay theirs)
        if (sem::fused_plan_set(M->host, layout, param, P) != SEM_OK) continue;
        if (named) P.own = false;
        // warm-up, then timed repetitions (the stage coefficients do not
        // change the work; qout is scratch here): one, and the others if it
        // took no more than half as long again as the best (of two, as a
        // single one may have been held up)
        auto stages = [&](int n, float& ms) {
            (void)hipEventRecord(e0, s);
            for (int r = 0; r < n && rc == SEM_OK; ++r)
                rc = sem::fused_stage_launch(M->d, P, 0.5, 0.5, 1e-3, qn, qs, qout, prec, s);
            (void)hipEventRecord(e1, s);
            const bool ok = rc == SEM_OK && hipEventSynchronize(e1) == hipSuccess &&
                            hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            ms /= float(n);
            return ok;
        };
        rc = sem::fused_stage_launch(M->d, P, 0.5, 0.5, 1e-3, qn, qs, qout, prec, s);
        float ms = 0.0f;
        bool ok = rc == SEM_OK && stages(1, ms);
        if (ok && best >= 0 && ms > 1.5f * best_t) {
            const float one = ms;
            ok = stages(1, ms);
            ms = std::min(one, ms);
        }
        if (ok && reps > 1 && (best < 0 || ms <= 1.5f * best_t)) {
            const float one = ms;
            ok = stages(reps - 1, ms);
            ms = (one + float(reps - 1) * ms) / float(reps);
        }
        if (ok) {
            // (ties go to the default)
            if (best < 0 || ms < (best == 0 && own ? 0.98f : 1.0f) * best_t) { best = int(ci); best_t = ms; }
            if (named && (best_named < 0 || ms < best_named_t)) { best_named = int(ci); best_named_t = ms; }
        }
        (void)hipStreamSynchronize(s);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (best < 0) return fail(SEM_ERR_HIP, "autotuning found no working configuration");
    // the plan of the fastest; a default one keeps the fastest order and chunk
    // for the stages that the owner kernel does not take, and a plan tuned for
    // those keeps the owner kernel for the others
    Tables& T = cand[best].first == SEM_LAYOUT_BLOCKS ? blks : cols;
    const bool default_wins = sem::fused_plan_owner(cand[best].first, cand[best].second);
    if (default_wins && best_named >= 0)
        (void)sem::fused_plan_set(M->host, cand[best_named].first, cand[best_named].second, T);
    else if ((rc = sem::fused_plan_set(M->host, cand[best].first, cand[best].second, T)) != SEM_OK)
        return fail(rc, "could not build the fused-stage tables");
    if (default_wins) {
        T.layout = SEM_LAYOUT_COLUMNS;
        T.by_default = true;
    } else if (own) {
        T.own = false;
    }
    HIPCHK(hipDeviceSynchronize());
    std::swap(M->fused, static_cast<sem::FusedPlan&>(T));
    ++M->epoch;
    if (best_lpc) *best_lpc = M->fused.t.layers_per_chunk;
    if (best_ms) *best_ms = best_t;
    return SEM_OK;
}

int sem_stage_autotune(sem_mesh* M, const double* qn, const double* qs, double* qout, int prec,
                       int reps, int* best_lpc, float* best_ms, void* stream) {
    return sem::guarded("sem_stage_autotune", [&] { return sem_stage_autotune_impl(M, qn, qs, qout, prec, reps, best_lpc, best_ms, stream); });
}

int sem_stage_get_tune(const sem_mesh* M, int* layers_per_chunk) {
    if (!M || !layers_per_chunk) return fail(SEM_ERR_ARG, "null argument");
    *layers_per_chunk = M->fused.t.layers_per_chunk;
    return SEM_OK;
}

int sem_mesh_get_epoch(const sem_mesh* M, int64_t* epoch) {
    if (!M || !epoch) return fail(SEM_ERR_ARG, "null argument");
    *epoch = M->epoch;
    return SEM_OK;
}

static int amr_flag_impl(const sem_mesh* M, const double* q, int criterion, const double* thr, int lvl_max,
             int8_t* ae, int8_t* ac, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!q || !ae || !ac) return fail(SEM_ERR_ARG, "null array");
    if (criterion != SEM_CRIT_SPEED && criterion != SEM_CRIT_VORTZ) return fail(SEM_ERR_ARG, "bad criterion");
    if (lvl_max < 0 || lvl_max > SEM_MAX_LEVEL) return fail(SEM_ERR_ARG, "lvl_max out of range");
    if (lvl_max > 0 && !thr) return fail(SEM_ERR_ARG, "null thresholds");
    sem::Thr T{};
    for (int l = 0; l < lvl_max; ++l) {
        T.v[l] = thr[l];
        if (l > 0 && thr[l] < thr[l - 1]) return fail(SEM_ERR_ARG, "thresholds must be non-decreasing");
    }
    const DevMesh& d = M->d;
    hipStream_t s = (hipStream_t)stream;
    switch (d.N) {
#define CASE(NN)                                                                        \
    case NN:                                                                            \
        hipLaunchKernelGGL((sem::k_amr_elem<NN + 1>), dim3(unsigned(d.n_col) * sem::pass_chunks<NN + 1>(d.n_z)), \
                           dim3(sem::pass_threads<NN + 1>()), 0, s, d, q, criterion, T, lvl_max, ae); \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
        default: return fail(SEM_ERR_N, "unsupported N");
    }
    hipLaunchKernelGGL(sem::k_amr_col, dim3((d.n_col + 255) / 256), dim3(256), 0, s, d, ae, ac);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int amr_flag(const sem_mesh* M, const double* q, int criterion, const double* thr, int lvl_max,
             int8_t* ae, int8_t* ac, void* stream) {
    return sem::guarded("amr_flag", [&] { return amr_flag_impl(M, q, criterion, thr, lvl_max, ae, ac, stream); });
}

// ------------------------------------------------------------ adaptation
static sem::MeshInput input_of(const sem_mesh_desc* d) {
    return sem::MeshInput{d->N, d->nx0, d->ny0, d->n_z, d->n_col, d->h_col_level, d->h_col_ix,
                          d->h_col_iy, d->Lx, d->Ly, d->h_z_edges, d->periodic_x != 0,
                          d->periodic_y != 0, d->f, d->g, d->R_d, d->c_p, d->p00};
}

static int sem_adapt_columns_impl(const sem_mesh_desc* desc, const int8_t* flags, int lvl_max, int32_t cap,
                      int32_t* lev, int32_t* ix, int32_t* iy, int32_t* n_out) {
    if (!desc || !flags || !n_out) return fail(SEM_ERR_ARG, "null argument");
    if (cap < 0 || (cap > 0 && (!lev || !ix || !iy))) return fail(SEM_ERR_ARG, "bad output arrays");
    std::vector<std::array<int32_t, 3>> out;
    std::string err;
    int rc = sem::adapt_layout(desc->nx0, desc->ny0, desc->periodic_x != 0, desc->periodic_y != 0,
                               desc->n_col, desc->h_col_level, desc->h_col_ix, desc->h_col_iy, flags,
                               lvl_max, out, err);
    if (rc != SEM_OK) return fail(rc, err);
    *n_out = int32_t(out.size());
    if (int64_t(out.size()) > cap)
        return fail(SEM_ERR_ARG, "output capacity " + std::to_string(cap) + " < " +
                                     std::to_string(out.size()) + " columns");
    for (size_t i = 0; i < out.size(); ++i) {
        lev[i] = out[i][0];
        ix[i] = out[i][1];
        iy[i] = out[i][2];
    }
    return SEM_OK;
}

int sem_adapt_columns(const sem_mesh_desc* desc, const int8_t* flags, int lvl_max, int32_t cap,
                      int32_t* lev, int32_t* ix, int32_t* iy, int32_t* n_out) {
    return sem::guarded("sem_adapt_columns", [&] { return sem_adapt_columns_impl(desc, flags, lvl_max, cap, lev, ix, iy, n_out); });
}

static int sem_transfer_plan_impl(const sem_mesh_desc* from, const sem_mesh_desc* to, int64_t* nnz,
                      int32_t* ptr, int32_t* src, double* w) {
    if (!from || !to || !nnz) return fail(SEM_ERR_ARG, "null argument");
    sem::HostMesh A, B;
    std::string err;
    int rc = sem::build_host_mesh(input_of(from), A, err);
    if (rc == SEM_OK) rc = sem::build_host_mesh(input_of(to), B, err);
    if (rc != SEM_OK) return fail(rc, err);
    sem::TransferRows T;
    if ((rc = sem::build_transfer(A, B, T, err)) != SEM_OK) return fail(rc, err);
    *nnz = int64_t(T.src.size());
    if (ptr) std::memcpy(ptr, T.ptr.data(), T.ptr.size() * sizeof(int32_t));
    if (src) std::memcpy(src, T.src.data(), T.src.size() * sizeof(int32_t));
    if (w) std::memcpy(w, T.w.data(), T.w.size() * sizeof(double));
    return SEM_OK;
}

int sem_transfer_plan(const sem_mesh_desc* from, const sem_mesh_desc* to, int64_t* nnz,
                      int32_t* ptr, int32_t* src, double* w) {
    return sem::guarded("sem_transfer_plan", [&] { return sem_transfer_plan_impl(from, to, nnz, ptr, src, w); });
}

static int sem_transfer_create_impl(const sem_mesh* from, const sem_mesh* to, sem_transfer** out) {
    if (!from || !to || !out) return fail(SEM_ERR_ARG, "null argument");
    *out = nullptr;
    sem::TransferRows T;
    std::string err;
    int rc = sem::build_transfer(from->host, to->host, T, err);
    if (rc != SEM_OK) return fail(rc, err);
    std::unique_ptr<sem_transfer> X(new sem_transfer());
    X->n_from = from->host.n_h;
    X->n_to = to->host.n_h;
    X->nzn = to->host.nzn;
    X->ldz = to->host.ldz;
    X->nnz = int64_t(T.src.size());
    for (int32_t s : T.src)
        if (s < 0 || s >= X->n_from) return fail(SEM_ERR_MESH, "transfer row source out of range");
    HIPCHK(hipMalloc(&X->ptr, T.ptr.size() * sizeof(int32_t)));
    HIPCHK(hipMemcpy(X->ptr, T.ptr.data(), T.ptr.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    if (X->nnz > 0) {
        HIPCHK(hipMalloc(&X->src, T.src.size() * sizeof(int32_t)));
        HIPCHK(hipMalloc(&X->w, T.w.size() * sizeof(double)));
        HIPCHK(hipMemcpy(X->src, T.src.data(), T.src.size() * sizeof(int32_t), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(X->w, T.w.data(), T.w.size() * sizeof(double), hipMemcpyHostToDevice));
    }
    // the rows a workgroup sums, longest first
    std::vector<int32_t> rows;
    auto len = [&](int32_t h) { return T.ptr[h + 1] - T.ptr[h]; };
    for (int32_t h = 0; h < X->n_to; ++h)
        if (len(h) > sem::TRANSFER_SHORT) rows.push_back(h);
    std::stable_sort(rows.begin(), rows.end(), [&](int32_t a, int32_t b) { return len(a) > len(b); });
    X->n_long = int(rows.size());
    if (X->n_long > 0) {
        HIPCHK(hipMalloc(&X->long_rows, rows.size() * sizeof(int32_t)));
        HIPCHK(hipMemcpy(X->long_rows, rows.data(), rows.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    }
    *out = X.release();
    return SEM_OK;
}

int sem_transfer_create(const sem_mesh* from, const sem_mesh* to, sem_transfer** out) {
    return sem::guarded("sem_transfer_create", [&] { return sem_transfer_create_impl(from, to, out); });
}

static int sem_transfer_apply_impl(const sem_transfer* X, const double* q_from, double* q_to, void* stream) {
    if (!X) return fail(SEM_ERR_ARG, "null transfer");
    if (!q_from || !q_to) return fail(SEM_ERR_ARG, "null array");
    if (q_from == q_to) return fail(SEM_ERR_ARG, "q_to must not alias q_from");
    if (X->n_to == 0) return SEM_OK;
    hipStream_t s = (hipStream_t)stream;
    const int64_t grid = X->n_long + (X->n_to * (X->ldz / 2) + 255) / 256;
    hipLaunchKernelGGL(sem::k_transfer, dim3(unsigned(grid)), dim3(256), 0, s, X->ptr, X->src, X->w, X->long_rows,
                       X->n_long, X->n_to, X->n_from, X->nzn, X->ldz, q_from, q_to);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int sem_transfer_apply(const sem_transfer* X, const double* q_from, double* q_to, void* stream) {
    return sem::guarded("sem_transfer_apply", [&] { return sem_transfer_apply_impl(X, q_from, q_to, stream); });
}

int sem_transfer_destroy(sem_transfer* X) {
    delete X;
    return SEM_OK;
}

}  // extern "C"
