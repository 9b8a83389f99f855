// Refinement forecaster, mesh side (gfx950): per-element features, the
// combination of forecast and criterion flags, and training labels.
//
// The paper's refinement criterion (Section 4.1) is a threshold on a field
// at the element's nodes; its closing section asks for better criteria.  The
// forecaster predicts, for every element, the refinement decision a few
// adaptation intervals ahead from 16 features of the element and its
// neighbours; its flags are combined with the plain criterion so that the
// criterion overrides every refinement the forecaster misses.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <unordered_map>

#include "handle.h"
#include "nodeval.h"
#include "rows.h"

namespace sem {

namespace {

struct Scale16 { float v[SEM_NFEAT]; };
struct ThrF { double v[SEM_MAX_LEVEL]; };

// accumulators of the element pass: 13 maxima (of squares where a square root
// is taken: it keeps their order) and one sum
enum { A_ZABS, A_UH, A_W, A_TMAX, A_TMIN, A_GP, A_GT, A_DIV, A_RMAX, A_RMIN, A_UHP, A_ZABSP,
       A_CRIT, A_NMAX, A_ZSUM = A_NMAX, A_N };

// square root of a maximum of squares (-infinity: of no number)
__device__ __forceinline__ double root(double x) { return x >= 0.0 ? sqrt(x) : x; }

}  // namespace

// Raw features of an element (element pass of nodeval.h):
//  0 level, 1 max|zeta|, 2 mean zeta, 3 max|u_h|, 4 max|w|, 5 max theta',
//  6 min theta', 7 max|grad p'|, 8 max|grad theta'|, 9 max|div u|,
//  10 rho' range, 11-12 (neighbour pass), 13 change of max|u_h| and
//  14 change of max|zeta| since q_prev, 15 the criterion's own flag;
// zeta = dv/dx - du/dy and every derivative element-local (tensor-product
// LGL derivative, as in the criterion; over terrain-following coordinates the
// physical derivative by the chain rule of the mapping: d/dx = box d/dx +
// a_x d/dzf, d/dy likewise, d/dz = g_s d/dzf, and p' from the per-node
// reference).  dem = number of thresholds the criterion's element maximum
// exceeds (the level the criterion asks for).
//
// 6,220 columns of 8 layers at N = 4 (three levels): 142 us, 0.56 GB read; 320
// with a workgroup per element and a thread per node, whose 14 results took a
// wave reduction each.  What is left is latency at ten waves per CU (LDS), half
// of it the wait for the nodes; VALU issue is 40 %.
template <int NP>
__global__ void __launch_bounds__(pass_threads<NP>(), NP <= 5 ? 3 : 2)
k_features(DevMesh m, const double* __restrict__ q, const double* __restrict__ qp,
           const int8_t* __restrict__ plain, int criterion, ThrF thr, int lvl_max, Scale16 sc,
           float* __restrict__ feat, double* __restrict__ aux, int8_t* __restrict__ dem) {
    constexpr int NP2 = NP * NP, NP3 = NP2 * NP, N = NP - 1;
    constexpr int PT = pass_threads<NP>(), ST = pass_stride<NP>(), TN = NP2 * ST, LZ = pass_layers<NP>();
    constexpr int RED = A_N * (PT + 1);
    // the tiles, then (after them) the threads' maxima
    __shared__ double2 buf[4 * TN > (RED + 1) / 2 ? 4 * TN : (RED + 1) / 2];
    __shared__ double sD[NP2], s_zs[NP2];     // s_zs, terrain: surface height per position
    __shared__ double s_max[LZ][A_N];
    double2 *t_uv = buf, *t_pt = buf + TN, *t_prev = buf + 2 * TN, *t_wr = buf + 3 * TN;
    double* red = reinterpret_cast<double*>(buf);
    const PassItem it = pass_item<NP>(m);
    const int c = it.c, nk = it.layers * N + 1, z0 = it.layer0 * N, tid = threadIdx.x;
    const bool ter = m.zs != nullptr;
    for (int x = tid; x < NP2; x += PT) {
        sD[x] = m.D[x];
        if (ter) {
            const int gz = m.gmap[c * NP2 + x];
            s_zs[x] = m.zs[gz >= 0 ? gz : m.n_h - gz - 1];
        }
    }
    // (a few nodes' loads at once; hanging positions then replace theirs)
    constexpr int U = 4;
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    for (int x0 = tid; x0 < NP2 * nk; x0 += U * PT) {
        int g[U], o[U], kz[U];
        double a[U][SEM_NFIELDS], b[U][2];
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const int x = min(x0 + s * PT, NP2 * nk - 1), pos = x / nk, kl = x - pos * nk;
            g[s] = m.gmap[c * NP2 + pos];
            o[s] = pos * ST + kl;
            kz[s] = z0 + kl;
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const int64_t r = int64_t(max(g[s], 0)) * m.ldz + kz[s];
#pragma unroll
            for (int f = 0; f < SEM_NFIELDS; ++f) a[s][f] = q[f * fs + r];
            b[s][0] = qp[fs + r];
            b[s][1] = qp[2 * fs + r];
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
            if (x0 + s * PT >= NP2 * nk) break;
            if (g[s] < 0) {
                node_values<0, SEM_NFIELDS>(m, q, g[s], kz[s], a[s]);
                node_values<1, 2>(m, qp, g[s], kz[s], b[s]);
            }
            // p' = p0 ((1 + rho'/rho0)(1 + theta'/theta0))^gamma - p0 without cancellation
            double p0, ra, tb;
            if (ter) {
                // per-node reference (hanging rows: the coarse face's interpolant)
                const int64_t fsr = int64_t(m.n_h + m.n_hh) * m.ldz;
                const int64_t r = int64_t(g[s] >= 0 ? g[s] : m.n_h - g[s] - 1) * m.ldz + kz[s];
                ra = a[s][0] * m.ref_n[fsr + r];
                tb = a[s][4] * m.ref_n[2 * fsr + r];
                p0 = m.ref_n[3 * fsr + r];
            } else {
                ra = a[s][0] * m.inv_rho0[kz[s]];
                tb = a[s][4] * m.inv_theta0[kz[s]];
                p0 = m.p0[kz[s]];
            }
            t_uv[o[s]] = double2{a[s][1], a[s][2]};
            t_pt[o[s]] = double2{p0 * pow1p_minus1(m, ra + tb + ra * tb), a[s][4]};
            t_prev[o[s]] = double2{b[s][0], b[s][1]};
            t_wr[o[s]] = double2{a[s][3], a[s][0]};
        }
    }
    __syncthreads();
    double acc[A_N];
#pragma unroll
    for (int r = 0; r < A_N; ++r) acc[r] = -INFINITY;
    acc[A_ZSUM] = 0.0;
    const int lay = tid / NP2, p = tid - lay * NP2;
    if (lay < it.layers) {
        const int i = p % NP, j = p / NP;
        const double sx = 2.0 / m.col_dx[c], sy = 2.0 / m.col_dy[c], szz = 2.0 / m.dz[it.layer0 + lay];
        double zx = 0, zy = 0, gs = 1.0;
        if (ter) {
            // terrain-following mapping: g_s = 1/(1 - zs/(H - z0)),
            // a_x = -g_s (H - zf)/(H - z0) dzs/dx, a_y likewise
            for (int mm = 0; mm < NP; ++mm) {
                zx += sD[i * NP + mm] * s_zs[mm + NP * j];
                zy += sD[j * NP + mm] * s_zs[i + NP * mm];
            }
            gs = 1.0 / (1.0 - s_zs[p] * m.inv_depth);
        }
#pragma unroll 1
        for (int k = 0; k < NP; ++k) {
            const int kl = lay * N + k;
            double vx = 0, uy = 0, ux = 0, vy = 0, wz = 0, px = 0, py = 0, pz = 0, tx = 0, ty = 0,
                   tz = 0, vpx = 0, upy = 0;
#pragma unroll
            for (int mm = 0; mm < NP; ++mm) {
                const double dxm = sD[i * NP + mm], dym = sD[j * NP + mm], dzm = m.D[k * NP + mm];
                const int ox = (mm + NP * j) * ST + kl, oy = (i + NP * mm) * ST + kl, oz = p * ST + lay * N + mm;
                const double2 xu = t_uv[ox], xp = t_pt[ox], yu = t_uv[oy], yp = t_pt[oy], zp = t_pt[oz];
                vx += dxm * xu.y; ux += dxm * xu.x; px += dxm * xp.x; tx += dxm * xp.y;
                vpx += dxm * t_prev[ox].y;
                uy += dym * yu.x; vy += dym * yu.y; py += dym * yp.x; ty += dym * yp.y;
                upy += dym * t_prev[oy].x;
                wz += dzm * t_wr[oz].x; pz += dzm * zp.x; tz += dzm * zp.y;
            }
            vx *= sx; ux *= sx; px *= sx; tx *= sx; vpx *= sx;
            uy *= sy; vy *= sy; py *= sy; ty *= sy; upy *= sy;
            wz *= szz; pz *= szz; tz *= szz;
            if (ter) {
                double uz = 0, vz = 0, upz = 0, vpz = 0;
                for (int mm = 0; mm < NP; ++mm) {
                    const double dzm = m.D[k * NP + mm];
                    const int oz = p * ST + lay * N + mm;
                    uz += dzm * t_uv[oz].x; vz += dzm * t_uv[oz].y;
                    upz += dzm * t_prev[oz].x; vpz += dzm * t_prev[oz].y;
                }
                uz *= szz; vz *= szz; upz *= szz; vpz *= szz;
                const double tg = m.tfac[z0 + kl] * gs;
                const double ax = -tg * zx * sx, ay = -tg * zy * sy;
                vx += ax * vz; ux += ax * uz; px += ax * pz; tx += ax * tz; vpx += ax * vpz;
                uy += ay * uz; vy += ay * vz; py += ay * pz; ty += ay * tz; upy += ay * upz;
                wz *= gs; pz *= gs; tz *= gs;
            }
            const int o = p * ST + kl;
            const double2 uv = t_uv[o], wr = t_wr[o], prev = t_prev[o];
            const double u = uv.x, v = uv.y, w = wr.x, rp = wr.y, tp = t_pt[o].y;
            const double zeta = vx - uy, zetap = vpx - upy;
            auto top = [&](int r, double x) { acc[r] = fmax(acc[r], x); };
            top(A_ZABS, fabs(zeta));
            acc[A_ZSUM] += zeta;
            top(A_UH, u * u + v * v);
            top(A_W, fabs(w));
            top(A_TMAX, tp);
            top(A_TMIN, -tp);
            top(A_GP, px * px + py * py + pz * pz);
            top(A_GT, tx * tx + ty * ty + tz * tz);
            top(A_DIV, fabs(ux + vy + wz));
            top(A_RMAX, rp);
            top(A_RMIN, -rp);
            top(A_UHP, prev.x * prev.x + prev.y * prev.y);
            top(A_ZABSP, fabs(zetap));
            top(A_CRIT, criterion == SEM_CRIT_SPEED ? u * u + v * v + w * w : zeta);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < A_N; ++r) red[r * (PT + 1) + tid] = acc[r];
    __syncthreads();
    for (int x = tid; x < it.layers * A_N; x += PT) {
        const int l = x / A_N, r = x - l * A_N;
        const double* y = red + r * (PT + 1) + l * NP2;
        double s = y[0];
        for (int n = 1; n < NP2; ++n) s = r == A_ZSUM ? s + y[n] : fmax(s, y[n]);
        const bool squares = r == A_UH || r == A_GP || r == A_GT || r == A_UHP ||
                             (r == A_CRIT && criterion == SEM_CRIT_SPEED);
        s_max[l][r] = squares ? root(s) : s;
    }
    __syncthreads();
    for (int x = tid; x < it.layers * SEM_NFEAT; x += PT) {
        const int l = x / SEM_NFEAT, r = x - l * SEM_NFEAT;
        const double* b = s_max[l];
        const int64_t e = int64_t(c) * m.n_z + it.layer0 + l;
        double f = 0.0;
        switch (r) {
            case 0: f = m.col_level[c]; break;
            case 1: f = b[A_ZABS]; break;
            case 2: f = b[A_ZSUM] / NP3; break;
            case 3: f = b[A_UH]; break;
            case 4: f = b[A_W]; break;
            case 5: f = b[A_TMAX]; break;
            case 6: f = -b[A_TMIN]; break;
            case 7: f = b[A_GP]; break;
            case 8: f = b[A_GT]; break;
            case 9: f = b[A_DIV]; break;
            case 10: f = b[A_RMAX] + b[A_RMIN]; break;
            case 13: f = b[A_UH] - b[A_UHP]; break;
            case 14: f = b[A_ZABS] - b[A_ZABSP]; break;
            case 15: f = plain[e]; break;
            default: break;
        }
        feat[e * SEM_NFEAT + r] = float(f * double(sc.v[r]));
        if (r < 2) aux[2 * e + r] = r == 0 ? b[A_ZABS] : b[A_UH];
        if (r == 2) {
            int d = 0;
            for (int lv = 1; lv <= lvl_max; ++lv)
                if (b[A_CRIT] > thr.v[lv - 1]) d = lv;
            dem[e] = int8_t(d);
        }
    }
}

// features 11 and 12: the largest max|zeta| and max|u_h| over the elements of
// the same layer in the horizontal neighbour columns
__global__ void k_features_nbr(DevMesh m, const double* __restrict__ aux, Scale16 sc,
                               float* __restrict__ feat) {
    const int64_t n = int64_t(m.n_col) * m.n_z;
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n;
         e += int64_t(gridDim.x) * blockDim.x) {
        const int c = int(e / m.n_z), layer = int(e % m.n_z);
        double zm = 0.0, um = 0.0;
        for (int r = m.nbr_ptr[c]; r < m.nbr_ptr[c + 1]; ++r) {
            const int64_t e2 = int64_t(m.nbr_col[r]) * m.n_z + layer;
            zm = fmax(zm, aux[2 * e2]);
            um = fmax(um, aux[2 * e2 + 1]);
        }
        feat[e * SEM_NFEAT + 11] = float(zm * double(sc.v[11]));
        feat[e * SEM_NFEAT + 12] = float(um * double(sc.v[12]));
    }
}

// forecast class (argmax of the logits, first maximum on ties: 0 coarsen,
// 1 keep, 2 refine), clamped to the level range, combined with the
// criterion's flag: refine if either refines, coarsen only if both coarsen
__global__ void k_forecast_elem(DevMesh m, const float* __restrict__ logits,
                                const int8_t* __restrict__ plain, int lvl_max,
                                int8_t* __restrict__ out) {
    const int64_t n = int64_t(m.n_col) * m.n_z;
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n;
         e += int64_t(gridDim.x) * blockDim.x) {
        const float* z = logits + 3 * e;
        int cls = 0;
        if (z[1] > z[cls]) cls = 1;
        if (z[2] > z[cls]) cls = 2;
        int f = cls - 1;
        const int lv = m.col_level[int(e / m.n_z)];
        if (f == 1 && lv >= lvl_max) f = 0;
        if (f == -1 && lv == 0) f = 0;
        const int p = plain[e];
        out[e] = int8_t((p == 1 || f == 1) ? 1 : ((p == -1 && f == -1) ? -1 : 0));
    }
}

__global__ void k_forecast_col(DevMesh m, const int8_t* __restrict__ ae, int8_t* __restrict__ ac) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < m.n_col) ac[c] = column_rule(m, ae, c);
}

// maximum horizontal wind sqrt(u^2 + v^2) over the unique nodes whose
// horizontal position lies in [x0, x1] x [y0, y1]: per-block maxima of the
// squares, then one block over the partial results (a maximum does not depend
// on order, and the root keeps it).  A thread per row and pair of levels in
// turn; bound by memory.
// 100,000 rows of 33 levels: 14 us; 44 with a thread per node, a division by
// the row length and a root each.
constexpr int WIND_BLOCKS = 256, WIND_THREADS = 1024;

__global__ void __launch_bounds__(WIND_THREADS)
k_max_wind(DevMesh m, const double* __restrict__ q, const double* __restrict__ hxy, double x0,
           double x1, double y0, double y1, double* __restrict__ part) {
    using vec = double __attribute__((ext_vector_type(2), aligned(8)));
    __shared__ double red[WIND_THREADS / 64];
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    const unsigned L = unsigned(m.nzn + 1) / 2;       // threads of a row
    const int64_t n = int64_t(m.n_h) * L;
    double best = 0.0;
    for (int64_t b = int64_t(blockIdx.x) * WIND_THREADS; b < n; b += int64_t(WIND_BLOCKS) * WIND_THREADS) {
        const int64_t first = b / L;
        const unsigned x = unsigned(b - first * L) + threadIdx.x, dh = x / L;
        const int64_t h = first + dh;
        if (h >= m.n_h) break;
        const int k = level_pair(int(x - dh * L) * 2, m.nzn);
        const double px = hxy[2 * h], py = hxy[2 * h + 1];
        if (px < x0 || px > x1 || py < y0 || py > y1) continue;
        const vec u = *reinterpret_cast<const vec*>(q + fs + h * m.ldz + k);
        const vec v = *reinterpret_cast<const vec*>(q + 2 * fs + h * m.ldz + k);
        best = fmax(best, fmax(u.x * u.x + v.x * v.x, u.y * u.y + v.y * v.y));
    }
    for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < WIND_THREADS / 64; ++w) best = fmax(best, red[w]);
        part[blockIdx.x] = best;
    }
}

__global__ void __launch_bounds__(256)
k_max_wind_final(const double* __restrict__ part, int n, double* __restrict__ out) {
    __shared__ double red[4];
    double best = 0.0;
    for (int t = threadIdx.x; t < n; t += blockDim.x) best = fmax(best, part[t]);
    for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) *out = sqrt(fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
}

}  // namespace sem

namespace {
using sem::fail;

inline uint64_t ckey(int l, int64_t x, int64_t y) {
    return (uint64_t(l) << 58) | (uint64_t(x) << 29) | uint64_t(y);
}
}  // namespace

extern "C" {

static int amr_features_impl(const sem_mesh* M, const double* q, const double* q_prev, const int8_t* plain,
                 int criterion, const double* thr, int lvl_max, const float* scale, float* feat,
                 int8_t* dem, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!M->have_ref && !M->d.zs)
        return fail(SEM_ERR_STATE, "neither sem_mesh_set_reference nor sem_mesh_set_terrain has been called");
    if (!q || !q_prev || !plain || !feat || !dem || !scale) return fail(SEM_ERR_ARG, "null array");
    if (criterion != SEM_CRIT_SPEED && criterion != SEM_CRIT_VORTZ) return fail(SEM_ERR_ARG, "bad criterion");
    if (lvl_max < 0 || lvl_max > SEM_MAX_LEVEL) return fail(SEM_ERR_ARG, "lvl_max out of range");
    if (lvl_max > 0 && !thr) return fail(SEM_ERR_ARG, "null thresholds");
    sem::ThrF T{};
    for (int l = 0; l < lvl_max; ++l) {
        T.v[l] = thr[l];
        if (l > 0 && thr[l] < thr[l - 1]) return fail(SEM_ERR_ARG, "thresholds must be non-decreasing");
    }
    sem::Scale16 S{};
    for (int r = 0; r < SEM_NFEAT; ++r) S.v[r] = scale[r];
    const sem::DevMesh& d = M->d;
    hipStream_t s = (hipStream_t)stream;
    const int nb = d.n_col * d.n_z;
    switch (d.N) {
#define CASE(NN)                                                                              \
    case NN:                                                                                  \
        hipLaunchKernelGGL((sem::k_features<NN + 1>), dim3(unsigned(d.n_col) * sem::pass_chunks<NN + 1>(d.n_z)), \
                           dim3(sem::pass_threads<NN + 1>()), 0, s, d, q,                     \
                           q_prev, plain, criterion, T, lvl_max, S, feat, M->feat_aux, dem);  \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
        default: return fail(SEM_ERR_N, "unsupported N");
    }
    HIPCHK(hipGetLastError());
    const int grid = std::max(1, std::min((nb + 255) / 256, 65536));
    hipLaunchKernelGGL(sem::k_features_nbr, dim3(grid), dim3(256), 0, s, d, M->feat_aux, S, feat);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int amr_features(const sem_mesh* M, const double* q, const double* q_prev, const int8_t* plain,
                 int criterion, const double* thr, int lvl_max, const float* scale, float* feat,
                 int8_t* dem, void* stream) {
    return sem::guarded("amr_features", [&] { return amr_features_impl(M, q, q_prev, plain, criterion, thr, lvl_max, scale, feat, dem, stream); });
}

static int amr_forecast_flags_impl(const sem_mesh* M, const float* logits, const int8_t* plain, int lvl_max,
                       int8_t* ae, int8_t* ac, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!logits || !plain || !ae || !ac) return fail(SEM_ERR_ARG, "null array");
    if (ae == plain) return fail(SEM_ERR_ARG, "d_adapt_elem must not alias d_plain_elem");
    if (lvl_max < 0 || lvl_max > SEM_MAX_LEVEL) return fail(SEM_ERR_ARG, "lvl_max out of range");
    const sem::DevMesh& d = M->d;
    hipStream_t s = (hipStream_t)stream;
    const int nb = d.n_col * d.n_z;
    const int grid = std::max(1, std::min((nb + 255) / 256, 65536));
    hipLaunchKernelGGL(sem::k_forecast_elem, dim3(grid), dim3(256), 0, s, d, logits, plain, lvl_max, ae);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(sem::k_forecast_col, dim3((d.n_col + 255) / 256), dim3(256), 0, s, d, ae, ac);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int amr_forecast_flags(const sem_mesh* M, const float* logits, const int8_t* plain, int lvl_max,
                       int8_t* ae, int8_t* ac, void* stream) {
    return sem::guarded("amr_forecast_flags", [&] { return amr_forecast_flags_impl(M, logits, plain, lvl_max, ae, ac, stream); });
}

static int sem_max_wind_impl(const sem_mesh* M, const double* q, double x0, double x1, double y0, double y1,
                 double* vmax, void* stream) {
    if (!M) return fail(SEM_ERR_ARG, "null mesh");
    if (!q || !vmax) return fail(SEM_ERR_ARG, "null array");
    if (!(x0 <= x1 && y0 <= y1)) return fail(SEM_ERR_ARG, "empty box");
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(sem::k_max_wind, dim3(sem::WIND_BLOCKS), dim3(sem::WIND_THREADS), 0, s, M->d, q, M->d_hxy,
                       x0, x1, y0, y1, M->wind_part);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(sem::k_max_wind_final, dim3(1), dim3(256), 0, s, M->wind_part,
                       sem::WIND_BLOCKS, vmax);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int sem_max_wind(const sem_mesh* M, const double* q, double x0, double x1, double y0, double y1,
                 double* vmax, void* stream) {
    return sem::guarded("sem_max_wind", [&] { return sem_max_wind_impl(M, q, x0, x1, y0, y1, vmax, stream); });
}

static int sem_forecast_labels_impl(const sem_mesh_desc* at, const sem_mesh_desc* later, const int8_t* dem_later,
                        int8_t* cls) {
    if (!at || !later || !dem_later || !cls) return fail(SEM_ERR_ARG, "null argument");
    if (at->n_z != later->n_z || at->nx0 != later->nx0 || at->ny0 != later->ny0 || at->n_z < 1)
        return fail(SEM_ERR_ARG, "the two layouts differ in base grid or layers");
    const int nz = at->n_z;
    // later columns, and the largest dem per layer over the descendants of
    // every coarser cell
    std::unordered_map<uint64_t, int> col;
    std::unordered_map<uint64_t, std::vector<int8_t>> below;
    col.reserve(size_t(later->n_col) * 2);
    for (int c = 0; c < later->n_col; ++c) {
        const int l = later->h_col_level[c];
        const int64_t x = later->h_col_ix[c], y = later->h_col_iy[c];
        if (l < 0 || l > SEM_MAX_LEVEL) return fail(SEM_ERR_MESH, "bad level in the later layout");
        col[ckey(l, x, y)] = c;
        for (int a = l - 1; a >= 0; --a) {
            auto& v = below[ckey(a, x >> (l - a), y >> (l - a))];
            if (v.empty()) v.assign(nz, int8_t(-1));
            for (int z = 0; z < nz; ++z) v[z] = std::max(v[z], dem_later[int64_t(c) * nz + z]);
        }
    }
    for (int c = 0; c < at->n_col; ++c) {
        const int l = at->h_col_level[c];
        const int64_t x = at->h_col_ix[c], y = at->h_col_iy[c];
        int found = -1;
        for (int a = l; a >= 0 && found < 0; --a) {
            auto it = col.find(ckey(a, x >> (l - a), y >> (l - a)));
            if (it != col.end()) found = it->second;
        }
        const std::vector<int8_t>* desc = nullptr;
        if (found < 0) {
            auto it = below.find(ckey(l, x, y));
            if (it == below.end()) return fail(SEM_ERR_MESH, "a column of the first layout is not covered by the later one");
            desc = &it->second;
        }
        for (int z = 0; z < nz; ++z) {
            const int d = found >= 0 ? dem_later[int64_t(found) * nz + z] : (*desc)[z];
            cls[int64_t(c) * nz + z] = int8_t(std::max(-1, std::min(1, d - l)) + 1);
        }
    }
    return SEM_OK;
}

int sem_forecast_labels(const sem_mesh_desc* at, const sem_mesh_desc* later, const int8_t* dem_later,
                        int8_t* cls) {
    return sem::guarded("sem_forecast_labels", [&] { return sem_forecast_labels_impl(at, later, dem_later, cls); });
}

}  // extern "C"
