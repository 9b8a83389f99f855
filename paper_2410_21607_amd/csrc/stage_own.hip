// Owner kernel of the fused Runge-Kutta stage (gfx950, FP64, box elements):
// every regular node (stage_fused.h) is computed whole, by the one column that
// owns it, in one launch.
//
// The column kernel of stage_fused.hip sums the shared nodes of neighbouring
// columns through memory: four colour launches, 25 of 16 rows of q_s read and
// of q_out written per column at N = 4, 9 of them read again.  Here a column
// computes the N x N positions at its left and lower sides and their share of
// every element around them.  What that needs from the neighbours is small: on
// a face between two columns of one level the elements' tendencies differ only
// in the derivative across it, so a face node takes the mean of the two
// columns' derivatives (equal masses), and the neighbour's comes from one line
// of N nodes per face node, the halo lines.  They are reduced to their sums of
// D(N, m) f_m while they are loaded, so that the tiles hold the column's own
// nodes only.  q_out is written once; q_s is read from beyond the L2 about 1.5
// times (most halo lines are in it: an XCD's columns are neighbours).
//
// A workgroup marches up its column in chunks of LPC elements, a thread per
// owned node:
//   * the loads of a chunk are requested while the previous one is computed;
//   * p' and the tiles (Section 2's pointwise fields) are formed; barrier;
//   * derivatives along z, x and y from the tiles, the tendency and the update;
//     a plane between two elements takes their z derivatives weighted by their
//     depths, the plane between two chunks through LDS; the last chunk also
//     finishes the top lid; barrier.
//
// What bounds it (N = 4, 64 x 64 x 16 elements): 178 us per stage against 231
// for the four colour launches, 0.69 GB of traffic per stage against 0.99
// (0.52 read, 0.18 written; 136 us at the copy rate).  Without any loads and
// stores the kernel takes 131 us, VALU issue is 40 % and LDS 31 % of the time,
// 10 of 12 waves per CU resident: memory and on-chip work overlap but for the
// latency of the chunk's chain load - tiles - barrier - derivatives.
#include "stage_fused.h"

#include <hip/hip_runtime.h>

#include "nodeval.h"
#include "rows.h"
#include "sem.h"

namespace sem {

namespace {

constexpr int NF = SEM_NFIELDS;

template <int NP, int LPC>
constexpr int own_threads() {
    constexpr int N = NP - 1, PARTS = N > 5 ? 2 : 1;
    constexpr int c = own_owned(N) * LPC * N, h = 2 * N * PARTS * LPC * N;
    return ((c > h ? c : h + 1) + 63) / 64 * 64;
}

// State arrays are read and written through buffer descriptors: a lane with
// nothing to load or store takes the offset NOWHERE (rows.h), which the hardware's
// range check drops, so that every load and store is issued unconditionally.  Behind
// a branch the compiler cannot count them and waits for all of them (the next
// chunk's loads and earlier stores included) at each use: 194 us per stage
// against 177 on 64 x 64 x 16 elements at N = 4.  32-bit byte offsets: the
// five fields have to fit in 2 GiB (own_fits).
using rsrc_t = __amdgpu_buffer_rsrc_t;
using u32x2 = __attribute__((ext_vector_type(2))) unsigned;
__device__ __forceinline__ rsrc_t state_rsrc(const double* p, int64_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0, int(n * 8), 0x00020000);
}
__device__ __forceinline__ double state_load(rsrc_t r, unsigned off, unsigned field) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, field, 0));
}
__device__ __forceinline__ void state_store(rsrc_t r, double x, unsigned off, unsigned field) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, off, field, 0);
}
// the state's descriptor sees a store of the caller's array, never one of the
// kernel's own loads: q_out aliases neither q_s nor q^n

// Three waves per SIMD: the FP64 chain needs about 150 registers; held to 128
// (four waves) it spills the requested loads and runs at 216 us.
template <int NP, int LPC>
__global__ void __launch_bounds__((own_threads<NP, LPC>()), 3)
k_stage_own(DevMesh m, OwnTables ot, double a, double b, double c, const double* __restrict__ qn,
            const double* __restrict__ qs, double* __restrict__ qo) {
    constexpr int N = NP - 1, P2 = own_owned(N), HS = own_positions(N);
    constexpr int NB = LPC * N;                   // levels of a full chunk below its top plane
    constexpr int WGT = own_threads<NP, LPC>();
    // roles while loading: a thread per halo line (or part of one, of HN
    // nodes) and level, the others the column's own nodes
    constexpr int PARTS = N > 5 ? 2 : 1, HN = (N + PARTS - 1) / PARTS;
    constexpr int HL = 2 * N * PARTS, HT = HL * NB, OT = WGT - HT;
    constexpr int PO = P2 + 2 * N;                // the column's positions in the tiles
    // their tile entries: levels below the top plane, then the top planes (of
    // the owned positions; in the last chunk, whose top is the lid, of all)
    constexpr int TN = PO * NB + HS;
    constexpr int OS = (TN + OT - 1) / OT, SLOTS = OS > HN ? OS : HN;
    static_assert(OT > 0, "threads for the column's own nodes");
    __shared__ double2 t_uv[TN], t_wt[TN], t_rp[TN];   // (u, v), (w, theta'), (rho, p')
    __shared__ double2 h_a[HT], h_b[HT], h_c[HT];      // halo sums: momentum across the face, u; v, w; theta', p'
    __shared__ double s_q[P2 * NB + P2];               // rho' of the owned nodes (the rest of their state is in the tiles)
    __shared__ double carry[2][6][P2];
    __shared__ double2 sDxy[P2 * NP];
    __shared__ double sD[NP * NP];
    __shared__ unsigned s_row[HS];                     // row_offset
    // what only the columns with hanging positions and far pressures need
    struct Slow {
        const int32_t *ptr, *src;
        const double* w;
        double gamma;
    };
    __shared__ Slow s_slow;
    __shared__ double s_bin[10];                       // C(gamma, n), n = 1..10
    // the mesh's level table: rho0, 1/rho0, 1/theta0, p0, dtheta0/dz, the share
    // of the element below in a plane between two (by their depths, which is
    // its share of the plane's lumped mass) per level; 2/dz per layer
    extern __shared__ double s_lev[];
    int tc = threadIdx.x;
    const int nzn = m.nzn;
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    const unsigned fb = unsigned(fs) * 8u;        // bytes of a field
    const rsrc_t rs = state_rsrc(qs, NF * fs), rn = state_rsrc(qn, NF * fs), ro = state_rsrc(qo, NF * fs);
    // columns of one XCD contiguous in the (Morton-ordered) list
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7;
    const int item = xcd * (G >> 3) + min(xcd, G & 7) + (blockIdx.x >> 3);

    for (int t = tc; t < HS; t += WGT) s_row[t] = ot.map[int64_t(item) * HS + t];
    for (int t = tc; t < 7 * nzn; t += WGT) s_lev[t] = m.lev[t];
    for (int t = tc; t < NP * NP; t += WGT) sD[t] = m.D[t];
    for (int t = tc; t < 2 * 6 * P2; t += WGT) (&carry[0][0][0])[t] = 0.0;
    if (tc < 10) s_bin[tc] = m.binom[tc + 1];
    if (tc == 0) s_slow = {m.hang_ptr, m.hang_src, m.hang_w, m.gamma};
    for (int t = tc; t < P2 * NP; t += WGT) {
        const int p = t / NP, k = t - p * NP;
        sDxy[t].x = m.D[(p % N) * NP + k];
        sDxy[t].y = m.D[(p / N) * NP + k];
    }
    const double sx = ot.sxy[2 * item], sy = ot.sxy[2 * item + 1];
    const unsigned long long mask = ot.mask[item];
    const bool hanging = ot.hang[item] != 0;
    __syncthreads();

    // position and level of the s-th node that thread t loads: a halo thread
    // the nodes of its line; the others the column's nodes position by
    // position, then the top planes.  nk: elements of the chunk times N (its
    // top level, -1 past the last chunk); tops: positions whose top plane is
    // loaded with a full chunk (all in the last one, whose top is the lid).
    // Selects only: a branch here would stand between the loads.
    auto place = [&](int t, int s, int nk, int tops, int& ps, int& kz) {
        const int l = t / NB, e = t - HT + s * OT, en = e / NB;
        const int kh = t - l * NB, kn = e - en * NB;
        const int line = l / PARTS, mm = s + (l - line * PARTS) * HN;
        const bool halo = t < HT;
        ps = halo ? PO + line * N + mm : en;
        kz = halo ? kh : kn;
        const int lim = halo & ((s >= HN) | (mm >= N)) ? -1 : s < OS ? nk : halo ? nk : -1;
        bool ok = kz <= lim;
        if ((s + 1) * OT > PO * NB) {             // a slot that holds top planes
            const bool top = !halo & (e >= PO * NB);
            const int pt = e - PO * NB;
            ps = top ? pt : ps;
            kz = top ? NB : kz;
            ok = top ? (nk == NB) & (pt < tops) : ok;
        }
        ps = ok ? ps : 0;
        kz = ok ? kz : 0;
        return ok;
    };
    double pf[SLOTS][NF];
    auto request = [&](int t, int L) {
        const int left = m.n_z - L, nk = left > 0 ? min(LPC, left) * N : -1;
        const int tops = left <= LPC ? HS : P2;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int ps, kz;
            const bool ok = place(t, s, nk, tops, ps, kz);
            const unsigned row = s_row[ps] + unsigned(L * N + kz) * 8u;
            const unsigned off = ok ? row : NOWHERE;
#pragma unroll
            for (int f = 0; f < NF; ++f) pf[s][f] = state_load(rs, off, f * fb);
        }
    };
    request(tc, 0);
    // (dropped stores, so that the first pass through the loop has the same
    // accesses outstanding as the others: the compiler then need not wait for
    // the stores of a chunk before the loads of the next are used)
#pragma unroll
    for (int f = 0; f < NF; ++f) state_store(ro, 0.0, NOWHERE, f * fb);

    for (int L0 = 0, ch = 0;; L0 += LPC, ++ch) {
        // the thread's index as the loop sees it: opaque, so that the addresses
        // derived from it are formed where they are used instead of being
        // held in registers across the loop
        asm volatile("" : "+v"(tc));
        const int nel = min(LPC, m.n_z - L0), nk = nel * N;
        const int L1 = L0 + nel;
        const bool last = L1 == m.n_z;
        const int tops = last ? HS : P2;
        const double* sb = s_lev + L0 * N;
        const double* sz8 = s_lev + 6 * nzn + L0;
        // one node's part of its halo line's sums; l: the thread's line part
        auto add_halo = [&](int s, int l, int kz, const double* q, double pp, double* d) {
            const int mm = s + l % PARTS * HN;
            const double cs = mm < N ? sD[N * NP + mm] : 0.0, u = q[1], v = q[2];
            d[0] += cs * ((sb[kz] + q[0]) * (l < N * PARTS ? u : v));
            d[1] += cs * u;
            d[2] += cs * v;
            d[3] += cs * q[3];
            d[4] += cs * q[4];
            d[5] += cs * pp;
        };
        auto put_halo = [&](const double* d) {
            h_a[tc] = double2{d[0], d[1]};
            h_b[tc] = double2{d[2], d[3]};
            h_c[tc] = double2{d[4], d[5]};
        };
        auto put_node = [&](int ps, int kz, const double* q, double pp) {
            const int o = kz == NB ? PO * NB + ps : ps * NB + kz;
            t_uv[o] = double2{q[1], q[2]};
            t_wt[o] = double2{q[3], q[4]};
            t_rp[o] = double2{sb[kz] + q[0], pp};
            if (ps < P2) s_q[kz == NB ? P2 * NB + ps : o] = q[0];
        };
        // pointwise fields of the loaded nodes (Section 2)
        bool far = false;
        if (!hanging) {
            // p' (pow1p_minus1's polynomial, the nodes side by side)
            double x[SLOTS], pr[SLOTS];
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                int ps, kz;
                const bool ok = place(tc, s, nk, tops, ps, kz);
                const double ra = pf[s][0] * sb[nzn + kz], tb = pf[s][4] * sb[2 * nzn + kz];
                x[s] = ra + tb + ra * tb;
                pr[s] = s_bin[9];
                far |= ok & !(fabs(x[s]) <= 1.0 / 64.0);
            }
#pragma unroll
            for (int n = 8; n >= 0; --n)
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) pr[s] = pr[s] * x[s] + s_bin[n];
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                int ps, kz;
                place(tc, s, nk, tops, ps, kz);
                pr[s] = sb[3 * nzn + kz] * (pr[s] * x[s]);
            }
            if (tc < HT) {
                double d[6] = {0, 0, 0, 0, 0, 0};
                const int l = tc / NB;
#pragma unroll
                for (int s = 0; s < HN; ++s) add_halo(s, l, tc - l * NB, pf[s], pr[s], d);
                put_halo(d);
            } else {
#pragma unroll
                for (int s = 0; s < OS; ++s) {
                    int ps, kz;
                    if (place(tc, s, nk, tops, ps, kz)) put_node(ps, kz, pf[s], pr[s]);
                }
            }
        }
        if (far || hanging) {
            // columns with hanging positions, which take the coarse face's
            // interpolant, and nodes whose pressure is outside the
            // polynomial's range (rare): node by node from the state
            const Slow S = s_slow;
            double d[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 1
            for (int s = 0; s < SLOTS; ++s) {
                int ps, kz;
                if (!place(tc, s, nk, tops, ps, kz)) continue;
                const unsigned r = s_row[ps];
                const bool direct = r < NOWHERE;
                const int hh = direct ? 0 : row_hanging(r);
                const int t0 = direct ? 0 : S.ptr[hh], t1 = direct ? 1 : S.ptr[hh + 1];
                double q[NF] = {0, 0, 0, 0, 0};
#pragma unroll 1
                for (int t = t0; t < t1; ++t) {
                    const double w = direct ? 1.0 : S.w[t];
                    const double* src = qs + (direct ? int64_t(r / 8u) : int64_t(S.src[t]) * m.ldz) + (L0 * N + kz);
#pragma unroll
                    for (int f = 0; f < NF; ++f) q[f] += w * src[f * fs];
                }
                const double ra = q[0] * sb[nzn + kz], tb = q[4] * sb[2 * nzn + kz];
                const double x = ra + tb + ra * tb;
                double pp = s_bin[9];
                for (int n = 8; n >= 0; --n) pp = pp * x + s_bin[n];
                pp = sb[3 * nzn + kz] * (fabs(x) <= 1.0 / 64.0 ? pp * x : pow1p_minus1_far(x, S.gamma));
                if (tc < HT) add_halo(s, tc / NB, kz, q, pp, d);
                else put_node(ps, kz, q, pp);
            }
            if (tc < HT) put_halo(d);
        }
        __syncthreads();
        asm volatile("" : "+v"(tc));
        // this thread's node, in natural order
        const int p = tc / NB, kzl = tc - p * NB;
        const bool lane_ok = p < P2;
        const int pc = lane_ok ? p : 0;
        const int i = pc % N, j = pc / N;
        const bool active = lane_ok && kzl < nk;
        // requested one phase early: the update base and the next chunk
        double base[NF];
        {
            const bool mine = active && ((mask >> pc) & 1) && a != 0.0;
            const unsigned an = mine ? s_row[pc] + unsigned(L0 * N + kzl) * 8u : NOWHERE;
#pragma unroll
            for (int f = 0; f < NF; ++f) base[f] = state_load(rn, an, f * fb);
        }
        request(tc, L1);
        // Sums over the taps of one direction, at entries o0 + k step (the last
        // at oN), of the six fields that a direction differentiates: the
        // momentum of its own velocity, u, v, w, theta', p'.  The empty asm
        // keeps the LDS reads of the next direction behind it.
        auto taps = [&](int o0, int step, int oN, auto coef, auto vel, double* d) {
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int ok = k < N ? o0 + k * step : oN;
                const double ck = coef(k);
                const double2 a1 = t_uv[ok], a2 = t_wt[ok], a3 = t_rp[ok];
                d[0] += ck * (a3.x * vel(a1, a2));
                d[1] += ck * a1.x;
                d[2] += ck * a1.y;
                d[3] += ck * a2.x;
                d[4] += ck * a2.y;
                d[5] += ck * a3.y;
            }
            asm volatile("" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]), "+v"(d[4]), "+v"(d[5]) : : "memory");
        };
        // z, of element el at its level kk, times w8
        auto taps_z = [&](int pc, int el, int kk, double w8, double* d) {
            const int o0 = pc * NB + el * N;
            const double sz = w8 * sz8[el];
            taps(o0, 1, el == LPC - 1 ? PO * NB + pc : o0 + N, [&](int k) { return sz * sD[kk * NP + k]; },
                 [](double2, double2 a2) { return a2.x; }, d);
        };
        // sums of halo line l at level kz of the chunk
        auto sums = [&](int l, int kz, double* d) {
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
                const int o = (l * PARTS + part) * NB + kz;
                const double2 y0 = h_a[o], y1 = h_b[o], y2 = h_c[o];
                d[0] += y0.x;
                d[1] += y0.y;
                d[2] += y1.x;
                d[3] += y1.y;
                d[4] += y2.x;
                d[5] += y2.y;
            }
        };
        // tendency of the node in tile entry o (rho' rp) from its z
        // derivatives, then its x and y ones: x0, xN, y0, yN, step give its
        // lines, halo its halo lines' sums.  A node on the column's left
        // (lower) face takes the mean of the two columns' x (y) derivatives.
        auto tendency = [&](int pc, int o, int x0, int xN, int y0, int yN, int step, auto halo, double rp, double dt0,
                            const double* z, double* R) {
            const int i = pc % N, j = pc / N;
            const double2 uv = t_uv[o], wt = t_wt[o], rq = t_rp[o];
            const double u = uv.x, v = uv.y, w = wt.x, ir = 1.0 / rq.x;
            R[0] = -z[0];
            R[1] = m.f * v - w * z[1];
            R[2] = -m.f * u - w * z[2];
            R[3] = -w * z[3] - z[5] * ir - rp * ir * m.g;
            R[4] = -w * z[4] - w * dt0;
#pragma unroll
            for (int dir = 0; dir < 2; ++dir) {
                const bool face = dir == 0 ? i == 0 : j == 0;
                double d[6] = {0, 0, 0, 0, 0, 0};
                if (face) {
                    const double cN = sD[NP * NP - 1];
                    halo(dir, d);
                    d[0] += cN * (rq.x * (dir == 0 ? u : v));
                    d[1] += cN * u;
                    d[2] += cN * v;
                    d[3] += cN * w;
                    d[4] += cN * wt.y;
                    d[5] += cN * rq.y;
                }
                taps(dir == 0 ? x0 : y0, dir == 0 ? step : N * step, dir == 0 ? xN : yN,
                     [&](int k) { return dir == 0 ? sDxy[pc * NP + k].x : sDxy[pc * NP + k].y; },
                     [&](double2 a1, double2) { return dir == 0 ? a1.x : a1.y; }, d);
                const double h = (face ? 0.5 : 1.0) * (dir == 0 ? sx : sy), vel = h * (dir == 0 ? u : v);
                R[0] -= d[0] * h;
                R[1] -= vel * d[1];
                R[2] -= vel * d[2];
                R[3] -= vel * d[3];
                R[4] -= vel * d[4];
                R[1 + dir] -= d[5] * (h * ir);
            }
        };
        auto update = [&](int o, double rp, unsigned ao, const double* base, const double* R) {
            const double2 uv = t_uv[o], wt = t_wt[o];
            const double q[NF] = {rp, uv.x, uv.y, wt.x, wt.y};
#pragma unroll
            for (int f = 0; f < NF; ++f) state_store(ro, a * base[f] + b * q[f] + c * R[f], ao, f * fb);
        };
        // (idle lanes compute the node of a valid one)
        // z: a plane between two elements takes their derivatives by weight.
        // The lanes of such planes run the pass of the element below; those of
        // the chunk's lowest plane, whose element below is in the previous
        // chunk, run the chunk's top element instead and hand it on.  With one
        // element per chunk no wave needs that second pass but the last one,
        // which runs it a lane per position.
        double R[NF];
        {
            const int kc = active ? kzl : 0, el = kc / N, kk = kc - el * N, o = pc * NB + kc;
            const double wl = sb[5 * nzn + kc];
            double z[6] = {0, 0, 0, 0, 0, 0};
            if constexpr (LPC == 1) {
                if (tc >= WGT - 64 && tc - (WGT - 64) < P2) {
                    const int pe = tc - (WGT - 64);
                    taps_z(pe, 0, N, 1.0, z);
#pragma unroll
                    for (int f = 0; f < 6; ++f) {
                        carry[ch & 1][f][pe] = z[f];
                        z[f] = 0.0;
                    }
                }
                if (kk == 0) {
#pragma unroll
                    for (int f = 0; f < 6; ++f) z[f] = wl * carry[~ch & 1][f][pc];
                }
            } else if (kk == 0) {
                taps_z(pc, kc == 0 ? nel - 1 : el - 1, N, kc == 0 ? 1.0 : wl, z);
                if (kc == 0) {
#pragma unroll
                    for (int f = 0; f < 6; ++f) {
                        const double up = z[f];
                        z[f] = wl * carry[~ch & 1][f][pc];
                        if (active) carry[ch & 1][f][pc] = up;
                    }
                }
            }
            taps_z(pc, el, kk, 1.0 - (kk == 0 ? wl : 0.0), z);
            tendency(pc, o, N * j * NB + kc, (P2 + j) * NB + kc, i * NB + kc, (P2 + N + i) * NB + kc, NB,
                     [&](int dir, double* d) { sums(dir == 0 ? j : N + i, kc, d); }, s_q[o], sb[4 * nzn + kc], z, R);
        }
        {
            // (the node again from the opaque index rather than held)
            asm volatile("" : "+v"(tc));
            const int p = tc / NB, pc = p < P2 ? p : 0, kzl = tc - p * NB;
            const bool mine = p < P2 && kzl < nk && ((mask >> pc) & 1);
            const int o = pc * NB + (kzl < nk ? kzl : 0);
            const unsigned ao = mine ? s_row[pc] + unsigned(L0 * N + kzl) * 8u : NOWHERE;
            if (L0 + kzl == 0) R[3] = 0.0;        // the bottom lid
            update(o, s_q[o], ao, base, R);
        }
        if (last) {
            // The top lid, a lane of the last wave per position: the last
            // element's z derivatives, this level's x and y ones.  (In the loop's exit and
            // from the opaque index, so that nothing is held for it across
            // the chunks.)
            asm volatile("" : "+v"(tc));
            if (LPC > 1) __syncthreads();
            if (tc >= WGT - 64 && tc - (WGT - 64) < P2) {
                const int pc = tc - (WGT - 64), i = pc % N, j = pc / N;
                const unsigned al = ((mask >> pc) & 1) ? s_row[pc] + unsigned(L1 * N) * 8u : NOWHERE;
                double bl[NF], z[6], RL[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) bl[f] = state_load(rn, a != 0.0 ? al : NOWHERE, f * fb);
#pragma unroll
                for (int f = 0; f < 6; ++f) z[f] = carry[ch & 1][f][pc];
                // entries of the top planes follow the other levels
                const bool full = nk == NB;
                const int st = full ? 1 : NB, e0 = full ? PO * NB : nk;
                const int ol = e0 + pc * st;
                const double rp = s_q[full ? P2 * NB + pc : ol];
                tendency(pc, ol, e0 + N * j * st, e0 + (P2 + j) * st, e0 + i * st, e0 + (P2 + N + i) * st, st,
                         [&](int dir, double* d) {
                             const int l = dir == 0 ? j : N + i;
                             if (!full) return sums(l, nk, d);
#pragma unroll
                             for (int s = 0; s < N; ++s) {
                                 const int oh = PO * NB + PO + l * N + s;
                                 const double cs = sD[N * NP + s];
                                 const double2 a1 = t_uv[oh], a2 = t_wt[oh], a3 = t_rp[oh];
                                 d[0] += cs * (a3.x * (dir == 0 ? a1.x : a1.y));
                                 d[1] += cs * a1.x;
                                 d[2] += cs * a1.y;
                                 d[3] += cs * a2.x;
                                 d[4] += cs * a2.y;
                                 d[5] += cs * a3.y;
                             }
                         }, rp, sb[4 * nzn + nk], z, RL);
                RL[3] = 0.0;
                update(ol, rp, al, bl, RL);
            }
            break;
        }
        __syncthreads();
    }
}

// (order, layers per chunk) instances, the fastest that was measured of each
// order: up to N = 4 chunks of 16 or 24 levels, at N = 5 and 6 of 10 and 6, which
// leave three workgroups per CU as N = 3 and 4 have; N = 7 and 8 have one (704 and
// 512 threads of about 150 registers).  us per stage with other chunks: N = 3 (64 x 64 x 16 elements) 4: 102,
// 8: 97; N = 4 8: 246, 4: 181; N = 5 (48 x 48 x 16) 1: 416, 2: 281, 4: 298;
// N = 6 (40 x 40 x 12) 1: 317, 2: 327; N = 7 (28 x 28 x 8) 1: 231, 2: 177: a
// layer's 56 bytes of a row keep every line waiting in the L2 for the next
// chunk, and more of them than it holds.
#define SEM_OWN_INSTANCES(X) X(2, 8) X(3, 8) X(4, 4) X(5, 2) X(6, 1) X(7, 2) X(8, 1)

}  // namespace

bool own_supported(int N) {
    switch (N) {
#define CASE(NN, LP) case NN: return true;
        SEM_OWN_INSTANCES(CASE)
#undef CASE
        default: return false;
    }
}

bool own_fits(int64_t n_h, int ldz, int nzn) { return NF * n_h * ldz * 8 < (int64_t(1) << 31) && nzn <= 512; }

int own_launch(const DevMesh& m, const OwnTables& ot, double a, double b, double c, const double* qn,
               const double* qs, double* qo, hipStream_t s) {
    if (ot.n == 0) return SEM_OK;
    const size_t lds = size_t(7) * m.nzn * sizeof(double);
    switch (m.N) {
#define CASE(NN, LP)                                                                                   \
    case NN:                                                                                           \
        hipLaunchKernelGGL((k_stage_own<NN + 1, LP>), dim3(ot.n), dim3(own_threads<NN + 1, LP>()), lds, s, \
                           m, ot, a, b, c, qn, qs, qo);                                                \
        break;
        SEM_OWN_INSTANCES(CASE)
#undef CASE
        default: return SEM_ERR_ARG;
    }
    return hipGetLastError() == hipSuccess ? SEM_OK : SEM_ERR_HIP;
}

}  // namespace sem
