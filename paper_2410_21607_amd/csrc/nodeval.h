// Device helpers shared by the HIP translation units: the value of one field
// at an element-local horizontal slot (through the hanging rows when the slot
// is a hanging point), the column rule of the refinement flags and the
// pressure ratio.
#pragma once

#include <hip/hip_runtime.h>

#include "devmesh.h"

namespace sem {

// value of field f at horizontal slot g (unique node or hanging point) and kz,
// interpolating hanging points through their rows
__device__ __forceinline__ double node_value(const DevMesh& m, const double* __restrict__ q,
                                             int g, int f, int kz) {
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    if (g >= 0) return q[f * fs + int64_t(g) * m.ldz + kz];
    const int hh = -g - 1;
    double s = 0.0;
    for (int t = m.hang_ptr[hh]; t < m.hang_ptr[hh + 1]; ++t)
        s += m.hang_w[t] * q[f * fs + int64_t(m.hang_src[t]) * m.ldz + kz];
    return s;
}

// the same for several fields of one array: out[f] is field F0 + f
template <int F0, int NV>
__device__ __forceinline__ void node_values(const DevMesh& m, const double* __restrict__ q, int g, int kz,
                                            double* out) {
    const int64_t fs = int64_t(m.n_h) * m.ldz;
    if (g >= 0) {
#pragma unroll
        for (int f = 0; f < NV; ++f) out[f] = q[(F0 + f) * fs + int64_t(g) * m.ldz + kz];
        return;
    }
    const int hh = -g - 1;
#pragma unroll
    for (int f = 0; f < NV; ++f) out[f] = 0.0;
    for (int t = m.hang_ptr[hh]; t < m.hang_ptr[hh + 1]; ++t) {
        const double w = m.hang_w[t];
        const int64_t o = int64_t(m.hang_src[t]) * m.ldz + kz;
#pragma unroll
        for (int f = 0; f < NV; ++f) out[f] += w * q[(F0 + f) * fs + o];
    }
}

// Element passes of the refinement side (flags, features): a workgroup takes
// `layers` stacked elements of a column (at most pass_layers), a thread per
// horizontal position and layer.  The nodes are loaded row by row, kz fastest
// and shared planes once, into tiles of pass_stride levels per position (odd,
// against bank conflicts); a thread then walks its position's N+1 nodes of one
// element and keeps the element's maxima in registers, so that they are
// reduced over (N+1)^2 threads and not (N+1)^3.
template <int NP>
constexpr int pass_layers() {
    return NP == 2 ? 16 : NP <= 4 ? 8 : NP == 5 ? 4 : NP == 6 ? 3 : NP == 7 ? 2 : 1;
}
template <int NP>
constexpr int pass_threads() {
    return (NP * NP * pass_layers<NP>() + 63) / 64 * 64;
}
template <int NP>
constexpr int pass_stride() {
    return (pass_layers<NP>() * (NP - 1) + 1) | 1;
}
// workgroups per column, and the layers each takes (balanced)
template <int NP>
__host__ __device__ constexpr int pass_chunks(int n_z) {
    return (n_z + pass_layers<NP>() - 1) / pass_layers<NP>();
}
struct PassItem {
    int c, layer0, layers;      // column, first layer, number of layers
};
template <int NP>
__device__ __forceinline__ PassItem pass_item(const DevMesh& m) {
    const int nc = pass_chunks<NP>(m.n_z), c = int(blockIdx.x) / nc, x = int(blockIdx.x) - c * nc;
    const int a = int(int64_t(x) * m.n_z / nc), b = int(int64_t(x + 1) * m.n_z / nc);
    return {c, a, b - a};
}

// Column rule of the refinement flags (Section 4.1 refines and coarsens whole
// columns): +1 if any element of column c is +1; -1 if every element of the
// column and of its three siblings is -1; else 0.
__device__ __forceinline__ int8_t column_rule(const DevMesh& m, const int8_t* __restrict__ ae, int c) {
    auto col_state = [&](int cc, bool& any_ref, bool& all_crs) {
        any_ref = false;
        all_crs = true;
        for (int z = 0; z < m.n_z; ++z) {
            const int8_t a = ae[cc * m.n_z + z];
            any_ref = any_ref || (a == 1);
            all_crs = all_crs && (a == -1);
        }
    };
    bool r, cr;
    col_state(c, r, cr);
    if (r) return 1;
    if (cr && m.sib[4 * c] >= 0) {
        bool ok = true;
        for (int s = 0; s < 4; ++s) {
            bool r2, c2;
            col_state(m.sib[4 * c + s], r2, c2);
            ok = ok && c2 && !r2;
        }
        if (ok) return -1;
    }
    return 0;
}

// (1+x)^gamma - 1 for the ideal-gas pressure ratio.  For |x| <= 1/64 the
// Taylor polynomial sum_{n=1..10} C(gamma, n) x^n is used (the first neglected
// term is below 2^-66 |gamma x|, far under one ulp); otherwise
// expm1(gamma log1p(x)).  That general branch is kept out of line: inlined,
// the compiler hoists its polynomial constants out of the chunk loop, where
// they hold about 30 registers for the whole kernel.
static __device__ __noinline__ double pow1p_minus1_far(double x, double gamma) {
    return expm1(gamma * log1p(x));
}
__device__ __forceinline__ double pow1p_minus1_near(const DevMesh& m, double x) {
    double s = m.binom[10];
#pragma unroll
    for (int n = 9; n >= 1; --n) s = s * x + m.binom[n];
    return s * x;
}
__device__ __forceinline__ double pow1p_minus1(const DevMesh& m, double x) {
    return fabs(x) <= 1.0 / 64.0 ? pow1p_minus1_near(m, x) : pow1p_minus1_far(x, m.gamma);
}

}  // namespace sem
