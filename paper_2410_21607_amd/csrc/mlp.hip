// Multilayer perceptron of the refinement forecaster (gfx950, FP32):
// 16 -> 64 -> 64 -> 3 with tanh, softmax cross-entropy, Adam.
//
// Parameters are one flat float array: W1[64][16], b1[64], W2[64][64], b2[64],
// W3[3][64], b3[3] (5443 floats, staged in LDS by every workgroup).
//
// A workgroup (four waves) takes tiles of 16 samples; wave w owns the 16 hidden
// units 16w..16w+15 of both layers.  The layers are matrix products with 16
// samples as columns, on the FP32 matrix instruction 16x16x4 (FP32 products
// and sums): a lane holds its unit's weights in registers as the A operand,
// the B operand is the input row or the LDS tile of the previous layer.  One
// thread per sample, as before, ran the 10,000 multiply-adds of a sample as
// one chain on n/64 waves: 4 workgroups for a training batch.
//
// Training step = three launches:
//   k_mlp_samples : forward pass, softmax, the per-sample back-propagated
//                   errors of the three layers and the sample's loss, written
//                   to the workspace;
//   k_mlp_grad    : the batch sum of every parameter's gradient: a workgroup
//                   per 16 x 16 tile of a weight matrix, on the FP64 matrix
//                   instruction (products of floats are exact in it), waves
//                   over interleaved samples combined in a fixed order
//                   (deterministic);
//   k_adam        : element-wise Adam update.
// Measured on an MI355X at 1024 samples: k_mlp_samples 7 us (63 before),
// k_mlp_grad 11 (38, a thread per parameter and batch segment); k_mlp_forward
// on 49,760 rows 16 us (58).  A training step is then paced by its three
// launches.
#include <cmath>
#include <cstdint>
#include <mutex>

#include "handle.h"

namespace sem {

namespace {

constexpr int NI = SEM_MLP_IN, NH = SEM_MLP_HIDDEN, NO = SEM_MLP_OUT;
constexpr int OW1 = 0, OB1 = OW1 + NH * NI, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NO * NH, NP = OB3 + NO;
static_assert(NP == SEM_MLP_NPARAM, "parameter count");
// workspace per sample: h1, h2, d1, d2 (64 each), d3 (3), loss (1)
constexpr int WH1 = 0, WH2 = WH1 + NH, WD1 = WH2 + NH, WD2 = WD1 + NH, WD3 = WD2 + NH,
              WL = WD3 + NO, WN = WL + 1;
static_assert(WN == SEM_MLP_WORK, "workspace per sample");

constexpr int TS = 16;             // samples per tile
constexpr int HS = NH + 4;         // LDS row stride of a sample's hidden values

using f4 = __attribute__((ext_vector_type(4))) float;
using d4 = __attribute__((ext_vector_type(4))) double;

// four consecutive floats: one 16-byte access where the caller's array is
// 16-byte aligned (AL), else four of 4 bytes (a view into a larger array)
template <bool AL>
__device__ __forceinline__ f4 ld4(const float* __restrict__ p) {
    if constexpr (AL) return *reinterpret_cast<const f4*>(p);
    else return f4{p[0], p[1], p[2], p[3]};
}
template <bool AL>
__device__ __forceinline__ void st4(float* __restrict__ p, f4 v) {
    if constexpr (AL) *reinterpret_cast<f4*>(p) = v;
    else { p[0] = v[0]; p[1] = v[1]; p[2] = v[2]; p[3] = v[3]; }
}

// lane = 16 g + c of wave w.  A operand of a step: row c, k = g; B: k = g,
// column c; accumulator: rows 4 g + 0..3, column c.  Step q has the products
// k = 4 q + g, and the instruction adds its four in that order, one rounding
// each: every sum is the chain over k = 0, 1, ... that a scalar loop forms, to
// the bit.  (Adam's first steps turn the rounding of a small gradient into a
// step of the learning rate, so that another order shows in the parameters.)
struct Lane { int w, g, c; };
__device__ __forceinline__ Lane lane_of(int t) { return {t >> 6, (t >> 4) & 3, t & 15}; }

// The 4 x 4 transpose of the values v[s] of the lanes g = 0..3 of a column:
// lane g's v[s] becomes lane s's v[g] (halves, then quarters of the wave
// exchanged).  Turns four consecutive values 16 t + 4 g + s into those of four
// steps, 16 t + 4 s + g, and back.
__device__ __forceinline__ f4 turn(f4 v) {
    using u2 = __attribute__((ext_vector_type(2))) unsigned;
    unsigned x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = __float_as_uint(v[s]);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const u2 y = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(x[s], x[s + 2], false, false));
        x[s] = y.x;
        x[s + 2] = y.y;
    }
#pragma unroll
    for (int s = 0; s < 4; s += 2) {
        const u2 y = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(x[s], x[s + 1], false, false));
        x[s] = y.x;
        x[s + 1] = y.y;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = __uint_as_float(x[s]);
    return v;
}
// Hidden values of a sample in LDS: value 16 t + 4 s + g at 16 t + 4 g + s, so
// that a lane's values of four steps are consecutive.
__device__ __forceinline__ void put_hidden(float* row, Lane l, f4 v) {
    *reinterpret_cast<f4*>(row + 16 * l.w + 4 * l.g) = turn(v);
}
// sum over the 64 hidden values: a += A[k] B[k]
__device__ __forceinline__ f4 chain(const float* A, const float* row, Lane l, f4 a) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f4 h = *reinterpret_cast<const f4*>(row + 16 * t + 4 * l.g);
#pragma unroll
        for (int s = 0; s < 4; ++s) a = __builtin_amdgcn_mfma_f32_16x16x4f32(A[4 * t + s], h[s], a, 0, 0, 0);
    }
    return a;
}
// this lane's share of the parameters
struct Weights {
    f4 w1, b1, b2, b3, w3[NO];     // w3: of the lane's hidden units
    float w2[16], z3[16];          // z3: row c of the output layer (c < NO)
    template <bool AL>
    __device__ __forceinline__ void load(const float* __restrict__ p, Lane l) {
        const int row = 16 * l.w + l.c, r4 = 16 * l.w + 4 * l.g;
        w1 = turn(ld4<AL>(p + OW1 + row * NI + 4 * l.g));
        b1 = ld4<AL>(p + OB1 + r4);
        b2 = ld4<AL>(p + OB2 + r4);
        const int o = min(l.c, NO - 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f4 a = turn(ld4<AL>(p + OW2 + row * NH + 16 * t + 4 * l.g));
            const f4 b = turn(ld4<AL>(p + OW3 + o * NH + 16 * t + 4 * l.g));
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                w2[4 * t + s] = a[s];
                z3[4 * t + s] = b[s];
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) b3[r] = p[OB3 + min(r, NO - 1)];
#pragma unroll
        for (int r = 0; r < NO; ++r) w3[r] = ld4<AL>(p + OW3 + r * NH + r4);
    }
};

struct Tile {
    float h1[TS][HS];              // first hidden layer, then reused for d2
    float h2[TS][HS];
};

// Hidden values of units 16w + 4g + 0..3 of sample c.  Two barriers; after the
// second T.h2 holds the second layer and T.h1 may be written again.
__device__ __forceinline__ void forward_tile(const Weights& W, f4 x, Lane l, Tile& T, f4& h1, f4& h2) {
    f4 a = W.b1;
#pragma unroll
    for (int s = 0; s < 4; ++s) a = __builtin_amdgcn_mfma_f32_16x16x4f32(W.w1[s], x[s], a, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) h1[r] = tanhf(a[r]);
    put_hidden(T.h1[l.c], l, h1);
    __syncthreads();
    a = chain(W.w2, T.h1[l.c], l, W.b2);
#pragma unroll
    for (int r = 0; r < 4; ++r) h2[r] = tanhf(a[r]);
    put_hidden(T.h2[l.c], l, h2);
    __syncthreads();
}
// the logits of sample c: rows 0..2 of the product, in the lanes of g = 0
__device__ __forceinline__ f4 logits_tile(const Weights& W, Lane l, const Tile& T) {
    return chain(W.z3, T.h2[l.c], l, W.b3);
}

}  // namespace

template <bool AL>
__global__ void __launch_bounds__(256)
k_mlp_forward(const float* __restrict__ p, const float* __restrict__ x, int64_t n,
              float* __restrict__ logits) {
    __shared__ Tile T;
    const Lane l = lane_of(threadIdx.x);
    Weights W;
    W.load<AL>(p, l);
    const int64_t nt = (n + TS - 1) / TS;
    int turn_of = 0;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const int64_t b = t * TS + l.c;
        f4 h1, h2;
        forward_tile(W, turn(ld4<AL>(x + min(b, n - 1) * NI + 4 * l.g)), l, T, h1, h2);
        // (a wave in turn; the next tile's second barrier frees T.h2)
        if (l.w == turn_of) {
            const f4 z = logits_tile(W, l, T);
            if (l.g == 0 && b < n)
#pragma unroll
                for (int o = 0; o < NO; ++o) logits[b * NO + o] = z[o];
        }
        turn_of = (turn_of + 1) & 3;
    }
}

template <bool AL>
__global__ void __launch_bounds__(256)
k_mlp_samples(const float* __restrict__ p, const float* __restrict__ x,
              const int8_t* __restrict__ cls, const int32_t* __restrict__ idx, int64_t n,
              int64_t n_rows, float* __restrict__ work) {
    __shared__ Tile T;
    const Lane l = lane_of(threadIdx.x);
    const float inv_n = 1.0f / float(n);
    Weights W;
    W.load<AL>(p, l);
    // the second layer transposed: row 16w + c of W2^T
    float wt[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) wt[q] = p[OW2 + (4 * q + l.g) * NH + 16 * l.w + l.c];
    const int64_t nt = (n + TS - 1) / TS;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const int64_t b = t * TS + l.c, bc = min(b, n - 1);
        const int64_t s = idx ? min(max(int64_t(idx[bc]), int64_t(0)), n_rows - 1) : bc;
        const int lab = min(max(int(cls[s]), 0), NO - 1);
        f4 h1, h2;
        forward_tile(W, turn(ld4<AL>(x + s * NI + 4 * l.g)), l, T, h1, h2);
        // (each wave forms the logits, whose lanes all need them)
        const f4 z = logits_tile(W, l, T);
        float z3[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) z3[o] = __shfl(z[o], l.c);
        // softmax and cross-entropy
        const float zm = fmaxf(z3[0], fmaxf(z3[1], z3[2]));
        float ex[NO], se = 0.0f, zl = z3[0];
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            ex[o] = expf(z3[o] - zm);
            se += ex[o];
            if (o == lab) zl = z3[o];
        }
        float d3[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) d3[o] = (ex[o] / se - (o == lab ? 1.0f : 0.0f)) * inv_n;
        // layer 2 error: (W3^T d3) * (1 - h2^2)
        f4 d2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float s2 = 0.0f;
#pragma unroll
            for (int o = 0; o < NO; ++o) s2 = fmaf(W.w3[o][r], d3[o], s2);
            d2[r] = s2 * (1.0f - h2[r] * h2[r]);
        }
        const int r4 = 16 * l.w + 4 * l.g;
        put_hidden(T.h1[l.c], l, d2);
        __syncthreads();
        // layer 1 error: (W2^T d2) * (1 - h1^2)
        const f4 a = chain(wt, T.h1[l.c], l, f4{0.0f, 0.0f, 0.0f, 0.0f});
        __syncthreads();               // the tile is written again by the next samples
        if (b >= n) continue;
        f4 d1;
#pragma unroll
        for (int r = 0; r < 4; ++r) d1[r] = a[r] * (1.0f - h1[r] * h1[r]);
        float* wb = work + b * WN;
        st4<AL>(wb + WH1 + r4, h1);
        st4<AL>(wb + WH2 + r4, h2);
        st4<AL>(wb + WD1 + r4, d1);
        st4<AL>(wb + WD2 + r4, d2);
        if (l.w == 0 && l.g == 0) {
#pragma unroll
            for (int o = 0; o < NO; ++o) wb[WD3 + o] = d3[o];
            wb[WL] = -(zl - zm - logf(se));
        }
    }
}

// Gradients as batch sums, and the mean loss.  A workgroup per 16 x 16 tile:
// 0-15 of W2 (rows d2, columns h1), 16-19 of W1 (d1, x), 20-23 of W3 (d3 and,
// as a fourth row, the loss; columns h2; 12 rows idle).  The biases and the
// loss are the row sums of the same operand, formed by the first tile of each
// row.  A wave takes every 16th group of four samples in order; the 16 waves'
// parts are added in wave order, so the result does not depend on scheduling.
constexpr int GRAD_TILES = 24, GRAD_WAVES = 16, GRAD_THREADS = 64 * GRAD_WAVES;

__global__ void __launch_bounds__(GRAD_THREADS)
k_mlp_grad(const float* __restrict__ x, const int32_t* __restrict__ idx, int64_t n,
           int64_t n_rows, const float* __restrict__ work, float* __restrict__ grad,
           float* __restrict__ loss) {
    __shared__ double part[GRAD_WAVES][256];
    __shared__ double rowsum[GRAD_WAVES][64];
    const int q = threadIdx.x, v = q >> 6, l = q & 63, g = l >> 4, c = l & 15;
    const int tile = blockIdx.x;
    const int kind = tile < 16 ? 2 : tile < 20 ? 1 : 3;          // weight matrix
    const int rb = kind == 2 ? tile / 4 : kind == 1 ? tile - 16 : 0;
    const int cb = kind == 2 ? tile % 4 : kind == 1 ? 0 : tile - 20;
    const int oa = kind == 2 ? WD2 + 16 * rb + c : kind == 1 ? WD1 + 16 * rb + c : WD3 + min(c, 3);
    const int ob = kind == 2 ? WH1 + 16 * cb + c : WH2 + 16 * cb + c;
    const bool row_ok = kind != 3 || c < 4;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    double rs = 0.0;
    const int64_t ns = (n + 3) / 4;
    // sixteen groups' operands are requested together: one at a time the loop
    // waits a round trip per group (14 against 11 us at 1024 samples)
    constexpr int U = 16;
    for (int64_t st = v; st < ns; st += U * GRAD_WAVES) {
        float av[U], bv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t bc = min(4 * (st + u * GRAD_WAVES) + g, n - 1);
            const float* wb = work + bc * WN;
            av[u] = wb[oa];
            if (kind == 1) {
                const int64_t sm = idx ? min(max(int64_t(idx[bc]), int64_t(0)), n_rows - 1) : bc;
                bv[u] = x[sm * NI + c];
            } else {
                bv[u] = wb[ob];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // past the batch both operands are zero (no 0 * inf)
            const bool in = 4 * (st + u * GRAD_WAVES) + g < n;
            const double da = (in && row_ok) ? double(av[u]) : 0.0, db = in ? double(bv[u]) : 0.0;
            rs += da;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(da, db, acc, 0, 0, 0);
        }
    }
    // accumulator: rows 4 r + g, column c
#pragma unroll
    for (int r = 0; r < 4; ++r) part[v][16 * (4 * r + g) + c] = acc[r];
    rowsum[v][l] = rs;
    __syncthreads();
    if (q < 256) {
        double t = 0.0;
        for (int k = 0; k < GRAD_WAVES; ++k) t += part[k][q];
        const int i = q >> 4, j = q & 15;
        if (kind == 2) grad[OW2 + (16 * rb + i) * NH + 16 * cb + j] = float(t);
        else if (kind == 1) grad[OW1 + (16 * rb + i) * NI + j] = float(t);
        else if (i < NO) grad[OW3 + i * NH + 16 * cb + j] = float(t);
    } else if (q < 256 + 16 && cb == 0) {
        const int i = q - 256;
        double t = 0.0;
        for (int k = 0; k < GRAD_WAVES; ++k)
            for (int h = 0; h < 4; ++h) t += rowsum[k][16 * h + i];
        if (kind == 2) grad[OB2 + 16 * rb + i] = float(t);
        else if (kind == 1) grad[OB1 + 16 * rb + i] = float(t);
        else if (i < NO) grad[OB3 + i] = float(t);
        else if (i == NO) *loss = float(t / double(n));
    }
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= NP) return;
    const float gr = g[r];
    const float mr = b1 * m[r] + (1.0f - b1) * gr;
    const float vr = b2 * v[r] + (1.0f - b2) * gr * gr;
    m[r] = mr;
    v[r] = vr;
    p[r] -= lr * (mr / c1) / (sqrtf(vr / c2) + eps);
}

// Workspace of mlp_backward_noalloc: one array per GPU, held until the
// process ends, shared by every call on that GPU (see sem.h).
static __device__ __align__(256) float scratch[size_t(SEM_MLP_NOALLOC_MAX) * SEM_MLP_WORK];

}  // namespace sem

namespace {
using sem::fail;

// device address of `scratch` on each GPU, looked up once per device with
// that device current (the host-side name is not a device address)
constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;

int scratch_for_current_device(float** out) {
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(SEM_ERR_HIP, "device index out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(sem::scratch)));
        if (!p) return fail(SEM_ERR_HIP, "no device address for the workspace array");
        g_scratch_ptr[dev] = static_cast<float*>(p);
    }
    *out = g_scratch_ptr[dev];
    return SEM_OK;
}

// tiles of 16 samples, at most eight workgroups per CU of a 256-CU GPU: each
// loads the 22 KB of parameters into its registers once
int grid_of(int64_t n) {
    const int64_t g = (n + sem::TS - 1) / sem::TS;
    return int(g < 1 ? 1 : g > 2048 ? 2048 : g);
}

bool aligned16(const void* a, const void* b, const void* c) {
    return ((uintptr_t(a) | uintptr_t(b) | uintptr_t(c)) & 15) == 0;
}

int launch_backward(const float* p, const float* x, int64_t n_rows, const int8_t* cls,
                    const int32_t* idx, int64_t n, float* work, float* grad, float* loss, hipStream_t s) {
    if (aligned16(p, x, work))
        hipLaunchKernelGGL(sem::k_mlp_samples<true>, dim3(grid_of(n)), dim3(256), 0, s, p, x, cls, idx, n,
                           n_rows, work);
    else
        hipLaunchKernelGGL(sem::k_mlp_samples<false>, dim3(grid_of(n)), dim3(256), 0, s, p, x, cls, idx, n,
                           n_rows, work);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(sem::k_mlp_grad, dim3(sem::GRAD_TILES), dim3(sem::GRAD_THREADS), 0, s, x, idx, n,
                       n_rows, work, grad, loss);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}
}  // namespace

extern "C" {

static int mlp_forward_impl(const float* p, const float* x, int64_t n, float* logits, void* stream) {
    if (!p || !logits || (n > 0 && !x)) return fail(SEM_ERR_ARG, "null array");
    if (n < 0) return fail(SEM_ERR_ARG, "negative sample count");
    if (n == 0) return SEM_OK;
    hipStream_t s = (hipStream_t)stream;
    if (aligned16(p, x, nullptr))
        hipLaunchKernelGGL(sem::k_mlp_forward<true>, dim3(grid_of(n)), dim3(256), 0, s, p, x, n, logits);
    else
        hipLaunchKernelGGL(sem::k_mlp_forward<false>, dim3(grid_of(n)), dim3(256), 0, s, p, x, n, logits);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int mlp_forward(const float* p, const float* x, int64_t n, float* logits, void* stream) {
    return sem::guarded("mlp_forward", [&] { return mlp_forward_impl(p, x, n, logits, stream); });
}

static int mlp_backward_impl(const float* p, const float* x, int64_t n_rows, const int8_t* cls,
                 const int32_t* idx, int64_t n, float* work, float* grad, float* loss, void* stream) {
    if (!p || !x || !cls || !work || !grad || !loss) return fail(SEM_ERR_ARG, "null array");
    if (n < 1) return fail(SEM_ERR_ARG, "empty batch");
    if (n_rows < 1 || (!idx && n > n_rows)) return fail(SEM_ERR_ARG, "batch larger than the data");
    return launch_backward(p, x, n_rows, cls, idx, n, work, grad, loss, (hipStream_t)stream);
}

int mlp_backward(const float* p, const float* x, int64_t n_rows, const int8_t* cls,
                 const int32_t* idx, int64_t n, float* work, float* grad, float* loss, void* stream) {
    return sem::guarded("mlp_backward", [&] { return mlp_backward_impl(p, x, n_rows, cls, idx, n, work, grad, loss, stream); });
}

static int mlp_backward_noalloc_impl(const float* p, const float* x, int64_t n_rows, const int8_t* cls,
                         const int32_t* idx, int64_t n, float* grad, float* loss, void* stream) {
    if (!p || !x || !cls || !grad || !loss) return fail(SEM_ERR_ARG, "null array");
    if (n < 1) return fail(SEM_ERR_ARG, "empty batch");
    if (n > SEM_MLP_NOALLOC_MAX)
        return fail(SEM_ERR_ARG, "batch larger than SEM_MLP_NOALLOC_MAX samples (use mlp_backward "
                                 "with a caller workspace)");
    if (n_rows < 1 || (!idx && n > n_rows)) return fail(SEM_ERR_ARG, "batch larger than the data");
    float* work = nullptr;
    int rc = scratch_for_current_device(&work);
    if (rc != SEM_OK) return rc;
    // the same two kernels as mlp_backward; k_mlp_samples writes every
    // workspace entry that k_mlp_grad reads (the first n samples), so nothing
    // left by an earlier call is read and no clearing is needed
    return launch_backward(p, x, n_rows, cls, idx, n, work, grad, loss, (hipStream_t)stream);
}

int mlp_backward_noalloc(const float* p, const float* x, int64_t n_rows, const int8_t* cls,
                         const int32_t* idx, int64_t n, float* grad, float* loss, void* stream) {
    return sem::guarded("mlp_backward_noalloc", [&] { return mlp_backward_noalloc_impl(p, x, n_rows, cls, idx, n, grad, loss, stream); });
}

static int mlp_adam_step_impl(float* p, const float* g, float* m, float* v, int t, float lr, float beta1,
                  float beta2, float eps, void* stream) {
    if (!p || !g || !m || !v) return fail(SEM_ERR_ARG, "null array");
    if (t < 1) return fail(SEM_ERR_ARG, "Adam step count starts at 1");
    if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps > 0.0f))
        return fail(SEM_ERR_ARG, "bad Adam hyper-parameters");
    const float c1 = float(1.0 - std::pow(double(beta1), t));
    const float c2 = float(1.0 - std::pow(double(beta2), t));
    hipLaunchKernelGGL(sem::k_adam, dim3((SEM_MLP_NPARAM + 255) / 256), dim3(256), 0,
                       (hipStream_t)stream, p, g, m, v, lr, beta1, beta2, eps, c1, c2);
    HIPCHK(hipGetLastError());
    return SEM_OK;
}

int mlp_adam_step(float* p, const float* g, float* m, float* v, int t, float lr, float beta1,
                  float beta2, float eps, void* stream) {
    return sem::guarded("mlp_adam_step", [&] { return mlp_adam_step_impl(p, g, m, v, t, lr, beta1, beta2, eps, stream); });
}

}  // extern "C"
