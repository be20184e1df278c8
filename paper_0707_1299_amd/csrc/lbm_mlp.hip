// Mobility-correction network: 4 -> 64 tanh -> 64 tanh -> 1 (linear output).
// Weights are held as bfloat16 for the forward pass and as FP32 master
// copies for training; every product accumulates in FP32.
//
// Parameter layout (flat, LBML_NPARAM = 4545):
//   W1[64][4] b1[64] W2[64][64] b2[64] W3[1][64] b3[1]
//
// Training is full-batch mean-squared error.  A block of four waves takes the
// samples sixteen at a time: the three 64 x 64 products of a batch (second
// layer, back-propagation through it, its weight gradient) run on the matrix
// cores in FP32, activations stay in LDS and every parameter's sum over the
// block's samples in registers.  One partial gradient per block goes to the
// work memory and a second kernel adds the partials in block order.  The split
// into blocks depends on the sample count alone, so repeated calls give
// bit-identical gradients.
#include <math.h>

#include <algorithm>
#include <mutex>

#include "../../include/lbm.h"
#include "lbm_device.h"

namespace {

constexpr int NP = 4545;
constexpr int O_W1 = 0, O_B1 = 256, O_W2 = 320, O_B2 = 4416, O_W3 = 4480, O_B3 = 4544;

__device__ __forceinline__ float bf16f(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// round to nearest, ties to even
__device__ __forceinline__ uint16_t f2bf16(float x)
{
    uint32_t b = __float_as_uint(x);
    if ((b & 0x7F800000u) == 0x7F800000u) return uint16_t((b >> 16) | ((b & 0xFFFFu) ? 0x40u : 0u));
    b += 0x7FFFu + ((b >> 16) & 1u);
    return uint16_t(b >> 16);
}

__global__ void k_round(const float* __restrict__ m, uint16_t* __restrict__ w, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = f2bf16(m[i]);
}

constexpr int SB = 16;                 // samples of a batch: one 16-wide matrix tile
constexpr int SP = SB + 1;             // LDS row stride of a 64 x 16 activation array (no bank conflicts)
constexpr int WP = 68;                 // LDS row stride of W2: rows 16 apart fall on distinct banks
constexpr int NPART = 4608;            // floats of one block's partial gradient: NP, the loss sum, padding

typedef float acc4 __attribute__((ext_vector_type(4)));

// Parameters as FP32 in LDS.
struct Weights {
    float4 W1[64];
    float b1[64], b2[64], W3[64];
    float W2[64 * WP];
    float b3;
};

__device__ __forceinline__ void stage(const uint16_t* __restrict__ w16, Weights& W)
{
    constexpr int PER = (NP + 255) / 256;
    uint16_t raw[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {    // all loads in flight before the first is used
        const int k = int(threadIdx.x) + 256 * j;
        raw[j] = k < NP ? w16[k] : uint16_t(0);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = int(threadIdx.x) + 256 * j;
        const float v = bf16f(raw[j]);
        if (k < O_B1) reinterpret_cast<float*>(W.W1)[k] = v;
        else if (k < O_W2) W.b1[k - O_B1] = v;
        else if (k < O_B2) W.W2[(k - O_W2) / 64 * WP + (k - O_W2) % 64] = v;
        else if (k < O_W3) W.b2[k - O_B2] = v;
        else if (k < O_B3) W.W3[k - O_W3] = v;
        else if (k == O_B3) W.b3 = v;
    }
    __syncthreads();
}

// Second-layer weights of wave w as the matrix instruction's first operand, held in registers for
// all batches: lane l gives row 16 w + l % 16 and, at step ks, the inner index 16 (l / 16) + ks (any
// order of the inner index serves, as long as both operands use it).
__device__ __forceinline__ void w2_rows(const Weights& W, float (&a)[16])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) a[ks] = W.W2[(16 * wave + (lane & 15)) * WP + 16 * (lane >> 4) + ks];
}

// First layer of the batch's samples into h1[unit][sample]; x: the input of sample threadIdx.x % 16.
__device__ __forceinline__ void layer1(const Weights& W, const float4 x, float* h1)
{
    const int s = threadIdx.x & 15, g = threadIdx.x >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = 16 * q + g;
        const float4 w = W.W1[j];
        h1[j * SP + s] = tanhf(fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, fmaf(w.x, x.x, W.b1[j])))));
    }
}

// 16 rows of a 64 x 64 matrix (operand a as w2_rows lays it out) times v[64][16]: lane l ends with
// rows 4 (l / 16) .. + 3 of the wave's sixteen, column (sample) l % 16.
__device__ __forceinline__ acc4 rows_times(const float (&a)[16], const float* v)
{
    const int lane = threadIdx.x & 63;
    acc4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks], v[(16 * (lane >> 4) + ks) * SP + (lane & 15)], c, 0, 0, 0);
    return c;
}

// Outputs of the batch's sixteen samples from the second layer's values h2 (rows as rows_times gives
// them): the wave sums W3 h2 over its lanes, the block over its waves.  yw: 4 x 16 floats.
__device__ __forceinline__ float layer3(const Weights& W, const float (&h2)[4], float* yw)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, u0 = 16 * wave + 4 * (lane >> 4);
    float y = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) y = fmaf(W.W3[u0 + r], h2[r], y);
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (lane < 16) yw[16 * wave + lane] = y;
    __syncthreads();
    const int s = lane & 15;
    return ((yw[s] + yw[16 + s]) + (yw[32 + s] + yw[48 + s])) + W.b3;
}

__device__ __forceinline__ float4 load_x(const float* __restrict__ x, long long i, bool live)
{
    return live ? make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// Bound by latency (a batch is a chain of two layers and a reduction), not by arithmetic: one batch of
// sixteen samples per block keeps the chain short and spreads a call over as many compute units as it
// has batches; past FWD_BLOCKS batches the blocks take several each, so the weights are staged
// once per block.  256 samples: 34.2 -> 5.1 us.
constexpr long long FWD_BLOCKS = 1024;

__global__ __launch_bounds__(256) void k_forward(const uint16_t* __restrict__ w16, long long n,
                                                 const float* __restrict__ x, float* __restrict__ y)
{
    __shared__ Weights W;
    __shared__ float h1[64 * SP], yw[64];
    stage(w16, W);
    float a[16];
    w2_rows(W, a);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, u0 = 16 * wave + 4 * (lane >> 4);
    for (long long b = blockIdx.x; b * SB < n; b += gridDim.x) {
        const long long i = b * SB + (threadIdx.x & 15);
        layer1(W, load_x(x, i, i < n), h1);
        __syncthreads();
        const acc4 z = rows_times(a, h1);
        float h2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) h2[r] = tanhf(z[r] + W.b2[u0 + r]);
        const float out = layer3(W, h2, yw);
        if (threadIdx.x < 16 && i < n) y[i] = out;
        // (the next batch writes h1 only after every wave has passed layer3's barrier, and yw only
        // after the barrier that follows its own first layer)
    }
}

// Sum over each 16-lane row of the wave, valid in the row's last lane.
__device__ __forceinline__ float row_sum(float v)
{
    v += lbm::dpp<0x111, 0xf, 0xf, true>(v);
    v += lbm::dpp<0x112, 0xf, 0xf, true>(v);
    v += lbm::dpp<0x114, 0xf, 0xf, true>(v);
    v += lbm::dpp<0x118, 0xf, 0xf, true>(v);
    return v;
}

// Gradient of the block's samples, `batches` consecutive batches from blockIdx.x * batches.  One block
// (gridDim.x == 1) writes the gradient and the loss themselves; otherwise block b writes its
// sums to part + NPART b.
// The three 64 x 64 products take 48 matrix instructions per wave and batch; the rest is two layers of
// tanh and four barriers.  1024 samples (32 blocks), with the sum over the blocks: 324 -> 13 us.
__global__ __launch_bounds__(256) void k_grad(const uint16_t* __restrict__ w16, long long n, long long batches,
                                              const float* __restrict__ x, const float* __restrict__ target,
                                              float* __restrict__ part, float* __restrict__ grad,
                                              float* __restrict__ loss)
{
    __shared__ Weights W;
    __shared__ float h1[64 * SP], d2[64 * SP], yw[64];
    stage(w16, W);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = lane & 15, g = lane >> 4, u0 = 16 * wave + 4 * g;
    float a[16], at[16];
    w2_rows(W, a);
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) at[ks] = W.W2[(16 * g + ks) * WP + 16 * wave + s];   // the transposed matrix's rows
    // sums over the block's samples: gW2 by matrix tiles (rows 16 wave .., columns 16 t ..), the others
    // per lane (the lane's sample, units u0 .. u0 + 3) and over the lanes at the end
    acc4 gW2[4];
    float gW1[4][4], gb1[4], gb2[4], gW3[4], gb3 = 0.0f, sq = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        gb1[r] = gb2[r] = gW3[r] = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) gW1[r][c] = gW2[r][c] = 0.0f;
    }
    const long long b0 = blockIdx.x * batches;
    for (long long b = b0; b < b0 + batches && b * SB < n; ++b) {
        const long long i = b * SB + s;
        const bool live = i < n;      // samples past the end: zero input, zero error
        const float4 xi = load_x(x, i, live);
        layer1(W, xi, h1);
        __syncthreads();
        const acc4 z = rows_times(a, h1);
        float h2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) h2[r] = tanhf(z[r] + W.b2[u0 + r]);
        const float out = layer3(W, h2, yw);
        const float res = live ? out - target[i] : 0.0f;
        const float dy = 2.0f * res / float(n);
        gb3 += dy;
        sq = fmaf(res, res, sq);
        // dz2_j = dy W3_j (1 - h2_j^2)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = dy * W.W3[u0 + r] * (1.0f - h2[r] * h2[r]);
            d2[(u0 + r) * SP + s] = d;
            gb2[r] += d;
            gW3[r] = fmaf(dy, h2[r], gW3[r]);
        }
        __syncthreads();
        // dz1_k = (sum_j W2_jk dz2_j) (1 - h1_k^2)
        const acc4 q = rows_times(at, d2);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float h = h1[(u0 + r) * SP + s];
            const float d = q[r] * (1.0f - h * h);
            gb1[r] += d;
            gW1[r][0] = fmaf(d, xi.x, gW1[r][0]);
            gW1[r][1] = fmaf(d, xi.y, gW1[r][1]);
            gW1[r][2] = fmaf(d, xi.z, gW1[r][2]);
            gW1[r][3] = fmaf(d, xi.w, gW1[r][3]);
        }
        // gW2_jk += sum over the batch of dz2_j h1_k
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const float e = d2[(16 * wave + s) * SP + 4 * g + ks];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                gW2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(e, h1[(16 * t + s) * SP + 4 * g + ks], gW2[t], 0, 0, 0);
        }
        __syncthreads();   // the next batch rewrites h1 and d2
    }
    const bool direct = gridDim.x == 1;
    float* o = direct ? grad : part + NPART * (long long)blockIdx.x;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[O_W2 + (u0 + r) * 64 + 16 * t + s] = gW2[t][r];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float v1 = row_sum(gb1[r]), v2 = row_sum(gb2[r]), v3 = row_sum(gW3[r]);
        float w[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) w[c] = row_sum(gW1[r][c]);
        if (s == 15) {
            o[O_B1 + u0 + r] = v1;
            o[O_B2 + u0 + r] = v2;
            o[O_W3 + u0 + r] = v3;
#pragma unroll
            for (int c = 0; c < 4; ++c) o[O_W1 + 4 * (u0 + r) + c] = w[c];
        }
    }
    const float t3 = row_sum(gb3), tq = row_sum(sq);   // every row of every wave holds the same sums
    if (threadIdx.x == 15) {
        o[O_B3] = t3;
        if (direct)
            *loss = tq / float(n);
        else
            o[NP] = tq;
    }
}

// Sums of nb partial gradients: a block takes 64 parameters, its wave w the w-th quarter of the
// partials in order; the four quarters are then added in order, all in FP64: the partials are FP32 sums of up to a few
// hundred samples, and their sum adds one rounding.
__global__ __launch_bounds__(256) void k_grad_sum(const float* __restrict__ part, int nb, long long n,
                                                  float* __restrict__ grad, float* __restrict__ loss)
{
    __shared__ double q[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;   // p < NPART
    const int per = (nb + 3) / 4, k0 = wave * per, k1 = min(nb, k0 + per);
    double v = 0.0;
    int k = k0;
    for (; k + 8 <= k1; k += 8) {
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = part[NPART * (long long)(k + j) + p];
#pragma unroll
        for (int j = 0; j < 8; ++j) v += double(t[j]);
    }
    for (; k < k1; ++k) v += double(part[NPART * (long long)k + p]);
    q[wave][lane] = v;
    __syncthreads();
    if (wave != 0) return;
    v = ((q[0][lane] + q[1][lane]) + q[2][lane]) + q[3][lane];
    if (p < NP)
        grad[p] = float(v);
    else if (p == NP)
        *loss = float(v / double(n));
}

__global__ void k_adam(float* __restrict__ m0, float* __restrict__ m1, float* __restrict__ v1,
                       const float* __restrict__ g, uint16_t* __restrict__ w16, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NP) return;
    const float gi = g[i];
    const float m = b1 * m1[i] + (1.0f - b1) * gi;
    const float v = b2 * v1[i] + (1.0f - b2) * gi * gi;
    m1[i] = m;
    v1[i] = v;
    const float mh = m / c1, vh = v / c2;
    const float w = m0[i] - lr * mh / (sqrtf(vh) + eps);
    m0[i] = w;
    w16[i] = f2bf16(w);
}

// Blocks of the gradient kernel for n samples: one per batch of SB samples, as far as the work memory
// (258 floats per sample) holds a partial gradient for each and GRAD_BLOCKS allows (the sum over the
// partials grows with the blocks, and 256 are one per compute unit).  Up to 35 samples one block does
// it all.
constexpr long long GRAD_BLOCKS = 256;

void launch_loss_grad(const uint16_t* d_w16, long long n, const float* d_x, const float* d_target, float* d_grad,
                      float* d_loss, float* d_work, hipStream_t s)
{
    const long long nbatch = (n + SB - 1) / SB;
    const long long most = std::max(1LL, std::min(GRAD_BLOCKS, 258 * n / NPART));
    const long long batches = (nbatch + most - 1) / most, nb = (nbatch + batches - 1) / batches;
    hipLaunchKernelGGL(k_grad, dim3((unsigned)nb), dim3(256), 0, s, d_w16, n, batches, d_x, d_target, d_work, d_grad,
                       d_loss);
    if (nb > 1)
        hipLaunchKernelGGL(k_grad_sum, dim3(NPART / 64), dim3(256), 0, s, (const float*)d_work, (int)nb, n, d_grad,
                           d_loss);
}

}  // namespace

// Work memory of lbml_loss_grad_static: a device array in the library itself, sized for
// LBML_STATIC_MAX_N samples (lbml_work_floats of that many).  Its name is a host-side stand-in:
// kernels receive the device address that hipGetSymbolAddress returns, taken once per device
// (with that device current) and kept in scratch_dev.  Every call on one device shares the array;
// the gradient pass writes every value it reads, so nothing needs clearing between calls.
static __device__ __align__(256) float scratch[258LL * LBML_STATIC_MAX_N];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
float* scratch_dev[MAX_DEVICES] = {};

int scratch_ptr(float** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return LB_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_dev[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return LB_ERR_HIP;
        scratch_dev[dev] = static_cast<float*>(p);
    }
    *out = scratch_dev[dev];
    return LB_OK;
}

}  // namespace

extern "C" {

int64_t lbml_work_floats(int64_t n) { return n < 0 ? -1 : 256 * n + 2 * n; }

int lbml_round_bf16(const float* d_master, uint16_t* d_w16, void* hip_stream)
{
    if (!d_master || !d_w16) return LB_ERR_ARG;
    hipLaunchKernelGGL(k_round, dim3((NP + 255) / 256), dim3(256), 0, (hipStream_t)hip_stream, d_master, d_w16, NP);
    return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP;
}

int lbml_forward(const uint16_t* d_w16, int64_t n, const float* d_x, float* d_y, void* hip_stream)
{
    if (n < 0 || (n > 0 && (!d_w16 || !d_x || !d_y))) return LB_ERR_ARG;
    if (n == 0) return LB_OK;
    const long long nb = std::min((long long)(n + SB - 1) / SB, FWD_BLOCKS);
    hipLaunchKernelGGL(k_forward, dim3((unsigned)nb), dim3(256), 0, (hipStream_t)hip_stream, d_w16, (long long)n, d_x,
                       d_y);
    return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP;
}

int lbml_loss_grad(const uint16_t* d_w16, int64_t n, const float* d_x, const float* d_target, float* d_grad,
                   float* d_loss, float* d_work, void* hip_stream)
{
    if (n <= 0 || !d_w16 || !d_x || !d_target || !d_grad || !d_loss || !d_work) return LB_ERR_ARG;
    (void)hipGetLastError();
    launch_loss_grad(d_w16, (long long)n, d_x, d_target, d_grad, d_loss, d_work, (hipStream_t)hip_stream);
    return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP;
}

int lbml_loss_grad_static(const uint16_t* d_w16, int64_t n, const float* d_x, const float* d_target, float* d_grad,
                          float* d_loss, void* hip_stream)
{
    if (n <= 0 || !d_w16 || !d_x || !d_target || !d_grad || !d_loss) return LB_ERR_ARG;
    if (n > LBML_STATIC_MAX_N) return LB_ERR_SIZE;
    float* work = nullptr;
    const int r = scratch_ptr(&work);
    if (r) return r;
    (void)hipGetLastError();
    launch_loss_grad(d_w16, (long long)n, d_x, d_target, d_grad, d_loss, work, (hipStream_t)hip_stream);
    return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP;
}

int lbml_adam_step(float* d_master, float* d_m, float* d_v, const float* d_grad, uint16_t* d_w16, int32_t t, float lr,
                   float beta1, float beta2, float eps, void* hip_stream)
{
    if (!d_master || !d_m || !d_v || !d_grad || !d_w16 || t < 1) return LB_ERR_ARG;
    const float c1 = 1.0f - powf(beta1, (float)t);
    const float c2 = 1.0f - powf(beta2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3((NP + 255) / 256), dim3(256), 0, (hipStream_t)hip_stream, d_master, d_m, d_v,
                       d_grad, d_w16, lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP;
}

}  // extern "C"
