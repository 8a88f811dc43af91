// Learned relaxation-time closure: MLP inference (FP32 MFMA), training
// kernels (loss and gradient in one pass, deterministic sums with Adam),
// coarse graining of a fine simulation onto a coarse one of the same
// elements, training targets, and their C entry points.
//
// Parameter blob (float32): mean[6], std[6], W1[64][6], b1[64], W2[64][64],
// b2[64], W3[64][64], b3[64], w4[64], b4[1], dtau_max[1]. The trainable
// parameters are the contiguous range W1 .. b4.
#include <mutex>
#include <cmath>
#include <string>
#include <vector>

#include "kernels_impl.h"
#include "ops.h"

namespace sel {

namespace {

constexpr int NF = 6, NH = 64;
constexpr int OFF_MEAN = 0, OFF_STD = 6, OFF_W1 = 12, OFF_B1 = OFF_W1 + NH * NF, OFF_W2 = OFF_B1 + NH,
              OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH * NH, OFF_W4 = OFF_B3 + NH,
              OFF_B4 = OFF_W4 + NH, OFF_DMAX = OFF_B4 + 1, BLOB = OFF_DMAX + 1;
constexpr int OFF_TRAIN = OFF_W1, NTRAIN = OFF_DMAX - OFF_W1;  // 8833

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float softplusf(float z) { return fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))); }

// tanh x = 1 - 2 / (exp(2x) + 1) with the hardware exp2 and reciprocal
// (absolute error about 1e-7; exp2 overflow gives the limits +-1)
__device__ __forceinline__ float tanh_fast(float x)
{
    const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);  // exp(2x) = 2^(2x / ln 2)
    return 1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f);
}

__device__ __forceinline__ float guard_dtau(float d, float tau, float dmax)
{
    // fallback to the plain method (0) for non-finite or out-of-range values
    return (d == d && d >= 0.f && d <= dmax * tau) ? d : 0.f;
}

// ------------------------------------------------------------ inference --
// Tiles of RW = 32 rows through 6 -> 64 -> 64 -> 64 -> 1, a workgroup of 4
// wavefronts per tile, with v_mfma_f32_16x16x4f32 for the three hidden layers.
// Wavefront w owns the hidden units 16 w .. 16 w + 15: its weight fragments stay
// in 34 registers over all tiles, and only the activations pass through LDS
// (two buffers of 8.5 KB, one barrier per layer), so that five workgroups share a
// CU and the tanh of some runs under the matrix products of others. Bound by
// the matrix units (14.5 us for 131 k rows) and the tanh (9 us), which overlap
// little. Tiles of 16 rows took 39 us for 131 k rows, of 64 rows 36.8, these 34.6.
// Few rows and sizes that leave k_mlp_lds a nearly empty last round take this
// kernel (mlp_in_lds).
constexpr int RW = 32;  // rows per tile
constexpr int RT = RW / 16;
// five resident workgroups per CU, each looping over its tiles
constexpr int64_t kInferMaxBlocks = 5 * 256;

__global__ void __launch_bounds__(256, 5) k_mlp(const float *__restrict__ P, const float *__restrict__ X, int64_t n,
                                                float tau, float *__restrict__ zout, float *__restrict__ dtau)
{
    constexpr int LD = 68;  // row stride: rows stay 16-byte aligned
    constexpr int RPW = RW / 4;  // output rows per wavefront
    __shared__ __attribute__((aligned(16))) float sH[2][RW][LD];
    __shared__ float sz[2][RW];
    const int tid = threadIdx.x, w = tid / 64, l = tid % 64, li = l & 15, lk = l >> 4;
    const int u = 16 * w + li;  // the lane's hidden unit
    // weight fragments: step ks of a product over 64 units takes unit 16 lk + ks
    float w1[2], wf[2][16], mean[2], istd[2], w4[RPW];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int c = 4 * ks + lk;
        w1[ks] = c < NF ? P[OFF_W1 + u * NF + c] : 0.f;
        mean[ks] = c < NF ? P[OFF_MEAN + c] : 0.f;
        istd[ks] = c < NF ? 1.f / P[OFF_STD + c] : 0.f;
    }
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        wf[0][ks] = P[OFF_W2 + u * NH + 16 * lk + ks];
        wf[1][ks] = P[OFF_W3 + u * NH + 16 * lk + ks];
    }
    // output layer: row RPW w + l % RPW of the tile, units RPW (l / RPW) .. + RPW - 1
#pragma unroll
    for (int c = 0; c < RPW; ++c) w4[c] = P[OFF_W4 + RPW * (l / RPW) + c];
    const float bias[3] = {P[OFF_B1 + u], P[OFF_B2 + u], P[OFF_B3 + u]};
    const float b4 = P[OFF_B4], dmax = P[OFF_DMAX];
    const int64_t tiles = (n + RW - 1) / RW;
    int turn = 0;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x, ++turn) {
        f4 acc[RT];
        // normalised inputs (columns 6 and 7 zero), hidden layer 1
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int64_t r = tile * RW + 16 * t + li;
            acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int c = 4 * ks + lk;
                const float x = (c < NF && r < n) ? (X[r * NF + c] - mean[ks]) * istd[ks] : 0.f;
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w1[ks], acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int layer = 0; layer < 3; ++layer) {
            float(*H)[LD] = sH[layer & 1];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) H[16 * t + 4 * lk + q][u] = tanh_fast(acc[t][q] + bias[layer]);
            __syncthreads();
            if (layer < 2) {
#pragma unroll
                for (int t = 0; t < RT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 16; ++ks)
#pragma unroll
                    for (int t = 0; t < RT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(H[16 * t + li][16 * lk + ks], wf[layer][ks],
                                                                     acc[t], 0, 0, 0);
            }
        }
        const int rr = RPW * w + l % RPW;
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < RPW; ++c) z += sH[0][rr][RPW * (l / RPW) + c] * w4[c];
#pragma unroll
        for (int k = RPW; k < 64; k *= 2) z += __shfl_xor(z, k);
        if (l < RPW) sz[turn & 1][rr] = z + b4;
        __syncthreads();  // layer 3 read before the next tile's layer 1 is written
        // softplus and guard for the whole tile by one wavefront, in turn (by
        // each of them for its own rows they were a third of the arithmetic)
        const int64_t r = tile * RW + l;
        if (w == (turn & 3) && l < RW && r < n) {
            const float zr = sz[turn & 1][l];
            if (zout) zout[r] = zr;
            if (dtau) dtau[r] = guard_dtau(tau * softplusf(zr), tau, dmax);
        }
    }
}

// The network with its weights in LDS: each wavefront runs tiles of RW rows
// of its own through all layers (A = activations, B = W^T, 2 x 4 output tiles of
// 16 x 16, activations re-laid out through LDS between layers). 71 KB of LDS,
// so two workgroups share a CU. A wavefront's LDS operations complete in order,
// so inside the row loop only compiler scheduling barriers separate the layers
// and the four wavefronts of a workgroup run independently. At most 1024
// workgroups, each looping over its tiles, so that one stages the weights
// for many tiles (4096 workgroups took 1.3% longer on 1.4 M rows).
constexpr int64_t kLdsBlocks = 1024;

// W2 and W3 into LDS by a workgroup of 256 threads: every load of a thread is
// issued before its first LDS store, so the workgroup waits for one memory
// round trip instead of one per loop iteration.
__device__ __forceinline__ void stage_hidden(const float *__restrict__ P, float (*sW2)[NH + 1],
                                             float (*sW3)[NH + 1], int tid)
{
    constexpr int PER = NH * NH / 256;
    float a[PER], b[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        a[i] = P[OFF_W2 + tid + 256 * i];
        b[i] = P[OFF_W3 + tid + 256 * i];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = tid + 256 * i;
        sW2[q / NH][q % NH] = a[i];
        sW3[q / NH][q % NH] = b[i];
    }
}

__global__ void __launch_bounds__(256) k_mlp_lds(const float *__restrict__ P, const float *__restrict__ X, int64_t n,
                                                 float tau, float *__restrict__ zout, float *__restrict__ dtau)
{
    __shared__ float sW1[NH][9];
    __shared__ float sW2[NH][NH + 1];
    __shared__ float sW3[NH][NH + 1];
    __shared__ float sb1[NH], sb2[NH], sb3[NH], sw4[NH];
    __shared__ float sH[4][RW][NH + 1];
    __shared__ float smean[NF], sistd[NF];
    const int tid = threadIdx.x;
    const float b4 = P[OFF_B4], dmax = P[OFF_DMAX];
    {
        // all loads first (one round trip), then the LDS stores
        float w1v[2], bv[4] = {0.f, 0.f, 0.f, 0.f}, mv = 0.f, sv = 1.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 256 * i, r = q / 8, c = q % 8;
            w1v[i] = (c < NF) ? P[OFF_W1 + r * NF + c] : 0.f;
        }
        if (tid < NH) {
            bv[0] = P[OFF_B1 + tid];
            bv[1] = P[OFF_B2 + tid];
            bv[2] = P[OFF_B3 + tid];
            bv[3] = P[OFF_W4 + tid];
        }
        if (tid < NF) {
            mv = P[OFF_MEAN + tid];
            sv = P[OFF_STD + tid];
        }
        stage_hidden(P, sW2, sW3, tid);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = tid + 256 * i;
            sW1[q / 8][q % 8] = w1v[i];
        }
        if (tid < NH) {
            sb1[tid] = bv[0];
            sb2[tid] = bv[1];
            sb3[tid] = bv[2];
            sw4[tid] = bv[3];
        }
        if (tid < NF) {
            smean[tid] = mv;
            sistd[tid] = 1.f / sv;
        }
    }
    __syncthreads();
    const int w = tid / 64, l = tid % 64;
    const int li = l & 15, lk = l >> 4;
    for (int64_t base = (int64_t)blockIdx.x * (4 * RW); base < n; base += (int64_t)gridDim.x * (4 * RW)) {
        // normalised inputs, K padded to 8: lane l fills row l % RW, columns 4 (l / RW) .. +3
        {
            const int rr = l % RW, c0 = 4 * (l / RW);
            const int64_t r = base + w * RW + rr;
#pragma unroll
            for (int c = c0; c < c0 + 4; ++c) {
                sH[w][rr][c] = (c < NF && r < n) ? (X[r * NF + c] - smean[c]) * sistd[c] : 0.f;
            }
        }
        __builtin_amdgcn_wave_barrier();
        f4 acc[RT][4];
        // hidden layer 1 (K = 8)
#pragma unroll
        for (int ti = 0; ti < RT; ++ti)
#pragma unroll
            for (int tj = 0; tj < 4; ++tj) acc[ti][tj] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            float a[RT], b[4];
#pragma unroll
            for (int t = 0; t < RT; ++t) a[t] = sH[w][16 * t + li][4 * ks + lk];
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t] = sW1[16 * t + li][4 * ks + lk];
#pragma unroll
            for (int ti = 0; ti < RT; ++ti)
#pragma unroll
                for (int tj = 0; tj < 4; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ti], b[tj], acc[ti][tj], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int ti = 0; ti < RT; ++ti)
#pragma unroll
            for (int tj = 0; tj < 4; ++tj)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = 16 * tj + li;
                    sH[w][16 * ti + 4 * lk + q][col] = tanh_fast(acc[ti][tj][q] + sb1[col]);
                }
        __builtin_amdgcn_wave_barrier();
        // hidden layers 2 and 3 (K = 64)
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            const float(*Wl)[NH + 1] = layer == 0 ? sW2 : sW3;
            const float *bl = layer == 0 ? sb2 : sb3;
#pragma unroll
            for (int ti = 0; ti < RT; ++ti)
#pragma unroll
                for (int tj = 0; tj < 4; ++tj) acc[ti][tj] = f4{0.f, 0.f, 0.f, 0.f};
            for (int ks = 0; ks < NH / 4; ++ks) {
                float a[RT], b[4];
#pragma unroll
                for (int t = 0; t < RT; ++t) a[t] = sH[w][16 * t + li][4 * ks + lk];
#pragma unroll
                for (int t = 0; t < 4; ++t) b[t] = Wl[16 * t + li][4 * ks + lk];
#pragma unroll
                for (int ti = 0; ti < RT; ++ti)
#pragma unroll
                    for (int tj = 0; tj < 4; ++tj)
                        acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ti], b[tj], acc[ti][tj], 0, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ti = 0; ti < RT; ++ti)
#pragma unroll
                for (int tj = 0; tj < 4; ++tj)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col = 16 * tj + li;
                        sH[w][16 * ti + 4 * lk + q][col] = tanh_fast(acc[ti][tj][q] + bl[col]);
                    }
            __builtin_amdgcn_wave_barrier();
        }
        // output layer: two lanes per row, halves of the 64 products
        {
            const int rr = l % RW, h = l / RW;
            float z = 0.f;
#pragma unroll 8
            for (int c = 32 * h; c < 32 * h + 32; ++c) z += sH[w][rr][c] * sw4[c];
            z += __shfl_xor(z, 32);
            z += b4;
            const int64_t r = base + w * RW + rr;
            if (h == 0 && r < n) {
                if (zout) zout[r] = z;
                if (dtau) dtau[r] = guard_dtau(tau * softplusf(z), tau, dmax);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Which of the two kernels takes n rows. k_mlp_lds deals 128 rows at a time to
// the 256 CUs and takes about 5.8 us for each such round of 32 k rows, k_mlp 32
// rows at a time and 1.5 us per 8 k rows: whichever has less to do in whole
// rounds, and the former for its slightly better rate (2 to 3%) where both have
// many. Measured, us with k_mlp_lds and k_mlp: 8 k rows 9.7 and 5.3, 16 k 9.8 and
// 7.6, 32 k 9.8 and 11.8, 33 k 14.9 and 13.0, 64 k 15.3 and 17.5, 98.4 k 27.5 and 24.7,
// 131.0 k 28.4 and 30.3, 131.3 k 33.2 and 31.5, 262 k 51.8 and 54.3, 1.4 M 261 and 270.
constexpr bool mlp_in_lds(int64_t n)
{
    return 4 * ((n + 32767) / 32768) <= (n + 8191) / 8192 + 1 + n / (1 << 19);
}

void launch_mlp(const float *P, const float *X, int64_t n, float tau, float *z, float *dtau, hipStream_t st)
{
    if (mlp_in_lds(n)) {
        const int64_t nb = (n + 4 * RW - 1) / (4 * RW);
        hipLaunchKernelGGL(k_mlp_lds, dim3((unsigned)(nb < kLdsBlocks ? nb : kLdsBlocks)), dim3(256), 0, st, P, X, n,
                           tau, z, dtau);
    } else {
        const int64_t nb = (n + RW - 1) / RW;
        hipLaunchKernelGGL(k_mlp, dim3((unsigned)(nb < kInferMaxBlocks ? nb : kInferMaxBlocks)), dim3(256), 0, st, P, X,
                           n, tau, z, dtau);
    }
}

// ------------------------------------------------------------- training --
// Rows per tile and workgroups of the gradient kernel: one tile of 16 rows each
// up to 256 workgroups (a minibatch of 4096 is one per CU), then several tiles
// per workgroup, up to 1024 workgroups. The split depends on n alone.
constexpr int TR = 16;
constexpr int64_t train_blocks(int64_t n)
{
    const int64_t t = (n + TR - 1) / TR;
    return t <= 256 ? t : t / 8 <= 256 ? 256 : t / 8 <= 1024 ? t / 8 : 1024;
}

// Work layout (floats): gradient [NTRAIN], loss partials [nblk] and the loss,
// gradient partials [nblk][NTRAIN].
struct TrainWork {
    float *grad, *part, *wpart;
};
constexpr int64_t work_floats(int64_t n) { return NTRAIN + train_blocks(n) + 1 + train_blocks(n) * NTRAIN; }

TrainWork carve_work(float *w, int64_t n)
{
    TrainWork t;
    t.grad = w;
    t.part = t.grad + NTRAIN;
    t.wpart = t.part + train_blocks(n) + 1;
    return t;
}

// Loss and gradient of the mean squared error of softplus(z) against y: forward,
// back-propagation and weight gradients of a tile of 16 rows in one pass, on
// v_mfma_f32_16x16x4f32, partial sums of one workgroup at a time. Wavefront w
// owns the hidden units 16 w .. 16 w + 15 of every layer:
//   forward   H_l[s][16w + li] = tanh(sum_k H_{l-1}[s][k] W_l[16w + li][k] + b_l)
//   backward  dz = (2/n) (softplus(z) - y) sigmoid(z), D3 = dz w4 (1 - H3^2),
//             D_l[s][16w + li] = (sum_k D_{l+1}[s][k] W_{l+1}[k][16w + li]) (1 - H_l^2)
//   gradient  G_l[16w + m][c] += sum_s D_l[s][16w + m] H_{l-1}[s][c]
// so its weight fragments (64 registers, loaded once) and gradient tiles (36)
// stay in registers over all its tiles; layers pass their activations and
// deltas through LDS (6 barriers a tile). A result's lane holds the rows
// 4 (l / 16) + q of its column; the sum over the samples takes them as its A
// operand as they are (sample 4 (l / 16) + ks in step ks), without LDS. Bound by
// latency: a minibatch of 4096 has one tile per CU. As five kernels (forward,
// backward, weight gradient, sum, Adam) over activations in memory and tiles of
// 128 rows on 32 CUs a step of 4096 rows took 57 us; with the sums and Adam in
// one more kernel it takes 20 (14.5 + 5.4).
__global__ void __launch_bounds__(256) k_train(const float *__restrict__ P, const float *__restrict__ X,
                                               const float *__restrict__ y, const int32_t *__restrict__ idx,
                                               int64_t n, float *__restrict__ part, float *__restrict__ wpart)
{
    constexpr int LD = 68;  // row stride: rows stay 16-byte aligned
    __shared__ __attribute__((aligned(16))) float sH[3][TR][LD], sD[2][TR][LD];
    __shared__ float sX[TR][17];
    const int tid = threadIdx.x, w = tid / 64, l = tid % 64, li = l & 15, lk = l >> 4;
    const int u = 16 * w + li;  // the lane's hidden unit
    // weight fragments: step ks of a product over 64 units takes unit 16 lk + ks
    float w1[2], wf[2][16], wb[2][16], w4k[16];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w1[ks] = 4 * ks + lk < NF ? P[OFF_W1 + u * NF + 4 * ks + lk] : 0.f;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const int k = 16 * lk + ks;
        wf[0][ks] = P[OFF_W2 + u * NH + k];
        wf[1][ks] = P[OFF_W3 + u * NH + k];
        wb[0][ks] = P[OFF_W3 + k * NH + u];
        wb[1][ks] = P[OFF_W2 + k * NH + u];
        w4k[ks] = P[OFF_W4 + k];
    }
    const float bias[3] = {P[OFF_B1 + u], P[OFF_B2 + u], P[OFF_B3 + u]};
    const float w4 = P[OFF_W4 + u], b4 = P[OFF_B4];
    float mean[2], istd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int c = 4 * ks + lk;
        mean[ks] = c < NF ? P[OFF_MEAN + c] : 0.f;
        istd[ks] = c < NF ? 1.f / P[OFF_STD + c] : 0.f;
    }
    f4 g1 = {0.f, 0.f, 0.f, 0.f}, g2[4], g3[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) g2[t] = g3[t] = f4{0.f, 0.f, 0.f, 0.f};
    float gb[3] = {0.f, 0.f, 0.f}, gw4 = 0.f, gb4 = 0.f, r2 = 0.f;
    const float two_n = 2.f / float(n);
    const int64_t tiles = (n + TR - 1) / TR;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        // the row of lane li, its inputs (columns lk and 4 + lk) and target
        // (past the end the last row again, with dz = 0: nothing that the rows
        // themselves don't hold, such as 0 times an infinite weight, gets into the sums)
        const int64_t r = tile * TR + li;
        const bool ok = r < n;
        const int64_t rc = ok ? r : n - 1, row = idx ? (int64_t)idx[rc] : rc;
        float a1[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int c = 4 * ks + lk;
            a1[ks] = c < NF ? (X[row * NF + c] - mean[ks]) * istd[ks] : 0.f;
        }
        const float yr = y[row];
        float h[3][4];
        f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[ks], w1[ks], acc, 0, 0, 0);
        if (w == 0) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) sX[li][4 * ks + lk] = a1[ks];
        }
        // hidden layers: activations to LDS, then the next layer's product
#pragma unroll
        for (int layer = 0; layer < 3; ++layer) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                h[layer][q] = tanh_fast(acc[q] + bias[layer]);
                sH[layer][4 * lk + q][u] = h[layer][q];
            }
            __syncthreads();
            if (layer < 2) {
                f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 16; ks += 2) {
                    c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(sH[layer][li][16 * lk + ks], wf[layer][ks], c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sH[layer][li][16 * lk + ks + 1], wf[layer][ks + 1], c1, 0,
                                                             0, 0);
                }
                acc = c0 + c1;
            }
        }
        // output, residual and dz of row li
        float z = 0.f;
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) z += sH[2][li][16 * lk + ks] * w4k[ks];
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        z += b4;
        const float res = ok ? softplusf(z) - yr : 0.f;
        const float dz = ok ? two_n * res / (1.f + expf(-z)) : 0.f;
        if (l < 16) {
            r2 += res * res;
            gb4 += dz;
        }
        float d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float dq = __shfl(dz, 4 * lk + q);
            gw4 += dq * h[2][q];
            d[q] = dq * w4 * (1.f - h[2][q] * h[2][q]);
            sD[0][4 * lk + q][u] = d[q];
            gb[2] += d[q];
        }
        __syncthreads();
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {  // D2 from D3 through W3, then D1 from D2 through W2
            f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 16; ks += 2) {
                c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[layer][li][16 * lk + ks], wb[layer][ks], c0, 0, 0, 0);
                c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sD[layer][li][16 * lk + ks + 1], wb[layer][ks + 1], c1, 0, 0,
                                                         0);
            }
            // weight gradient of the layer above with its own deltas
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float b = sH[1 - layer][4 * lk + ks][16 * t + li];
                    if (layer == 0) g3[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[ks], b, g3[t], 0, 0, 0);
                    else g2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[ks], b, g2[t], 0, 0, 0);
                }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float hq = h[1 - layer][q];
                d[q] = (c0[q] + c1[q]) * (1.f - hq * hq);
                if (layer == 0) sD[1][4 * lk + q][u] = d[q];
                gb[1 - layer] += d[q];
            }
            if (layer == 0) __syncthreads();
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            g1 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[ks], li < 8 ? sX[4 * lk + ks][li] : 0.f, g1, 0, 0, 0);
        __syncthreads();  // the tile's LDS is free again
    }
    // gradient row 16 w + 4 lk + q, column 16 t + li of each tile
    float *__restrict__ out = wpart + (int64_t)blockIdx.x * NTRAIN;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = 16 * w + 4 * lk + q;
        if (li < NF) out[OFF_W1 - OFF_TRAIN + m * NF + li] = g1[q];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            out[OFF_W2 - OFF_TRAIN + m * NH + 16 * t + li] = g2[t][q];
            out[OFF_W3 - OFF_TRAIN + m * NH + 16 * t + li] = g3[t][q];
        }
    }
    // column sums over the four row quarters
    float v[4] = {gb[0], gb[1], gb[2], gw4};
    constexpr int off[4] = {OFF_B1, OFF_B2, OFF_B3, OFF_W4};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] += __shfl_xor(v[k], 16);
        v[k] += __shfl_xor(v[k], 32);
        if (l < 16) out[off[k] - OFF_TRAIN + u] = v[k];
    }
    if (w == 0) {
#pragma unroll
        for (int k = 8; k > 0; k >>= 1) {
            r2 += __shfl_xor(r2, k);
            gb4 += __shfl_xor(gb4, k);
        }
        if (l == 0) {
            out[OFF_B4 - OFF_TRAIN] = gb4;
            part[blockIdx.x] = r2;
        }
    }
}

// The partials summed (32 parameters per workgroup, eight runs of consecutive
// partials each, the runs added in order: the result depends on n alone), then
// with ADAM the update (Kingma & Ba, bias-corrected), else the gradient to grad.
// The workgroup after the last parameter sums the loss partials into *loss.
template <bool ADAM>
__global__ void __launch_bounds__(256) k_train_sum(const float *__restrict__ wpart, const float *__restrict__ part,
                                                   int nb, int64_t n, float *__restrict__ grad,
                                                   float *__restrict__ loss, float *P, float *m, float *v, int64_t t,
                                                   float lr, float b1, float b2, float eps)
{
    __shared__ float sh[8][32];
    const int c = threadIdx.x % 32, seg = threadIdx.x / 32;
    const int per = (nb + 7) / 8, k0 = seg * per, k1 = k0 + per < nb ? k0 + per : nb;
    const bool is_loss = blockIdx.x == (NTRAIN + 31) / 32;
    const int q = blockIdx.x * 32 + c;
    float s = 0.f;
    if (is_loss) {
        for (int k = k0 + c; k < k1; k += 32) s += part[k];
#pragma unroll
        for (int k = 16; k > 0; k >>= 1) s += __shfl_xor(s, k, 32);
    } else if (q < NTRAIN) {
#pragma unroll 16
        for (int k = k0; k < k1; ++k) s += wpart[(int64_t)k * NTRAIN + q];
    }
    sh[seg][c] = s;
    __syncthreads();
    if (seg) return;
    for (int k = 1; k < 8; ++k) s += sh[k][c];
    if (is_loss) {
        if (c == 0) loss[0] = s / float(n);
        return;
    }
    if (q >= NTRAIN) return;
    if constexpr (ADAM) {
        const float mq = b1 * m[q] + (1.f - b1) * s;
        const float vq = b2 * v[q] + (1.f - b2) * s * s;
        m[q] = mq;
        v[q] = vq;
        const float mh = mq / (1.f - powf(b1, float(t)));
        const float vh = vq / (1.f - powf(b2, float(t)));
        P[OFF_TRAIN + q] -= lr * mh / (sqrtf(vh) + eps);
    } else {
        grad[q] = s;
    }
}

// gradient partials and loss partials of n samples into T
void launch_gradient(const float *P, const float *X, const float *y, const int32_t *idx, int64_t n, TrainWork T,
                     hipStream_t st)
{
    hipLaunchKernelGGL(k_train, dim3((unsigned)train_blocks(n)), dim3(256), 0, st, P, X, y, idx, n, T.part, T.wpart);
}

constexpr unsigned kSumBlocks = (NTRAIN + 31) / 32 + 1;

// --------------------------------------------------------- coarse graining --
// One workgroup per element, one thread per fine node; the projection matrix
// Pm[ic][jf] is applied along r, s (and t) through LDS (sizes change per pass).
template <int DIM, int Q, typename T, bool DEV>
__global__ void k_coarse(NodeMap Mf, const T *ff, NodeMap Mc, T *fc, const double *Pm, int nf1, int nc1, double rho0)
{
    __shared__ double b0[1024], b1[1024];
    __shared__ double sP[kMaxN1 * kMaxN1];
    const int64_t e = blockIdx.x;
    const int p = threadIdx.x;
    const int npf = blockDim.x;
    for (int q = p; q < nc1 * nf1; q += npf) sP[q] = Pm[q];
    const int i = p % nf1, j = (p / nf1) % nf1, k = (DIM == 3) ? p / (nf1 * nf1) : 0;
    bool ownf;
    const SIdx sf = Mf.sidx(e, p, ownf);
    bool ownc = false;
    SIdx sc{0, 0};
    const bool on_coarse = i < nc1 && j < nc1 && (DIM == 2 || k < nc1);
    if (on_coarse) sc = Mc.sidx(e, i + nc1 * j + (DIM == 3 ? nc1 * nc1 * k : 0), ownc);
    for (int a = 0; a < Q; ++a) {
        b0[p] = double(ff[sf.base + (int64_t)a * sf.stride]);
        __syncthreads();
        if (i < nc1) {  // along r: [nc1][nf1][nf1]
            double v = 0.0;
            for (int c = 0; c < nf1; ++c) v += sP[i * nf1 + c] * b0[c + nf1 * j + nf1 * nf1 * k];
            b1[i + nc1 * j + nc1 * nf1 * k] = v;
        }
        __syncthreads();
        double v = 0.0;
        if (i < nc1 && j < nc1) {  // along s: [nc1][nc1][nf1]
            for (int c = 0; c < nf1; ++c) v += sP[j * nf1 + c] * b1[i + nc1 * c + nc1 * nf1 * k];
        }
        if (DIM == 3) {
            __syncthreads();
            if (i < nc1 && j < nc1) b0[i + nc1 * j + nc1 * nc1 * k] = v;
            __syncthreads();
            if (on_coarse) {
                v = 0.0;
                for (int c = 0; c < nf1; ++c) v += sP[k * nf1 + c] * b0[i + nc1 * j + nc1 * nc1 * c];
            }
        }
        if (on_coarse && ownc) fc[sc.base + (int64_t)a * sc.stride] = T(v);
        __syncthreads();
    }
    (void)rho0;
}

// Training target per coarse element: P(u), P(u u) from the fine state,
// S-bar from P(u) with the coarse metric, tau_sgs = P(uu) - P(u) P(u),
// nu_t = max(0, -<dev tau_sgs : S-bar> / <2 S-bar : S-bar>), dtau* = nu_t / (c_s^2 dt),
// written as y = dtau* / tau (the target of softplus(z)) on every coarse node.
template <int DIM, int Q, typename T, bool DEV>
__global__ void k_targets(NodeMap Mf, const T *ff, const double *Pm, int nf1, int nc1, const T *Gmc,
                          const double *wJc, const double *Dc, double rho0, double dtc, double tauc, float *y)
{
    constexpr int NFLD = DIM + DIM * (DIM + 1) / 2;
    __shared__ double b0[1024], b1[1024];
    __shared__ double sP[kMaxN1 * kMaxN1];
    __shared__ double cf[NFLD][512];
    const int64_t e = blockIdx.x;
    const int p = threadIdx.x;
    const int npf = blockDim.x;
    const int ncp = (DIM == 3) ? nc1 * nc1 * nc1 : nc1 * nc1;
    for (int q = p; q < nc1 * nf1; q += npf) sP[q] = Pm[q];
    const int i = p % nf1, j = (p / nf1) % nf1, k = (DIM == 3) ? p / (nf1 * nf1) : 0;
    bool own;
    const SIdx sf = Mf.sidx(e, p, own);
    double m = 0, jv[3] = {0, 0, 0};
    static_for<0, Q>([&](auto AA) {
        constexpr int a = decltype(AA)::value;
        const double v = double(ff[sf.base + (int64_t)a * sf.stride]);
        m += v;
        if constexpr (lat_e<DIM, Q>(a, 0) != 0) jv[0] += lat_e<DIM, Q>(a, 0) * v;
        if constexpr (lat_e<DIM, Q>(a, 1) != 0) jv[1] += lat_e<DIM, Q>(a, 1) * v;
        if constexpr (lat_e<DIM, Q>(a, 2) != 0) jv[2] += lat_e<DIM, Q>(a, 2) * v;
    });
    const double rho = DEV ? rho0 + m : m;
    double fld[NFLD];
    for (int c = 0; c < DIM; ++c) fld[c] = jv[c] / rho;
    {
        int q = DIM;
        for (int r = 0; r < DIM; ++r)
            for (int c = r; c < DIM; ++c) fld[q++] = fld[r] * fld[c];
    }
    const bool on_coarse = i < nc1 && j < nc1 && (DIM == 2 || k < nc1);
    const int pc = i + nc1 * j + (DIM == 3 ? nc1 * nc1 * k : 0);
    for (int q = 0; q < NFLD; ++q) {
        b0[p] = fld[q];
        __syncthreads();
        if (i < nc1) {
            double v = 0.0;
            for (int c = 0; c < nf1; ++c) v += sP[i * nf1 + c] * b0[c + nf1 * j + nf1 * nf1 * k];
            b1[i + nc1 * j + nc1 * nf1 * k] = v;
        }
        __syncthreads();
        double v = 0.0;
        if (i < nc1 && j < nc1)
            for (int c = 0; c < nf1; ++c) v += sP[j * nf1 + c] * b1[i + nc1 * c + nc1 * nf1 * k];
        if (DIM == 3) {
            __syncthreads();
            if (i < nc1 && j < nc1) b0[i + nc1 * j + nc1 * nc1 * k] = v;
            __syncthreads();
            if (on_coarse) {
                v = 0.0;
                for (int c = 0; c < nf1; ++c) v += sP[k * nf1 + c] * b0[i + nc1 * j + nc1 * nc1 * c];
            }
        }
        if (on_coarse) cf[q][pc] = v;
        __syncthreads();
    }
    double num = 0.0, den = 0.0;
    if (on_coarse) {
        const int idx[3] = {i, j, k};
        const int str[3] = {1, nc1, nc1 * nc1};
        double du[3][3] = {};
        for (int mm = 0; mm < DIM; ++mm) {
            const int b = pc - idx[mm] * str[mm];
            for (int c = 0; c < nc1; ++c) {
                const double dq = Dc[idx[mm] * nc1 + c];
                for (int q = 0; q < DIM; ++q) du[q][mm] += dq * cf[q][b + c * str[mm]];
            }
        }
        const double wj = wJc[e * ncp + pc];
        double A[3][3] = {};
        for (int mm = 0; mm < DIM; ++mm)
            for (int q = 0; q < DIM; ++q) {
                const double drdx = double(Gmc[(e * DIM * DIM + mm * DIM + q) * ncp + pc]) / wj;
                for (int c = 0; c < DIM; ++c) A[c][q] += du[c][mm] * drdx;
            }
        double S[3][3] = {}, tau[3][3] = {};
        int q = DIM;
        for (int r = 0; r < DIM; ++r)
            for (int c = r; c < DIM; ++c) {
                tau[r][c] = tau[c][r] = cf[q][pc] - cf[r][pc] * cf[c][pc];
                ++q;
            }
        double tr = 0.0;
        for (int r = 0; r < DIM; ++r) tr += tau[r][r];
        for (int r = 0; r < DIM; ++r)
            for (int c = 0; c < DIM; ++c) {
                S[r][c] = 0.5 * (A[r][c] + A[c][r]);
                const double td = tau[r][c] - (r == c ? tr / DIM : 0.0);
                num += wj * td * S[r][c];
                den += wj * 2.0 * S[r][c] * S[r][c];
            }
    }
    b0[p] = num;  // b0 and b1 are free after the last pass
    b1[p] = den;
    __syncthreads();
    if (p == 0) {
        double sn = 0.0, sd = 0.0;
        for (int q = 0; q < npf; ++q) {
            sn += b0[q];
            sd += b1[q];
        }
        const double nut = (sd > 0.0) ? fmax(0.0, -sn / sd) : 0.0;
        b0[0] = nut / (dtc / 3.0) / tauc;
    }
    __syncthreads();
    if (p < ncp) y[e * ncp + p] = float(b0[0]);
}

template <int DIM, int Q, typename T, bool DEV>
NodeMap nodemap_of(const sel_sim *s)
{
    NodeMap M;
    M.pcode = s->pcode;
    M.bmap = s->bmap;
    M.bown = s->bown;
    M.E = s->E;
    M.Gi = s->Gi;
    M.QGi = (int64_t)Q * s->Gi;
    M.NP = s->np;
    M.NI = s->nint;
    M.NB = s->nbe;
    M.Q = Q;
    return M;
}

template <int DIM, int Q, typename T, bool DEV>
int run_coarse(const sel_sim *f, sel_sim *c, const double *dP, bool targets, float *y)
{
    const dim3 grid((unsigned)f->E), block((unsigned)f->np);
    if (!targets) {
        hipLaunchKernelGGL((k_coarse<DIM, Q, T, DEV>), grid, block, 0, c->stream, nodemap_of<DIM, Q, T, DEV>(f),
                           static_cast<const T *>(f->f[f->cur]), nodemap_of<DIM, Q, T, DEV>(c),
                           static_cast<T *>(c->f[c->cur]), dP, f->n1, c->n1, f->p.rho0);
    } else {
        hipLaunchKernelGGL((k_targets<DIM, Q, T, DEV>), grid, block, 0, c->stream, nodemap_of<DIM, Q, T, DEV>(f),
                           static_cast<const T *>(f->f[f->cur]), dP, f->n1, c->n1, static_cast<const T *>(c->Gm),
                           c->wJ, c->geoD, f->p.rho0, c->p.dt, c->tau, y);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        set_error(std::string("coarse-graining launch failed: ") + hipGetErrorString(err));
        return SEL_EDEVICE;
    }
    return SEL_OK;
}

int coarse_dispatch(const sel_sim *f, sel_sim *c, const double *dP, bool targets, float *y)
{
    const bool f32 = f->prec == SEL_FP32_DEV;
    if (f->dim == 2 && f->Q == 9)
        return f32 ? run_coarse<2, 9, float, true>(f, c, dP, targets, y) : run_coarse<2, 9, double, false>(f, c, dP, targets, y);
    if (f->dim == 3 && f->Q == 27)
        return f32 ? run_coarse<3, 27, float, true>(f, c, dP, targets, y)
                   : run_coarse<3, 27, double, false>(f, c, dP, targets, y);
    if (f->dim == 3 && f->Q == 19)
        return f32 ? run_coarse<3, 19, float, true>(f, c, dP, targets, y)
                   : run_coarse<3, 19, double, false>(f, c, dP, targets, y);
    set_error("coarse graining: unsupported lattice");
    return SEL_EUNSUPPORTED;
}

int check_pair(const sel_sim *f, const sel_sim *c)
{
    if (!f || !c) {
        set_error("coarse graining: null simulation");
        return SEL_EINVAL;
    }
    if (f->dim != c->dim || f->Q != c->Q || f->prec != c->prec || f->E != c->E || c->N > f->N) {
        set_error("coarse graining: simulations must share dim, lattice, storage and elements, coarse N <= fine N");
        return SEL_EINVAL;
    }
    if (f->np > 1024 || c->np > 512) {
        set_error("coarse graining: order too high (fine np <= 1024, coarse np <= 512)");
        return SEL_EUNSUPPORTED;
    }
    return SEL_OK;
}

}  // namespace

int launch_mlp_infer(sel_sim *s)
{
    const int64_t n = s->Gtot;
    launch_mlp(s->cl_params, s->cl_X, n, float(s->tau), nullptr, s->cl_dtau, s->stream);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        set_error(std::string("closure inference launch failed: ") + hipGetErrorString(err));
        return SEL_EDEVICE;
    }
    return SEL_OK;
}

}  // namespace sel

using sel::set_error;

extern "C" int64_t sel_closure_len(void) { return sel::BLOB; }

extern "C" int sel_closure_set(sel_sim *s, const float *params, int64_t len)
{
    if (!s) {
        set_error("sel_closure_set: null sim");
        return SEL_EINVAL;
    }
    if (!params) {
        s->closure_on = false;
        return SEL_OK;
    }
    if (!s->closure_space) {
        set_error("sel_closure_set: the simulation was created without closure buffers (pass a blob to sel_init)");
        return SEL_ESTATE;
    }
    if (len != sel::BLOB) {
        set_error("sel_closure_set: blob length must be sel_closure_len()");
        return SEL_EINVAL;
    }
    if (hipMemcpyAsync(s->cl_params, params, sizeof(float) * len, hipMemcpyHostToDevice, s->stream) != hipSuccess ||
        hipStreamSynchronize(s->stream) != hipSuccess) {
        set_error("sel_closure_set: upload failed");
        return SEL_EDEVICE;
    }
    s->closure_on = true;
    return SEL_OK;
}

extern "C" int sel_closure_features(sel_sim *s, float *d_X)
{
    if (!s || !d_X) {
        set_error("sel_closure_features: null argument");
        return SEL_EINVAL;
    }
    return sel::find_ops(s->dim, s->N, s->Q, s->prec)->features(s, d_X, 0, 0);
}

extern "C" int sel_closure_dtau(sel_sim *s, float *d_dtau)
{
    if (!s || !d_dtau) {
        set_error("sel_closure_dtau: null argument");
        return SEL_EINVAL;
    }
    if (!s->closure_on) {
        set_error("sel_closure_dtau: no closure attached");
        return SEL_ESTATE;
    }
    if (int rc = sel::find_ops(s->dim, s->N, s->Q, s->prec)->features(s, s->cl_X, 1, 0)) return rc;
    if (int rc = sel::launch_mlp_infer(s)) return rc;
    if (hipMemcpyAsync(d_dtau, s->cl_dtau, sizeof(float) * s->Gtot, hipMemcpyDeviceToDevice, s->stream) != hipSuccess) {
        set_error("sel_closure_dtau: copy failed");
        return SEL_EDEVICE;
    }
    return SEL_OK;
}

static int projection_on_device(const sel_sim *f, const sel_sim *c, double **dP)
{
    std::vector<double> Pm((size_t)c->n1 * f->n1);
    if (sel::build_projection(f->N, c->N, Pm.data())) {
        set_error("coarse graining: projection table");
        return SEL_EINVAL;
    }
    if (hipMalloc(dP, sizeof(double) * Pm.size()) != hipSuccess) {
        set_error("coarse graining: allocation failed");
        return SEL_ENOMEM;
    }
    if (hipMemcpyAsync(*dP, Pm.data(), sizeof(double) * Pm.size(), hipMemcpyHostToDevice, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        (void)hipFree(*dP);
        set_error("coarse graining: upload failed");
        return SEL_EDEVICE;
    }
    return SEL_OK;
}

extern "C" int sel_coarse_grain(const sel_sim *fine, sel_sim *coarse)
{
    if (int rc = sel::check_pair(fine, coarse)) return rc;
    double *dP = nullptr;
    if (int rc = projection_on_device(fine, coarse, &dP)) return rc;
    int rc = hipStreamSynchronize(fine->stream) == hipSuccess ? SEL_OK : SEL_EDEVICE;
    if (!rc) rc = sel::coarse_dispatch(fine, coarse, dP, false, nullptr);
    if (!rc && hipStreamSynchronize(coarse->stream) != hipSuccess) rc = SEL_EDEVICE;
    (void)hipFree(dP);
    return rc;
}

extern "C" int sel_closure_targets(const sel_sim *fine, sel_sim *coarse, float *d_y)
{
    if (!d_y) {
        set_error("sel_closure_targets: null output");
        return SEL_EINVAL;
    }
    if (int rc = sel::check_pair(fine, coarse)) return rc;
    double *dP = nullptr;
    if (int rc = projection_on_device(fine, coarse, &dP)) return rc;
    int rc = hipStreamSynchronize(fine->stream) == hipSuccess ? SEL_OK : SEL_EDEVICE;
    if (!rc) rc = sel::coarse_dispatch(fine, coarse, dP, true, d_y);
    if (!rc && hipStreamSynchronize(coarse->stream) != hipSuccess) rc = SEL_EDEVICE;
    (void)hipFree(dP);
    return rc;
}

extern "C" int sel_mlp_forward(const float *d_params, const float *d_X, int64_t n, double tau, float *d_z,
                               float *d_dtau, void *stream)
{
    if (!d_params || !d_X || n < 0) {
        set_error("sel_mlp_forward: bad argument");
        return SEL_EINVAL;
    }
    if (n == 0) return SEL_OK;
    sel::launch_mlp(d_params, d_X, n, float(tau), d_z, d_dtau, static_cast<hipStream_t>(stream));
    if (hipGetLastError() != hipSuccess) {
        set_error("sel_mlp_forward: launch failed");
        return SEL_EDEVICE;
    }
    return SEL_OK;
}

extern "C" int64_t sel_mlp_work_floats(int64_t n) { return sel::work_floats(n); }

// one Adam step with the training work memory at d_work (both entry points)
static int train_step(const char *who, float *d_params, float *d_m, float *d_v, const float *d_X, const float *d_y,
                      const int32_t *d_idx, int64_t n, int64_t t, double lr, double b1, double b2, double eps,
                      float *d_work, double *loss, void *stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    sel::TrainWork T = sel::carve_work(d_work, n);
    float *dloss = T.part + sel::train_blocks(n);
    sel::launch_gradient(d_params, d_X, d_y, d_idx, n, T, st);
    hipLaunchKernelGGL(sel::k_train_sum<true>, dim3(sel::kSumBlocks), dim3(256), 0, st, T.wpart, T.part,
                       (int)sel::train_blocks(n), n, T.grad, dloss, d_params, d_m, d_v, t, float(lr), float(b1),
                       float(b2), float(eps));
    if (hipGetLastError() != hipSuccess) {
        set_error(std::string(who) + ": launch failed");
        return SEL_EDEVICE;
    }
    if (loss) {
        float h = 0.f;
        if (hipMemcpyAsync(&h, dloss, sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            set_error(std::string(who) + ": device error");
            return SEL_EDEVICE;
        }
        *loss = h;
    }
    return SEL_OK;
}

extern "C" int sel_mlp_train_step(float *d_params, float *d_m, float *d_v, const float *d_X, const float *d_y,
                                  const int32_t *d_idx, int64_t n, int64_t t, double lr, double b1, double b2, double eps, float *d_work,
                                  double *loss, void *stream)
{
    if (!d_params || !d_m || !d_v || !d_X || !d_y || !d_work || n < 1 || t < 1) {
        set_error("sel_mlp_train_step: bad argument");
        return SEL_EINVAL;
    }
    return train_step("sel_mlp_train_step", d_params, d_m, d_v, d_X, d_y, d_idx, n, t, lr, b1, b2, eps, d_work, loss,
                      stream);
}

// ------------------------------------------------ allocation-free training --
// The training work memory of sel_mlp_train_step_noalloc: one file-scope
// device array (each GPU the library runs on holds its own copy until the
// process ends). Host code never passes the array's name to a kernel (on the
// host it only stands for the symbol): the device address is looked up once
// per device with hipGetSymbolAddress, on the first call made with that
// device current, and kept per device. Every call writes each value of the
// work memory it later reads (gradient partials, loss), so nothing needs clearing
// between calls.
constexpr int64_t kNoAllocRows = 4096;
constexpr int64_t kNoAllocFloats = sel::work_floats(kNoAllocRows);
static __device__ __align__(256) float scratch[kNoAllocFloats];

static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float *g_scratch_ptr[kMaxDevices] = {};

static int scratch_of_current_device(float **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        set_error("sel_mlp_train_step_noalloc: no usable current device");
        return SEL_EDEVICE;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error(std::string("sel_mlp_train_step_noalloc: hipGetSymbolAddress failed: ") + hipGetErrorString(e));
            return SEL_EDEVICE;
        }
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return SEL_OK;
}

extern "C" int sel_mlp_train_step_noalloc(float *d_params, float *d_m, float *d_v, const float *d_X,
                                          const float *d_y, const int32_t *d_idx, int64_t n, int64_t t, double lr,
                                          double b1, double b2, double eps, double *loss, void *stream)
{
    if (!d_params || !d_m || !d_v || !d_X || !d_y || n < 1 || t < 1) {
        set_error("sel_mlp_train_step_noalloc: bad argument");
        return SEL_EINVAL;
    }
    if (n > kNoAllocRows) {
        set_error("sel_mlp_train_step_noalloc: at most 4096 rows per call (its fixed work memory); use "
                  "sel_mlp_train_step with a work buffer for larger minibatches");
        return SEL_EINVAL;
    }
    float *work = nullptr;
    if (int rc = scratch_of_current_device(&work)) return rc;
    return train_step("sel_mlp_train_step_noalloc", d_params, d_m, d_v, d_X, d_y, d_idx, n, t, lr, b1, b2, eps, work,
                      loss, stream);
}

extern "C" int sel_mlp_gradient(const float *d_params, const float *d_X, const float *d_y, const int32_t *d_idx,
                                int64_t n, float *d_work, float *d_grad, double *loss, void *stream)
{
    if (!d_params || !d_X || !d_y || !d_work || !d_grad || n < 1) {
        set_error("sel_mlp_gradient: bad argument");
        return SEL_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    sel::TrainWork T = sel::carve_work(d_work, n);
    float *dloss = T.part + sel::train_blocks(n);
    sel::launch_gradient(d_params, d_X, d_y, d_idx, n, T, st);
    hipLaunchKernelGGL(sel::k_train_sum<false>, dim3(sel::kSumBlocks), dim3(256), 0, st, T.wpart, T.part,
                       (int)sel::train_blocks(n), n, T.grad, dloss, nullptr, nullptr, nullptr, 0, 0.f, 0.f, 0.f, 0.f);
    if (hipGetLastError() != hipSuccess) {
        set_error("sel_mlp_gradient: launch failed");
        return SEL_EDEVICE;
    }
    if (hipMemcpyAsync(d_grad, T.grad, sizeof(float) * sel::NTRAIN, hipMemcpyDeviceToDevice, st) != hipSuccess) {
        set_error("sel_mlp_gradient: copy failed");
        return SEL_EDEVICE;
    }
    if (loss) {
        float h = 0.f;
        if (hipMemcpyAsync(&h, dloss, sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            set_error("sel_mlp_gradient: device error");
            return SEL_EDEVICE;
        }
        *loss = h;
    }
    return SEL_OK;
}
