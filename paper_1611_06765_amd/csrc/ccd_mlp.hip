// ccd_mlp.hip -- training and inference kernels of the warm-start network
// (include/ccd_mlp.h): forward on a feature buffer (FP32 or BF16 MFMA), loss
// and gradient (FP32 MFMA), and the Adam update of Kingma and Ba (2015),
// Algorithm 1.  Gradients are summed in a fixed order (per-block partials,
// then one reduction), so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "../../include/ccd_mlp.h"
#include "ccd_internal.h"
#include "mlp_net.h"

using namespace mlp;

namespace {

#define MLP_TRY(x)                                                                      \
    do {                                                                                \
        hipError_t e_ = (x);                                                            \
        if (e_ != hipSuccess) {                                                         \
            ccd::set_error(std::string(#x) + ": " + hipGetErrorString(e_));             \
            return CCD_EHIP;                                                            \
        }                                                                               \
    } while (0)

// ---- forward on a buffer of packed features -----------------------------------
// A wave takes NT tiles of four amplitudes (16 rows) at a time, the next ones'
// features on their way meanwhile, and a grid of the blocks that fit the chip at
// once (three per compute unit in BF16 at 168 registers, two in FP32) strides over
// them, so W2 is staged once per resident block.  1 037 776 amplitudes in BF16: 240 ->
// 176 us a call in a long row of calls, 257 -> 192 waited for.  By step, in bursts of
// five calls after an idle GPU, which take longer: 275 us with one tile at a time, 2048
// blocks and the accumulators in the AGPR file, 225 with two, 208 with 168 plain
// registers (four tiles 226, at two waves a SIMD; the next step's layer 1 issued among
// this step's MFMAs 220); 60 000 amplitudes 33 -> 22 us.  FP32 1336 -> 1220.  What is
// left is the activations' VALU time beside the MFMAs (see tile_predict).
template <bool BF16, int NT>
__global__ void __launch_bounds__(256, 3) k_mlp_fwd(const float* __restrict__ P, const float* __restrict__ feat,
                                                 int64_t n, float* __restrict__ y) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const Lds s = lds_carve<BF16>(lds);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr int kAmps = 4 * NT;
    const int64_t ngrp = (n + kAmps - 1) / kAmps, step = (int64_t)gridDim.x * 4;
    float4 nx[NT][2];
    auto fetch = [&](int64_t t) {
#pragma unroll
        for (int k = 0; k < NT; k++) {
            const int64_t e = kAmps * t + 4 * k + ((lane & 15) >> 2);
            nx[k][0] = nx[k][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (e < n) {
                nx[k][0] = *(const float4*)&feat[e * kPack];
                nx[k][1] = *(const float4*)&feat[e * kPack + 4];
            }
        }
    };
    int64_t t = (int64_t)blockIdx.x * 4 + w;
    fetch(t);
    lds_load<BF16>(P, s, threadIdx.x, 256);
    __syncthreads();
    for (; t < ngrp; t += step) {
        float f[NT][kPack], yp[NT];
#pragma unroll
        for (int k = 0; k < NT; k++) {
            const float4 a = nx[k][0], b = nx[k][1];
            f[k][0] = a.x; f[k][1] = a.y; f[k][2] = a.z; f[k][3] = a.w;
            f[k][4] = b.x; f[k][5] = b.y; f[k][6] = b.z; f[k][7] = b.w;
        }
        fetch(t + step);
        tile_predict<BF16, NT>(f, s, lane, yp);
#pragma unroll
        for (int k = 0; k < NT; k++) {
            const int64_t eo = kAmps * t + 4 * k + (lane >> 4);
            if ((lane & 15) == 0 && eo < n) y[eo] = yp[k];
        }
    }
}

// ---- loss and gradient ----------------------------------------------------------
// A block takes chunks of kCh = 16 amplitudes (64 rows = 16 amplitudes x 4 swap
// variants) of the batch, `nc` chunks in a row.  Wave w = (rt, ch): row tile
// rt = w / 2 (amplitudes 4 rt .. 4 rt + 3 of the chunk) and column half ch =
// w % 2 of the 128 x 128 layer.  Per chunk:
//   h1 = relu(W1 x + b1)                      (VALU, into LDS)
//   z2 = h1 W2^T + b2, g = W3 relu(z2)        (MFMA, W2 in LDS)
//   y = sum_k sign_k g_k / 4, dL/dg_k = sign_k (y - y*) / (4 M)
//   dz2 = dg W3 relu'(z2)                     (into LDS)
//   dW2 += dz2^T h1                            (MFMA 32x32x2, two tiles per wave held in registers)
//   dh1 = dz2 W2, dz1 = dh1 relu'(z1)         (MFMA; relu'(z1) = [h1 > 0])
//   dW1 += dz1^T x, db1 += sum dz1, db2 += sum dz2, dW3 += dg^T relu(z2)
// The block's sums go to its row of the partial-gradient buffer.
//
// Bound by the FP32 MFMA rate: 6.3 MFLOP per chunk, 11 us of one compute unit at
// the measured 141 TFLOP/s of all 256.  W2, h1 and dz2 take 137 KB of LDS, one
// block per compute unit, so a batch is cut into at most kMaxBlk = 256 blocks and
// a block loops over chunks only past 4096 amplitudes; eight waves (two per SIMD)
// cover each other's LDS reads.  Batch 4096: 110 us in 64 blocks of eight serial
// 32-row chunks, 30 us in 256 blocks of one 64-row chunk; what is left beside the
// products is staging W2, the gathered features and 18 MB of partial rows.
constexpr int kCh = 16;        // amplitudes per chunk
constexpr int kMaxBlk = 256;   // partial-gradient rows: one block per compute unit
constexpr int kGradThreads = 512;
constexpr int kLdH = kW + 4;

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // the parameters need no more than float alignment
// D = A B + C for 32x32x2 FP32 tiles: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32] and receives D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32]
__device__ __forceinline__ f16v mfma_f32_32(float a, float b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__host__ __device__ constexpr size_t grad_lds_bytes() {
    return (size_t)(kW * kLd32 + 2 * 4 * kCh * kLdH + kCh * kPack + 2 * kCh + 2 * 4 * kCh) * 4;
}

// Indices of `order` outside [0, n_rows) are skipped (the amplitude counts as
// absent) and counted in *bad.
__global__ void __launch_bounds__(kGradThreads) k_mlp_grad(
    const float* __restrict__ P, const float* __restrict__ feat, const float* __restrict__ target,
    const int32_t* __restrict__ order, int64_t base, int64_t n, int64_t n_rows, int nc, float inv_m,
    float* __restrict__ work, float* __restrict__ work_loss, int32_t* __restrict__ bad) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float* W2 = (float*)lds;                 // [128][kLd32]
    float* H1 = W2 + kW * kLd32;             // [64][kLdH]
    float* DZ2 = H1 + 4 * kCh * kLdH;        // [64][kLdH]
    float* Fs = DZ2 + 4 * kCh * kLdH;        // [16][8]
    float* Ys = Fs + kCh * kPack;            // [16]
    float* Vs = Ys + kCh;                    // [16] 1 = amplitude present
    float* Gs = Vs + kCh;                    // [2][64]

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, rt = w >> 1, ch = w & 1;
    const int r16 = lane & 15, kq = lane >> 4;
    const int64_t e0 = (int64_t)blockIdx.x * nc * kCh;
    const int64_t e1 = std::min<int64_t>(n, e0 + (int64_t)nc * kCh);

    // feature q of amplitude el of the chunk at e (threads 0 .. 127), loaded one
    // chunk ahead; q = 0 also carries the target and the presence flag
    float nf = 0.f, ny = 0.f, nv = 0.f;
    auto fetch = [&](int64_t e) {
        if (tid < kCh * kPack) {
            const int el = tid >> 3, q = tid & 7;
            const int64_t li = e + el;
            int64_t gi = li < e1 ? (order ? (int64_t)order[base + li] : base + li) : -1;
            if (li < e1 && (gi < 0 || gi >= n_rows)) {
                if (q == 0) atomicAdd(bad, 1);
                gi = -1;
            }
            const bool ok = gi >= 0;
            nf = ok ? feat[gi * kPack + q] : 0.f;
            nv = ok ? 1.f : 0.f;
            ny = ok && q == 0 ? target[gi] : 0.f;
        }
    };
    fetch(e0);
    // W2 is on its way while the first chunk's layer 1 runs
    constexpr int kW2Per = kW * kW / (4 * kGradThreads);
    f4v w2r[kW2Per];
#pragma unroll
    for (int k = 0; k < kW2Per; k++) w2r[k] = *(const f4u*)&P[OFF_W2 + 4 * (tid + kGradThreads * k)];
    // layer-1 weights of unit tid % 128, and b2 / W3 of this lane's four columns
    const int c1 = tid & 127;
    float w1[7];
#pragma unroll
    for (int q = 0; q < 7; q++) w1[q] = P[OFF_W1 + c1 * kPack + q];
    const float b1 = P[OFF_B1 + c1];
    float b2[4], w3[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int col = (ch * 4 + j) * 16 + r16;
        b2[j] = P[OFF_B2 + col];
        w3[j] = P[OFF_W3 + col];
    }

    // dW2 tiles: rows 32 (w / 2), columns 32 (2 (w % 2) + u), u = 0, 1
    f16v aW2[2];
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int i = 0; i < 16; i++) aW2[u][i] = 0.f;
    float aW3[4] = {0.f, 0.f, 0.f, 0.f}, aB2[4] = {0.f, 0.f, 0.f, 0.f}, aB1[4] = {0.f, 0.f, 0.f, 0.f};
    float aW1[4][7];
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
        for (int q = 0; q < 7; q++) aW1[j][q] = 0.f;
    // in 64 bits: a lane adds a term per chunk, and a block's run of chunks grows with the batch
    double loss = 0.0;

    for (int64_t e = e0; e < e1; e += kCh) {
        __syncthreads();  // previous chunk done with Fs, H1, DZ2, Gs
        if (tid < kCh * kPack) {
            Fs[tid] = nf;
            if ((tid & 7) == 0) { Ys[tid >> 3] = ny; Vs[tid >> 3] = nv; }
        }
        __syncthreads();
        if (e + kCh < e1) fetch(e + kCh);
        // layer 1 into LDS: unit c1, rows tid / 128 + 4 m (variant tid / 128 of amplitude m)
        {
            const int k = tid >> 7;
#pragma unroll 4
            for (int el = 0; el < kCh; el++) {
                float x[7];
                variant_inputs(&Fs[el * kPack], k, x);
                float z = b1;
#pragma unroll
                for (int q = 0; q < 7; q++) z += w1[q] * x[q];
                H1[(4 * el + k) * kLdH + c1] = act(z);
            }
        }
        if (e == e0) {
#pragma unroll
            for (int k = 0; k < kW2Per; k++) {
                const int q = 4 * (tid + kGradThreads * k);
                *(f4v*)&W2[(q >> 7) * kLd32 + (q & 127)] = w2r[k];
            }
        }
        __syncthreads();
        // layer 2 and the wave's share of g
        f4v z2[4];
#pragma unroll
        for (int j = 0; j < 4; j++) z2[j] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int st = 0; st < 32; st++) {
            const float a = H1[(rt * 16 + r16) * kLdH + 4 * st + kq];
#pragma unroll
            for (int j = 0; j < 4; j++)
                z2[j] = mfma_f32(a, W2[((ch * 4 + j) * 16 + r16) * kLd32 + 4 * st + kq], z2[j]);
        }
        float gp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                z2[j][i] += b2[j];
                gp[i] += act(z2[j][i]) * w3[j];
            }
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) gp[i] += __shfl_xor(gp[i], o);
        if (r16 == 0)
#pragma unroll
            for (int i = 0; i < 4; i++) Gs[ch * 4 * kCh + rt * 16 + 4 * kq + i] = gp[i];
        __syncthreads();
        // residual of amplitude el = 4 rt + kq; dL/dg of its four rows
        const int el = rt * 4 + kq;
        float g[4];
#pragma unroll
        for (int i = 0; i < 4; i++) g[i] = Gs[4 * el + i] + Gs[4 * kCh + 4 * el + i];
        const float yp = 0.25f * ((g[0] - g[1]) - (g[2] - g[3]));
        const float res = Vs[el] != 0.f ? yp - Ys[el] : 0.f;
        if (ch == 0 && r16 == 0) loss += (double)(0.5f * res * res * inv_m);
        float dg[4];
#pragma unroll
        for (int i = 0; i < 4; i++) dg[i] = variant_sign(i) * 0.25f * res * inv_m;
        // dz2, dW3, db2
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int col = (ch * 4 + j) * 16 + r16;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float dz = dg[i] * w3[j] * dact(z2[j][i]);
                aW3[j] += dg[i] * act(z2[j][i]);
                aB2[j] += dz;
                DZ2[(rt * 16 + 4 * kq + i) * kLdH + col] = dz;
            }
        }
        __syncthreads();
        // dW2 += dz2^T h1 over the chunk's 64 rows
        {
            const int r32 = lane & 31, kh = lane >> 5;
#pragma unroll 8
            for (int st = 0; st < 2 * kCh; st++) {
                const int r = 2 * st + kh;
                const float av = DZ2[r * kLdH + 32 * rt + r32];
#pragma unroll
                for (int u = 0; u < 2; u++)
                    aW2[u] = mfma_f32_32(av, H1[r * kLdH + 32 * (2 * ch + u) + r32], aW2[u]);
            }
        }
        // dh1 = dz2 W2 for rows of tile rt, k-tiles ch*4 .. ch*4+3
        f4v dh[4];
#pragma unroll
        for (int j = 0; j < 4; j++) dh[j] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int st = 0; st < 32; st++) {
            const float a = DZ2[(rt * 16 + r16) * kLdH + 4 * st + kq];
#pragma unroll
            for (int j = 0; j < 4; j++)
                dh[j] = mfma_f32(a, W2[(4 * st + kq) * kLd32 + (ch * 4 + j) * 16 + r16], dh[j]);
        }
        // dz1 = dh1 relu'(z1), rows 4 el + i (variant i of amplitude el)
        float xv[4][7];
#pragma unroll
        for (int i = 0; i < 4; i++) variant_inputs(&Fs[el * kPack], i, xv[i]);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int c = (ch * 4 + j) * 16 + r16;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float dz1 = dh[j][i] * dact(H1[(4 * el + i) * kLdH + c]);
                aB1[j] += dz1;
#pragma unroll
                for (int q = 0; q < 7; q++) aW1[j][q] += dz1 * xv[i][q];
            }
        }
    }
    // ---- block sums -> partial-gradient row of this block
    float* out = work + (size_t)blockIdx.x * kParams;
    // lane groups kq hold partial sums over their rows: reduce over kq
#pragma unroll
    for (int j = 0; j < 4; j++) {
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            aW3[j] += __shfl_xor(aW3[j], o);
            aB2[j] += __shfl_xor(aB2[j], o);
            aB1[j] += __shfl_xor(aB1[j], o);
#pragma unroll
            for (int q = 0; q < 7; q++) aW1[j][q] += __shfl_xor(aW1[j][q], o);
        }
    }
    // the waves of row tiles 1 .. 3 hand their column sums to row tile 0's of
    // the same half, which adds them in tile order
    __syncthreads();
    float* X = H1;  // [3 row tiles][128 columns][10] scratch
    if (rt > 0 && kq == 0) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float* q = X + ((rt - 1) * kW + (ch * 4 + j) * 16 + r16) * 10;
            q[0] = aW3[j]; q[1] = aB2[j]; q[2] = aB1[j];
#pragma unroll
            for (int f = 0; f < 7; f++) q[3 + f] = aW1[j][f];
        }
    }
    __syncthreads();
    if (rt == 0 && kq == 0) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int col = (ch * 4 + j) * 16 + r16;
            float v[10] = {aW3[j], aB2[j], aB1[j]};
#pragma unroll
            for (int f = 0; f < 7; f++) v[3 + f] = aW1[j][f];
            for (int t = 0; t < 3; t++)
#pragma unroll
                for (int f = 0; f < 10; f++) v[f] += X[(t * kW + col) * 10 + f];
            out[OFF_W3 + col] = v[0];
            out[OFF_B2 + col] = v[1];
            out[OFF_B1 + col] = v[2];
#pragma unroll
            for (int f = 0; f < 7; f++) out[OFF_W1 + col * kPack + f] = v[3 + f];
            out[OFF_W1 + col * kPack + 7] = 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int i = 0; i < 16; i++)
            out[OFF_W2 + (32 * rt + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3)) * kW + 32 * (2 * ch + u) + (lane & 31)] =
                aW2[u][i];
    // b3 cancels in the antisymmetrised output; padding stays zero
    if (tid < kParams - OFF_B3) out[OFF_B3 + tid] = 0.f;
    // loss: lanes r16 == 0 of waves ch == 0 hold it
    loss += __shfl_xor(loss, 16);
    loss += __shfl_xor(loss, 32);
    double* Ls = (double*)Gs;
    if (ch == 0 && lane == 0) Ls[rt] = loss;
    __syncthreads();
    if (tid == 0) work_loss[blockIdx.x] = (float)((Ls[0] + Ls[1]) + (Ls[2] + Ls[3]));
}

// sum of the block partials (fixed order: four quarters of the rows, each in
// row order, then the quarters in order); mode 0 writes the gradient, mode 1
// applies one Adam step.  A block owns 64 parameters, one wave per quarter with
// 16 row loads in flight (256 rows, 18 MB: 5.7 us; one thread per parameter over
// 64 rows took 18 us, a serial chain of loads); the last block adds the batch loss
// to acc[0].
constexpr int kRedParams = 64, kRedBlocks = (kParams + kRedParams - 1) / kRedParams + 1;
__global__ void __launch_bounds__(256) k_mlp_reduce(const float* __restrict__ work, const float* __restrict__ work_loss,
                                                    int nblk, int mode, float* __restrict__ grad, float* __restrict__ P,
                                                    float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                                    float b2, float eps, float bc1, float bc2, double* acc) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        if (w > 0) return;
        double l = 0.0;
        for (int b = lane; b < nblk; b += 64) l += (double)work_loss[b];
        for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
        if (lane == 0) acc[0] += l;
        return;
    }
    __shared__ float sh[4][kRedParams];
    const int p = blockIdx.x * kRedParams + lane;
    const int per = (nblk + 3) / 4, lo = w * per, hi = min(nblk, lo + per);
    float g = 0.f;
    if (p < kParams) {
        const float* q = work + p;
        int b = lo;
        for (; b + 16 <= hi; b += 16) {
            float x[16];
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = q[(size_t)(b + k) * kParams];
#pragma unroll
            for (int k = 0; k < 16; k++) g += x[k];
        }
        for (; b < hi; b++) g += q[(size_t)b * kParams];
    }
    sh[w][lane] = g;
    __syncthreads();
    if (w > 0 || p >= kParams) return;
    g = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
    if (mode == 0) {
        grad[p] = g;
    } else {
        const float mn = b1 * m[p] + (1.f - b1) * g;
        const float vn = b2 * v[p] + (1.f - b2) * g * g;
        m[p] = mn;
        v[p] = vn;
        P[p] -= lr * (mn / bc1) / (sqrtf(vn / bc2) + eps);
    }
}

__global__ void k_mlp_zero(double* acc, int32_t* bad) {
    acc[0] = 0.0;
    bad[0] = 0;
}

struct Work {
    float* part;
    float* loss;
    double* acc;
    int32_t* bad;   // count of out-of-range indices
};

// A work area holds one partial-gradient row per block: at most kMaxBlk, one per
// chunk of a small batch.  (The size grows with n, so an area made for n serves
// every smaller batch.)
size_t bytes_of_rows(int64_t rows) {
    return (size_t)rows * kParams * 4 + (size_t)((rows + 63) / 64) * 256 + 256;
}
int64_t rows_for(int64_t n) { return std::max<int64_t>(1, std::min<int64_t>(kMaxBlk, (n + kCh - 1) / kCh)); }
size_t work_bytes_for(int64_t n) { return bytes_of_rows(rows_for(n)); }

// The blocks of a batch of n and the chunks of each.  An area of only one row
// per 64 amplitudes is taken too, with fewer blocks.
struct Split {
    int nblk, nc;
};
Split split_for(int64_t n, size_t bytes) {
    int64_t rows = rows_for(n);
    if (bytes < bytes_of_rows(rows)) rows = std::max<int64_t>(1, std::min(rows, (n + 63) / 64));
    const int64_t nch = (n + kCh - 1) / kCh, nc = (nch + rows - 1) / rows;
    return {(int)((nch + nc - 1) / nc), (int)nc};
}
bool work_fits(int64_t n, size_t bytes) {
    return bytes >= work_bytes_for(n) || bytes >= bytes_of_rows(std::max<int64_t>(1, (n + 63) / 64));
}

Work carve(void* w, int rows) {
    Work k;
    k.part = (float*)w;
    k.loss = k.part + (size_t)rows * kParams;
    k.acc = (double*)((char*)w + bytes_of_rows(rows) - 256);
    k.bad = (int32_t*)(k.acc + 1);
    return k;
}

ccd_status grad_attrs() {
    static bool done = false;
    if (done) return CCD_OK;
    MLP_TRY(hipFuncSetAttribute((const void*)k_mlp_grad, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)grad_lds_bytes()));
    MLP_TRY(hipFuncSetAttribute((const void*)k_mlp_fwd<false, 1>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes<false>()));
    MLP_TRY(hipFuncSetAttribute((const void*)k_mlp_fwd<false, 2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_bytes<false>()));
    done = true;
    return CCD_OK;
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

}  // namespace

extern "C" {

ccd_status ccd_mlp_forward(const float* params, const float* feat, int64_t n, int32_t precision, float* y,
                           void* stream) {
    if (!params || (n > 0 && (!feat || !y)) || n < 0 ||
        (precision != CCD_PREC_FP32 && precision != CCD_PREC_BF16)) {
        ccd::set_error("ccd_mlp_forward: need params, feat, y, n >= 0 and precision FP32 or BF16");
        return CCD_EINVAL;
    }
    if (!aligned(params, 16) || !aligned(feat, 16)) {
        ccd::set_error("ccd_mlp_forward: params and feat must be 16-byte aligned");
        return CCD_EINVAL;
    }
    if (n == 0) return CCD_OK;
    ccd_status s = grad_attrs();
    if (s != CCD_OK) return s;
    // two tiles a wave once one each would give every wave of the chip two to four: below
    // that half as many waves would only be slower (100 amplitudes in FP32 16.6 -> 20.4 us)
    const int64_t ntile = (n + 3) / 4;
    const bool bf16 = precision == CCD_PREC_BF16, two = ntile > 4096;
    const int64_t waves = two ? (ntile + 1) / 2 : ntile;
    const int grid = (int)std::min<int64_t>((waves + 3) / 4, bf16 ? 768 : 512);
    const auto k = bf16 ? (two ? k_mlp_fwd<true, 2> : k_mlp_fwd<true, 1>)
                        : (two ? k_mlp_fwd<false, 2> : k_mlp_fwd<false, 1>);
    hipLaunchKernelGGL(k, dim3(grid), dim3(256), bf16 ? lds_bytes<true>() : lds_bytes<false>(), (hipStream_t)stream,
                       params, feat, n, y);
    MLP_TRY(hipGetLastError());
    return CCD_OK;
}

ccd_status ccd_mlp_work_size(int64_t n, size_t* bytes) {
    if (!bytes || n < 1) {
        ccd::set_error("ccd_mlp_work_size: need n >= 1 and bytes");
        return CCD_EINVAL;
    }
    *bytes = work_bytes_for(n);
    return CCD_OK;
}

ccd_status ccd_mlp_loss_grad(const float* params, const float* feat, const float* target, int64_t n, float* grad,
                             double* loss, void* work, size_t work_bytes, void* stream) {
    if (!params || !feat || !target || !grad || !work || n < 1) {
        ccd::set_error("ccd_mlp_loss_grad: NULL argument or n < 1");
        return CCD_EINVAL;
    }
    if (!work_fits(n, work_bytes) || !aligned(work, 256)) {
        ccd::set_error("ccd_mlp_loss_grad: work buffer too small or not 256-byte aligned");
        return CCD_EINVAL;
    }
    ccd_status s = grad_attrs();
    if (s != CCD_OK) return s;
    const Split sp = split_for(n, work_bytes);
    const Work k = carve(work, sp.nblk);
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_mlp_zero, dim3(1), dim3(1), 0, st, k.acc, k.bad);
    hipLaunchKernelGGL(k_mlp_grad, dim3(sp.nblk), dim3(kGradThreads), grad_lds_bytes(), st, params, feat, target,
                       (const int32_t*)nullptr, (int64_t)0, n, n, sp.nc, 1.0f / (float)n, k.part, k.loss, k.bad);
    hipLaunchKernelGGL(k_mlp_reduce, dim3(kRedBlocks), dim3(256), 0, st, k.part, k.loss, sp.nblk, 0, grad,
                       (float*)nullptr, (float*)nullptr, (float*)nullptr, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f, k.acc);
    MLP_TRY(hipGetLastError());
    if (loss) {
        MLP_TRY(hipMemcpyAsync(loss, k.acc, 8, hipMemcpyDeviceToHost, st));
        MLP_TRY(hipStreamSynchronize(st));
    }
    return CCD_OK;
}

ccd_status ccd_mlp_train(float* params, float* adam_m, float* adam_v, int64_t* step, const float* feat,
                         const float* target, int64_t n_rows, const int32_t* order, int64_t n_order,
                         const ccd_adam_opts* o, void* work, size_t work_bytes, double* mean_loss, void* stream) {
    if (!params || !adam_m || !adam_v || !step || !feat || !target || !order || !o || !work || n_rows < 1) {
        ccd::set_error("ccd_mlp_train: NULL argument or n_rows < 1");
        return CCD_EINVAL;
    }
    if (o->batch < 1 || n_order < o->batch || !(o->lr > 0.f) || !(o->beta1 >= 0.f && o->beta1 < 1.f) ||
        !(o->beta2 >= 0.f && o->beta2 < 1.f) || !(o->eps > 0.f) || *step < 0) {
        ccd::set_error("ccd_mlp_train: need 1 <= batch <= n_order, lr > 0, 0 <= beta < 1, eps > 0, step >= 0");
        return CCD_EINVAL;
    }
    if (!work_fits(o->batch, work_bytes) || !aligned(work, 256)) {
        ccd::set_error("ccd_mlp_train: work buffer smaller than ccd_mlp_work_size(batch) or misaligned");
        return CCD_EINVAL;
    }
    ccd_status s = grad_attrs();
    if (s != CCD_OK) return s;
    const Split sp = split_for(o->batch, work_bytes);
    const Work k = carve(work, sp.nblk);
    const int64_t nsteps = n_order / o->batch;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_mlp_zero, dim3(1), dim3(1), 0, st, k.acc, k.bad);
    for (int64_t q = 0; q < nsteps; q++) {
        const int64_t t = *step + 1;
        const float bc1 = (float)(1.0 - std::pow((double)o->beta1, (double)t));
        const float bc2 = (float)(1.0 - std::pow((double)o->beta2, (double)t));
        hipLaunchKernelGGL(k_mlp_grad, dim3(sp.nblk), dim3(kGradThreads), grad_lds_bytes(), st, params, feat, target, order,
                           q * o->batch, (int64_t)o->batch, n_rows, sp.nc, 1.0f / (float)o->batch, k.part, k.loss, k.bad);
        hipLaunchKernelGGL(k_mlp_reduce, dim3(kRedBlocks), dim3(256), 0, st, k.part, k.loss, sp.nblk, 1,
                           (float*)nullptr, params, adam_m, adam_v, o->lr, o->beta1, o->beta2, o->eps, bc1, bc2,
                           k.acc);
        MLP_TRY(hipGetLastError());
        *step = t;
    }
    double acc = 0.0;
    int32_t bad = 0;
    MLP_TRY(hipMemcpyAsync(&acc, k.acc, 8, hipMemcpyDeviceToHost, st));
    MLP_TRY(hipMemcpyAsync(&bad, k.bad, 4, hipMemcpyDeviceToHost, st));
    MLP_TRY(hipStreamSynchronize(st));
    if (mean_loss) *mean_loss = acc / (double)nsteps;
    if (bad) {
        ccd::set_error("ccd_mlp_train: " + std::to_string(bad) + " indices of order outside [0, n_rows) were skipped");
        return CCD_EINVAL;
    }
    return CCD_OK;
}

}  // extern "C"
