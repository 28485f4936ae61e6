// mlp.hip -- training and packing of the opacity surrogate on gfx950.
//
// Training minimises L = (1/B) sum_b sum_o (y_bo - t_bo)^2 / 2 over
// mini-batches of table coordinates, targets t = (log10 kappa_table - mean)
// / std from bilinear lookups of the bound table.  One block handles 64
// samples: layers 1 and 3 on the vector ALU in FP32, the 64x64 products of the
// forward pass (W2 h1) and of back-propagation (dL/dh1 = W2^T dz2 and dL/dW2 =
// sum_s dz2 h1^T) on the bfloat16 matrix cores (v_mfma_f32_32x32x16_bf16, FP32
// accumulation) with each operand split into a high part and a remainder,
// keeping hi*hi + hi*lo + lo*hi (about 16 significant bits per product), the
// small layers on the vector ALU.  Per-block gradients go to a partial buffer
// that one kernel reduces in a fixed order before the Adam update (Kingma &
// Ba 2015), so training is deterministic.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "m1_internal.h"
#include "mlp_device.h"

namespace m1 {

constexpr int NP = M1_MLP_NPARAM;
// parameter offsets in the flat vector (W1 b1 W2 b2 W3 b3 Ws)
constexpr int P_W1 = 0, P_B1 = 128, P_W2 = 192, P_B2 = 4288, P_W3 = 4352, P_B3 = 4480, P_WS = 4482;
// transposed W2 fragments for back-propagation, after the inference pack
constexpr int MLP_OFF_W2THI = MLP_PACK_FLOATS, MLP_OFF_W2TLO = MLP_PACK_FLOATS + 2048;
// then a copy of the flat parameters, from which the inference entries are derived
constexpr int MLP_OFF_THETA = MLP_PACK_FLOATS + 4096;
constexpr int MLP_TRAIN_PACK = MLP_OFF_THETA + NP;
constexpr int LDS_STRIDE = 65;

// ---------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------

// Fragment slot of A-operand element (m, k) of a 64x64 matrix for
// v_mfma_f32_32x32x16_bf16: tile mt = m / 32, k-step ks = k / 16, lane =
// 32 ((k % 16) / 8) + m % 32, element e = k % 8.
__host__ __device__ __forceinline__ int frag_slot(int m, int k)
{
    const int mt = m >> 5, ks = k >> 4, lane = ((k & 15) >> 3) * 32 + (m & 31), e = k & 7;
    return ((mt * 4 + ks) * 64 + lane) * 8 + e;
}

// The inference form's LDS image in the packed network, from the flat
// parameters: the split fragments of A2 = s W2 (s = MLP_TANH_SCALE), one W2
// element per thread, and the layer-1, bias and output entries
// (mlp_image_entry).  16 blocks of 256 threads.
__global__ void __launch_bounds__(256) k_mlp_pack_infer(const float *theta, float *pk)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int u = t >> 6, k = t & 63;
    MlpShared &img = *reinterpret_cast<MlpShared *>(pk + MLP_OFF_IMG);
    const float v = MLP_TANH_SCALE * theta[P_W2 + t];
    const __bf16 h = to_bf16(v);
    reinterpret_cast<__bf16 *>(&img.w2[0][0][0][0])[frag_slot(u, k)] = h;
    reinterpret_cast<__bf16 *>(&img.w2[1][0][0][0])[frag_slot(u, k)] = to_bf16(v - float(h));
    mlp_image_entry(theta + P_W1, theta + P_B1, theta + P_B2, theta + P_W3, img, t);
}

// One parameter's entries in the packed network (all but the inference image).
__device__ __forceinline__ void pack_param(float *pk, int i, float w)
{
    if (i < P_B1) pk[MLP_OFF_W1 + i] = w;
    else if (i < P_W2) pk[MLP_OFF_B1 + (i - P_B1)] = w;
    else if (i < P_B2) {
        const int u = (i - P_W2) >> 6, k = (i - P_W2) & 63;
        const __bf16 h = to_bf16(w), l = to_bf16(w - float(h));
        reinterpret_cast<__bf16 *>(pk + MLP_OFF_W2HI)[frag_slot(u, k)] = h;
        reinterpret_cast<__bf16 *>(pk + MLP_OFF_W2LO)[frag_slot(u, k)] = l;
        reinterpret_cast<__bf16 *>(pk + MLP_OFF_W2THI)[frag_slot(k, u)] = h;
        reinterpret_cast<__bf16 *>(pk + MLP_OFF_W2TLO)[frag_slot(k, u)] = l;
    } else if (i < P_W3) pk[MLP_OFF_B2 + (i - P_B2)] = w;
    else if (i < P_B3) pk[MLP_OFF_W3 + (i - P_W3)] = w;
    else if (i < P_WS) pk[MLP_OFF_B3 + (i - P_B3)] = w;
    else pk[MLP_OFF_WS + (i - P_WS)] = w;
}

// The entries other than the inference image from the flat parameters at
// MLP_OFF_THETA, and the normalisation.  With `adam` ([3][NP]) also the start of
// a training run: two moments of zero and the parameters.
constexpr int PACK_BLOCKS = (NP + 255) / 256;

__global__ void __launch_bounds__(256) k_mlp_pack(float *pk, float4 norm, float *adam)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 4) pk[MLP_OFF_NORM + i] = i == 0 ? norm.x : i == 1 ? norm.y : i == 2 ? norm.z : norm.w;
    if (i >= NP) return;
    const float w = pk[MLP_OFF_THETA + i];
    pack_param(pk, i, w);
    if (adam) {
        adam[i] = 0.f;
        adam[NP + i] = 0.f;
        adam[2 * NP + i] = w;
    }
}

// Parameters and normalisation to the device and k_mlp_pack, in the context's
// stream; theta must stay as it is until the stream is synchronised.  What the
// caller queued on the default stream (the samples, say) is waited for, also
// where the context's stream does not wait for that one by itself.
static hipError_t upload_network(m1_ctx *c, const float *theta, const double *norm, float *adam)
{
    hipError_t e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(c->mlp_dev + MLP_OFF_THETA, theta, NP * sizeof(float), hipMemcpyHostToDevice, c->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_pack, dim3(PACK_BLOCKS), dim3(256), 0, c->stream, c->mlp_dev,
                       make_float4(float(norm[0]), float(norm[1]), float(norm[2]), float(norm[3])), adam);
    return hipGetLastError();
}

static hipError_t mlp_buffer(m1_ctx *c)
{
    if (c->mlp_dev) return hipSuccess;
    return device_alloc(reinterpret_cast<void **>(&c->mlp_dev), MLP_TRAIN_PACK * sizeof(float));
}

int mlp_pack(m1_ctx *c, const float *theta, const double *norm)
{
    if (mlp_buffer(c) != hipSuccess) {
        set_error("MLP buffer allocation failed");
        return -2;
    }
    std::vector<float> host(theta, theta + NP);
    hipError_t e = upload_network(c, host.data(), norm, nullptr);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mlp_pack_infer, dim3(16), dim3(256), 0, c->stream, c->mlp_dev + MLP_OFF_THETA,
                           c->mlp_dev);
        e = hipGetLastError();
    }
    const hipError_t es = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) {
        set_error(std::string("MLP upload: ") + hipGetErrorString(e));
        return -3;
    }
    c->mlp_theta.swap(host);
    for (int i = 0; i < 4; ++i) c->op.norm[i] = norm[i];
    c->op.mlp = c->mlp_dev;
    return 0;
}

// ---------------------------------------------------------------------------
// forward + backward of 64 samples
// ---------------------------------------------------------------------------

struct TrainArgs {
    const float *pk;       // packed current network (inference + transposed frags)
    const float *samples;  // [n][2] table coordinates
    long n_train;
    long offset;
    float inv_batch;
    OpacityParams op;      // table (targets) and axes
    float *partial;        // [nblk][NP]
    float *loss_part;      // [nblk]
};

// value of v in a lane given by a wavefront-uniform number
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ void split8(const float v[8], bf16x8 &h, bf16x8 &l)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 b = to_bf16(v[e]);
        h[e] = b;
        l[e] = to_bf16(v[e] - float(b));
    }
}

__device__ __forceinline__ f32x16 mfma3(const bf16x8 &ah, const bf16x8 &al, const bf16x8 &bh, const bf16x8 &bl,
                                        f32x16 acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc, 0, 0, 0);
    return acc;
}

// Sums over the 64 samples in their order: of column[s] weight[s] (weights the
// same in every lane, 16-byte aligned) and of column[s].
__device__ __forceinline__ float dot64(const float *column, const float *weight)
{
    const float4 *wt = reinterpret_cast<const float4 *>(weight);
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < 64; s += 4) {
        const float4 x = wt[s / 4];
        acc += column[s * LDS_STRIDE] * x.x;
        acc += column[(s + 1) * LDS_STRIDE] * x.y;
        acc += column[(s + 2) * LDS_STRIDE] * x.z;
        acc += column[(s + 3) * LDS_STRIDE] * x.w;
    }
    return acc;
}

__device__ __forceinline__ float sum64(const float *column)
{
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < 64; ++s) acc += column[s * LDS_STRIDE];
    return acc;
}

// What bounds it: latency.  A batch is a few dozen to a few hundred blocks, each
// a chain of small dependent products, so the work of 64 samples is spread over
// the wavefronts of a block: the first four hold one 32 x 32 tile each of the
// three 64 x 64 products (and layer 1 of 16 samples each), the fifth the table
// targets, the loss and the output bias and shortcut, the last three, while the
// first four multiply, one sum over samples per hidden layer each (the two
// weights and the bias).  Every sum keeps the order of one lane per parameter.
// A training step at batch 4096 (64 blocks), one wavefront per 64 samples -> this
// with the deeper reduction below: 27.3 -> 10.7 us (this kernel 18.3 -> 6.5 us: 13,200
// cycles, of them 4,400 up to the end of layer 1, most of it the first loads,
// and 4,100 in the two products of back-propagation); 2368 samples 24.0 -> 11.3 us.
// A block takes 69 KB of LDS: two per compute unit.
constexpr int TRAIN_THREADS = 512;

__global__ void __launch_bounds__(TRAIN_THREADS) k_mlp_fwd_bwd(TrainArgs a)
{
    __shared__ float H1[64 * LDS_STRIDE], H2[64 * LDS_STRIDE], DZ1[64 * LDS_STRIDE], DZ2[64 * LDS_STRIDE];
    __shared__ float4 W3q[32];              // W3[2][64]
    __shared__ float4 DYq[32], X1q[48];     // [2][64] dL/dy and [3][64] x0, x1, 1, by sample
    __shared__ float PART[2][2][64];        // [output][half of the units][sample]
    const float *W3 = reinterpret_cast<const float *>(W3q);
    float *DY = reinterpret_cast<float *>(DYq), *X1 = reinterpret_cast<float *>(X1q);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, l32 = lane & 31;
    const int mt = (w >> 1) & 1, nt = w & 1;   // the wavefront's tile (wavefronts 0..3)
    const bool tiles = w < 4, head = w == 4;
    const float *p = a.pk;
    float *out = a.partial + (long)blockIdx.x * NP;

    // wavefronts 0..3: lane % 16 is the sample within the wavefront's 16;
    // the others: one sample a lane
    const int s0 = tiles ? 16 * w + (lane & 15) : lane;
    long sidx = a.offset + (long)blockIdx.x * 64 + s0;
    if (sidx >= a.n_train) sidx %= a.n_train;
    const float lr = a.samples[2 * sidx], lt = a.samples[2 * sidx + 1];
    const float x0 = 2.0f * (lr - float(a.op.lr0)) / float(a.op.lr1 - a.op.lr0) - 1.0f;
    const float x1 = 2.0f * (lt - float(a.op.lt0)) / float(a.op.lt1 - a.op.lt0) - 1.0f;

    bf16x8 w2h[4], w2l[4], wth[4], wtl[4];   // rows 32 mt.. of W2 and of W2^T
    float4 b2[4];
    float b3[2], ws[4];
    if (tiles) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int f = (mt * 4 + ks) * 64 + lane;
            w2h[ks] = reinterpret_cast<const bf16x8 *>(p + MLP_OFF_W2HI)[f];
            w2l[ks] = reinterpret_cast<const bf16x8 *>(p + MLP_OFF_W2LO)[f];
            wth[ks] = reinterpret_cast<const bf16x8 *>(p + MLP_OFF_W2THI)[f];
            wtl[ks] = reinterpret_cast<const bf16x8 *>(p + MLP_OFF_W2TLO)[f];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) b2[q] = *reinterpret_cast<const float4 *>(p + MLP_OFF_B2 + mlp_unit(mt, 4 * q, g));
        // layer 1: lane = unit
        const float2 w1 = reinterpret_cast<const float2 *>(p + MLP_OFF_W1)[lane];
        const float b1 = p[MLP_OFF_B1 + lane];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float y0 = lane_value(x0, j), y1 = lane_value(x1, j);
            H1[(16 * w + j) * LDS_STRIDE + lane] = fast_tanh(w1.x * y0 + w1.y * y1 + b1);
        }
    } else if (head) {
#pragma unroll
        for (int q = 0; q < 2; ++q) b3[q] = p[MLP_OFF_B3 + q];
#pragma unroll
        for (int q = 0; q < 4; ++q) ws[q] = p[MLP_OFF_WS + q];
    } else {
        if (w == 7 && lane < 32) W3q[lane] = reinterpret_cast<const float4 *>(p + MLP_OFF_W3)[lane];
        X1[64 * (w - 5) + lane] = w == 5 ? x0 : w == 6 ? x1 : 1.0f;
    }
    __syncthreads();

    // layer 2, Z2^T = W2 H1^T
    float h2[16];
    float t0 = 0.f, t1 = 0.f;
    if (tiles) {
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            float v[8];
            bf16x8 bh, bl;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = H1[(32 * nt + l32) * LDS_STRIDE + 16 * ks + 8 * g + e];
            split8(v, bh, bl);
            acc = mfma3(w2h[ks], w2l[ks], bh, bl, acc);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float h = fast_tanh(acc[i] + reinterpret_cast<const float *>(b2)[i]);
            h2[i] = h;
            H2[(32 * nt + l32) * LDS_STRIDE + mlp_unit(mt, i, g)] = h;
        }
    } else if (head) {
        double tP, tR;
        table_lookup<double>(a.op, double(lr), double(lt), tP, tR);
        t0 = float((tP - a.op.norm[0]) / a.op.norm[1]);
        t1 = float((tR - a.op.norm[2]) / a.op.norm[3]);
    }
    __syncthreads();

    // output layer: one sample a lane, wavefront = output and half of the units
    if (tiles) {
        const int o = w & 1, half = w >> 1;
        float part = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int u = mlp_unit(m, i, half);
                part += W3[64 * o + u] * H2[lane * LDS_STRIDE + u];
            }
        PART[o][half][lane] = part;
    }
    __syncthreads();

    float lossl = 0.f;
    if (head) {
        const float y0 = PART[0][0][lane] + PART[0][1][lane] + b3[0] + ws[0] * x0 + ws[1] * x1;
        const float y1 = PART[1][0][lane] + PART[1][1][lane] + b3[1] + ws[2] * x0 + ws[3] * x1;
        const float e0 = y0 - t0, e1 = y1 - t1;
        lossl = 0.5f * (e0 * e0 + e1 * e1) * a.inv_batch;
        DY[lane] = e0 * a.inv_batch;
        DY[64 + lane] = e1 * a.inv_batch;
    }
    __syncthreads();

    // dz2 = (W3^T dy) * (1 - h2^2)
    if (tiles) {
        const float d0 = DY[32 * nt + l32], d1 = DY[64 + 32 * nt + l32];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int u = mlp_unit(mt, i, g);
            DZ2[(32 * nt + l32) * LDS_STRIDE + u] = (W3[u] * d0 + W3[64 + u] * d1) * (1.0f - h2[i] * h2[i]);
        }
    }
    __syncthreads();

    float sum2 = 0.f;
    if (tiles) {
        // dL/dh1^T = W2^T dz2^T: A = W2^T, B[k = u][n = s]
        f32x16 dh;
#pragma unroll
        for (int i = 0; i < 16; ++i) dh[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            float v[8];
            bf16x8 bh, bl;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = DZ2[(32 * nt + l32) * LDS_STRIDE + 16 * ks + 8 * g + e];
            split8(v, bh, bl);
            dh = mfma3(wth[ks], wtl[ks], bh, bl, dh);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int q = (32 * nt + l32) * LDS_STRIDE + mlp_unit(mt, i, g);
            const float h = H1[q];
            DZ1[q] = dh[i] * (1.0f - h * h);
        }
    } else if (!head) {
        // lane = unit: dL/dW3[o][u] = sum_s dy_o h2[s][u] (o = 0, 1) and dL/db2[u]
        sum2 = w < 7 ? dot64(H2 + lane, DY + 64 * (w - 5)) : sum64(DZ2 + lane);
    } else {
        // dL/db3 and dL/dWs: lanes 0..5 are (output, input or bias)
        const int o = lane < 3 ? 0 : 1, q = lane < 6 ? lane - 3 * o : 0;
        float acc = 0.f;
#pragma unroll
        for (int s = 0; s < 64; s += 4) {
            const float4 d = DYq[16 * o + s / 4], x = X1q[16 * q + s / 4];
            acc += d.x * x.x;
            acc += d.y * x.y;
            acc += d.z * x.z;
            acc += d.w * x.w;
        }
        if (lane < 6) out[q == 2 ? P_B3 + o : P_WS + o * 2 + q] = acc;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lossl += __shfl_xor(lossl, o);
        if (lane == 0) a.loss_part[blockIdx.x] = lossl;
    }
    __syncthreads();

    if (tiles) {
        // dL/dW2 = dz2^T h1 with K = samples: A[m = u][k = s], B[k = s][n = k_in]
        f32x16 gw;
#pragma unroll
        for (int i = 0; i < 16; ++i) gw[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            float va[8], vb[8];
            bf16x8 ah, al, bh, bl;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int s = 16 * ks + 8 * g + e;
                va[e] = DZ2[s * LDS_STRIDE + 32 * mt + l32];
                vb[e] = H1[s * LDS_STRIDE + 32 * nt + l32];
            }
            split8(va, ah, al);
            split8(vb, bh, bl);
            gw = mfma3(ah, al, bh, bl, gw);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) out[P_W2 + mlp_unit(mt, i, g) * 64 + 32 * nt + l32] = gw[i];
    } else if (!head) {
        // lane = unit: dL/dW1 (x0, x1) and dL/db1
        const float sum1 = w < 7 ? dot64(DZ1 + lane, X1 + 64 * (w - 5)) : sum64(DZ1 + lane);
        out[w < 7 ? P_W3 + 64 * (w - 5) + lane : P_B2 + lane] = sum2;
        out[w < 7 ? P_W1 + 2 * lane + (w - 5) : P_B1 + lane] = sum1;
    }
}

// ---------------------------------------------------------------------------
// gradient reduction (fixed order), Adam, repacking
// ---------------------------------------------------------------------------

struct AdamArgs {
    float *theta, *m, *v;
    const float *partial;
    int nblk;
    float lr, b1, b2, eps, c1, c2;
    float *pk;
    const float *loss_part;
    float *loss_hist;
    long step;
};

// Sum of the nblk per-block partial gradients of parameter i, in a
// fixed order shared by the Adam and gradient kernels (so both produce the
// same bits): a 256-thread block owns 64 consecutive parameters (one per
// lane); wavefront w adds the partials of the contiguous quarter
// [w q, w q + q) of the blocks in order, and the first wavefront adds the
// four quarter sums in order w = 0..3.  Returns the sum in the threads of
// the first wavefront (i < NP); the other threads return 0.
constexpr int RED_PARAMS = 64, RED_BLOCKS = (NP + RED_PARAMS - 1) / RED_PARAMS;

__device__ __forceinline__ float reduce_partials(const float *partial, int nblk, int i, float (&sh)[4][64])
{
    constexpr int DEEP = 16;   // loads in flight (one after the other took 8.4 us at 64 blocks, now 3.8)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = (nblk + 3) >> 2;
    const int b0 = w * q, b1 = b0 + q < nblk ? b0 + q : nblk;
    float g = 0.f;
    if (i < NP) {
        int b = b0;
        for (; b + DEEP <= b1; b += DEEP) {
            float v[DEEP];
#pragma unroll
            for (int e = 0; e < DEEP; ++e) v[e] = partial[(long)(b + e) * NP + i];
#pragma unroll
            for (int e = 0; e < DEEP; ++e) g += v[e];
        }
        for (; b < b1; ++b) g += partial[(long)b * NP + i];
    }
    sh[w][lane] = g;
    __syncthreads();
    if (w != 0) return 0.f;
    return ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
}

// Sum of the loss parts in their order, by one wavefront: 64 loaded at once,
// then added one by one.
__device__ __forceinline__ float sum_loss(const float *part, int nblk)
{
    const int lane = threadIdx.x & 63;
    float L = 0.f;
    for (int b = 0; b < nblk; b += 64) {
        const float v = b + lane < nblk ? part[b + lane] : 0.f;
        const int m = nblk - b < 64 ? nblk - b : 64;
        for (int l = 0; l < m; ++l) L += lane_value(v, l);
    }
    return L;
}

__global__ void __launch_bounds__(256) k_mlp_adam(AdamArgs a)
{
    __shared__ float sh[4][64];
    const int i = blockIdx.x * RED_PARAMS + (threadIdx.x & 63);
    if (blockIdx.x == RED_BLOCKS) {   // one more block for the loss
        const float L = sum_loss(a.loss_part, a.nblk);
        if (threadIdx.x == 0) a.loss_hist[a.step] = L;
        return;
    }
    const int ic = i < NP ? i : NP - 1;
    const float m0 = a.m[ic], v0 = a.v[ic], th0 = a.theta[ic];
    const float g = reduce_partials(a.partial, a.nblk, i, sh);
    if (threadIdx.x >= 64 || i >= NP) return;
    const float m = a.b1 * m0 + (1.f - a.b1) * g;
    const float v = a.b2 * v0 + (1.f - a.b2) * g * g;
    a.m[i] = m;
    a.v[i] = v;
    const float w = th0 - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
    a.theta[i] = w;
    // refresh the packed network used by the next forward pass
    pack_param(a.pk, i, w);
}

__global__ void __launch_bounds__(256) k_mlp_reduce(const float *partial, int nblk, const float *loss_part,
                                                    float *grad, float *loss)
{
    __shared__ float sh[4][64];
    const int i = blockIdx.x * RED_PARAMS + (threadIdx.x & 63);
    if (blockIdx.x == RED_BLOCKS) {
        const float L = sum_loss(loss_part, nblk);
        if (threadIdx.x == 0) *loss = L;
        return;
    }
    const float g = reduce_partials(partial, nblk, i, sh);
    if (threadIdx.x < 64 && i < NP) grad[i] = g;
}

// ---------------------------------------------------------------------------
// held-out error against the table
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256) k_mlp_eval(const float *pk, const float *samples, long n, OpacityParams op,
                                                  float *blockmax)
{
    __shared__ float sh[2][256];
    __shared__ MlpShared w;
    mlp_stage(pk, w, threadIdx.x, blockDim.x);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const long id = blockIdx.x * 256L + threadIdx.x;
    const long idc = id < n ? id : n - 1;
    const float lr = samples[2 * idc], lt = samples[2 * idc + 1];
    const float x0 = 2.0f * (lr - float(op.lr0)) / float(op.lr1 - op.lr0) - 1.0f;
    const float x1 = 2.0f * (lt - float(op.lt0)) / float(op.lt1 - op.lt0) - 1.0f;
    float y0, y1;
    mlp_forward_shared(pk, w, x0, x1, lane, y0, y1);
    double tP, tR;
    table_lookup<double>(op, double(lr), double(lt), tP, tR);
    const double dP = double(y0 * pk[MLP_OFF_NORM + 1] + pk[MLP_OFF_NORM + 0]) - tP;
    const double dR = double(y1 * pk[MLP_OFF_NORM + 3] + pk[MLP_OFF_NORM + 2]) - tR;
    float mP = 0.f, mR = 0.f;
    if (id < n) {
        mP = float(fabs(exp10(dP) - 1.0));
        mR = float(fabs(exp10(dR) - 1.0));
    }
    sh[0][threadIdx.x] = mP;
    sh[1][threadIdx.x] = mR;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sh[0][threadIdx.x] = fmaxf(sh[0][threadIdx.x], sh[0][threadIdx.x + s]);
            sh[1][threadIdx.x] = fmaxf(sh[1][threadIdx.x], sh[1][threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        blockmax[2 * blockIdx.x] = sh[0][0];
        blockmax[2 * blockIdx.x + 1] = sh[1][0];
    }
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------

// mean / std of each table and the least-squares plane t = b + w0 x0 + w1 x1
// (normalised units) used to initialise the linear shortcut, from one pass over
// the differences from the first node (four interleaved sums each: one chain
// of additions takes four times as long).  Taken when a table is bound, where
// its values are at hand: a training run took 76 us to read a 128 x 128 table back
// and 81 us for its sums.
void mlp_table_stats(const float *kP, const float *kR, int nr, int nt, double norm[4], float lin[2][3])
{
    const double n = double(nr) * nt, di = 2.0 / (nr - 1), dj = 2.0 / (nt - 1);
    double f1 = 0, f2 = 0, g1 = 0, g2 = 0;      // node coordinates: sums and sums of squares
    for (int i = 0; i < nr; ++i) f1 += di * i - 1.0, f2 += (di * i - 1.0) * (di * i - 1.0);
    for (int j = 0; j < nt; ++j) g1 += dj * j - 1.0, g2 += (dj * j - 1.0) * (dj * j - 1.0);
    for (int o = 0; o < 2; ++o) {
        const float *T = o ? kR : kP;
        const double ref = T[0];
        double S = 0, S2 = 0, SF = 0, SG = 0;   // sums of d, d^2, d x0, d x1
        for (int j = 0; j < nt; ++j) {
            const float *row = T + (long)j * nr;
            double s[4] = {0, 0, 0, 0}, q[4] = {0, 0, 0, 0}, w[4] = {0, 0, 0, 0};
            int i = 0;
            for (; i + 4 <= nr; i += 4)
                for (int e = 0; e < 4; ++e) {
                    const double d = row[i + e] - ref;
                    s[e] += d;
                    q[e] += d * d;
                    w[e] += d * (di * (i + e) - 1.0);
                }
            for (; i < nr; ++i) {
                const double d = row[i] - ref;
                s[0] += d;
                q[0] += d * d;
                w[0] += d * (di * i - 1.0);
            }
            const double r = (s[0] + s[1]) + (s[2] + s[3]);
            S += r;
            S2 += (q[0] + q[1]) + (q[2] + q[3]);
            SF += (w[0] + w[1]) + (w[2] + w[3]);
            SG += (dj * j - 1.0) * r;
        }
        const double dm = S / n, var = S2 / n - dm * dm, sd = var > 0 ? std::sqrt(var) : 1.0;
        norm[2 * o] = ref + dm;
        norm[2 * o + 1] = sd;
        // normal equations of the plane fit on the node grid
        double A[3][3] = {{n, f1 * nt, g1 * nr}, {f1 * nt, f2 * nt, f1 * g1}, {g1 * nr, f1 * g1, g2 * nr}};
        double b[3] = {(S - n * dm) / sd, (SF - dm * f1 * nt) / sd, (SG - dm * g1 * nr) / sd};
        for (int piv = 0; piv < 3; ++piv)          // Gaussian elimination (SPD, no pivoting)
            for (int r = piv + 1; r < 3; ++r) {
                const double m = A[r][piv] / A[piv][piv];
                for (int q = piv; q < 3; ++q) A[r][q] -= m * A[piv][q];
                b[r] -= m * b[piv];
            }
        double x[3];
        for (int r = 2; r >= 0; --r) {
            double s3 = b[r];
            for (int q = r + 1; q < 3; ++q) s3 -= A[r][q] * x[q];
            x[r] = s3 / A[r][r];
        }
        lin[o][0] = float(x[0]);
        lin[o][1] = float(x[1]);
        lin[o][2] = float(x[2]);
    }
}

int mlp_train(m1_ctx *c, const m1_train_cfg *cfg, m1_train_report *rep)
{
    std::vector<float> th(cfg->theta_init, cfg->theta_init + NP);
    if (!cfg->keep_init)
        for (int o = 0; o < 2; ++o) {
            th[P_B3 + o] = c->tab_lin[o][0];
            th[P_WS + 2 * o] = c->tab_lin[o][1];
            th[P_WS + 2 * o + 1] = c->tab_lin[o][2];
        }
    const int nblk = cfg->batch / 64;
    const long n_eval_blocks = (cfg->n_eval + 255) / 256;
    // what comes back, in one copy: the trained parameters, the loss of each
    // step, the held-out maxima.  The host buffer first: a failed host
    // allocation then leaves no device buffer behind
    const size_t nres = size_t(NP) + cfg->steps + 2 * n_eval_blocks;
    std::vector<float> res(nres);
    float *buf = nullptr;
    const size_t nbuf = 2 * size_t(NP) + nres + size_t(nblk) * NP + nblk;
    if (mlp_buffer(c) != hipSuccess) {
        set_error("MLP buffer allocation failed");
        return int(M1_EDEVICE);
    }
    if (device_alloc(reinterpret_cast<void **>(&buf), nbuf * sizeof(float)) != hipSuccess) {
        set_error("m1_mlp_train: allocation failed");
        return int(M1_ENOMEM);
    }
    float *mom = buf, *vel = buf + NP, *theta = buf + 2 * NP;   // as k_mlp_pack sets them
    float *loss_hist = theta + NP, *evmax = loss_hist + cfg->steps;
    float *partial = theta + nres, *loss_part = partial + size_t(nblk) * NP;
    OpacityParams op = c->op;
    for (int i = 0; i < 4; ++i) op.norm[i] = c->tab_norm[i];
    op.mlp = c->mlp_dev;
    hipError_t e = upload_network(c, th.data(), op.norm, buf);
    hipEvent_t ev0, ev1;
    hipEventCreate(&ev0);
    hipEventCreate(&ev1);
    hipEventRecord(ev0, c->stream);
    TrainArgs ta;
    ta.pk = c->mlp_dev;
    ta.samples = cfg->samples;
    ta.n_train = cfg->n_train;
    ta.inv_batch = 1.0f / float(cfg->batch);
    ta.op = op;
    ta.partial = partial;
    ta.loss_part = loss_part;
    AdamArgs aa;
    aa.theta = theta;
    aa.m = mom;
    aa.v = vel;
    aa.partial = partial;
    aa.nblk = nblk;
    aa.b1 = float(cfg->beta1);
    aa.b2 = float(cfg->beta2);
    aa.eps = float(cfg->eps);
    aa.pk = c->mlp_dev;
    aa.loss_part = loss_part;
    aa.loss_hist = loss_hist;
    for (long s = 0; s < cfg->steps && e == hipSuccess; ++s) {
        ta.offset = (s * (long)cfg->batch) % cfg->n_train;
        hipLaunchKernelGGL(k_mlp_fwd_bwd, dim3(nblk), dim3(TRAIN_THREADS), 0, c->stream, ta);
        const double frac = cfg->steps > 1 ? double(s) / double(cfg->steps - 1) : 1.0;
        aa.lr = float(cfg->lr_final + 0.5 * (cfg->lr - cfg->lr_final) * (1.0 + std::cos(M_PI * frac)));
        aa.c1 = float(1.0 - std::pow(cfg->beta1, double(s + 1)));
        aa.c2 = float(1.0 - std::pow(cfg->beta2, double(s + 1)));
        aa.step = s;
        hipLaunchKernelGGL(k_mlp_adam, dim3(RED_BLOCKS + 1), dim3(256), 0, c->stream, aa);
        e = hipGetLastError();
    }
    hipEventRecord(ev1, c->stream);
    if (e == hipSuccess) {
        // the inference entries of the trained network
        hipLaunchKernelGGL(k_mlp_pack_infer, dim3(16), dim3(256), 0, c->stream, theta, c->mlp_dev);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mlp_eval, dim3((unsigned)n_eval_blocks), dim3(256), 0, c->stream, c->mlp_dev,
                           cfg->samples + 2 * cfg->n_train, cfg->n_eval, op, evmax);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(res.data(), theta, nres * sizeof(float), hipMemcpyDeviceToHost, c->stream);
    const hipError_t es = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) e = es;
    float ms = 0.f;
    hipEventElapsedTime(&ms, ev0, ev1);
    hipEventDestroy(ev0);
    hipEventDestroy(ev1);
    hipFree(buf);
    if (e != hipSuccess) {
        // the packed network is part-trained by now: the one in use before, if
        // any, goes back
        if (!c->mlp_theta.empty()) mlp_pack(c, std::vector<float>(c->mlp_theta).data(), c->op.norm);
        set_error(std::string("m1_mlp_train: ") + hipGetErrorString(e));
        return int(M1_EDEVICE);
    }
    const float *hist = res.data() + NP, *em = hist + cfg->steps;
    double L = 0;
    const long tail = std::min<long>(100, cfg->steps);
    for (long s = cfg->steps - tail; s < cfg->steps; ++s) L += hist[s];
    rep->final_loss = L / tail;
    rep->max_rel_err_P = 0;
    rep->max_rel_err_R = 0;
    for (long b = 0; b < n_eval_blocks; ++b) {
        rep->max_rel_err_P = std::max<double>(rep->max_rel_err_P, em[2 * b]);
        rep->max_rel_err_R = std::max<double>(rep->max_rel_err_R, em[2 * b + 1]);
    }
    rep->seconds = ms * 1e-3;
    std::copy(res.begin(), res.begin() + NP, th.begin());
    c->op = op;
    c->mlp_theta.swap(th);   // packed device copy already holds the trained network
    return 0;
}

int mlp_gradient(m1_ctx *c, const float *samples, long n, const float *theta, float *grad, double *loss)
{
    if (mlp_pack(c, theta, c->op.norm) != 0) return int(M1_EDEVICE);
    const int nblk = int(n / 64);
    float *buf = nullptr;
    const size_t nbuf = size_t(nblk) * NP + nblk + NP + 1;
    if (device_alloc(reinterpret_cast<void **>(&buf), nbuf * sizeof(float)) != hipSuccess) {
        set_error("m1_mlp_gradient: allocation failed");
        return int(M1_ENOMEM);
    }
    float *partial = buf, *loss_part = buf + size_t(nblk) * NP, *g = loss_part + nblk, *L = g + NP;
    TrainArgs ta;
    ta.pk = c->mlp_dev;
    ta.samples = samples;
    ta.n_train = n;
    ta.inv_batch = 1.0f / float(n);
    ta.op = c->op;
    // a launch takes fewer than 2^32 threads: 2^22 blocks at a time
    constexpr int BLOCKS = 1 << 22;
    hipError_t e = hipSuccess;
    for (int b = 0; b < nblk && e == hipSuccess; b += BLOCKS) {
        ta.offset = 64L * b;
        ta.partial = partial + size_t(b) * NP;
        ta.loss_part = loss_part + b;
        hipLaunchKernelGGL(k_mlp_fwd_bwd, dim3(std::min(BLOCKS, nblk - b)), dim3(TRAIN_THREADS), 0, c->stream, ta);
        e = hipGetLastError();
    }
    float Lh = 0.f;
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_mlp_reduce, dim3(RED_BLOCKS + 1), dim3(256), 0, c->stream, partial, nblk,
                           loss_part, g, L);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(grad, g, NP * sizeof(float), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(&Lh, L, sizeof(float), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    hipFree(buf);
    if (e != hipSuccess) {
        set_error(std::string("m1_mlp_gradient: ") + hipGetErrorString(e));
        return int(M1_EDEVICE);
    }
    *loss = Lh;
    return 0;
}

} // namespace m1
