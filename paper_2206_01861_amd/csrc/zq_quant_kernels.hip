// Quantization kernels of libzq (gfx950):
//   * group-wise weight quantization, INT8 and packed INT4 (Sec. 4.1, App. A.2)
//   * LayerNorm / bias+GeLU / identity fused with token-wise INT8 quantization
//     (Sec. 4.1; Sec. 4.3 and App. D, "Operation Fusion for Token-wise
//     Activation Quantization").
// All of them are bound by HBM traffic: reads are 16-byte vectors, coalesced
// along the row; a row is read once and stays in registers between the
// reduction that finds its scale and the pass that emits its codes.
#include "zq_device.h"
#include "zq_internal.h"

#include <limits.h>

namespace zq {

int compute_units();                                    // of the current device

// ---------------------------------------------------------------------------
// Row front-ends.  A row is handled by TPR threads (one wave, or a whole
// workgroup of 256 or more), each holding VPT vectors of 8 elements in registers.
// ---------------------------------------------------------------------------

template <int TPR>
__device__ __forceinline__ float row_sum(float v, float *lds) {
    v = wave_sum(v);
    if (TPR > kWave) {
        const int w = threadIdx.x / kWave;
        __syncthreads();
        if ((threadIdx.x % kWave) == 0) lds[w] = v;
        __syncthreads();
        v = lds[0] + lds[1] + lds[2] + lds[3];
#pragma unroll
        for (int i = 4; i < TPR / kWave; ++i) v += lds[i];
    }
    return v;
}

template <int TPR>
__device__ __forceinline__ float row_max(float v, float *lds) {
    v = wave_max(v);
    if (TPR > kWave) {
        const int w = threadIdx.x / kWave;
        __syncthreads();
        if ((threadIdx.x % kWave) == 0) lds[w] = v;
        __syncthreads();
        v = fmaxf(fmaxf(lds[0], lds[1]), fmaxf(lds[2], lds[3]));
#pragma unroll
        for (int i = 4; i < TPR / kWave; ++i) v = fmaxf(v, lds[i]);
    }
    return v;
}

// Vector idx of a row: y where it is wanted, and the codes.
__device__ __forceinline__ void store_row_vector(const float (&v)[8], float inv, int row, int K, int idx,
                                                 int8_t *__restrict__ xq, void *__restrict__ y_out, int y_dtype) {
    if (y_out != nullptr) {
        if (y_dtype == 1) {
            float4 *yo = reinterpret_cast<float4 *>(reinterpret_cast<float *>(y_out) + (size_t)row * K) + 2 * idx;
            yo[0] = make_float4(v[0], v[1], v[2], v[3]);
            yo[1] = make_float4(v[4], v[5], v[6], v[7]);
        } else {
            half8 h;
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = (half_t)v[e];
            reinterpret_cast<half8 *>(reinterpret_cast<half_t *>(y_out) + (size_t)row * K)[idx] = h;
        }
    }
    uint32_t q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = quant_code_bits(v[e], inv);
    reinterpret_cast<uint2 *>(xq + (size_t)row * K)[idx] =
        make_uint2(pack4_code_bits(q[0], q[1], q[2], q[3]), pack4_code_bits(q[4], q[5], q[6], q[7]));
}

constexpr int row_block(int tpr) { return tpr > 256 ? tpr : 256; }      // threads of a workgroup

template <int OP, int TPR, int VPT>
__global__ __launch_bounds__(row_block(TPR)) void rowquant_kernel(const half8 *__restrict__ in, const half8 *__restrict__ p0,
                                                       const half8 *__restrict__ p1, float eps, int M, int K,
                                                       int8_t *__restrict__ xq, float *__restrict__ s_tok,
                                                       void *__restrict__ y_out, int y_dtype) {
    __shared__ float lds[row_block(TPR) / kWave];
    constexpr int RPB = row_block(TPR) / TPR;
    const int t = threadIdx.x % TPR;
    const int row = blockIdx.x * RPB + threadIdx.x / TPR;
    if (TPR <= kWave && row >= M) return;   // whole waves leave together; no block barrier is used
    const int nvec = K >> 3;
    const half8 *rin = in + (size_t)row * nvec;

    constexpr bool kGelu = (OP == kOpGeluErf || OP == kOpGeluTanh);
    // Every load of the row and (for up to four vectors per thread) of its parameters is issued before
    // the first result is waited for: vectors past the end of the row read vector 0 instead of being
    // skipped, so that no branch separates the loads and one memory round trip covers them all.
    constexpr bool kPre = (VPT <= 4) && (OP == kOpLayerNorm || kGelu);
    bool ok[VPT];
    int idc[VPT];
    uint32x4_t raw[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int idx = i * TPR + t;
        ok[i] = idx < nvec;
        idc[i] = ok[i] ? idx : 0;
        raw[i] = __builtin_bit_cast(uint32x4_t, rin[idc[i]]);
    }
    uint32x4_t pa[kPre ? VPT : 1], pb[kPre ? VPT : 1];
    if (kPre && OP == kOpLayerNorm) {
        // gamma is always there; without beta, gamma is loaded a second time (a cache hit) and not
        // used, which keeps the loads free of branches
        const half8 *q1 = p1 != nullptr ? p1 : p0;
#pragma unroll
        for (int i = 0; i < (kPre ? VPT : 0); ++i) {
            pa[i] = __builtin_bit_cast(uint32x4_t, p0[idc[i]]);
            pb[i] = __builtin_bit_cast(uint32x4_t, q1[idc[i]]);
        }
    } else if (kPre && p0 != nullptr) {
#pragma unroll
        for (int i = 0; i < (kPre ? VPT : 0); ++i) pa[i] = __builtin_bit_cast(uint32x4_t, p0[idc[i]]);
    }

    float v[VPT][8];
    if (!kGelu) {
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const half8 h = __builtin_bit_cast(half8, raw[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] = ok[i] ? (float)h[e] : 0.0f;
        }
    }

    if (OP == kOpLayerNorm) {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < VPT; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[i][e];
        const float mean = row_sum<TPR>(s, lds) / (float)K;
        float ss = 0.0f;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if (ok[i]) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float d = v[i][e] - mean;
                    ss += d * d;
                }
            }
        }
        const float var = row_sum<TPR>(ss, lds) / (float)K;
        const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if (ok[i]) {
                const half8 g = kPre ? __builtin_bit_cast(half8, pa[kPre ? i : 0]) : p0[idc[i]];
                if (p1 != nullptr) {
                    const half8 b = kPre ? __builtin_bit_cast(half8, pb[kPre ? i : 0]) : p1[idc[i]];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[i][e] = (v[i][e] - mean) * rstd * (float)g[e] + (float)b[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[i][e] = (v[i][e] - mean) * rstd * (float)g[e];
                }
            }
        }
    } else if (kGelu) {
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if (ok[i]) {
                if (p0 != nullptr) {
                    const uint32x4_t b = kPre ? pa[kPre ? i : 0] : __builtin_bit_cast(uint32x4_t, p0[idc[i]]);
#pragma unroll
                    for (int d = 0; d < 4; ++d) add2_f16_f32(raw[i][d], b[d], v[i][2 * d], v[i][2 * d + 1]);
                } else {
                    const half8 h = __builtin_bit_cast(half8, raw[i]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[i][e] = (float)h[e];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) v[i][e] = (OP == kOpGeluErf) ? gelu_erf(v[i][e]) : gelu_tanh(v[i][e]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[i][e] = 0.0f;
            }
        }
    }

    // Token-wise scale (Sec. 4.1): absmax of the row, from registers.
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < VPT; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(v[i][e]));
    a = row_max<TPR>(a, lds);
    float scale, inv;
    quant_scales(a, 127.0f, scale, inv);
    if (t == 0) s_tok[row] = scale;

#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int idx = i * TPR + t;
        if (ok[i]) store_row_vector(v[i], inv, row, K, idx, xq, y_out, y_dtype);
    }
}

// GeLU without a bias for up to as many rows as there are compute units: a row is cut into gridDim.x parts, one workgroup
// each.  One compute unit works 18 VALU instructions an element off at 64 a cycle, 0.96 us for 8192 elements, while the
// others idle.  The parts of a row agree on its scale without exchanging anything, because each of them reads the whole row:
// GeLU of an FP16 input rises from where it passes kGeluNegMax on, and below zero it stays under kGeluNegMax in size, so the
// row's absmax is the GeLU of its largest input (two elements per instruction) once that is above kGeluNegMax.  A row of
// smaller inputs is worked off whole by each part.  The computed functions have both properties over every finite FP16
// value, so the scale has the bits that the maximum over all results has; with a bias the argument is any fp32 value,
// where neighbours may round the other way.  us per call, a workgroup per row / parts: 1x8192 3.3 / 2.6, 27x8192 3.7 / 2.6,
// 16x16384 5.0 / 2.7, 64x24576 6.9 / 4.6, 5x6400 3.5 / 2.6, 256x16384 6.8 / 5.5.
constexpr float kGeluNegMax = 0.1702f;               // erf form: 0.16997, tanh form: 0.17004
constexpr int16_t kHalfInfBits = 0x7c00;

template <int OP>
__device__ __forceinline__ float gelu_op(float u) {
    return OP == kOpGeluErf ? gelu_erf(u) : gelu_tanh(u);
}

template <int OP, int NT, int VPT>
__global__ __launch_bounds__(NT) void gelu_parts_kernel(const uint32x4_t *__restrict__ in, int K, int own,
                                                        int8_t *__restrict__ xq, float *__restrict__ s_tok,
                                                        void *__restrict__ y_out, int y_dtype) {
    __shared__ float lds[NT / kWave];
    const int t = threadIdx.x;
    const int row = blockIdx.y;
    const int nvec = K >> 3;
    const uint32x4_t *rin = in + (size_t)row * nvec;
    // This part's vectors, the first `own` of a thread, then the others'.  Vectors past the end read vector 0.
    const int first = (int)blockIdx.x * own;
    uint32x4_t raw[VPT];
    int idx[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int slot = first + i < VPT ? first + i : first + i - VPT;
        idx[i] = slot * NT + t;
        raw[i] = rin[idx[i] < nvec ? idx[i] : 0];
    }
    // The bits of non-negative FP16 numbers order like 16-bit integers, those of negative ones are below all of them.
    typedef int16_t short2_t __attribute__((ext_vector_type(2)));
    short2_t m2 = {0, 0};
#pragma unroll
    for (int i = 0; i < VPT; ++i)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t two = raw[i][d];              // (a bit cast of the element itself reads element 0)
            m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(short2_t, two));
        }
    // A positive NaN is above infinity and hides the other inputs of its thread: it counts as infinity here, and a row with
    // either is worked off whole, where NaNs raise no maximum (the other values of such a row keep their codes).
    const int16_t top = m2[0] > m2[1] ? m2[0] : m2[1];
    float a = gelu_op<OP>(row_max<NT>(top > kHalfInfBits ? INFINITY : (float)__builtin_bit_cast(half_t, top), lds));
    if (!(a > kGeluNegMax && a < INFINITY)) {
        a = 0.0f;
        for (int i = t; i < nvec; i += NT) {
            const half8 h = __builtin_bit_cast(half8, rin[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(gelu_op<OP>((float)h[e])));
        }
        a = row_max<NT>(a, lds);
    }
    float scale, inv;
    quant_scales(a, 127.0f, scale, inv);
    if (t == 0 && blockIdx.x == 0) s_tok[row] = scale;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        if (i >= own) break;
        if (idx[i] < nvec) {
            const half8 h = __builtin_bit_cast(half8, raw[i]);
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = gelu_op<OP>((float)h[e]);
            store_row_vector(v, inv, row, K, idx[i], xq, y_out, y_dtype);
        }
    }
}

template <int OP, int TPR, int VPT>
static hipError_t launch_rq(const void *in, const void *p0, const void *p1, float eps, int M, int K, int8_t *xq,
                            float *s_tok, void *y_out, int y_dtype, hipStream_t st) {
    constexpr int RPB = row_block(TPR) / TPR;
    const int blocks = (M + RPB - 1) / RPB;
    hipLaunchKernelGGL((rowquant_kernel<OP, TPR, VPT>), dim3(blocks), dim3(row_block(TPR)), 0, st,
                       reinterpret_cast<const half8 *>(in), reinterpret_cast<const half8 *>(p0),
                       reinterpret_cast<const half8 *>(p1), eps, M, K, xq, s_tok, y_out, y_dtype);
    return hipGetLastError();
}

// Threads of a row, 0: GeLU in parts (gelu_parts_kernel).  bias: GeLU's.
//
// GeLU in parts: not rows that are one part of the same threads as here, with the search for the largest input on top (67x2000
// 2.40 / 2.53, 12x512 2.2 / 2.4); from 528 to 1024 values one part has 256 threads for the one wave here (3 % ahead).
//
// Short rows: one wave per row, four rows per workgroup.  Up to 2048 values where a workgroup per row would be many
// rounds of them: no barrier in the three reductions (LayerNorm 2048x2048 5.9 -> 5.1 us, 2048x1280 5.3 -> 4.2,
// 8192x2048 16.4 -> 14.0; at 512 rows level, at 5 rows 2.7 -> 2.9; 4096 values are 25 % slower that way).  The
// arithmetic of GeLU wants more waves: 2100x1920 5.2 -> 5.6.
//
// Longer rows: a workgroup shares one row, with up to four vectors per thread: six to sixteen of 256 threads are too few
// waves for the arithmetic of GeLU (300x16384 7.8 -> 6.5 us, 300x24576 10.9 -> 8.4, 2048x24576 33.5 -> 31.9; LayerNorm
// 2048x12288 21.2 -> 20.3).  With enough rows to keep the chip full either way the smaller
// workgroups are ahead, 256 threads / more (GeLU 16384x10240 93 / 97 us, 16384x24576 215 / 218, tanh form 220 / 229;
// LayerNorm 16384x10240 107.5 / 112), and for LayerNorm, whose parameters take registers too, everywhere on rows of more
// than 16384 values (4096x24576 68 / 98).  Its rows of up to 16384 values fit the chip at once with 256 threads, four workgroups a compute unit,
// where two of 512 do not: 513 to 1280 rows and, where the fourth vector of a thread is half empty, up to 2048 stay with 256
// (571x12752 7.1 / 8.1, 900x12608 9.0 / 9.9, 1645x8496 11.2 / 11.8; 1480x16304 17.8 / 15.9).  The plain quantizer gains (8192x24576 110 / 103) but for
// 257 to 512 rows of more than 16384 values, which 256 threads take at once (366x32256 6.7 / 7.4, 489x31456 7.8 / 8.9), and many of the
// longest (3522x26208 44.7 / 49.5), and so does GeLU with a bias,
// whose loads go out with the row's for up to four vectors only (16384x24576 252 / 220, 4096x10240 34.4 / 33.3).
int row_threads(RowOp op, int M, int K, bool bias) {
    const int nvec = K / 8;
    const bool gelu = op == kOpGeluErf || op == kOpGeluTanh;
    const bool one_part = nvec <= 64 || (nvec > 64 * 2 && nvec <= 256);
    if (gelu && !bias && !one_part && M <= compute_units()) return 0;
    if (nvec <= 64 * 2 || (M > 512 && !gelu && nvec <= 64 * 4)) return 64;
    if (nvec <= 256 * 4) return 256;
    if (op != kOpIdentity && !bias && M > 2048) return 256;
    if (op == kOpIdentity && nvec > 512 * 4 && ((M > 256 && M <= 512) || (M > 3072 && K > 24576))) return 256;
    if (op == kOpLayerNorm && (nvec > 512 * 4 || (M > 512 && (M <= 1280 || K <= 11264)))) return 256;
    return nvec <= 512 * 4 ? 512 : 1024;
}

// The vectors a thread holds: the fewest of those built that cover the row.  Built is what row_threads can ask for.
template <int OP>
static hipError_t launch_rq_op(const void *in, const void *p0, const void *p1, float eps, int M, int K, int8_t *xq,
                               float *s_tok, void *y_out, int y_dtype, int threads, hipStream_t st) {
    constexpr bool kGelu = OP == kOpGeluErf || OP == kOpGeluTanh;
    const int nvec = K / 8;
#define ZQ_RQ(TPR, VPT) \
    if (nvec <= (TPR) * (VPT)) return launch_rq<OP, TPR, VPT>(in, p0, p1, eps, M, K, xq, s_tok, y_out, y_dtype, st)
    switch (threads) {
        case 64:
            ZQ_RQ(64, 1);
            ZQ_RQ(64, 2);
            if constexpr (!kGelu) {
                ZQ_RQ(64, 3);
                ZQ_RQ(64, 4);
            }
            break;
        case 256:
            ZQ_RQ(256, 1);
            ZQ_RQ(256, 2);
            ZQ_RQ(256, 3);
            ZQ_RQ(256, 4);
            if constexpr (OP != kOpIdentity) {
                ZQ_RQ(256, 6);
                ZQ_RQ(256, 8);
            }
            ZQ_RQ(256, 12);
            ZQ_RQ(256, 16);
            break;
        case 512:
            ZQ_RQ(512, 3);
            ZQ_RQ(512, 4);
            break;
        case 1024:
            if constexpr (OP != kOpLayerNorm) {
                ZQ_RQ(1024, 3);
                ZQ_RQ(1024, 4);
            }
            break;
    }
#undef ZQ_RQ
    return hipErrorInvalidValue;
}

template <int OP, int NT, int VPT>
static hipError_t launch_gelu_parts_t(const void *in, int M, int K, int parts, int8_t *xq, float *s_tok, void *y_out,
                                      int y_dtype, hipStream_t st) {
    const int own = (VPT + parts - 1) / parts;          // vectors of a thread
    hipLaunchKernelGGL((gelu_parts_kernel<OP, NT, VPT>), dim3((VPT + own - 1) / own, M), dim3(NT), 0, st,
                       reinterpret_cast<const uint32x4_t *>(in), K, own, xq, s_tok, y_out, y_dtype);
    return hipGetLastError();
}

// Parts: as many as a compute unit each holds, one vector per thread at least.  Rows of up to 4096 values leave something to
// part with 256 threads only (64x3072 2.5 us, with 512 2.7), longer ones have fewer parts that read the row with 512
// (64x24576 4.6 us, with 256 threads 7.1, with 1024 4.9).
template <int OP>
static hipError_t launch_gelu_parts(const void *in, int M, int K, int cus, int8_t *xq, float *s_tok, void *y_out,
                                    int y_dtype, hipStream_t st) {
    const int nvec = K / 8;
#define ZQ_GP(NT, VPT) return launch_gelu_parts_t<OP, NT, VPT>(in, M, K, cus / M, xq, s_tok, y_out, y_dtype, st)
    if (nvec <= 256 * 1) ZQ_GP(256, 1);
    if (nvec <= 256 * 2) ZQ_GP(256, 2);
    if (nvec <= 512 * 2) ZQ_GP(512, 2);
    if (nvec <= 512 * 3) ZQ_GP(512, 3);
    if (nvec <= 512 * 4) ZQ_GP(512, 4);
    if (nvec <= 512 * 6) ZQ_GP(512, 6);
    if (nvec <= 512 * 8) ZQ_GP(512, 8);
#undef ZQ_GP
    return hipErrorInvalidValue;
}

hipError_t launch_rowquant(RowOp op, const void *in, const void *p0, const void *p1, float eps, int M, int K,
                           int8_t *xq, float *s_tok, void *y_out, int y_dtype, hipStream_t st) {
    const int threads = row_threads(op, M, K, op != kOpLayerNorm && p0 != nullptr);
    if (threads == 0) {
        const int cus = compute_units();
        return op == kOpGeluErf ? launch_gelu_parts<kOpGeluErf>(in, M, K, cus, xq, s_tok, y_out, y_dtype, st)
                                : launch_gelu_parts<kOpGeluTanh>(in, M, K, cus, xq, s_tok, y_out, y_dtype, st);
    }
    switch (op) {
        case kOpLayerNorm: return launch_rq_op<kOpLayerNorm>(in, p0, p1, eps, M, K, xq, s_tok, y_out, y_dtype, threads, st);
        case kOpGeluErf: return launch_rq_op<kOpGeluErf>(in, p0, p1, eps, M, K, xq, s_tok, y_out, y_dtype, threads, st);
        case kOpGeluTanh: return launch_rq_op<kOpGeluTanh>(in, p0, p1, eps, M, K, xq, s_tok, y_out, y_dtype, threads, st);
        case kOpIdentity: return launch_rq_op<kOpIdentity>(in, p0, p1, eps, M, K, xq, s_tok, y_out, y_dtype, threads, st);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Stand-alone dequantization of an INT32 accumulator tensor: the separate
// kernel of the unfused pipeline (Fig. 2, left) that the GeMM epilogue
// replaces (fp32 arithmetic, one FP16 rounding).
// One thread per four consecutive columns (a group holds a multiple of 16).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dequant_kernel(const int32x4 *__restrict__ acc, const float *__restrict__ s_tok,
                                                      const float *__restrict__ s_w, int gs,
                                                      const half_t *__restrict__ bias, int M, int N,
                                                      half4 *__restrict__ out) {
    const int nq = N >> 2;
    const long total = (long)M * nq;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int m = (int)(i / nq);
        const int n = (int)(i - (long)m * nq) * 4;
        const int32x4 v = acc[i];
        const float sc = s_tok[m] * s_w[n / gs];
        half4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float f = (float)v[e] * sc;
            if (bias != nullptr) f += (float)bias[n + e];
            o[e] = (half_t)f;
        }
        out[i] = o;
    }
}

hipError_t launch_dequant(const int32_t *acc, const float *s_tok, const float *s_w, int groups, const void *bias, int M,
                          int N, void *out, hipStream_t st) {
    const long total = (long)M * (N / 4);
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(dequant_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<const int32x4 *>(acc),
                       s_tok, s_w, N / groups, reinterpret_cast<const half_t *>(bias), M, N,
                       reinterpret_cast<half4 *>(out));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Group-wise weight quantization.  A group is a contiguous chunk of gs*K fp16
// values.
//
// Groups of up to 16 MB, as a rule (one_pass_pays): wq_group_kernel, one pass over the weights.  A group
// is cut into slices of at most 64 KB, one workgroup each, which keeps its
// slice in registers while the workgroups of the group agree on their maximum.
// Bound: HBM, 2 + bits/8 bytes per weight.  Up to five workgroups on a compute
// unit keep 80 MB in flight on the chip, so that loads of later groups cover
// the exchange of earlier ones.  Reading the weights twice (absmax, then
// codes) against this, weights from HBM, per call: INT8 12288x4096 57 -> 34 us
// (4.4 TB/s), 24576x6144 157 -> 98, 4096x4096 34 -> 17; INT4 16384x4096 63 -> 41,
// 8192x2048 32 -> 16; 512 threads or 48 KB slices measured level or behind.
//
// The exchange is one 32-bit word per group: the maximum (15 bits, the pattern
// of |fp16|) above the count of slices that arrived and the count of those
// that have read the maximum (8 bits each, hence at most 255 slices).  A slice
// either raises the maximum and counts itself in one compare-and-swap or, if
// it raises nothing, in one addition.  The word stands in the first 128-byte
// line of the group's codes: nothing is allocated, and the words of different
// groups lie far apart (side by side in s_w they shared a memory channel, and
// 12288x4096 took 146 us).  Nobody stores that line's codes except the slice
// that reads the maximum last, which makes them from the weights once more.
// All accesses to the words are agent-scope atomics, and no other memory is
// exchanged.  A slice's wait ends because the workgroups of a group have
// consecutive ids, are started in order of their ids and fit the chip several
// times over; should it last longer than the polls it is given, the workgroup
// reads the whole group for the maximum itself, so that the result never
// depends on it.
//
// Else: clear, absmax (integer atomic max on the fp32 bit pattern,
// exact and order independent), quantize, and turn absmax into the scale in
// place; the weights are read twice.  s_w is the scratch here.
// ---------------------------------------------------------------------------

constexpr int kWqThreads = 256;
constexpr int kWqVecs = 16;                             // 16-byte vectors of a slice per thread
constexpr int kWqMaxSlices = 255;                       // eight bits of the exchange word
constexpr int kWqPolls = 1 << 16;                       // some 90 ms
constexpr int kWqSleep = 12;                            // 768 cycles between polls (4: more traffic, 32: later, both 3 % behind)
constexpr int kWqLine = 128;
// Where the line of a group's exchange word begins in its codes.
__device__ __forceinline__ int wq_line_offset(const void *codes) {
    return (int)(-reinterpret_cast<uintptr_t>(codes) & (kWqLine - 1));
}

__global__ void wq_clear_line_kernel(uint8_t *wq, long group_bytes, int groups) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= groups) return;
    uint8_t *codes = wq + i * group_bytes;
    *reinterpret_cast<uint32_t *>(codes + wq_line_offset(codes)) = 0u;
}

// The largest |fp16| pattern of a vector, merged into the two halves of m.
typedef uint16_t ushort2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ ushort2_t absmax_pattern(ushort2_t m, uint32x4_t v) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
        m = __builtin_elementwise_max(m, __builtin_bit_cast(ushort2_t, v[e] & 0x7fff7fffu));
    return m;
}
// ... of the workgroup, in every thread.
__device__ __forceinline__ uint32_t block_max_pattern(ushort2_t m, uint32_t *lds) {
    const uint32_t w = wave_max_u32(m[0] > m[1] ? m[0] : m[1]);
    __syncthreads();
    if ((threadIdx.x % kWave) == 0) lds[threadIdx.x / kWave] = w;
    __syncthreads();
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < kWqThreads / kWave; ++i) r = lds[i] > r ? lds[i] : r;
    return r;
}
__device__ __forceinline__ float pattern_to_float(uint32_t p) { return (float)__builtin_bit_cast(half_t, (uint16_t)p); }

template <int BITS>
__device__ __forceinline__ void store_codes(void *wq, long i, uint32x4_t v, float inv) {
    const half8 h = __builtin_bit_cast(half8, v);
    uint32_t q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = quant_code_bits((float)h[e], inv);
    if (BITS == 8) {
        reinterpret_cast<uint2 *>(wq)[i] =
            make_uint2(pack4_code_bits(q[0], q[1], q[2], q[3]), pack4_code_bits(q[4], q[5], q[6], q[7]));
    } else {
        uint32_t p = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) p |= (q[e] & 0xfu) << (4 * e);   // even k in the low nibble
        reinterpret_cast<uint32_t *>(wq)[i] = p;
    }
}

template <int BITS, int VPT>
__global__ __launch_bounds__(kWqThreads) void wq_group_kernel(const uint32x4_t *__restrict__ w, long chunk_vecs,
                                                              int slices, int slice_vecs, int polls,
                                                              void *wq, float *__restrict__ s_w) {
    __shared__ uint32_t lds[kWqThreads / kWave], lds_max;
    const int g = blockIdx.x / slices;
    const long first = (long)(blockIdx.x % slices) * slice_vecs;
    const int n = (int)(chunk_vecs - first < slice_vecs ? chunk_vecs - first : slice_vecs);   // at least 1
    const long base = g * chunk_vecs + first;

    // Vectors past the end of the slice read its first one again, so that no branch separates the loads.  Streaming
    // loads: no later access finds the weights in a cache (24576x6144 109 -> 98 us).
    uint32x4_t raw[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int idx = i * kWqThreads + (int)threadIdx.x;
        raw[i] = __builtin_nontemporal_load(w + base + (idx < n ? idx : 0));
    }
    ushort2_t mv = {0, 0};
#pragma unroll
    for (int i = 0; i < VPT; ++i) mv = absmax_pattern(mv, raw[i]);
    uint32_t m = block_max_pattern(mv, lds);

    const float qmax = (BITS == 8) ? 127.0f : 7.0f;
    constexpr int CB = BITS;                                // bytes of eight codes
    uint8_t *codes = static_cast<uint8_t *>(wq) + g * chunk_vecs * CB;
    const int line = wq_line_offset(codes);
    uint32_t *word = reinterpret_cast<uint32_t *>(codes + line);
    int skip = INT_MAX;                                     // the first of the vectors whose codes the line will hold
    if (slices > 1) {
        constexpr uint32_t kExpired = ~0u;
        if (first == 0) skip = line / CB;
        if (threadIdx.x == 0) {
            uint32_t cur = 0;
            for (;;) {                                      // a failed swap means that another slice arrived
                const uint32_t want = (m << 16) | ((cur & 0xffffu) + 0x100u);
                if (__hip_atomic_compare_exchange_strong(word, &cur, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)) {
                    cur = want;
                    break;
                }
                if ((cur >> 16) >= m) {
                    cur = __hip_atomic_fetch_add(word, 0x100u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 0x100u;
                    break;
                }
            }
            while (((cur >> 8) & 0xffu) != (uint32_t)slices && polls-- > 0) {
                __builtin_amdgcn_s_sleep(kWqSleep);
                cur = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            lds_max = ((cur >> 8) & 0xffu) == (uint32_t)slices ? cur >> 16 : kExpired;
        }
        __syncthreads();
        m = lds_max;
        if (m == kExpired) {
            ushort2_t all = {0, 0};
            for (long i = threadIdx.x; i < chunk_vecs; i += kWqThreads) all = absmax_pattern(all, w[g * chunk_vecs + i]);
            m = block_max_pattern(all, lds);
        }
    }
    float scale, inv;
    quant_scales(pattern_to_float(m), qmax, scale, inv);
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int idx = i * kWqThreads + (int)threadIdx.x;
        if (idx < n && (unsigned)(idx - skip) >= (unsigned)(kWqLine / CB)) store_codes<BITS>(wq, base + idx, raw[i], inv);
    }
    if (threadIdx.x >= kWave) return;
    uint32_t read = (uint32_t)slices - 1u;                  // slices that have read the maximum before this one
    if (slices > 1 && threadIdx.x == 0)
        read = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffu;
    if (__builtin_amdgcn_readfirstlane(read) != (uint32_t)slices - 1u) return;
    if (threadIdx.x == 0) s_w[g] = scale;
    if (slices > 1 && threadIdx.x < kWqLine / CB) {
        const long i = g * chunk_vecs + line / CB + threadIdx.x;
        store_codes<BITS>(wq, i, w[i], inv);
    }
}

__global__ void wq_clear_kernel(uint32_t *amax_bits, int groups) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < groups) amax_bits[i] = 0u;
}

__global__ __launch_bounds__(kWqThreads) void wq_absmax_kernel(const uint32x4_t *__restrict__ w, long chunk_vecs,
                                                               long slice_vecs, uint32_t *__restrict__ amax_bits) {
    __shared__ uint32_t lds[kWqThreads / kWave];
    const int g = blockIdx.y;
    const long lo = (long)blockIdx.x * slice_vecs;
    long hi = lo + slice_vecs;
    if (hi > chunk_vecs) hi = chunk_vecs;
    ushort2_t m = {0, 0};
    for (long i = lo + threadIdx.x; i < hi; i += kWqThreads) m = absmax_pattern(m, w[g * chunk_vecs + i]);
    const uint32_t r = block_max_pattern(m, lds);
    if (threadIdx.x == 0) atomicMax(amax_bits + g, __float_as_uint(pattern_to_float(r)));   // non-negative floats order like their bits
}

template <int BITS>
__global__ __launch_bounds__(kWqThreads) void wq_quant_kernel(const uint32x4_t *__restrict__ w, long chunk_vecs,
                                                              long slice_vecs, const float *__restrict__ amax,
                                                              void *__restrict__ wq) {
    const int g = blockIdx.y;
    const long lo = (long)blockIdx.x * slice_vecs;
    long hi = lo + slice_vecs;
    if (hi > chunk_vecs) hi = chunk_vecs;
    const float qmax = (BITS == 8) ? 127.0f : 7.0f;
    float scale, inv;
    quant_scales(amax[g], qmax, scale, inv);
    const long gbase = (long)g * chunk_vecs;
    for (long i = lo + threadIdx.x; i < hi; i += kWqThreads) store_codes<BITS>(wq, gbase + i, w[gbase + i], inv);
}

__global__ void wq_finalize_kernel(float *s_w, int groups, float qmax) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < groups) {
        float scale, inv;
        quant_scales(s_w[i], qmax, scale, inv);
        s_w[i] = scale;
    }
}

template <int BITS, int VPT>
static hipError_t launch_wq_group(const void *w, long chunk_vecs, int groups, int polls, void *wq, float *s_w,
                                  hipStream_t st) {
    const int most = kWqThreads * VPT;
    const int p = (int)((chunk_vecs + most - 1) / most);
    const int slice_vecs = (int)((chunk_vecs + p - 1) / p);
    const int slices = (int)((chunk_vecs + slice_vecs - 1) / slice_vecs);       // every slice holds a vector
    if (slices > 1)
        hipLaunchKernelGGL(wq_clear_line_kernel, dim3((groups + 255) / 256), dim3(256), 0, st, static_cast<uint8_t *>(wq),
                           chunk_vecs * BITS, groups);
    hipLaunchKernelGGL((wq_group_kernel<BITS, VPT>), dim3((unsigned)(groups * slices)), dim3(kWqThreads), 0, st,
                       reinterpret_cast<const uint32x4_t *>(w), chunk_vecs, slices, slice_vecs, polls, wq, s_w);
    return hipGetLastError();
}

// One pass where it is faster than two, measured over 4000 sizes (1 to 300 groups of 0.2 to 255 slices, weights from HBM,
// replayed graphs).  The time of two passes over time of one:  slices 8, 32, 64, 96, 128, 192, 255
//     1 group     0.9  1.0  1.1  1.2  1.3  1.3  1.4         12 groups   2.0  3.1  2.1  1.5  1.2  0.7  0.6
//     4 groups    1.2  1.8  2.4  2.0  1.7  1.2  0.9         48 groups   2.6  1.9  1.2  0.9  0.8  0.6  0.5
// A group of many slices leaves the chip together when its last one has arrived, and the next groups' loads start together:
// some 5 workgroups per compute unit hold the loads of later groups only while a group is a small part of them (INT8
// 12800x12640 in 25 groups 182 us in two passes, 360 in one).  A few slices in all are too little work for the exchange (one
// group of 229376 INT4 weights 8.2 us in two passes, 10.0 in one), but issued as a call of its own, as weights are, that is
// two launches instead of four: 12.1 and 7.9.
static bool one_pass_pays(int groups, long slices, int cus) {
    if (slices > (cus < kWqMaxSlices ? cus : kWqMaxSlices)) return false;
    return slices <= 80 || groups * slices <= (2500 - 7 * slices) * cus / 256;
}

template <int BITS>
static hipError_t launch_wq(const void *w, int N, int K, int groups, bool wait, void *wq, float *s_w, hipStream_t st) {
    const long chunk_vecs = (long)(N / groups) * K / 8;
    // the slices of a group have to run at once: each needs a fifth of a compute unit's registers, so one per compute
    // unit always fits
    const int cus = compute_units();
    if (one_pass_pays(groups, (chunk_vecs + kWqThreads * kWqVecs - 1) / (kWqThreads * kWqVecs), cus)) {
        const int polls = wait ? kWqPolls : 0;
        if (chunk_vecs <= kWqThreads * 4) return launch_wq_group<BITS, 4>(w, chunk_vecs, groups, polls, wq, s_w, st);
        if (chunk_vecs <= kWqThreads * 8) return launch_wq_group<BITS, 8>(w, chunk_vecs, groups, polls, wq, s_w, st);
        return launch_wq_group<BITS, kWqVecs>(w, chunk_vecs, groups, polls, wq, s_w, st);
    }
    // enough slices per group to put a few thousand workgroups in flight
    long P = (4096 + groups - 1) / groups;
    const long max_p = (chunk_vecs + 255) / 256;
    if (P > max_p) P = max_p;
    const long slice_vecs = (chunk_vecs + P - 1) / P;
    const dim3 grid((unsigned)P, (unsigned)groups);
    const int cb = (groups + 255) / 256;
    const uint32x4_t *wv = reinterpret_cast<const uint32x4_t *>(w);
    hipLaunchKernelGGL(wq_clear_kernel, dim3(cb), dim3(256), 0, st, reinterpret_cast<uint32_t *>(s_w), groups);
    hipLaunchKernelGGL(wq_absmax_kernel, grid, dim3(kWqThreads), 0, st, wv, chunk_vecs, slice_vecs,
                       reinterpret_cast<uint32_t *>(s_w));
    hipLaunchKernelGGL(wq_quant_kernel<BITS>, grid, dim3(kWqThreads), 0, st, wv, chunk_vecs, slice_vecs, s_w, wq);
    hipLaunchKernelGGL(wq_finalize_kernel, dim3(cb), dim3(256), 0, st, s_w, groups, BITS == 8 ? 127.0f : 7.0f);
    return hipGetLastError();
}

hipError_t launch_weight_quant(const void *w, int N, int K, int groups, int bits, bool wait, void *wq, float *s_w,
                               hipStream_t st) {
    return bits == 8 ? launch_wq<8>(w, N, K, groups, wait, wq, s_w, st) : launch_wq<4>(w, N, K, groups, wait, wq, s_w, st);
}

}  // namespace zq
