// GeMM for one to four tokens on the vector ALUs (v_dot4_i32_i8): INT8 activations, INT8 or packed INT4 weights, any
// legal K (Sec. 4.3: at small batch the latency is the time to load the weights).
//
// Bound: HBM, and around it latency.  A 16-row matrix-core operand wants its rows in neighbouring lanes: loads of 64
// bytes a row, sixteen cross-lane permutations per stage of 256 values, and sums of 1.5 KB per wave through LDS.  For a
// token or two the products are few enough for the vector ALUs, which take the weights as they lie: sixteen lanes read 256
// contiguous bytes of a row, a wave's load four rows, a workgroup's rows are eight, and piece p of 256 bytes of K belongs to
// wave p % NW.  A wave asks for all its pieces (up to four at a time) before it waits, sums over its sixteen lanes with four
// DPP steps and hands one number per row and token to the epilogue.  Small workgroups deal the rows evenly and keep up to 32
// waves on a compute unit.  us per call in a replayed graph, weights from HBM, before (direct or streaming) / this kernel:
//   1 token, INT8: 2048x2048 3.1 / 2.6, 8192x2048 5.2 / 4.8, 2048x8192 6.6 / 4.9, 6400x1600 4.7 / 3.9, 4096x16384 16.0 / 13.0,
//     24576x6144 27.6 / 25.8 (5.8 TB/s); INT4: 16384x4096 8.4 / 7.8, 2048x8192 5.1 / 3.8
//   2 tokens: 8192x2048 5.4 / 5.0, 2048x8192 6.6 / 5.1; INT4 6144x2048 3.7 / 3.5
// Sixteen rows a workgroup measured 3 to 15 % slower, four 5 % slower on average.
#include <type_traits>

#include "zq_device.h"
#include "zq_internal.h"

namespace zq {

namespace {

constexpr int kPiece = 256;                    // bytes of a weight row that sixteen lanes read at once
[[maybe_unused]] constexpr int kGroups = 2;    // groups of four rows of a workgroup
constexpr int kRows = 4 * kGroups;

template <int CTRL>
__device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

}  // namespace

// MT: tokens, CH: pieces that a wave asks for at once, NW: waves, rounds: CH pieces each.
template <int MT, int WBITS, int CH, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_vector_kernel(
    const uint8_t *__restrict__ xq, const uint8_t *__restrict__ wq, int M, int N, int K, int rounds, int gs, int act,
    const float *__restrict__ s_tok, const float *__restrict__ s_w, const half_t *__restrict__ bias,
    half_t *__restrict__ out, int32_t *__restrict__ acc_out) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the launch stub
    constexpr int XL = 8 / WBITS;              // 16-byte activation loads per weight load
    static_assert(kRows * MT <= 64 * NW, "a thread per output");
    __shared__ int32_t part[NW][MT][kRows];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int c = lane % 16, r = lane / 16;
    const int n_base = (int)blockIdx.x * kRows;
    const int wrow = WBITS == 8 ? K : K / 2;
    const __amdgpu_buffer_rsrc_t rs_w =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(wq), 0, (int)((size_t)N * wrow), kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rs_x =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(xq), 0, (int)((size_t)M * K), kRsrcFlags);
    constexpr uint32_t kNowhere = 0x80000000u; // past the end of either buffer: loads give 0
    uint32_t voff_w[kGroups], voff_x[MT];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const int n = n_base + 4 * g + r;
        voff_w[g] = n < N ? (uint32_t)(n * wrow + 16 * c) : kNowhere;
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) voff_x[m] = m < M ? (uint32_t)(m * K + 16 * XL * c) : kNowhere;
    // thread t < kRows * MT finishes row t % kRows of token t / kRows
    const int t = threadIdx.x;
    const int em = t / kRows, en = n_base + t % kRows;
    const bool mine = em < MT && em < M && en < N;
    float e_sc = 0.0f, e_b = 0.0f;

    int acc[kGroups][MT];
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[g][m] = 0;
    auto load = [&](__amdgpu_buffer_rsrc_t rs, uint32_t vo, int so) __attribute__((always_inline)) {
        return __builtin_bit_cast(int32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)vo, so, 0));
    };
    auto round = [&](int b, auto first_c) __attribute__((always_inline)) {
        int32x4 w[CH][kGroups], x[CH][MT][XL];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int p = (wave + (b * CH + i) * NW) * kPiece;
            const int off = p < wrow ? p : 0;
            const bool in = p + 16 * c < wrow; // past the end of the row: zeros
#pragma unroll
            for (int g = 0; g < kGroups; ++g) w[i][g] = load(rs_w, in ? voff_w[g] : kNowhere, off);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int l = 0; l < XL; ++l) x[i][m][l] = load(rs_x, (in ? voff_x[m] : kNowhere) + 16 * l, XL * off);
        }
        if constexpr (decltype(first_c)::value) {          // the epilogue's operands come with the first pieces
            if (mine) {
                e_sc = s_tok[em] * s_w[en / gs];
                if (bias != nullptr) e_b = (float)bias[en];
            }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if constexpr (WBITS == 8) {
#pragma unroll
                for (int g = 0; g < kGroups; ++g)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[g][m] = __builtin_amdgcn_sdot4(w[i][g][e], x[i][m][0][e], acc[g][m], false);
            } else {
                // even and odd nibbles as int8 values times 16; the activations are sorted the same way
                int even[MT][4], odd[MT][4];
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t lo = (uint32_t)x[i][m][e / 2][2 * (e % 2)], hi = (uint32_t)x[i][m][e / 2][2 * (e % 2) + 1];
                        even[m][e] = (int)__builtin_amdgcn_perm(hi, lo, 0x06040200u);
                        odd[m][e] = (int)__builtin_amdgcn_perm(hi, lo, 0x07050301u);
                    }
#pragma unroll
                for (int g = 0; g < kGroups; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t d = (uint32_t)w[i][g][e];
                        const int we = (int)((d << 4) & 0xf0f0f0f0u), wo = (int)(d & 0xf0f0f0f0u);
#pragma unroll
                        for (int m = 0; m < MT; ++m) {
                            acc[g][m] = __builtin_amdgcn_sdot4(we, even[m][e], acc[g][m], false);
                            acc[g][m] = __builtin_amdgcn_sdot4(wo, odd[m][e], acc[g][m], false);
                        }
                    }
            }
        }
    };
    round(0, std::true_type{});
    for (int b = 1; b < rounds; ++b) round(b, std::false_type{});

#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            int v = acc[g][m];
            v = dpp_add<kDppXor1>(v);
            v = dpp_add<kDppXor2>(v);
            v = dpp_add<kDppHalfMirror>(v);
            v = dpp_add<kDppMirror>(v);
            if (c == 0) part[wave][m][4 * g + r] = v;
        }
    __syncthreads();
    if (mine) {
        int v = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += part[w][em][t % kRows];
        if constexpr (WBITS == 4) v >>= 4;     // exact: every product carried the factor 16
        const float f = apply_activation(__builtin_fmaf((float)v, e_sc, e_b), act);
        out[(size_t)em * N + en] = (half_t)f;
        if (acc_out != nullptr) acc_out[(size_t)em * N + en] = v;
    }
#endif
}

namespace {

template <int MT, int WBITS, int CH, int NW>
hipError_t launch_vector_t(const GemmArgs &a, int rounds, hipStream_t st) {
    hipLaunchKernelGGL((gemm_vector_kernel<MT, WBITS, CH, NW>), dim3((a.N + kRows - 1) / kRows), dim3(64 * NW), 0, st,
                       reinterpret_cast<const uint8_t *>(a.xq), static_cast<const uint8_t *>(a.wq), a.M, a.N, a.K, rounds,
                       a.N / a.groups, a.act, a.s_tok, a.s_w, static_cast<const half_t *>(a.bias),
                       static_cast<half_t *>(a.out), a.acc_out);
    return hipGetLastError();
}

// Eight waves, four where a row has no piece for more; the pieces of a wave in as few rounds as four at a time make, and
// rounds of the same size.
template <int MT, int WBITS>
hipError_t launch_vector(const GemmArgs &a, hipStream_t st) {
    const int pieces = ((WBITS == 8 ? a.K : a.K / 2) + kPiece - 1) / kPiece;
    if (pieces <= 4) return launch_vector_t<MT, WBITS, 1, 4>(a, 1, st);
    const int per_wave = (pieces + 7) / 8;
    const int rounds = (per_wave + 3) / 4;
    switch ((per_wave + rounds - 1) / rounds) {
        case 1: return launch_vector_t<MT, WBITS, 1, 8>(a, rounds, st);
        case 2: return launch_vector_t<MT, WBITS, 2, 8>(a, rounds, st);
        case 3: return launch_vector_t<MT, WBITS, 3, 8>(a, rounds, st);
        default: return launch_vector_t<MT, WBITS, 4, 8>(a, rounds, st);
    }
}

}  // namespace

// One token: everywhere (the route of a call leaves nine pieces against more than 4096 rows to streaming, see direct_pays).  More tokens cost a 16-byte
// activation load each where the weights cost two, so the line is drawn where the kernels with matrix cores pay more for
// something else, few rows against a long K above all.  us, before / this kernel, over 110 random shapes:
//   2 tokens, INT8   1792x7168 6.5 / 4.7, 5664x1888 4.8 / 4.1, 8832x2944 9.0 / 7.6, 4736x18944 20.2 / 19.9; beyond: 2560x9216
//                    7.5 / 8.2 (320 workgroups on 256 compute units); 12288x4096, see direct_pays
//             INT4   896x3584 3.2 / 2.8, 6144x2048 3.7 / 3.5; beyond: 3072x768 2.6 / 2.8, 6016x6016 6.9 / 7.1, 13056x4352 9.5 / 11.3
//   3, 4 tokens INT8 768x2560 3.4 / 3.1, 1696x6784 6.4 / 5.5; beyond: 6144x2048 4.9 / 4.9, 3840x3840 5.1 / 5.6
//             INT4   none: 1536x6144 4.1 / 4.2, 18048x6016 13.2 / 23.2
//
// A K of a piece or two of 256 bytes leaves waves idle in every workgroup, which many rows make many of: not INT4 up to K 1024
// above 16384 rows (1 token 31536x256 3.5 / 4.7, 26400x768 4.6 / 5.2, 29440x1024 4.9 / 5.6; 1152 and more 0.91 of the time), nor at 2
// tokens up to K 1024 (3328x1024 2.5 / 2.7, 8192x1024 3.0 / 3.2), nor INT8 of one piece above 20480 rows at 2 tokens, 28672 at 1
// (2 tokens 29024x256 4.2 / 4.9, 1 token 31424x256 4.2 / 4.5).
bool vector_pays(int M, int N, int K, int w_bits) {
    if (w_bits == 4 && M == 1 && N > 16384 && K <= 1024) return false;
    if (w_bits == 8 && K <= kPiece && N > (M == 1 ? 28672 : 20480)) return false;
    if (M == 1) return true;
    if (M == 2) {
        if (w_bits == 8) return !(N > 2048 && N <= 3072 && K > 8192) && !(K % 4096 == 0 && N > 8192 && N <= 12288);
        return N <= 2048 || (N <= 8192 && K > 1024 && K <= 4096);
    }
    return M <= 4 && w_bits == 8 && N <= 2048 && K >= 2560;
}

hipError_t launch_gemm_vector(const GemmArgs &a, hipStream_t st) {
    if (a.M < 1 || a.M > 4) return hipErrorInvalidValue;
    if (a.w_bits == 8) {
        if (a.M == 1) return launch_vector<1, 8>(a, st);
        if (a.M == 2) return launch_vector<2, 8>(a, st);
        return launch_vector<4, 8>(a, st);
    }
    if (a.M == 1) return launch_vector<1, 4>(a, st);
    if (a.M == 2) return launch_vector<2, 4>(a, st);
    return hipErrorInvalidValue;               // (see vector_pays)
}

}  // namespace zq
