// Dot products of sample bits (+-1) with real class rows, exact to 2^-55 of a slice's largest element: the forward step of
// cosine inference and of online training (arXiv 2206.04746, Sec. III).
//
// A double-precision product on this chip runs at the vector unit's rate wherever it is sent, 64 times slower than 8-bit whole
// numbers on the matrix cores.  So a slice of a row (512 dimensions) is turned into whole numbers of 56 bits, relative to its
// largest element, and those into seven signed digits of 8 bits: sums of +-digit are exact in 32 bits, and the
// dot product is the digits' sums put together in fp64, one rounding of 2^-53 where an fp64 sum has one per dimension.  An
// element down to 2^-30 of the slice's largest loses nothing, a smaller one at most 2^-55 of that.  2947 samples, 6 classes, D = 10000: the fp64
// form took 20 us, this 8 (cosine inference 24.4 and 13.2 with the finish).  What bounds it: bytes made of bits, and a block's own digits
// before its first product.
//
// grid (slices, tiles of samples, chunks of classes), eight waves.  The block forms the digits of its rows in LDS, in the
// order in which the matrix instruction takes them; a wave has 16 samples (RT of these), whose bits become bytes of 1 and -1 on the way: a
// 32-bit word of a sample is eight registers, dimension 8 j + r in byte j of register r.  P digits of 16 / P
// classes share a tile of 16 columns.
#include <algorithm>

#include "hdc_internal.h"
#include "online_weight.h"

namespace hdc {

namespace {

constexpr int kWaves = 8, kThreads = kWaves * kWave, kDigits = 7;
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kBlocks = 4, kDims = 128 * kBlocks;   // of a slice

template <int P>
struct Shape {
    static constexpr int kClasses = 16 / P;                     // of a chunk
    static constexpr int kTiles = (kDigits + P - 1) / P;
    static constexpr int kUnits = kBlocks * 32 * kClasses;      // fours of dimensions of a class
    static constexpr int kPerThread = kUnits / kThreads;
};

// Turns the lanes of a row of 16 by N: lane i takes lane i + N.
template <int N>
__device__ __forceinline__ double from_lane(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + 16 - N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + 16 - N, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// part[slice * stride + n * step_n + c * step_c].  The blocks of one tile more, where wanted, form the squared-norm partials.
template <int P, int RT>
__global__ __launch_bounds__(kThreads) void row_dots_kernel(const uint32_t *__restrict__ hv, int64_t nb, int W, const float *__restrict__ acc,
                                                            int D, int C, int per, double *__restrict__ part, int64_t stride, int64_t step_n,
                                                            int64_t step_c, double *__restrict__ normpart, int G) {
    using S = Shape<P>;
    __shared__ __align__(16) uint32_t digits[kBlocks * 2 * S::kTiles][kWave][4];
    __shared__ uint32_t largest[2][S::kClasses];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int c0 = blockIdx.z * S::kClasses, slices = (D + kDims - 1) / kDims;
    const int s0 = blockIdx.x * per, s1 = min(s0 + per, slices);
    const int64_t first = (int64_t)blockIdx.y * (kWaves * 16 * RT);
    if (first >= nb) {   // squared norms, a wave to 64 dimensions
        for (int c = c0; c < min(c0 + S::kClasses, C); ++c)
            for (int g = s0 * (kDims / kWave) + wave; g < min(s1 * (kDims / kWave), G); g += kWaves) {
                const int d = g * kWave + lane;
                const double v = d < D ? (double)acc[(int64_t)c * D + d] : 0.0;
                double q = v * v;
                for (int off = 1; off < kWave; off <<= 1) q += __shfl_xor(q, off, kWave);
                if (lane == 0) normpart[(int64_t)c * G + g] = q;
            }
        return;
    }
    if (tid < 2 * S::kClasses) (&largest[0][0])[tid] = 0;
    const int col = lane & 15, kg = lane >> 4;
    int64_t row[RT];     // this lane's sample of a tile
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int64_t n = first + (wave * RT + t) * 16 + col;
        row[t] = (n < nb ? n : nb - 1) * W;
    }
    const bool idle = first + (int64_t)wave * RT * 16 >= nb;   // no sample of this wave's
    double total[RT][4] = {};
    for (int sl = s0; sl < s1; ++sl) {
        const int d0 = sl * kDims;
        // A unit is four dimensions 8 j + r of a word and a class; its place in u: r % 4, class, r / 4, word, so that lanes
        // write to LDS side by side.
        constexpr int kStep = 4 * S::kClasses;
        uint32_t x[S::kPerThread][4];   // bits of the elements
#pragma unroll
        for (int i = 0; i < S::kPerThread; ++i) {
            const int u = tid + i * kThreads, c = u / 4 % S::kClasses, at = d0 + u / (2 * kStep) * 32 + u / kStep % 2 * 4 + u % 4;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[i][j] = c0 + c < C && at + 8 * j < D ? __float_as_uint(acc[(int64_t)(c0 + c) * D + at + 8 * j]) : 0u;
        }
        uint32_t word[RT][kBlocks];
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) word[t][b] = hv[row[t] + min(d0 / 32 + 4 * b + kg, W - 1)];
        __syncthreads();   // the digits before have been read
        uint32_t *const most = largest[(sl - s0) & 1];
#pragma unroll
        for (int i = 0; i < S::kPerThread; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) m = max(m, x[i][j] & 0x7FFFFFFFu);
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));   // quad_perm 1,0,3,2
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));   // quad_perm 2,3,0,1
            if constexpr (kStep <= 16) m = max(m, (uint32_t)__shfl_xor((int)m, 16, kWave));
            if constexpr (kStep <= 32) m = max(m, (uint32_t)__shfl_xor((int)m, 32, kWave));
            if (lane < kStep && lane % 4 == 0) atomicMax(&most[lane / 4], m);
        }
        __syncthreads();
        if (tid < S::kClasses) largest[(sl - s0 + 1) & 1][tid] = 0;
#pragma unroll
        for (int i = 0; i < S::kPerThread; ++i) {
            const int u = tid + i * kThreads, c = u / 4 % S::kClasses, b = u / (8 * kStep), k = u / (2 * kStep) % 4, r = u / kStep % 2 * 4 + u % 4;
            // the slice's largest element is below 2^(top - 126): times this, below 2^54
            const double scale = __builtin_ldexp(1.0, 54 + 126 - max((int)(most[c] >> 23), 1));
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double v = (double)__uint_as_float(x[i][j]) * scale, upper = rint(v * 0x1p-32);   // both exact
                const int64_t low = (int64_t)(int)rint(fma(upper, -0x1p32, v));
                const uint64_t whole = ((uint64_t)(uint32_t)(int)upper << 32) + (uint64_t)low + 0x80808080808080ull;   // byte k less 128 is digit k
                lo[j] = (uint32_t)whole ^ 0x80808080u;
                hi[j] = (uint32_t)(whole >> 32) ^ 0x808080u;
            }
            // byte k of the four elements into one word
            const uint32_t a01 = __builtin_amdgcn_perm(lo[1], lo[0], 0x05010400), a23 = __builtin_amdgcn_perm(lo[3], lo[2], 0x05010400);
            const uint32_t b01 = __builtin_amdgcn_perm(lo[1], lo[0], 0x07030602), b23 = __builtin_amdgcn_perm(lo[3], lo[2], 0x07030602);
            const uint32_t e01 = __builtin_amdgcn_perm(hi[1], hi[0], 0x05010400), e23 = __builtin_amdgcn_perm(hi[3], hi[2], 0x05010400);
            const uint32_t f01 = __builtin_amdgcn_perm(hi[1], hi[0], 0x07030602), f23 = __builtin_amdgcn_perm(hi[3], hi[2], 0x07030602);
            const uint32_t out[8] = {__builtin_amdgcn_perm(a23, a01, 0x05040100), __builtin_amdgcn_perm(a23, a01, 0x07060302),
                                     __builtin_amdgcn_perm(b23, b01, 0x05040100), __builtin_amdgcn_perm(b23, b01, 0x07060302),
                                     __builtin_amdgcn_perm(e23, e01, 0x05040100), __builtin_amdgcn_perm(e23, e01, 0x07060302),
                                     __builtin_amdgcn_perm(f23, f01, 0x05040100), 0u};
#pragma unroll
            for (int w = 0; w < S::kTiles * P; ++w)   // (an eighth digit, where a tile has room for one, is zero)
                digits[(b * 2 + r / 4) * S::kTiles + w / P][k * 16 + w % P * S::kClasses + c][r % 4] = out[w];
        }
        __syncthreads();
        if (idle) continue;
        v4i sum[RT][S::kTiles] = {};
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            v4i ops[RT][2];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int r = 0; r < 8; ++r)   // a bit picks 1 or -1
                    ops[t][r / 4][r % 4] = (int)__builtin_amdgcn_perm(0u, 0x01FFu, word[t][b] >> r & 0x01010101u);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int w = 0; w < S::kTiles; ++w) {
                    const v4i d = *reinterpret_cast<const v4i *>(digits[(b * 2 + h) * S::kTiles + w][lane]);
#pragma unroll
                    for (int t = 0; t < RT; ++t) sum[t][w] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ops[t][h], d, sum[t][w], 0, 0, 0);
                }
        }
        const int c = col % S::kClasses;
        const uint32_t top = most[c];
        const double unit = __builtin_ldexp(1.0, max((int)(top >> 23), 1) - 126 - 54);
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double v;
                if constexpr (P == 1) {   // (sums of 512 digits: two of them go together in 32 bits)
                    v = (double)sum[t][6][i];
#pragma unroll
                    for (int w = 4; w >= 0; w -= 2) v = fma(v, 65536.0, (double)(sum[t][w][i] + 256 * sum[t][w + 1][i]));
                } else if constexpr (P == 2) {
                    v = (double)sum[t][3][i];
#pragma unroll
                    for (int w = 2; w >= 0; --w) v = fma(v, 65536.0, (double)sum[t][w][i]);
                    v = fma(from_lane<8>(v), 256.0, v);
                } else {
                    v = fma((double)sum[t][1][i], 4294967296.0, (double)sum[t][0][i]);
                    v = fma(from_lane<4>(v), 256.0, v);
                    v = fma(from_lane<8>(v), 65536.0, v);
                }
                v *= unit;
                if (__builtin_expect(top >= 0x7F800000u, 0)) {   // an element that is no number or infinite: one after another
                    v = 0.0;
                    const int64_t n = first + (wave * RT + t) * 16 + 4 * kg + i;
                    if (n < nb && c0 + c < C)
                        for (int d = d0; d < min(d0 + kDims, D); ++d) {
                            const double a = (double)acc[(int64_t)(c0 + c) * D + d];
                            v += hv[n * W + d / 32] >> (d % 32) & 1 ? a : -a;
                        }
                }
                total[t][i] += v;
            }
    }
    // register i of lane 16 q + col: sample 4 q + i
    if (col < S::kClasses && c0 + col < C) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t n = first + (wave * RT + t) * 16 + 4 * kg + i;
                if (n < nb) part[blockIdx.x * stride + n * step_n + (c0 + col) * step_c] = total[t][i];
            }
    }
}

int digits_of_a_tile(int C) { return C <= 4 ? 4 : C <= 8 ? 2 : 1; }

}  // namespace

int row_dots_slices(int D, int most) { return std::min((D + kDims - 1) / kDims, most); }

int launch_row_dots(hdc_ctx_impl *c, const uint32_t *hv, int64_t nb, const float *acc, double *part, int64_t stride, int64_t step_n,
                    int64_t step_c, double *normpart, int most, int *slices, hipStream_t s) {
    const int C = c->p.C, D = c->p.D, G = (D + kWave - 1) / kWave, P = digits_of_a_tile(C), all = (D + kDims - 1) / kDims;
    const int64_t chunks = P == 1 ? (C + 15) / 16 : 1, blocks = (nb + 127) / 128 * chunks * all;
    // Two tiles of samples a wave where that leaves four blocks a compute unit: the digits are formed half as often.  Then as many
    // slices to a block as leave three: the fewer partial sums to be read again.
    const bool two = blocks >= 8 * (int64_t)c->num_cus;
    const int64_t fit = blocks / (two ? 2 : 1) / (3 * (int64_t)c->num_cus);
    const int per = (int)std::max<int64_t>((all + most - 1) / most, std::min<int64_t>(all, fit));
    *slices = (all + per - 1) / per;
    const int64_t tile = kWaves * 16 * (two ? 2 : 1);
    const dim3 grid((unsigned)*slices, (unsigned)((nb + tile - 1) / tile + (normpart ? 1 : 0)), (unsigned)chunks);
#define HDC_ROW_DOTS(P, RT) \
    hipLaunchKernelGGL((row_dots_kernel<P, RT>), grid, dim3(kThreads), 0, s, hv, nb, c->W, acc, D, C, per, part, stride, step_n, step_c, normpart, G)
    if (P == 4) {
        if (two) HDC_ROW_DOTS(4, 2); else HDC_ROW_DOTS(4, 1);
    } else if (P == 2) {
        if (two) HDC_ROW_DOTS(2, 2); else HDC_ROW_DOTS(2, 1);
    } else {
        if (two) HDC_ROW_DOTS(1, 2); else HDC_ROW_DOTS(1, 1);
    }
#undef HDC_ROW_DOTS
    HDC_HIP(hipGetLastError());
    return HDC_OK;
}

}  // namespace hdc
