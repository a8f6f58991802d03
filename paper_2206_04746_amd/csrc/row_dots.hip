// Dot products of sample bits (+-1) with real class rows, of a slice rounded once: the forward step of cosine inference and of
// online training (arXiv 2206.04746, Sec. III).
//
// A double-precision product on this chip runs at the vector unit's rate wherever it is sent, 64 times slower than 8-bit whole
// numbers on the matrix cores.  So a slice of a row (512 dimensions) is turned into whole numbers of 56 bits, relative to its
// largest element, and those into seven signed digits of 8 bits: sums of +-digit are exact in 32 bits, and the dot product is
// the digits' sums put together in fp64, one rounding of 2^-53 where an fp64 sum has one per dimension.  2947 samples, 6 classes,
// D = 10000: the fp64 form took 20 us, this 8 (cosine inference 25.6 and 14.8 with the finish).  What bounds it: bytes made of bits,
// and a block's own digits before its first product.
//
// Digits hold an element whole if its last bit is no less than 2^-53 of the largest one's power of two: every element down to 2^-30
// of the largest.  A row of a slice with one that they do not hold, or that is no number or infinite, is summed in fp64 on the
// matrix cores instead: the same call with one such element takes 26 us, with one in every row of every slice 39 (26 classes: 33.8, 38
// and 80, and 82 in the fp64 form).
//
// grid (slices, tiles of samples, chunks of classes), eight waves.  The block forms the digits of its rows in LDS, in the
// order in which the matrix instruction takes them; a wave has 16 samples (RT of these), whose bits become bytes of 1 and -1 on the way: a
// 32-bit word of a sample is eight registers, dimension 8 j + r in byte j of register r.  P digits of 16 / P
// classes share a tile of 16 columns.
#include <algorithm>

#include "hdc_internal.h"
#include "online_weight.h"
#include "row_digits.h"

namespace hdc {

namespace {

constexpr int kWaves = 8, kThreads = kWaves * kWave, kDigits = 7;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

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
__device__ __forceinline__ int from_lane(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + 16 - N, 0xF, 0xF, true);
}

// part[slice * stride + n * step_n + c * step_c].  The blocks of one tile more, where wanted, form the squared-norm partials.
// (Six waves a SIMD, 80 registers, where one tile a wave lets them: three blocks a compute unit.  8000 samples, 6 classes, D = 10000: 19.9 us
// a cosine call, with the 82 registers it would take otherwise 21.1.)
template <int P, int RT>
__global__ __launch_bounds__(kThreads, P > 1 && RT == 1 ? 6 : 2) void row_dots_kernel(const uint32_t *__restrict__ hv, int64_t nb, int W, const float *__restrict__ acc,
                                                            int D, int C, int per, double *__restrict__ part, int64_t stride, int64_t step_n,
                                                            int64_t step_c, double *__restrict__ normpart, int G) {
    using S = Shape<P>;
    __shared__ __align__(16) uint32_t digits[kBlocks * 2 * S::kTiles][kWave][4];
    __shared__ uint32_t largest[2][S::kClasses];   // element of a slice; bit 31: digits leave out some of an element
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
        uint32_t least = ~0u;   // (a thread's elements are of one class: kThreads is a multiple of a word's units)
#pragma unroll
        for (int i = 0; i < S::kPerThread; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                m = max(m, x[i][j] & 0x7FFFFFFFu);
                least = min(least, (x[i][j] & 0x7FFFFFFFu) - 1);
            }
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));   // quad_perm 1,0,3,2
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));   // quad_perm 2,3,0,1
            if constexpr (kStep <= 16) m = max(m, (uint32_t)__shfl_xor((int)m, 16, kWave));
            if constexpr (kStep <= 32) m = max(m, (uint32_t)__shfl_xor((int)m, 32, kWave));
            if (lane < kStep && lane % 4 == 0) atomicMax(&most[lane / 4], m);
        }
        __syncthreads();
        if (tid < S::kClasses) largest[(sl - s0 + 1) & 1][tid] = 0;
        const int own = tid / 4 % S::kClasses;
        const uint32_t top_of = most[own] >> 23 & 255;   // (255, with an element that is no number or infinite: digits of no meaning)
        const double scale = digits_scale(top_of);
#pragma unroll
        for (int i = 0; i < S::kPerThread; ++i) {
            const int u = tid + i * kThreads, b = u / (8 * kStep), k = u / (2 * kStep) % 4, r = u / kStep % 2 * 4 + u % 4;
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) digits_of((double)__uint_as_float(x[i][j]) * scale, lo[j], hi[j]);
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
                digits[(b * 2 + r / 4) * S::kTiles + w / P][k * 16 + w % P * S::kClasses + own][r % 4] = out[w];
        }
        if (__builtin_expect(!digits_hold(least, top_of), 0)) {
            bool all = true;
#pragma unroll
            for (int i = 0; i < S::kPerThread; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double v = (double)__uint_as_float(x[i][j]) * scale;
                    all &= v == rint(v);
                }
            if (!all) atomicOr(&most[own], 0x80000000u);
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
        const bool exact = top < 0x7F800000u;
        const double unit = exact ? __builtin_ldexp(1.0, max((int)(top >> 23), 1) - 126 - 54) : 0.0;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // (sums of 512 digits: two of them go together in 32 bits)
                int s01, s23, s45, s6;
                if constexpr (P == 1) {
                    s01 = sum[t][0][i] + 256 * sum[t][1][i], s23 = sum[t][2][i] + 256 * sum[t][3][i];
                    s45 = sum[t][4][i] + 256 * sum[t][5][i], s6 = sum[t][6][i];
                } else if constexpr (P == 2) {
                    s01 = sum[t][0][i] + 256 * from_lane<8>(sum[t][0][i]), s23 = sum[t][1][i] + 256 * from_lane<8>(sum[t][1][i]);
                    s45 = sum[t][2][i] + 256 * from_lane<8>(sum[t][2][i]), s6 = sum[t][3][i];
                } else {
                    s01 = sum[t][0][i] + 256 * from_lane<4>(sum[t][0][i]), s45 = sum[t][1][i] + 256 * from_lane<4>(sum[t][1][i]);
                    s23 = from_lane<8>(s01), s6 = from_lane<8>(sum[t][1][i]);
                }
                total[t][i] += sum_of_digits(s01, s23, s45, s6) * unit;
            }
        if (__builtin_expect(__ballot(!exact) != 0, 0)) {   // classes that digits do not hold: in fp64
            // Lanes of row kg of 16 have words kg, kg + 4 ... of the slice.  What comes out as sample 4 i + kg is to be sample 4 kg + i.
            const int64_t tile = first + (int64_t)wave * RT * 16 + 4 * (col % 4) + col / 4;
            const float *const values = acc + (int64_t)min(c0 + c, C - 1) * D;
            v4d all_of[RT] = {};
            float x[2][8];   // of eight dimensions, and the next eight
            uint32_t bits[2][RT];
            auto ask = [&](int h, float(&to)[8], uint32_t(&word_of)[RT]) {
                const int d = d0 + 32 * (4 * (h / 4) + kg) + 8 * (h & 3);
#pragma unroll
                for (int t = 0; t < RT; ++t) word_of[t] = hv[min(tile + 16 * t, nb - 1) * W + min(d / 32, W - 1)] >> 8 * (h & 3);
                if (d + 8 <= D) {
                    __builtin_memcpy(to, values + d, sizeof(to));
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) to[j] = d + j < D ? values[d + j] : 0.0f;
                }
            };
            auto add = [&](const float(&from)[8], const uint32_t(&word_of)[RT]) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const double a = exact || col >= S::kClasses ? 0.0 : (double)from[j];
#pragma unroll
                    for (int t = 0; t < RT; ++t)
                        all_of[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(word_of[t] >> j & 1 ? 1.0 : -1.0, a, all_of[t], 0, 0, 0);
                }
            };
            ask(0, x[0], bits[0]);
#pragma unroll 1
            for (int h = 0; h < 4 * kBlocks; h += 2) {
                ask(h + 1, x[1], bits[1]);
                add(x[0], bits[0]);
                ask(h + 2, x[0], bits[0]);   // (past the slice: not used)
                add(x[1], bits[1]);
            }
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) total[t][i] += all_of[t][i];
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
