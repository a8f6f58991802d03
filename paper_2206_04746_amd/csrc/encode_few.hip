// ID-Level encoding (arXiv 2206.04746, Sec. III, Eq. 1) of a few samples: one launch.
//
// For a handful of samples encoding is latency: launches, and how long the one block that works on a
// stretch of a sample takes to see its operands.  The kernels for many samples quantise in a launch of
// their own, give a wave 64 word columns - five blocks a sample at D = 10000 - and copy a level slice into
// LDS first; where they leave level-invariant dimensions out, a third launch puts those back.  Here a block
// takes 16 word columns of one sample, quantises the sample itself, and its lanes split the features as
// well: lane (share, word) bundles every SHARES-th feature of its word, with level words straight from
// the cache, and the shares' bit-sliced counts are added up by lane exchanges and one LDS round.  All
// dimensions are bundled.  561 features, D = 10000, whole calls: one sample 23.4 -> 17.3 us (12.4 us of
// kernels -> 5.6), 64 samples back to back 12.6 -> 9.4 us.
#include <algorithm>

#include "bundle.h"

namespace hdc {

constexpr int kFewWords = 16;   // word columns of a block: 64 bytes of a table row
constexpr int kFewBatch = 8;    // features whose words are asked for together

// pl += other, P planes each
template <int P>
__device__ __forceinline__ void add_planes(uint32_t *pl, const uint32_t *other) {
    uint32_t carry = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const uint32_t a = pl[i], b = other[i];
        pl[i] = xor3(a, b, carry);
        carry = maj3(a, b, carry);
    }
}
// The sum over the four lanes of a word (lanes w, w + 16, w + 32, w + 48), in all of them.
template <int P>
__device__ __forceinline__ void add_lane_groups(uint32_t *pl) {
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
        uint32_t other[P];
#pragma unroll
        for (int i = 0; i < P; ++i) other[i] = (uint32_t)__shfl_xor((int)pl[i], off, kWave);
        add_planes<P>(pl, other);
    }
}

// grid (stretches of 16 words, samples).  LDS: level-row byte offsets [votes rounded up to 2], u16, then the
// waves' counts [WAVES][P][16].
template <int P, int WAVES, bool kU8>
__global__ __launch_bounds__(WAVES *kWave) void encode_few_kernel(
    const void *__restrict__ feats, int F, int votes, int Fp, int L, const float *__restrict__ lo,
    const float *__restrict__ scale, const uint32_t *__restrict__ item, const uint32_t *__restrict__ level,
    uint32_t *__restrict__ hv, int W, uint32_t bias) {
    constexpr int T = WAVES * kWave, kShares = WAVES * 4;
    extern __shared__ uint32_t sm[];
    uint16_t *rows = reinterpret_cast<uint16_t *>(sm);
    uint32_t *counts = sm + (votes + 1) / 2;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), word = lane & (kFewWords - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int share = wave * 4 + (lane >> 4);
    const int col = blockIdx.x * kFewWords + word;
    // this lane's word of row r of the two slice-major tables: + r * 256 bytes
    const size_t slice = (size_t)(blockIdx.x / (kSliceWords / kFewWords));
    const int in_slice = (blockIdx.x % (kSliceWords / kFewWords)) * kFewWords + word;
    const uint32_t *ids = item + slice * Fp * kSliceWords + in_slice;
    const char *levels = reinterpret_cast<const char *>(level + slice * L * kSliceWords + in_slice);

    uint32_t id[kFewBatch];
    auto load_ids = [&](int f0) {
#pragma unroll
        for (int k = 0; k < kFewBatch; ++k) id[k] = ids[(size_t)std::min(f0 + k * kShares, votes - 1) * kSliceWords];
    };
    load_ids(share);   // on their way while the block quantises
    const size_t row = (size_t)blockIdx.y * F;
    for (int f = tid; f < votes; f += T) {
        uint32_t b = 0;   // (the tie vote of an even F sits in bin 0)
        if (f < F)
            b = kU8 ? (uint32_t)reinterpret_cast<const uint8_t *>(feats)[row + f] * (uint32_t)L >> 8
                    : bin_f32(reinterpret_cast<const float *>(feats)[row + f], lo[f], scale[f], L);
        rows[f] = (uint16_t)(b * (kSliceWords * 4));
    }
    __syncthreads();

    uint32_t pl[P];
#pragma unroll
    for (int i = 0; i < P; ++i) pl[i] = share == 0 && ((bias >> i) & 1u) ? 0xffffffffu : 0u;
    for (int f0 = share; f0 - share < votes; f0 += kFewBatch * kShares) {   // every lane makes the same trips
        if (f0 != share) load_ids(f0);
        uint32_t x[kFewBatch];
#pragma unroll
        for (int k = 0; k < kFewBatch; ++k)
            x[k] = *reinterpret_cast<const uint32_t *>(levels + rows[std::min(f0 + k * kShares, votes - 1)]);
#pragma unroll
        for (int k = 0; k < kFewBatch; ++k) x[k] = f0 + k * kShares < votes ? x[k] ^ id[k] : 0u;
        ripple<3, P>(pl, Tree<3, 0>::run(pl, x));
    }
    add_lane_groups<P>(pl);
    if (lane < kFewWords)
#pragma unroll
        for (int i = 0; i < P; ++i) counts[(wave * P + i) * kFewWords + word] = pl[i];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int j = 0; j < WAVES / 4; ++j) {   // a lane group adds up a quarter of the waves
        uint32_t x[P];
#pragma unroll
        for (int i = 0; i < P; ++i) x[i] = counts[(((lane >> 4) * (WAVES / 4) + j) * P + i) * kFewWords + word];
        if (j == 0)
#pragma unroll
            for (int i = 0; i < P; ++i) pl[i] = x[i];
        else
            add_planes<P>(pl, x);
    }
    add_lane_groups<P>(pl);
    if (lane < kFewWords && col < W) hv[(int64_t)blockIdx.y * W + col] = pl[P - 1];
}

template <int WAVES>
static int launch_few(hdc_ctx_impl *c, const void *feats, int N, uint32_t *hv, int P, uint32_t bias, hipStream_t s) {
    const dim3 grid((unsigned)((c->W + kFewWords - 1) / kFewWords), (unsigned)N), block(WAVES * kWave);
    const size_t lds = (size_t)((c->votes + 1) / 2 + WAVES * P * kFewWords) * 4;
    ProfScope prof(c, HDC_K_ENCODE, s);
#define HDC_FEW(P_, U8)                                                                                           \
    hipLaunchKernelGGL((encode_few_kernel<P_, WAVES, U8>), grid, block, lds, s, feats, c->p.F, c->votes, c->Fp, c->p.L, \
                       c->lo_d, c->scale_d, c->item_d, c->level_d, hv, c->W, bias)
    const bool u8 = c->p.feat_dtype == HDC_U8;
    switch (P) {
        case 8: if (u8) HDC_FEW(8, true); else HDC_FEW(8, false); break;
        case 10: if (u8) HDC_FEW(10, true); else HDC_FEW(10, false); break;
        default: if (u8) HDC_FEW(12, true); else HDC_FEW(12, false); break;
    }
#undef HDC_FEW
    HDC_HIP(hipGetLastError());
    return HDC_OK;
}

bool try_encode_few(hdc_ctx_impl *c, const void *feats, int64_t N, uint32_t *hv, bool sparse, hipStream_t s, int *rc) {
    // A block costs about 1.1 ns + 6.8 ns per thousand features of the chip's time (31 to 784 features,
    // D = 2048 to 20000), the other kernels 7 us more than this one's launch: below that sum.
    // From 1024 samples on a matrix kernel takes any model that it can, with one launch more.
    const int64_t blocks = (int64_t)((c->W + kFewWords - 1) / kFewWords) * N;
    if (N >= 1024 || blocks * (c->p.F + 160) > 1 << 20) return false;
    // The sparse encoder's two launches take 8.6 us whatever they find: a model of a few features is there
    // sooner (F = 3, bytes, unrelated levels: 6400 blocks 10.9 us, 4800 blocks 9.1; at F = 64 4680 blocks 8.6).
    if (sparse && blocks > 4400) return false;
    int P;
    uint32_t bias;
    majority_planes(c, &P, &bias);
    if (P > 12) return false;
    // eight waves share a sample's features while there are blocks for two rounds of the chip at most
    *rc = blocks <= 2 * c->num_cus ? launch_few<8>(c, feats, (int)N, hv, P, bias, s)
                                   : launch_few<4>(c, feats, (int)N, hv, P, bias, s);
    return true;
}

}  // namespace hdc
