// Online training, per sample and in small batches, as a few parallel steps per block of up to 256
// samples (arXiv 2206.04746, Sec. III Eqs. 2-3, caption of Fig. 1; Sec. VI-D2 for batches).
//
// The method is a dependency chain: a sample's cosines need the class rows as the sample (or batch)
// before left them.  But a row only ever moves along samples, so within a block of samples
//     <acc_c before m, s_m> = <acc_c at the block's start, s_m> + sum over earlier n of k_n,c <s_n, s_m>
// and the whole chain can be walked on the scalar products of the samples with one another, which
// do not depend on the rows.  Four kernels:
//   online_gram_kernel   once per call: <s_n, s_m> of all pairs of a block
//   online_dots_kernel   per block: <acc_c, s_m> against the rows as they stand (fp64), which do not hold the
//                        block before yet: what that adds comes from the samples' products
//   online_chain_kernel  per block, one workgroup: cosines, predictions and weights of all samples; its other
//                        workgroups apply the updates of the block before to the rows element by element, in
//                        sample order, one fp32 rounding per update (per batch: one per batch), and form the
//                        rows' new squared norms
//   online_rows_kernel   the same updates for the last block (for every one, before the next, where a weight could overflow)
// Calls of more than 1024 samples of up to 32 classes go in blocks of 2048 (online_spread.hip), with their products from
// online_gram_kernel here in strips of 16 columns.  Other per-sample calls of up to 16 classes take online_wide_kernel for the chain, which walks the block as a whole, with the
// row updates of the block before as its other workgroups (wide_takes).
// The dot products stay fp64 sums of the same fp32 rows and fp32 weights.  They leave out the fp32 rounding of the u <= 512
// updates of a row made since the block before began: at most 2^-24 of an element each, so u 2^-24 of a cosine at the very
// most and about sqrt(u) 2^-24 as a rule.  Largest over 36 to 180 models each, D = 33 to 4096, 1 to 16 classes, 1200 samples
// up to 35 % from their prototype: 2.6e-7 from zero rows (2.5e-8 at D = 10000, 6 classes), 3.4e-6 from rows of size 1e6; 7.1e-6
// and 5.6e-4 for a few cosines where samples drive rows of up to 80 and of up to 1000 times their prototype through zero
// (with only the updates since the block itself began: 2.0e-7, 1.8e-6, 7.1e-6, 1.2e-4).
// That is no distance from the method.  Against the method in 64 bits (largest over the same models, the walk by samples,
// which rounds the rows at every step / this): cosines 2.3e-7 / 1.7e-7, 7.6e-6 / 5.0e-6, 5.2e-6 / 6.5e-7, 3.6e-4 / 1.2e-4;
// rows, relative 2-norm, 1.1e-6 / 9.3e-7, 1.8e-5 / 1.8e-5, 2.0e-6 / 1.5e-6, and 6.5e-6 / 1.3e-5 through zero from 1000 prototypes
// (in the geometric mean 9.4e-7 / 1.2e-6).  On the GPU, 1 to 16 classes, D = 1000 to 12000, 1000 to 1500 samples from zero rows:
// rows 1.43e-7 to 5.47e-7, blocks that begin from their own rows 1.42e-7 to 5.46e-7.  But the two forms may part where two
// cosines agree that closely, also where samples that repeat make rows proportional.
//
// Walking the chain sample after sample on one workgroup took 3.6 us per sample (two block barriers
// and a block-wide sum for each).
#include <algorithm>

#include "online_lanes.h"

namespace hdc {

constexpr int kChainBlock = 256;                    // most samples of a block
constexpr int kSub = 64;                            // samples of a sub-block: one per lane
constexpr int kSubs = kChainBlock / kSub;
constexpr int kTile = kSub * kSub;                  // products of one pair of sub-blocks
constexpr int kTiles = kSubs * (kSubs + 1) / 2;     // pairs (a, b), a <= b, at b (b + 1) / 2 + a
constexpr int64_t kHeldBlocks = 64;                 // blocks whose columns and products are held at a time (32: sets of 8193 to 16384 samples 4 to 6 % slower in three epochs)
constexpr float kTameRate = 1e30f;                  // a learning rate below which no weight overflows
constexpr int kChainMaxWaves = 16;
constexpr int kSlices = 10;                         // most slices the dimensions are split into

// ---- the order of a block's products in online_wide_kernel (below) --------------------------------
constexpr int kWideWaves = 8, kWideRows = 96, kWideClasses = 16;   // rows of a wave: room for
constexpr int kNoSample = kChainBlock;   // its weight is zero
// Groups of rows: 640 rows and the filling of 4 C classes are 184 groups of four at most (8 classes), 352 of two (16).
__host__ __device__ constexpr int wide_group(int C) { return C <= 8 ? 4 : 2; }
__host__ __device__ constexpr int wide_rows(int GR) { return GR == 4 ? 92 : 88; }   // of a wave, therefore
// Places in LDS for sums over a wave's rows from its first one on, one for every run of groups of a class in a wave.
// The last two: one that holds zero, one nobody reads.
__host__ __device__ constexpr int wide_places(int C) { return kSubs * C + kWideWaves + 2; }

struct WideOrder {                       // of a block, from its labels
    uint16_t src[kWideWaves][kWideRows]; // a wave's rows: sample, kNoSample where a class is filled up
    uint16_t to[kWideWaves][kSub];       // places of its groups' sums
    uint16_t sum[kWideClasses][kSubs][8];// a class's sum in a target sub-block: that of place [0] less that of place [1], and those of
                                         // [2] to [5] in the waves it goes on in; [6]: it goes on in more than one
    uint16_t row[kSubs][kChainBlock];    // 96 wave + row of a sample in a target sub-block's list, ~0: none
    int32_t rows;                        // of a wave: at least 64, so that a list of 256 touches no more than five waves
    int32_t pad[3];
};

// A wave's rows as they lie in memory: [wave][row / 8][lane][row % 8], 16 bytes a lane and load.
constexpr int kWideImage = kWideWaves * kWideRows * kSub;
__host__ __device__ constexpr int wide_place(int row, int lane) {   // row: 96 wave + its row
    return ((row >> 3) * kSub + lane) * 8 + (row & 7);
}

// Writes the order of one block (256 threads).  A list: the samples of a class among those up to the end of a target
// sub-block; lists stand at C j + c, their groups one after another are dealt to the waves in equal numbers.
__device__ void write_order(const int32_t *__restrict__ labels, int nb, int C, WideOrder *__restrict__ out) {
    __shared__ WideOrder o;
    __shared__ int cnt[kSubs][kWideClasses];
    __shared__ int first[kSubs * kWideClasses], run[kSubs * kWideClasses];   // a list's first group and run
    const int t = threadIdx.x, lane = t & (kWave - 1), a = t >> 6;
    const int GR = wide_group(C), zero = wide_places(C) - 2, lists = kSubs * C;
    int y = t < nb ? labels[t] : -1;
    y = y >= 0 && y < C ? y : -1;
    int rank = 0;
    for (int c = 0; c < C; ++c) {
        const uint64_t m = __ballot(y == c);
        if (y == c) rank = __popcll(m & ((1ull << lane) - 1));
        if (lane == 0) cnt[a][c] = __popcll(m);
    }
    for (int i = t; i < kWideWaves * kWideRows; i += kChainBlock) (&o.src[0][0])[i] = kNoSample;
    for (int i = t; i < kSubs * kChainBlock; i += kChainBlock) (&o.row[0][0])[i] = 0xFFFF;
    for (int i = t; i < kWideWaves * kSub; i += kChainBlock) (&o.to[0][0])[i] = (uint16_t)(zero + 1);
    __syncthreads();
    if (a == 0) {   // a lane to a list
        const int j = lane / C, c = lane % C;
        int groups = 0;
        if (lane < lists)
            for (int i = 0; i <= j; ++i) groups += cnt[i][c];
        groups = (groups + GR - 1) / GR;
        const int end = lane_sum(groups), g0 = end - groups;
        const int per = max((__builtin_amdgcn_readlane(end, kWave - 1) + kWideWaves - 1) / kWideWaves, kSub / GR);   // groups of a wave
        const int w0 = g0 / per, w1 = groups ? (end - 1) / per : w0 - 1, runs = w1 - w0 + 1;
        const int r0 = lane_sum(runs) - runs;
        if (lane < lists) {
            first[lane] = g0;
            run[lane] = r0;
            uint16_t *sum = o.sum[c][j];
            sum[0] = (uint16_t)(runs ? r0 : zero);
            sum[1] = (uint16_t)(runs && g0 % per ? r0 - 1 : zero);   // (the run before it in the wave)
            for (int i = 2; i < 6; ++i) sum[i] = (uint16_t)(runs >= i ? r0 + i - 1 : zero);
            sum[6] = runs > 2;
            sum[7] = 0;
        }
        if (lane == 0) o.rows = per * GR;
    }
    __syncthreads();
    if (y >= 0) {
        const int per = o.rows / GR;
        int r = rank;
        for (int i = 0; i < a; ++i) r += cnt[i][y];
        for (int j = a; j < kSubs; ++j) {
            const int list = j * C + y, g = first[list] + r / GR, w = g / per, u = g % per * GR + r % GR;
            o.src[w][u] = (uint16_t)t;
            o.row[j][t] = (uint16_t)(w * kWideRows + u);
            o.to[w][g % per] = (uint16_t)(run[list] + w - first[list] / per);
        }
    }
    __syncthreads();
    for (int i = t; i < (int)(sizeof(WideOrder) / 4); i += kChainBlock)
        reinterpret_cast<uint32_t *>(out)[i] = reinterpret_cast<const uint32_t *>(&o)[i];
}

// ---- the samples' bits, dimension group by dimension group ----------------------------------------
// col[g][n] = bits 64 g .. 64 g + 63 of sample n: the steps below work on one group of all samples of a
// block, which row by row would be 8 bytes out of every 4 W (the rows step took 16 us like that, most of
// it in these loads).  Bits past D are dropped here: the products count every bit of a word.  A block
// turns 64 samples x 16 groups through LDS.  grid (sample tiles, group tiles, and where there are orders to
// write a row more: block after block of samples)
constexpr int kColGroups = 16;
template <bool WIDE>
__global__ __launch_bounds__(256) void online_columns_kernel(const uint32_t *__restrict__ hv, int64_t N, int W,
                                                             uint32_t last_mask, int G, int64_t ld,
                                                             uint64_t *__restrict__ col,
                                                             const int32_t *__restrict__ labels, int C,
                                                             WideOrder *__restrict__ order) {
    if (WIDE && (int)blockIdx.y * kColGroups >= G) {
        const int64_t n = (int64_t)blockIdx.x * kChainBlock;
        if (n < N) write_order(labels + n, (int)(N - n < kChainBlock ? N - n : kChainBlock), C, order + blockIdx.x);
        return;
    }
    __shared__ uint32_t tile[kSub][2 * kColGroups + 1];
    const int t = threadIdx.x;
    const int64_t n0 = (int64_t)blockIdx.x * kSub;
    const int g0 = blockIdx.y * kColGroups;
#pragma unroll
    for (int r = 0; r < kSub / 8; ++r) {
        const int sm = r * 8 + (t >> 5), w = 2 * g0 + (t & 31);
        const uint32_t x = (n0 + sm < N && w < W) ? hv[(n0 + sm) * W + w] : 0u;
        tile[sm][t & 31] = w == W - 1 ? x & last_mask : x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kColGroups / 4; ++i) {
        const int gg = (t >> 6) + 4 * i, sm = t & 63;
        if (g0 + gg < G)
            col[(int64_t)(g0 + gg) * ld + n0 + sm] = (uint64_t)tile[sm][2 * gg] | ((uint64_t)tile[sm][2 * gg + 1] << 32);
    }
}

// ---- products of the samples of a block ---------------------------------------------------------
// grid (pair (a, b) of sub-blocks, then the pairs of a block with the next one if they are wanted, block).  <s_n, s_m> = D - 2 popcount(h_n ^ h_m) is stored as
// (D >> 1) - popcount, which fits 16 bits up to D = 65535.  popcount(h_n ^ h_m) = |h_n| + |h_m| - 2 <h_n, h_m>,
// the last term a product of 0/1 vectors on 4-bit floats: a nibble with one bit set is worth 0.5, 1 or 2,
// so the bits stay where they are in one operand and carry the reciprocal in the other (search_mfma.hip
// tells the whole of it); a step is 64 dimensions, a word per lane.  The eight waves split the dimensions
// and add up 64 x 64 whole numbers in LDS.  7352 samples at D = 10000: XOR and popcount on the
// vector unit took 59 us, this 15.
constexpr int kGramWaves = 8, kGramPitch = kSub + 8;   // (the two halves of a wave add to different banks)
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

enum class Products { kTiles, kWide, kStrips };   // for online_chain_kernel, online_wide_kernel, online_spread_kernel

template <Products FOR>
__global__ __launch_bounds__(kGramWaves *kWave) void online_gram_kernel(const uint64_t *__restrict__ col, int64_t ld,
                                                                        int64_t N, int D, int G, int block,
                                                                        int16_t *__restrict__ gram,
                                                                        const WideOrder *__restrict__ order,
                                                                        int16_t *__restrict__ image, int16_t *__restrict__ pairs) {
    __shared__ int sum[kSub][kGramPitch];
    __shared__ int ones[2][kSub];
    constexpr bool WIDE = FOR == Products::kWide;
    const bool pair = FOR != Products::kStrips && (int)blockIdx.x >= kTiles;   // sub-block a of this block, b of the next one
    int a, b = 0;
    if (pair) {
        a = ((int)blockIdx.x - kTiles) / kSubs;
        b = ((int)blockIdx.x - kTiles) % kSubs;
    } else {
        while ((b + 1) * (b + 2) / 2 <= (int)blockIdx.x) ++b;
        a = (int)blockIdx.x - b * (b + 1) / 2;
    }
    const int64_t n0 = (int64_t)blockIdx.y * block, m0 = n0 + (pair ? block : 0);   // first sample of the rows' block, of the columns'
    const int nb = (int)(N - m0 < block ? N - m0 : block);
    if (b * kSub >= nb) return;
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t >> 6;
    const int r = lane & 31, half = lane >> 5;   // this lane's sample of a tile of 32, and its word of a group
    for (int i = t; i < kSub * kGramPitch; i += kGramWaves * kWave) (&sum[0][0])[i] = 0;
    if (t < 2 * kSub) (&ones[0][0])[t] = 0;
    const uint32_t *src[4];   // rows a 64 + r, + 32; columns b 64 + r, + 32
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = (i < 2 ? a : b) * kSub + 32 * (i & 1) + r;
        src[i] = reinterpret_cast<const uint32_t *>(col + (i < 2 ? n0 : m0) + (pair && i < 2 ? n : min(n, nb - 1))) + half;   // (a block with a next one is full; what is past it nobody asks for)
    }
    v16f dot[2][2] = {};
    int pop[4] = {0, 0, 0, 0};
    constexpr int U = 4;   // groups a trip; those past the last read as zeros
    for (int g0 = wave; g0 < G; g0 += U * kGramWaves) {
        uint32_t x[U][4];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[k][i] = src[i][2 * (int64_t)min(g0 + k * kGramWaves, G - 1) * ld];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            v8i op[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[k][i] = g0 + k * kGramWaves < G ? x[k][i] : 0u;
                pop[i] += __popc(x[k][i]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t u = x[k][i], v = x[k][2 + i];
                op[i] = v8i{(int)(u & 0x11111111u), (int)(u & 0x22222222u), (int)(u & 0x44444444u),
                            (int)((u >> 1) & 0x44444444u), 0, 0, 0, 0};
                op[2 + i] = v8i{(int)((v << 2) & 0x44444444u), (int)(v & 0x22222222u), (int)((v >> 2) & 0x11111111u),
                                (int)((v >> 3) & 0x11111111u), 0, 0, 0, 0};
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    dot[i][j] =
                        __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(op[i], op[2 + j], dot[i][j], 4, 4, 0, 0, 0, 0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) atomicAdd(&ones[i >> 1][32 * (i & 1) + r], pop[i]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < 16; ++k)   // register k: row 8 (k / 4) + 4 half + k % 4, column r
                atomicAdd(&sum[32 * i + 8 * (k / 4) + 4 * half + k % 4][32 * j + r], (int)dot[i][j][k]);
    __syncthreads();
    if constexpr (FOR == Products::kStrips) {   // eight of a row to a thread: 16 samples' columns after one another, by rows
        static_assert(kTile == 8 * kGramWaves * kWave, "a thread to eight products");
        const int u = t >> 3, v = 8 * (t & 7), n = a * kSub + u, strip = (b * kSub + v) / kStripCols;
        u32x4 out;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int lo = (D >> 1) - ones[0][u] - ones[1][v + 2 * k] + 2 * sum[u][v + 2 * k];
            const int hi = (D >> 1) - ones[0][u] - ones[1][v + 2 * k + 1] + 2 * sum[u][v + 2 * k + 1];
            out[k] = (uint32_t)(uint16_t)lo | (uint32_t)hi << 16;
        }
        if (n < kStripCols * (strip + 1))
            *reinterpret_cast<u32x4 *>(gram + (int64_t)blockIdx.y * kSpanProducts + strip_start(strip) + n * kStripCols + (v & 8)) = out;
        return;
    }
    int16_t *out = pair ? pairs + ((int64_t)blockIdx.y * kSubs * kSubs + ((int)blockIdx.x - kTiles)) * kTile
                        : gram + ((int64_t)blockIdx.y * kTiles + blockIdx.x) * kTile;
    for (int i = t; i < kTile; i += kGramWaves * kWave) {
        const int u = i / kSub, v = i % kSub;
        const int half = (D >> 1) - ones[0][u] - ones[1][v] + 2 * sum[u][v];
        if (WIDE && !pair) {   // for online_wide_kernel the whole product (D <= 32767) where it counts, and it in the row that holds it
            const int whole = a < b || u < v ? 2 * half + (D & 1) : 0, row = order[blockIdx.y].row[b][a * kSub + u];
            out[i] = (int16_t)whole;
            if (row != 0xFFFF) image[(int64_t)blockIdx.y * kWideImage + wide_place(row, v)] = (int16_t)whole;
        } else {
            out[i] = (int16_t)half;
        }
    }
}

// ---- dot products against the rows at the block's start -----------------------------------------
// grid (slices of the dimensions and, where wanted, the block before; tiles of 16 samples; of 16 classes), 8 waves a block that
// split the slice.  On the matrix cores in fp64: their rate equals the vector unit's on this chip, but
// the sum over the dimensions comes with the instruction, where the vector form spends a cross-lane
// sum per (sample, class).  Any assignment of dimensions to the instruction's K positions will
// do as long as both operands agree: lane 16 q + i takes dimensions 16 q .. 16 q + 15 of a group of
// 64, so that it loads 64 consecutive bytes of row i and 16 bits of sample i.  Output
// part[slice][class][sample].
constexpr int kDotWaves = 8;
typedef double f64x4 __attribute__((ext_vector_type(4)));

// One more slice where the rows do not yet hold the updates of the block before: what those add to 16 samples'
// products, from the products of samples and that block's weights (lane 16 q + i: sample i, one of four samples before).
__device__ __forceinline__ f64x4 add_block_before(const int16_t *__restrict__ pairs, const OnlineWeight *__restrict__ recs, int before, int D, double *lds) {
    static_assert(kDotWaves * kWave == 2 * kChainBlock, "a thread to half a row of 16");
    int16_t(*g)[16] = reinterpret_cast<int16_t(*)[16]>(lds);                 // 8 KB
    OnlineWeight *r = reinterpret_cast<OnlineWeight *>(lds + 1024);          // 4 KB
    const int t = threadIdx.x, n0 = t >> 1, b = blockIdx.y / 4, v = 16 * (blockIdx.y % 4) + 8 * (t & 1);
    *reinterpret_cast<u32x4 *>(&g[n0][8 * (t & 1)]) =
        *reinterpret_cast<const u32x4 *>(pairs + (((n0 / kSub) * kSubs + b) * kSub + n0 % kSub) * kSub + v);
    if (t < kChainBlock) r[t] = t < before ? recs[t] : OnlineWeight{-1, -1, 0.0f, 0.0f};
    __syncthreads();
    const int q = (t & (kWave - 1)) >> 4, i = t & 15, c = blockIdx.z * 16 + i;
    f64x4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kChainBlock / kDotWaves / 4; ++s) {
        const int n = (t / kWave) * (kChainBlock / kDotWaves) + 4 * s + q;
        const OnlineWeight w = r[n];
        const float k = w.y == c ? w.w_y : w.pred == c ? -w.w_p : 0.0f;
        sum = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(2 * (int)g[n][i] + (D & 1)), (double)k, sum, 0, 0, 0);
    }
    __syncthreads();
    return sum;
}

__global__ __launch_bounds__(kDotWaves *kWave) void online_dots_kernel(const uint64_t *__restrict__ col,
                                                                       int64_t ld, int nb,
                                                                       const float *__restrict__ acc, int D, int C,
                                                                       int slice, int slices, const int16_t *__restrict__ pairs,
                                                                       const OnlineWeight *__restrict__ recs, int before,
                                                                       double *__restrict__ part) {
    __shared__ __align__(16) double red[kDotWaves][256];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int q = lane >> 4, i = lane & 15;
    int n = blockIdx.y * 16 + i;
    n = n < nb ? n : nb - 1;
    const int c = blockIdx.z * 16 + i;
    const uint16_t *h = reinterpret_cast<const uint16_t *>(col) + 4 * (int64_t)n + q;   // this lane's 16 bits of a group
    const float *row = acc + (int64_t)(c < C ? c : C - 1) * D;
    const int share = slice / kDotWaves;   // a multiple of 64
    const int lo = blockIdx.x * slice + wave * share;
    const int hi = lo + share < D ? lo + share : D;
    f64x4 sum = {0.0, 0.0, 0.0, 0.0};
    if ((int)blockIdx.x == slices) sum = add_block_before(pairs, recs, before, D, &red[0][0]);   // (lo is past D)
    for (int d0 = lo; d0 < hi; d0 += kWave) {
        const int d = d0 + 16 * q;
        const uint32_t inv = ~(uint32_t)h[(int64_t)(d0 >> 6) * ld * 4];   // bit k: the sign of dimension d + k
        float x[16];
        if (d + 16 <= D) {
            __builtin_memcpy(x, row + d, sizeof(x));
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float v = row[d + k < D ? d + k : D - 1];
                x[k] = d + k < D ? v : 0.0f;
            }
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int hi32 = (int)(((inv << (31 - k)) & 0x80000000u) | 0x3FF00000u);
            sum = __builtin_amdgcn_mfma_f64_16x16x4f64(__hiloint2double(hi32, 0), (double)x[k], sum, 0, 0, 0);
        }
    }
    // register r of lane 16 q + i: sample 4 r + q, class i
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(4 * r + q) * 16 + i] = sum[r];
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 256) {
        const int cc = blockIdx.z * 16 + (t >> 4), m = blockIdx.y * 16 + (t & 15);
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kDotWaves; ++w) s += red[w][(t & 15) * 16 + (t >> 4)];
        if (cc < C) part[((int64_t)blockIdx.x * C + cc) * kChainBlock + m] = s;
    }
}

// ---- the rows ------------------------------------------------------------------------------------
// A block per group of 64 dimensions, waves deal the classes among them.  A lane keeps one element of
// a row in a register and takes the updates that name its class in sample order: the listed samples'
// weight and 64 bits come by lane reads, so nothing in the loop waits for memory.  Per sample one fp32
// add (the method's rounding); in batches an fp64 sum per batch and one rounding.
template <bool BATCH>
__device__ __forceinline__ void update_rows(int g, const uint64_t *__restrict__ col, int64_t ld, int nb, int batch,
                                            const OnlineWeight *__restrict__ recs, float *acc, int D, int C, int G,
                                            double *__restrict__ normpart) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int d = g * kWave + lane;
    OnlineWeight rec[kSubs];
    uint64_t bits[kSubs];
#pragma unroll
    for (int j = 0; j < kSubs; ++j) {
        const int n = min(j * kSub + lane, nb - 1);
        rec[j] = recs[n];
        bits[j] = col[(int64_t)g * ld + n];
    }
    for (int c = wave; c < C; c += nw) {
        float a = d < D ? acc[(int64_t)c * D + d] : 0.0f;
        double delta = 0.0;
        int end = batch;   // first sample of the next batch
#pragma unroll
        for (int j = 0; j < kSubs; ++j) {
            const OnlineWeight r = rec[j];
            const int lo = (int)(uint32_t)bits[j], hi = (int)(uint32_t)(bits[j] >> 32);
            const float w = r.y == c ? r.w_y : r.pred == c ? -r.w_p : 0.0f;
            uint64_t list = __ballot(w != 0.0f && j * kSub + lane < nb);
            while (list) {
                constexpr int U = 4;   // entries at a time; past the list's end weight 0
                float x[U];
                int n[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = list ? __builtin_ctzll(list) : 0;
                    const float v = list ? lane_f32(w, i) : 0.0f;
                    n[u] = list ? j * kSub + i : 0;
                    const uint64_t mask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(lo, i) |
                                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, i) << 32;
                    x[u] = __builtin_amdgcn_inverse_ballot_w64(mask) ? v : -v;   // (waits for the lane reads; inline assembly would not)
                    list &= list - 1;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if constexpr (BATCH) {
                        if (n[u] >= end) {   // uniform
                            a = (float)((double)a + delta);
                            delta = 0.0;
                            end = (n[u] / batch + 1) * batch;
                        }
                        delta += (double)x[u];
                    } else {
                        a = __fadd_rn(a, x[u]);
                    }
                }
            }
        }
        if (BATCH) a = (float)((double)a + delta);
        double q = 0.0;
        if (d < D) {
            acc[(int64_t)c * D + d] = a;
            q = (double)a * (double)a;
        }
        q = lane_prefix(q);
        if (lane == kWave - 1) normpart[(int64_t)c * G + g] = q;
    }
}

// grid (groups)
template <bool BATCH>
__global__ __launch_bounds__(kChainMaxWaves *kWave) void online_rows_kernel(
    const uint64_t *__restrict__ col, int64_t ld, int nb, int batch, const OnlineWeight *__restrict__ recs, float *acc,
    int D, int C, int G, double *__restrict__ normpart) {
    update_rows<BATCH>((int)blockIdx.x, col, ld, nb, batch, recs, acc, D, C, G, normpart);
}

// What a chain's launch needs to run the row updates of the block before beside it, a workgroup to a group of dimensions.
struct BlockBefore {
    const uint64_t *col;
    int64_t ld;
    int nb;
    const OnlineWeight *recs;
    float *acc;
    double *normpart;
};

// ---- the chain -----------------------------------------------------------------------------------
// The product of samples n < m from a block's tiles, which hold them whole or as online_gram_kernel's halves.
struct TileProduct {
    static constexpr bool kPanels = false;
    const int16_t *prod;
    int odd;
    bool halves;
    __device__ int operator()(int n, int m) const {
        const int b = m / kSub, g = prod[b * (b + 1) / 2 * kTile + n * kSub + m % kSub];
        return halves ? 2 * g + odd : g;
    }
};

// What walk_subs keeps in LDS.
template <int CPW, int WAVES>
struct ChainShared {
    double best[2][WAVES][kSub];
    double cosy[2][kSub];
    int pred[CPW > 1 ? 2 : 1][CPW > 1 ? WAVES : 1][kSub];
    OnlineWeight rec[kChainBlock];
    uint2 list[WAVES][kChainBlock];   // a wave's own: weight and place of the samples that name its class
};

// One workgroup; wave w has classes w CPW .. w CPW + CPW - 1, lane m of it sample m of the sub-block.
//
// Sub-block after sub-block: the samples' weights k_n,c (nonzero for the label's class and a wrong
// prediction's) are found as the fixed point of
//     dot_m,c  = D0_m,c + sum over n < m of k_n,c <s_n, s_m>
//     |acc_c|^2 before m = its value at the sub-block's start + sum over n < m of 2 k_n,c dot_n,c + k_n,c^2 D
//     cosines, prediction, k_m,.
// by plain iteration from k = 0.  It is triangular - pass t leaves the first t samples final - so the
// fixed point is unique, is what the walk sample by sample gives, and at most 64 passes reach it;
// because one sample moves the cosines of the others little, four or five do (the last one only
// finds that no weight changed in any bit), 8 to 18 in the first few sub-blocks of a zero model.  A pass
// costs about two samples of a walk.  In batches (BATCH) only samples of earlier batches count
// for dot and norm of a sample; the number of batch starts in a sub-block bounds the passes.
//
// What bounds it is latency, so: everything that comes from memory is asked for at the start, by
// sixteen waves (those without classes leave then); a wave sums over the samples that name its class
// only (a ballot lists them) and keeps their products in registers from pass to pass, for as
// long as the list is the same; the best cosine of each wave meets the others' in LDS, where every wave
// takes the same decision for all 64 samples: one barrier a pass (two LDS areas in turn).
//
// Rows or weights that are infinite or no numbers: the passes add samples that do not count with factor
// zero, which is no longer nothing then, and the order of the classes matters to a comparison.  A block that
// starts from such rows is walked sample by sample (walk_block), and so is every block if the learning rate
// could make a weight overflow; else a weight, at most 2 or twice the rate, stays finite.
//
// HALVES: the tiles are what online_gram_kernel leaves for this kernel, else for online_wide_kernel.  WARM: the passes of
// a sub-block begin from the weights in s.rec, not from zero (they end in the same place).  `start`: dot products against
// the rows at the block's start (used up).  `norm`: squared norms there, then at its end.
template <int CPW, bool BATCH, bool HALVES, bool WARM, int WAVES>
__device__ __forceinline__ void walk_subs(const int16_t *prod, int nb, int batch, int C, int D, float lr, double inv_root_d,
                                          int (&label)[kSubs], double (&start)[CPW][kSubs], double (&norm)[CPW], ChainShared<CPW, WAVES> &s,
                                          OnlineWeight *__restrict__ out) {
    constexpr int kKept = CPW == 1 || WAVES <= kWideWaves ? 24 : CPW == 2 ? 12 : 4;   // list entries of a class whose products stay in registers
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int subs = (nb + kSub - 1) / kSub;
    const int used = (C + CPW - 1) / CPW;   // waves that have classes
    const int odd = D & 1;
    const double dd = (double)D;
    auto whole = [&](int16_t g) { return HALVES ? 2 * (int)g + odd : (int)g; };

    // adds w_i <s_i, s_lane> over the listed samples i < lane of the diagonal tile to `all`, and to `some` where i < lim
    auto walk = [&](uint64_t list, double w, const int16_t *tile, int lim, double &all, double &some) {
        constexpr int U = 8;   // entries at a time; past the list's end weight 0
        while (list) {
            int at[U], g[U];
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                at[u] = (__ffsll((long long)list) - 1) & (kSub - 1);
                const double x = lane_f64(w, at[u]);
                v[u] = list ? x : 0.0;
                list &= list - 1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) g[u] = whole(tile[at[u] * kSub + lane]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (BATCH) some = fma(v[u], (double)(at[u] < lim ? g[u] : 0), some);
                all = fma(v[u], (double)(at[u] < lane ? g[u] : 0), all);
            }
        }
    };

    double nrm[CPW], nrm_fb[CPW];
#pragma unroll
    for (int k = 0; k < CPW; ++k) nrm[k] = nrm_fb[k] = norm[k];
    int buf = 0;
    for (int j = 0; j < subs; ++j) {
        const int m0 = j * kSub, m = m0 + lane;
        int y = label[0];
        const int fb = BATCH ? m / batch * batch : m;   // first sample that does not count for this one
        int passes = kSub;
        if (BATCH) passes = 1 + (m0 + kSub - 1) / batch - m0 / batch;
        double d0[CPW], d0_all[CPW];
#pragma unroll
        for (int k = 0; k < CPW; ++k) d0[k] = d0_all[k] = start[k][0];
#pragma unroll
        for (int i = 0; i + 1 < kSubs; ++i) {   // the next sub-block's move up
            label[i] = label[i + 1];
#pragma unroll
            for (int k = 0; k < CPW; ++k) start[k][i] = start[k][i + 1];
        }
        // What the sub-blocks before this one add: their entries of the class side by side in the
        // wave's own list, then eight at a time (every lane reads the same entry and its own product).
        if (j > 0) {
            const int16_t *tiles = prod + j * (j + 1) / 2 * kTile + lane;   // row n of tile a is row a 64 + n here
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                const int c = wave * CPW + k;
                int entries = 0;
                for (int a = 0; a < j; ++a) {
                    const OnlineWeight r = s.rec[a * kSub + lane];
                    const float w = r.y == c ? r.w_y : r.pred == c ? -r.w_p : 0.0f;
                    const uint64_t list = __ballot(w != 0.0f);
                    const int at = entries + __popcll(list & ((1ull << lane) - 1));
                    if (w != 0.0f) s.list[wave][at] = make_uint2(__float_as_uint(w), (uint32_t)(a * kSub + lane));
                    entries += __popcll(list);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                for (int e = 0; e < entries; e += 8) {
                    uint2 x[8];
                    int g[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = s.list[wave][min(e + u, entries - 1)];
#pragma unroll
                    for (int u = 0; u < 8; ++u) g[u] = whole(tiles[x[u].y * kSub]);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double v = e + u < entries ? (double)__uint_as_float(x[u].x) : 0.0;
                        if (BATCH) d0[k] = fma(v, (double)((int)x[u].y < fb ? g[u] : 0), d0[k]);
                        d0_all[k] = fma(v, (double)g[u], d0_all[k]);
                    }
                }
                if (!BATCH) d0[k] = d0_all[k];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();   // the list is rewritten for the next class
            }
        }
        const int16_t *diag = prod + (j * (j + 1) / 2 + j) * kTile;
        float wy = 0.0f, wp = 0.0f;
        int pred = -1;
        if constexpr (WARM) {
            const OnlineWeight r = s.rec[m];
            wy = r.w_y;
            wp = r.w_p;
            pred = r.pred;
        }
        double before[CPW] = {}, total[CPW] = {};   // what the sub-block adds to the squared norms, before each sample and in all
        uint64_t known[CPW] = {};      // the list whose first products are kept: entry u is sample at[][u]
        int at[CPW][kKept] = {};
        double kept[CPW][kKept] = {};
        auto norms = [&](int k, double &dot) {
            const int c = wave * CPW + k;
            const float wf = y == c ? wy : pred == c ? -wp : 0.0f;
            const double w = (double)wf;
            const uint64_t list = __ballot(wf != 0.0f);
            const int entries = __popcll(list);
            double all = d0_all[k], all1 = 0.0;
            dot = d0[k];
            uint64_t rest = list;
            const bool renew = list != known[k];
            known[k] = list;
#pragma unroll
            for (int q = 0; q < kKept; q += 4) {
                if (entries > q) {   // uniform, like renew
                    if (renew) {
#pragma unroll
                        for (int u = q; u < q + 4; ++u) {
                            at[k][u] = (__ffsll((long long)rest) - 1) & (kSub - 1);   // past the end the last sample: nobody comes after it
                            rest &= rest - 1;
                        }
#pragma unroll
                        for (int u = q; u < q + 4; ++u) {
                            const int g = whole(diag[at[k][u] * kSub + lane]);
                            kept[k][u] = (double)(at[k][u] < lane ? g : 0);
                        }
                    }
#pragma unroll
                    for (int u = q; u < q + 4; ++u) {
                        const double v = lane_f64(w, at[k][u]);
                        if (BATCH) dot = fma(v, at[k][u] < fb - m0 ? kept[k][u] : 0.0, dot);
                        if (u & 1)
                            all1 = fma(v, kept[k][u], all1);
                        else
                            all = fma(v, kept[k][u], all);
                    }
                }
            }
            all += all1;
            if (entries > kKept) {
                rest = list;
#pragma unroll
                for (int u = 0; u < kKept; ++u) rest &= rest - 1;
                walk(rest, w, diag, fb - m0, all, dot);
            }
            if (!BATCH) dot = all;
            const double sum = lane_prefix(wf != 0.0f ? w * (2.0 * all + w * dd) : 0.0);
            before[k] = lane_before(sum);
            total[k] = lane_f64(sum, kWave - 1);
        };
        bool settled = false;
        for (int pass = 1; !settled && pass <= passes; ++pass) {
            double best = -4.0;
            int arg = 0;
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                const int c = wave * CPW + k;
                if (c < C) {
                    double dot;
                    norms(k, dot);
                    double nn = nrm[k] + before[k];
                    if (BATCH) nn = fb >= m0 ? nrm[k] + __shfl(before[k], fb - m0, kWave) : nrm_fb[k];
                    const double cs = nn > 0.0 ? dot * refined_rsq(nn) * inv_root_d : 0.0;
                    if (y == c) s.cosy[buf][lane] = cs;
                    if (cs > best) {
                        best = cs;
                        arg = c;
                    }
                }
            }
            s.best[buf][wave][lane] = best;
            if constexpr (CPW > 1) s.pred[buf][wave][lane] = arg;
            __syncthreads();
            const double cos_y = s.cosy[buf][lane];
            best = -4.0;
            arg = 0;
            for (int w0 = 0; w0 < used; w0 += 8) {   // eight waves' bests at a time (the last one repeats: it cannot win twice)
                double v[8];
                int p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    p[u] = min(w0 + u, used - 1);
                    v[u] = s.best[buf][p[u]][lane];
                    if constexpr (CPW > 1) p[u] = s.pred[buf][p[u]][lane];
                }
                const double top = fmax(fmax(fmax(v[0], v[1]), fmax(v[2], v[3])), fmax(fmax(v[4], v[5]), fmax(v[6], v[7])));
                int first = p[7];
#pragma unroll
                for (int u = 6; u >= 0; --u) first = v[u] == top ? p[u] : first;
                if (top > best) {
                    best = top;
                    arg = first;
                }
            }
            float wy1 = 0.0f, wp1 = 0.0f;
            int pred1 = -1;
            if (y >= 0) {
                wy1 = (float)(1.0 - cos_y);
                if (arg != y) {
                    pred1 = arg;
                    wp1 = (float)((double)lr * (1.0 - best));
                }
            }
            settled = __ballot(wy1 != wy || wp1 != wp || pred1 != pred) == 0;
            wy = wy1;
            wp = wp1;
            pred = pred1;
            buf ^= 1;
        }
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            double dot;
            if (!settled) norms(k, dot);   // the last pass used the weights of the one before
            if (BATCH) {
                const int next = (m0 + kSub) / batch * batch;   // where the next sub-block's first batch begins
                if (next >= m0 && next < m0 + kSub) nrm_fb[k] = nrm[k] + lane_f64(before[k], next - m0);
            }
            nrm[k] += total[k];
            if (BATCH && (m0 + kSub) % batch == 0) nrm_fb[k] = nrm[k];
        }
        if (wave == 0) {
            const OnlineWeight r = {y, pred, wy, wp};
            s.rec[m] = r;
            if (m < nb) out[m] = r;
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < CPW; ++k) norm[k] = nrm[k];
}

template <int CPW, bool BATCH>
__global__ __launch_bounds__(kChainMaxWaves *kWave) void online_chain_kernel(
    const int16_t *__restrict__ gram, const double *__restrict__ part, int slices, int nb, int batch,
    const int32_t *__restrict__ labels, const double *__restrict__ normpart, int G, int C, int D, float lr,
    double inv_root_d, OnlineWeight *__restrict__ out, double *grown, bool ahead, BlockBefore before_it) {
    if (blockIdx.x) {
        update_rows<BATCH>((int)blockIdx.x - 1, before_it.col, before_it.ld, before_it.nb, batch, before_it.recs, before_it.acc, D, C, G,
                           before_it.normpart);
        return;
    }
    extern __shared__ __align__(16) int16_t prod[];   // the tiles of the block's sub-blocks
    __shared__ ChainShared<CPW, kChainMaxWaves> s;
    __shared__ int s_odd[kChainMaxWaves];   // a wave's rows are not finite
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int subs = (nb + kSub - 1) / kSub;
    const int used = (C + CPW - 1) / CPW;   // waves that have classes
    constexpr int kCopies = kTiles * kTile * 2 / 16 / (kChainMaxWaves * kWave);
    uint4 copy[kCopies];
    const int units = subs * (subs + 1) / 2 * (kTile * 2 / 16);
#pragma unroll
    for (int u = 0; u < kCopies; ++u)
        copy[u] = reinterpret_cast<const uint4 *>(gram)[min(tid + u * kChainMaxWaves * kWave, units - 1)];
    double nrm[CPW];   // squared norms before the sub-block; and where the batch that runs into it began
    double at_start[CPW];           // before the block
    double start[CPW][kSubs];       // dot products against the rows at the block's start
    int label[kSubs];
    bool odd_rows = false;
#pragma unroll
    for (int j = 0; j < kSubs; ++j) {
        const int y = labels[min(j * kSub + lane, nb - 1)];
        label[j] = j * kSub + lane < nb && y >= 0 && y < C ? y : -1;
    }
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = wave * CPW + k;
        nrm[k] = at_start[k] = 0.0;
#pragma unroll
        for (int j = 0; j < kSubs; ++j) start[k][j] = 0.0;
        if (c < C) {
            double sum = 0.0;
            for (int g0 = 0; g0 < G; g0 += 4 * kWave) {
                double p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = normpart[(int64_t)c * G + min(g0 + i * kWave + lane, G - 1)];
#pragma unroll
                for (int i = 0; i < 4; ++i) sum += g0 + i * kWave + lane < G ? p[i] : 0.0;
            }
            double x[kSlices + 1][kSubs];
#pragma unroll
            for (int i = 0; i <= kSlices; ++i)
#pragma unroll
                for (int j = 0; j < kSubs; ++j)
                    x[i][j] = part[((int64_t)min(i, slices - 1) * C + c) * kChainBlock + j * kSub + lane];
#pragma unroll
            for (int i = 0; i <= kSlices; ++i)
#pragma unroll
                for (int j = 0; j < kSubs; ++j) start[k][j] += i < slices ? x[i][j] : 0.0;
            nrm[k] = lane_f64(lane_prefix(sum), kWave - 1) + (ahead ? grown[c] : 0.0);
            at_start[k] = nrm[k];
            odd_rows |= !(nrm[k] < __builtin_inf());
        }
    }
    if (lane == 0) s_odd[wave] = odd_rows;
#pragma unroll
    for (int u = 0; u < kCopies; ++u)
        if (tid + u * kChainMaxWaves * kWave < units)
            reinterpret_cast<uint4 *>(prod)[tid + u * kChainMaxWaves * kWave] = copy[u];
    __syncthreads();
    if (wave >= used) return;   // (an ended wave takes no part in later barriers)
    if (__builtin_expect(__ballot(lane < used && s_odd[lane]) != 0 || !(fabsf(lr) < kTameRate), 0)) {   // the same in every wave
        walk_block<CPW, BATCH>(TileProduct{prod, D & 1, true}, part, kChainBlock, slices, nb, batch, labels, normpart, ahead ? grown : nullptr, grown, G, C, D, lr,
                               inv_root_d, s.rec, s.cosy[0]);
        for (int n = tid; n < nb; n += used * kWave) out[n] = s.rec[n];
        return;
    }
    walk_subs<CPW, BATCH, true, false, kChainMaxWaves>(prod, nb, batch, C, D, lr, inv_root_d, label, start, nrm, s, out);
#pragma unroll
    for (int k = 0; k < CPW; ++k)
        if (lane == 0 && wave * CPW + k < C) grown[wave * CPW + k] = nrm[k] - at_start[k];
}

// ---- the chain of a whole block at once ------------------------------------------------------------
// One workgroup, per sample (not in batches), up to 16 classes.  The same fixed point as in online_chain_kernel, over all
// samples of a block together: four or five passes settle 256 samples where the sub-blocks one after another take
// sixteen (from rows of zeros nine to twenty where those take 24 to 37; what predictions that are wrong make of it is told at
// kWideMostWrong).  7352 samples x 3 epochs, 6 classes, D = 10000: 29.2 us a block -> 16.4 with the rows of the block before
// beside it, of which five are spent before the first pass.
//
// A pass takes the block's whole triangle of products, 640 rows of 64 (source sample x targets of a sub-block).  They
// stay in registers for all passes, as fp64: eight waves of up to 92 rows, listed sub-block after sub-block and class
// after class (write_order), each class filled up to whole groups of GR rows.  A weight reaches all lanes with the
// multiply-add itself (a row-wise broadcast of its 64-bit operand: no lane read), and after every group the running sum
// goes to its class's place in LDS, so that there is no branch in it: a class's sum is the difference of two places.  A
// jump costs 20 clocks, as much as four rows; a branch where a class ends took 280 a group, this way 70.  Class c
// belongs to wave c % 8, whose lanes form its dot products, the squared norms before each sample (prefix sums) and the
// cosines of all four sub-blocks; wave j decides for the samples of sub-block j.  Three barriers, 5600 clocks a pass:
// rows 1600, cosines 1800 to 2600, decisions 1250.  A class wrongly predicted for a sample takes that sample's products
// from LDS, as the list changes from pass to pass.
//
// All of it has to stay within 256 registers: a kernel that spills waits 4 us longer for its launch.

// Where about half the predictions are wrong a block needs 30 to 70 passes, nearly as many as its sub-blocks together,
// and each costs up to twice as much (the lists of wrong ones).  From more wrong ones than this of 64 in half its
// sub-blocks, or after so many passes, a block is finished by walk_subs, from the weights as they are.  Microseconds for
// 2000 samples, whole passes only / this / online_chain_kernel:
//   labels at random, samples 10 % from their prototype, D = 10000: 2 classes 2652 1812 1867, 3 3117 1736 1782,
//   6 1667 1036 1073, 8 1297 834 846, 10 1462 1016 885, 12 1215 941 847, 16 1168 844 843; half of them at random, 30 %:
//   2 406 409 640, 3 384 386 528, 6 512 480 486, 8 547 492 481, 10 664 663 599, 16 748 640 662; right labels, 45 %, D = 1000:
//   3 311 311 454, 6 416 377 436, 12 655 596 552, 16 827 659 630
// (Nine to twelve classes are two a wave on five or six waves here, where the other kernel has a wave for each.)  24, 28, 36
// and 44 instead of 32, over 56 such calls for each of 2 to 16 classes: in the mean within 1 % of this, and 2 % and 5 % slower.
constexpr int kWideMostWrong = 32, kWidePasses = 20;

template <int CPW, int GR>
__global__ __launch_bounds__(kWideWaves *kWave) void online_wide_kernel(
    const int16_t *__restrict__ gram, const int16_t *__restrict__ image, const WideOrder *__restrict__ order,
    double *part, int slices, int nb, const int32_t *__restrict__ labels,
    const double *__restrict__ normpart, int G, int C, int D, float lr, double inv_root_d, OnlineWeight *__restrict__ out,
    double *grown, bool ahead, BlockBefore before) {
    if (blockIdx.x) {
        update_rows<false>((int)blockIdx.x - 1, before.col, before.ld, before.nb, 1, before.recs, before.acc, D, C, G, before.normpart);
        return;
    }
    extern __shared__ __align__(16) int16_t prod[];   // the tiles of the block's sub-blocks, then s_place [wide_places], s_cos [4 C], s_start [4 C]
    __shared__ double s_wy[kChainBlock + 2];
    __shared__ uint2 s_wrong[kChainBlock];   // class wrongly predicted, or -1, and its weight
    __shared__ double s_grown[kWideClasses];   // what the block adds to a class's squared norm
    __shared__ int s_odd[kWideWaves];
    __shared__ int2 s_any[kSubs];            // of a sub-block's samples: whether a weight changed; how many predictions are wrong
    constexpr int kRows = wide_rows(GR);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int subs = (nb + kSub - 1) / kSub;
    const int tiles = subs * (subs + 1) / 2, places = wide_places(C);
    double(*s_place)[kSub] = reinterpret_cast<double(*)[kSub]>(prod + tiles * kTile);
    double(*s_cos)[kSub] = s_place + places;            // [4 c + j]
    // dot products against the rows at the block's start: in LDS, or (two classes a wave: it is full) where they came from
    double(*start)[kSub] = CPW == 1 ? s_cos + kSubs * C : reinterpret_cast<double(*)[kSub]>(part);

    // Everything from memory at once, in the order in which it is needed: 300 KB take the longer part of the time
    // before the first pass, and what the later passes need comes in during that one.
    int label[kSubs];
#pragma unroll
    for (int i = 0; i < kSubs; ++i) label[i] = labels[min(i * kSub + lane, nb - 1)];
    double p[CPW][4];
#pragma unroll
    for (int k = 0; k < CPW; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) p[k][i] = normpart[(int64_t)min(wave + k * kWideWaves, C - 1) * G + min(i * kWave + lane, G - 1)];
    constexpr int kAtOnce = 3, kThreads = kWideWaves * kWave;   // elements of part a thread has in flight, a load for each slice
    double first[kAtOnce][kSlices + 1];
    const int elements = C * kChainBlock;
    auto ask = [&](int e0, double(&v)[kAtOnce][kSlices + 1]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u)
#pragma unroll
            for (int i = 0; i <= kSlices; ++i) v[u][i] = part[(int64_t)min(i, slices - 1) * elements + min(e0 + u * kThreads, elements - 1)];
    };
    auto take = [&](int e0, const double(&v)[kAtOnce][kSlices + 1]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i <= kSlices; ++i) s += i < slices ? v[u][i] : 0.0;
            if (e0 + u * kThreads < elements) (&start[0][0])[e0 + u * kThreads] = s;
        }
    };
    ask(tid, first);
    uint4 raw[(kRows + 7) / 8];
#pragma unroll
    for (int i = 0; i < (kRows + 7) / 8; ++i)
        raw[i] = reinterpret_cast<const uint4 *>(image)[(wave * (kWideRows / 8) + i) * kSub + lane];
    uint32_t wsrc[kWideRows / 32];   // the samples whose weights this lane broadcasts, two to a register
#pragma unroll
    for (int i = 0; i < kWideRows / 32; ++i)
        wsrc[i] = (uint32_t)order->src[wave][32 * i + (lane & 15)] | (uint32_t)order->src[wave][32 * i + 16 + (lane & 15)] << 16;
    const int to = order->to[wave][lane];
    const int rows = order->rows;
    uint32_t sum_at[CPW];   // lane 8 j + i: place i of sub-block j
#pragma unroll
    for (int k = 0; k < CPW; ++k) sum_at[k] = order->sum[min(wave + k * kWideWaves, C - 1)][(lane >> 3) & (kSubs - 1)][lane & 7];
    constexpr int kCopies = kTiles * kTile * 2 / 16 / (kWideWaves * kWave);
    u32x4 copy[kCopies];
    const int units = tiles * (kTile * 2 / 16);
#pragma unroll
    for (int u = 0; u < kCopies; ++u)
        copy[u] = reinterpret_cast<const u32x4 *>(gram)[min(tid + u * kThreads, units - 1)];

    take(tid, first);
    for (int e = tid + kAtOnce * kThreads; e < elements; e += kAtOnce * kThreads) {
        ask(e, first);
        take(e, first);
    }
    bool odd_rows = false, zero_rows = true;
    uint64_t mine[CPW][kSubs];   // samples with the class's label
    double nrm[CPW];
#pragma unroll
    for (int i = 0; i < kSubs; ++i) label[i] = i * kSub + lane < nb && label[i] >= 0 && label[i] < C ? label[i] : -1;
    int y = -1;   // of the sample this lane decides for
#pragma unroll
    for (int i = 0; i < kSubs; ++i) y = wave == i ? label[i] : y;
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = wave + k * kWideWaves;
#pragma unroll
        for (int j = 0; j < kSubs; ++j) mine[k][j] = __ballot(label[j] == c);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) s += i * kWave + lane < G ? p[k][i] : 0.0;
        for (int g = 4 * kWave + lane; g < G; g += kWave) s += normpart[(int64_t)min(c, C - 1) * G + g];
        nrm[k] = lane_f64(lane_prefix(s), kWave - 1) + (ahead ? grown[min(c, C - 1)] : 0.0);
        odd_rows |= !(nrm[k] < __builtin_inf());
        zero_rows &= nrm[k] == 0.0;
    }
    if (lane == 0) s_odd[wave] = odd_rows ? 1 : zero_rows ? 0 : 2;
    if (tid < kChainBlock + 2) s_wy[tid] = 0.0;
    if (tid < kChainBlock) s_wrong[tid] = make_uint2(~0u, 0u);   // (past the last sub-block nobody decides)
    if (tid < kWideClasses) s_grown[tid] = 0.0;
    if (tid < kSubs) s_any[tid] = make_int2(0, 0);   // (past the last sub-block nobody writes)
    if (tid < kSub) s_place[places - 2][tid] = 0.0;
    __syncthreads();
    const int kind = s_odd[lane & (kWideWaves - 1)];
    const bool zero_model = __ballot(kind != 0) == 0;
    const bool strange = __ballot(kind == 1) != 0 || !(fabsf(lr) < kTameRate);

    float wy = 0.0f, wp = 0.0f;
    int pred = -1;
    bool wrong_ones = false, hard = false;
    // Predictions and weights from s_cos, after a barrier; false: no weight has changed.  (With guess, labels count as
    // predictions: rows of zeros would say class 0 of every sample.  The passes end in the same place from any start.)
    auto decide = [&](int l, bool guess) __attribute__((always_inline)) {
        if (wave < subs) {
            const double cos_y = s_cos[kSubs * max(y, 0) + wave][l];
            double best = -4.0;
            int arg = 0;
            for (int c0 = 0; c0 < C; c0 += 8) {   // eight at a time (the last one repeats: it cannot win twice)
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = s_cos[kSubs * min(c0 + u, C - 1) + wave][l];
                const double top = fmax(fmax(fmax(v[0], v[1]), fmax(v[2], v[3])), fmax(fmax(v[4], v[5]), fmax(v[6], v[7])));
                int first = 7;
#pragma unroll
                for (int u = 6; u >= 0; --u) first = v[u] == top ? u : first;
                if (top > best) {
                    best = top;
                    arg = c0 + first;
                }
            }
            float wy1 = 0.0f, wp1 = 0.0f;
            int pred1 = -1;
            if (y >= 0) {
                wy1 = (float)(1.0 - cos_y);
                if (arg != y && !guess) {
                    pred1 = arg;
                    wp1 = (float)((double)lr * (1.0 - best));
                }
            }
            const uint64_t changed = __ballot(wy1 != wy || wp1 != wp || pred1 != pred), wrong = __ballot(pred1 >= 0);
            wy = wy1;
            wp = wp1;
            pred = pred1;
            s_wy[wave * kSub + l] = (double)wy;
            s_wrong[wave * kSub + l] = make_uint2((uint32_t)pred, __float_as_uint(wp));
            if (l == 0) s_any[wave] = make_int2(changed != 0, __popcll(wrong));
        }
        __syncthreads();
        const int v = reinterpret_cast<const int *>(s_any)[l & (2 * kSubs - 1)];
        const uint64_t any = __ballot(v != 0);   // the same in every wave
        wrong_ones = (any & 0xAA) != 0;
        hard = 2 * __popcll(__ballot(v > kWideMostWrong) & 0xAA) >= subs;
        return (any & 0x55) != 0;
    };
    // the first pass: no sample of the block counts yet
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = wave + k * kWideWaves;
        const double r = nrm[k] > 0.0 ? refined_rsq(nrm[k]) * inv_root_d : 0.0;
        if (c < C) {
#pragma unroll
            for (int i = 0; i < kSubs; ++i) s_cos[kSubs * c + i][lane] = start[kSubs * c + i][lane] * r;
        }
    }
    __syncthreads();
    bool going = decide(lane, zero_model);

#pragma unroll
    for (int u = 0; u < kCopies; ++u) reinterpret_cast<u32x4 *>(prod)[min(tid + u * kThreads, units - 1)] = copy[u];
    double kept[kRows];
#pragma unroll
    for (int i = 0; i < (kRows + 7) / 8; ++i) {
        const uint32_t q[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (8 * i + u < kRows) kept[8 * i + u] = (double)(int)(int16_t)(q[u >> 1] >> (16 * (u & 1)));
    }
    if (__builtin_expect(strange, 0)) {
        __syncthreads();
        OnlineWeight *rec = reinterpret_cast<OnlineWeight *>(&s_place[0][0]);   // (4 KB of at least 7)
        walk_block<CPW, false>(TileProduct{prod, 0, false}, part, kChainBlock, CPW == 1 ? slices : 1, nb, 1, labels, normpart, ahead ? grown : nullptr, grown, G, C, D,
                               lr, inv_root_d, rec, s_wy);
        for (int n = tid; n < nb; n += kWideWaves * kWave) out[n] = rec[n];
        return;
    }
    const double dd = (double)D;
    int column[kSubs];   // first tile of a target sub-block; past the last one, of that
#pragma unroll
    for (int i = 0; i < kSubs; ++i) column[i] = min(i, subs - 1) * (min(i, subs - 1) + 1) / 2 * kTile;
    for (int pass = 1; going && !hard && pass <= kWidePasses; ++pass) {
        int l = lane;
        asm volatile("" : "+v"(l));   // (addresses are formed anew in a pass: kept over all, they would not fit the registers)
        {
            double w[kWideRows / 16];
#pragma unroll
            for (int i = 0; i < kWideRows / 16; ++i) w[i] = s_wy[wsrc[i / 2] >> (16 * (i & 1)) & 0xFFFFu];
            int at = to * (kSub * (int)sizeof(double)), used = __builtin_amdgcn_readfirstlane(rows);
            asm volatile("" : "+v"(at), "+s"(used));   // (what follows from these is not kept over the passes: a hundred scalars, which spill)
            double sum = 0.0;
            char *base = reinterpret_cast<char *>(&s_place[0][l]);
            each<kWideRows / 16>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
                if (16 * i < used)
                    each<(kRows - 16 * i < 16 ? kRows - 16 * i : 16) / GR>([&](auto q_) {
                        constexpr int g = 16 / GR * i + decltype(q_)::value;
                        add_rows<g * GR % 16, GR>(sum, w[i], kept + g * GR);
                        *reinterpret_cast<double *>(base + __builtin_amdgcn_readlane(at, g)) = sum;
                    });
            });
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = wave + k * kWideWaves;
            if (c < C) {
                double dot[kSubs], wd[kSubs];
#pragma unroll
                for (int i = 0; i < kSubs; ++i) {
                    dot[i] = start[kSubs * c + i][l];
                    const double v = s_wy[i * kSub + l];
                    wd[i] = __builtin_amdgcn_inverse_ballot_w64(mine[k][i]) ? v : 0.0;
                }
                {
#pragma unroll
                    for (int i0 = 0; i0 < kSubs; i0 += 2) {   // (two at a time: more would not fit the registers)
                        double v[2][3];
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int u = 0; u < 3; ++u) v[i][u] = s_place[__builtin_amdgcn_readlane(sum_at[k], 8 * (i0 + i) + u)][l];
#pragma unroll
                        for (int i = 0; i < 2; ++i) dot[i0 + i] += (v[i][0] - v[i][1]) + v[i][2];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (__builtin_expect(__ballot((l & 7) == 6 && l < 8 * kSubs && sum_at[k]) != 0, 0)) {
#pragma unroll
                        for (int i = 0; i < kSubs; ++i)
#pragma unroll
                            for (int u = 3; u < 6; ++u) dot[i] += s_place[__builtin_amdgcn_readlane(sum_at[k], 8 * i + u)][l];
                    }
                }
                if (wrong_ones) {
#pragma unroll
                    for (int a = 0; a < kSubs; ++a) {
                        const uint2 r = s_wrong[a * kSub + l];
                        const double wx = -(double)__uint_as_float(r.y);
                        uint64_t list = __ballot((int)r.x == c);
                        if ((int)r.x == c) wd[a] = wx;
                        while (list) {
                            constexpr int U = 4;   // samples at a time; past the list's end weight 0
                            int n[U], g[U][kSubs];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                n[u] = list ? __builtin_ctzll(list) : -1;
                                list &= list - 1;
#pragma unroll
                                for (int i = a; i < kSubs; ++i) g[u][i] = prod[column[i] + a * kTile + (n[u] & (kSub - 1)) * kSub + l];
                            }
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const double z = lane_f64(wx, n[u] & (kSub - 1)), v = n[u] >= 0 ? z : 0.0;
#pragma unroll
                                for (int i = a; i < kSubs; ++i) dot[i] = fma(v, (double)g[u][i], dot[i]);
                            }
                        }
                    }
                }
                double run[kSubs];   // what the samples up to each add to the squared norm
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kSubs; ++i) run[i] = lane_prefix(wd[i] * fma(wd[i], dd, 2.0 * dot[i]));
                double base = nrm[k];   // of the squared norm: at the sub-block's start
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kSubs; ++i) {
                    const double nn = base + lane_before(run[i]);
                    base += lane_f64(run[i], kWave - 1);
                    s_cos[kSubs * c + i][l] = nn > 0.0 ? dot[i] * refined_rsq(nn) * inv_root_d : 0.0;
                }
                if (l == 0) s_grown[c] = base - nrm[k];
            }
        }
        __syncthreads();
        going = decide(l, false);
    }
    if (__builtin_expect(!going, 1)) {
        if (wave < subs && wave * kSub + lane < nb) out[wave * kSub + lane] = OnlineWeight{y, pred, wy, wp};
        if (tid < C) grown[tid] = s_grown[tid];
        return;
    }
    // sub-block after sub-block, from the weights as they are
    double from[CPW][kSubs], norm[CPW];
#pragma unroll
    for (int k = 0; k < CPW; ++k)
        if (lane == 0 && wave + k * kWideWaves < C) s_grown[wave + k * kWideWaves] = nrm[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = min(wave * CPW + k, C - 1);
        norm[k] = s_grown[c];
#pragma unroll
        for (int i = 0; i < kSubs; ++i) from[k][i] = start[kSubs * c + i][lane];
    }
    __syncthreads();
    ChainShared<CPW, kWideWaves> &s = reinterpret_cast<ChainShared<CPW, kWideWaves> &>(s_place[0][0]);
    if (wave < subs) s.rec[wave * kSub + lane] = OnlineWeight{y, pred, wy, wp};
    __syncthreads();
    if (wave * CPW >= C) return;
#pragma unroll
    for (int i = 0; i < kSubs; ++i) label[i] = i < subs ? s.rec[i * kSub + lane].y : -1;
    walk_subs<CPW, false, false, true, kWideWaves>(prod, nb, 1, C, D, lr, inv_root_d, label, from, norm, s, out);
#pragma unroll
    for (int k = 0; k < CPW; ++k)
        if (lane == 0 && wave * CPW + k < C) grown[wave * CPW + k] = norm[k] - s_grown[wave * CPW + k];
}

// ---- host side -------------------------------------------------------------------------------------
static int chain_slice(int D) {   // dimensions of a slice: up to ten slices, whole groups of 64 per wave
    int s = (D + kSlices - 1) / kSlices;
    s = (s + kDotWaves * kWave - 1) / (kDotWaves * kWave) * (kDotWaves * kWave);
    return s;
}

// Samples whose columns are held at a time: within 64 MB.
int64_t held_samples(int G) {
    const int64_t fit = ((int64_t)64 << 20) / ((int64_t)G * (int64_t)sizeof(uint64_t)) / kSub * kSub;
    return std::min(fit, kHeldBlocks * kChainBlock);
}

void launch_columns(hdc_ctx_impl *c, const uint32_t *hv, int64_t n, int64_t ld, hipStream_t s) {
    const int G = (c->p.D + kWave - 1) / kWave;
    hipLaunchKernelGGL(online_columns_kernel<false>, dim3((unsigned)((n + kSub - 1) / kSub), (unsigned)((G + kColGroups - 1) / kColGroups)),
                       dim3(256), 0, s, hv, n, c->W, c->last_word_mask, G, ld, c->oc_col_d, nullptr, c->p.C, nullptr);
}

void launch_strips(hdc_ctx_impl *c, int64_t n, int64_t ld, int block, int16_t *strips, hipStream_t s) {
    const int subs = (int)((std::min<int64_t>(n, block) + kSub - 1) / kSub);
    hipLaunchKernelGGL(online_gram_kernel<Products::kStrips>, dim3((unsigned)(subs * (subs + 1) / 2), (unsigned)((n + block - 1) / block)),
                       dim3(kGramWaves * kWave), 0, s, c->oc_col_d, ld, n, c->p.D, (c->p.D + kWave - 1) / kWave, block, strips, nullptr,
                       nullptr, nullptr);
}

bool online_chain_takes(const hdc_ctx_impl *c) { return c->p.C <= 4 * kChainMaxWaves && c->p.D <= 65535; }

// A block of 256 samples costs as much as this many batches the other way, three launches each.  The fewer the
// classes, the longer the list of samples that name one; at two and four classes a wave the passes spill; at large
// D a batch costs more, a block hardly.  1020 samples, time of the blocks over that of the batches, at 32, 42, 51, 64
// and 85 samples a batch:
//   C = 1:  D = 1000 0.74 0.96 1.12 1.05 1.52   10000 0.71 0.95 1.03 1.01 1.39   40000 0.62 0.92 0.92 1.11 1.27
//   C = 2:  D = 1000 0.59 0.79 0.90 0.85 1.24    4000 0.57 0.75 0.84 0.85 1.17   40000 0.51 0.73 0.79 0.84 1.03
//   C = 4:  D = 1000 0.49 0.66 0.73 0.78 1.04    4000 0.48 0.63 0.72 0.76 1.02   10000 0.45 0.58 0.66 0.71 0.96
//   C = 10: D = 1000 0.37 0.53 0.59 0.60 0.86    4000 0.36 0.53 0.59 0.60 0.87   10000 0.34 0.49 0.55 0.56 0.78
//   C = 33: D = 1000 0.54 0.74 0.83 0.83 1.17    4000 0.55 0.77 0.83 0.84 1.19   10000 0.43 0.59 0.67 0.68 0.94
// The line below was drawn when a block was three launches, and is on the careful side of two: of 3128 calls it decides (1 to
// 64 classes, D = 100 to 65535, 4 to 1500 samples, batches of 1 to 85) 14 are more than 5 % faster in batches, the worst
// 1.21 times, and 194 more than 5 % faster in blocks, the worst 1.7 times.
static double batches_per_block(int C, int D) {
    if (D < 512 && C <= 10) return C == 1 ? 4.0 : C <= 4 ? 3.2 : 2.0;   // few dimensions: the passes settle sooner
    const double small = C == 1 ? 7.0 : C == 2 ? 4.7 : C <= 5 ? 3.9 : C <= 16 ? 3.05 : 3.7;
    return small / (1.0 + D / (C <= 2 ? 45e3 : C <= 5 ? 30e3 : C <= 10 ? 45e3 : 22e3));
}

// A block that is not full costs a third of a full one and its share of the rest; but a call costs two
// batches more, a last block of a few samples (260 at 85 a batch) as much as any.  (Of 723 calls of two or three batches, or
// of so few a block, 601 would be more than 5 % faster in blocks, half of them 1.2 times and more.)
bool online_chain_pays(const hdc_ctx_impl *c, int64_t N, int64_t batch) {
    if (3 * batch > kChainBlock) return false;   // (two batches a block or one: not measured)
    const int64_t block = kChainBlock / batch * batch, batches = (N + batch - 1) / batch, rest = N % block;
    const double blocks = (double)(N / block) + (rest ? 0.35 + 0.65 * (double)rest / (double)block : 0.0);
    return batches >= 2 * ((N + block - 1) / block) + 2 && (double)batches >= batches_per_block(c->p.C, c->p.D) * blocks;
}

// Per-sample calls whose blocks are walked as a whole (online_wide_kernel).  A product has to fit 16 bits; a learning rate
// that can make a weight overflow leaves the walk sample by sample, and that to the other kernel.  The first blocks of a
// zero model take more passes the more classes, and long lists of one to three classes are what the sub-blocks pay for.
// Time by sub-blocks over time of this way, samples 10 and 30 % from their prototype, every tenth label at random, D = 1000:
//   C = 1:  129 samples 1.41 1.40, 520 2.15 2.12    C = 3: 129 1.08 1.07, 520 1.20 1.25    C = 5: 200 1.02 1.15, 385 1.03 1.10
//   C = 8:  300 0.90 0.88, 520 0.94 0.97, 769 1.00 1.03    C = 12: 520 0.98 1.06, 1281 1.07 1.16    C = 16: 520 0.96 1.04, 1025 1.02 1.13,
//   1793 1.09 1.19
// and, 2000 samples, 6 classes, D = 10000: 1.42 without false labels, 1.20 with a third of them false, 1.01 with half of them or
// with labels at random; 10 classes 1.36, 1.11, 0.92, 0.89 (two classes a wave on five waves: at kWideMostWrong).
// A block costs as much whatever part of it has samples: five classes and more go this way if a first block is two thirds
// full, nine and more if all are on the average.  8 epochs, D = 64 to 10000, every tenth or third label at random, time this way
// over time by sub-blocks (over time by sub-blocks with three launches a block):
//   6 classes: 129 samples 0.95 to 1.09, 200 0.79 to 0.96, 300 0.91 to 1.07 (0.84 to 1.01), 400 0.83 to 0.96
//   8 classes: 129 1.05 to 1.13, 200 0.92 to 0.97, 300 1.01 to 1.13 (0.92 to 1.08), 400 0.90 to 0.99
//   10 classes: 129 1.02 to 1.15, 200 0.87 to 1.02, 300 1.01 to 1.16 (0.95 to 1.13), 400 0.86 to 1.05
static bool wide_takes(const hdc_ctx_impl *c, int64_t N, int32_t epochs, float lr) {
    const int C = c->p.C;
    const int64_t blocks = (N + kChainBlock - 1) / kChainBlock;
    return C <= kWideClasses && c->p.D <= 32767 && N > 2 * kSub && N * epochs > 2 * kSub * (C - 2) &&
           (C <= 4 || 3 * N >= 2 * kChainBlock * (C <= kWideWaves ? 1 : blocks)) && fabsf(lr) < kTameRate;
}

// (the tests call it, for contexts without the scratch of longer blocks)
int reserve_online_blocks(hdc_ctx_impl *c) {
    if (c->oc_ready) return HDC_OK;
    const int C = c->p.C, D = c->p.D;
    const int G = (D + kWave - 1) / kWave, slice = chain_slice(D), slices = (D + slice - 1) / slice;
    HDC_HIP(hipSetDevice(c->device));
    // one allocation (each takes half a millisecond), the parts at multiples of 256 bytes
    struct { void **at; size_t bytes; } parts[] = {
        {(void **)&c->oc_col_d, (size_t)G * held_samples(G) * sizeof(uint64_t)},
        {(void **)&c->oc_gram_d, (size_t)kHeldBlocks * kTiles * kTile * sizeof(int16_t)},
        {(void **)&c->oc_pairs_d, (size_t)(kHeldBlocks - 1) * kSubs * kSubs * kTile * sizeof(int16_t)},
        {(void **)&c->oc_image_d, (size_t)kHeldBlocks * kWideImage * sizeof(int16_t)},
        {(void **)&c->oc_order_d, (size_t)kHeldBlocks * sizeof(WideOrder)},
        {(void **)&c->oc_part_d, (size_t)(slices + 1) * C * kChainBlock * sizeof(double)},
        {(void **)&c->oc_rec_d, (size_t)2 * kChainBlock * sizeof(OnlineWeight)},
        {(void **)&c->oc_norm_d, (size_t)C * (G + 1) * sizeof(double)},
    };
    size_t want = 0;
    for (const auto &p : parts) want += (p.bytes + 255) / 256 * 256;
    int rc = grow(&c->oc_mem_d, &c->oc_mem_bytes, want);
    char *next = c->oc_mem_d;
    for (const auto &p : parts) {
        *p.at = next;
        if (next) next += (p.bytes + 255) / 256 * 256;
    }
    if (rc == HDC_OK) rc = grow(&c->on_bits_d, &c->on_bits_bytes, (size_t)kOnlineWords * sizeof(uint32_t));
    if (rc == HDC_OK) rc = grow(&c->ob_norm_d, &c->ob_norm_bytes, (size_t)C * G * sizeof(double));
    c->oc_ready = rc == HDC_OK;
    if (rc == HDC_ENOMEM) {   // all or nothing: what is left of the memory is for the other ways
        (void)hipFree(c->oc_mem_d);
        c->oc_mem_d = nullptr;
        c->oc_mem_bytes = 0;
    }
    return rc;
}

// (Long calls go in blocks of 256 where the memory for longer ones cannot be had.)
int reserve_online_chain(hdc_ctx_impl *c) {
    if (c->oc_ready && c->os_ready) return HDC_OK;
    int rc = reserve_online_blocks(c);
    if (rc == HDC_OK) {
        rc = reserve_online_spread(c);
        if (rc == HDC_ENOMEM) rc = HDC_OK;
    }
    return rc;
}

bool online_chain_ready(hdc_ctx_impl *c, hipStream_t s, int *rc) {
    *rc = HDC_OK;
    if (!online_chain_takes(c)) return false;
    if (!c->oc_ready && !stream_captured(s)) *rc = reserve_online_chain(c);
    if (*rc == HDC_ENOMEM) *rc = HDC_OK;
    return c->oc_ready;
}

// A block's chain, with the row updates of the block before beside it if the rows do not hold those yet (ahead).
struct ChainCall {
    int64_t b;               // block of those that are held
    int slices, nb, batch, G;
    const int32_t *labels;
    float lr;
    const double *norm;      // squared-norm partials of the rows
    bool ahead;
    BlockBefore before;
    OnlineWeight *recs;      // out
};

template <int CPW, bool BATCH>
static int launch_chain(hdc_ctx_impl *c, const ChainCall &a, hipStream_t s) {
    auto kern = online_chain_kernel<CPW, BATCH>;
    const int slot = (CPW == 1 ? 0 : CPW == 2 ? 2 : 4) + (BATCH ? 1 : 0);
    if (!c->oc_attr_set[slot]) {
        HDC_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kTiles * kTile * (int)sizeof(int16_t)));
        c->oc_attr_set[slot] = true;
    }
    const int subs = (a.nb + kSub - 1) / kSub;
    hipLaunchKernelGGL(kern, dim3(a.ahead ? 1u + (unsigned)a.G : 1u), dim3(kChainMaxWaves * kWave),
                       (size_t)(subs * (subs + 1) / 2) * kTile * sizeof(int16_t), s, c->oc_gram_d + a.b * kTiles * kTile, c->oc_part_d,
                       a.slices + (a.ahead ? 1 : 0), a.nb, a.batch, a.labels, a.norm, a.G, c->p.C, c->p.D, a.lr,
                       1.0 / sqrt((double)c->p.D), a.recs, c->oc_norm_d + (int64_t)c->p.C * a.G, a.ahead, a.before);
    HDC_HIP(hipGetLastError());
    return HDC_OK;
}

template <int CPW, int GR>
static int launch_wide(hdc_ctx_impl *c, const ChainCall &a, hipStream_t s) {
    auto kern = online_wide_kernel<CPW, GR>;
    const int slot = CPW == 1 ? 6 : 7, C = c->p.C, per_place = kSub * (int)sizeof(double);
    const int most = CPW * kWideWaves, cosines = kSubs * (CPW == 1 ? 2 : 1);   // places beside the runs' for a class: cosines, starts
    auto behind = [&](int classes) {   // the products: the places, or what a walk by sub-blocks keeps there
        return std::max((wide_places(classes) + cosines * classes) * per_place, (int)sizeof(ChainShared<CPW, kWideWaves>));
    };
    if (!c->oc_attr_set[slot]) {
        HDC_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kTiles * kTile * (int)sizeof(int16_t) + behind(most)));
        c->oc_attr_set[slot] = true;
    }
    const int subs = (a.nb + kSub - 1) / kSub;
    hipLaunchKernelGGL(kern, dim3(a.ahead ? 1u + (unsigned)a.G : 1u), dim3(kWideWaves * kWave),
                       (size_t)(subs * (subs + 1) / 2) * kTile * sizeof(int16_t) + behind(C), s,
                       c->oc_gram_d + a.b * kTiles * kTile, c->oc_image_d + a.b * kWideImage,
                       static_cast<const WideOrder *>(c->oc_order_d) + a.b, c->oc_part_d, a.slices + (a.ahead ? 1 : 0), a.nb, a.labels,
                       a.norm, a.G, C, c->p.D, a.lr, 1.0 / sqrt((double)c->p.D), a.recs, c->oc_norm_d + (int64_t)C * a.G, a.ahead,
                       a.before);
    HDC_HIP(hipGetLastError());
    return HDC_OK;
}

// The blocks of samples that are held.  Two launches a block: the chain of block b beside the row updates of block b - 1,
// then the products of block b + 1 with the rows as those left them, and with block b's updates by the samples' own
// products.  (Rows, products and chain one after another took 27 us a block instead of 22, per sample, 6 classes, D = 10000;
// 36 instead of 30 in batches of 64.)  A learning rate that can make a weight overflow leaves that: each block after the rows.
template <bool BATCH>
static int walk_held(hdc_ctx_impl *c, const int32_t *labels, int64_t N, float lr, int batch, bool wide, float *acc, int64_t ld,
                     int *norm_at, hipStream_t s) {
    const int C = c->p.C, D = c->p.D;
    const int G = (D + kWave - 1) / kWave, slice = chain_slice(D), slices = (D + slice - 1) / slice;
    const int block = kChainBlock / batch * batch;   // whole batches
    double *norm[2] = {c->ob_norm_d, c->oc_norm_d};  // squared norms: of the rows before the last update, and after
    const int64_t blocks = (N + block - 1) / block;
    const bool beside = fabsf(lr) < kTameRate;
    OnlineWeight *const all = static_cast<OnlineWeight *>(c->oc_rec_d);   // of an even block, and of an odd one
    for (int64_t b = 0; b < blocks; ++b) {
        const int nb = (int)(N - b * block < block ? N - b * block : block);
        OnlineWeight *recs = all + b % 2 * kChainBlock;
        const OnlineWeight *recs_before = all + (b + 1) % 2 * kChainBlock;
        const uint64_t *col = c->oc_col_d + b * block;
        const bool ahead = beside && b > 0;   // the rows do not hold the block before yet
        {
            ProfScope prof(c, HDC_K_ONLINE_FWD, s, BATCH);
            hipLaunchKernelGGL(online_dots_kernel,
                               dim3((unsigned)(slices + (ahead ? 1 : 0)), (unsigned)((nb + 15) / 16), (unsigned)((C + 15) / 16)),
                               dim3(kDotWaves * kWave), 0, s, col, ld, nb, acc, D, C, slice, slices,
                               ahead ? c->oc_pairs_d + (b - 1) * kSubs * kSubs * kTile : nullptr, recs_before, block, c->oc_part_d);
        }
        HDC_HIP(hipGetLastError());
        const ChainCall a = {b, slices, nb, batch, G, labels + b * block, lr, norm[*norm_at], ahead,
                             {col - (ahead ? block : 0), ld, block, recs_before, acc, norm[*norm_at ^ 1]}, recs};
        {
            ProfScope prof(c, HDC_K_ONLINE, s, BATCH), with(c, HDC_K_ONLINE_BWD, s, BATCH && ahead);
            int rc;
            if (wide)
                rc = C <= kWideWaves ? launch_wide<1, wide_group(kWideWaves)>(c, a, s) : launch_wide<2, wide_group(2 * kWideWaves)>(c, a, s);
            else if (C <= kChainMaxWaves)
                rc = launch_chain<1, BATCH>(c, a, s);
            else if (C <= 2 * kChainMaxWaves)
                rc = launch_chain<2, BATCH>(c, a, s);
            else
                rc = launch_chain<4, BATCH>(c, a, s);
            if (rc != HDC_OK) return rc;
        }
        if (ahead) *norm_at ^= 1;
        if (!beside || b + 1 == blocks) {
            const unsigned waves = (unsigned)(C < 4 ? 4 : C < kChainMaxWaves ? C : kChainMaxWaves);
            ProfScope prof(c, HDC_K_ONLINE_BWD, s, BATCH);
            hipLaunchKernelGGL(online_rows_kernel<BATCH>, dim3((unsigned)G), dim3(waves * kWave), 0, s, col, ld, nb, batch, recs, acc, D,
                               C, G, norm[*norm_at ^ 1]);
            HDC_HIP(hipGetLastError());
            *norm_at ^= 1;
        }
    }
    return HDC_OK;
}

template <bool BATCH>
static int walk_blocks(hdc_ctx_impl *c, const uint32_t *hv, const int32_t *labels, int64_t N, int32_t epochs, float lr,
                       int batch, float *acc, hipStream_t s) {
    const int C = c->p.C, D = c->p.D, W = c->W;
    const int G = (D + kWave - 1) / kWave;
    const bool wide = !BATCH && wide_takes(c, N, epochs, lr);
    ProfScope walk(c, HDC_K_ONLINE, s, !BATCH);   // a walk by samples as a whole; of batches each block's three steps
    ProfScope which(c, HDC_K_ONLINE_WIDE, s, wide);
    int rc = launch_norm(c, acc, G, s);
    if (rc != HDC_OK) return rc;
    const int block = kChainBlock / batch * batch;   // whole batches
    const int64_t ld = held_samples(G), held = std::min(ld / block, kHeldBlocks) * block;
    int norm_at = 0;   // which of the two arrays of squared norms is that of the rows
    for (int32_t e = 0; e < epochs; ++e)
        for (int64_t h0 = 0; h0 < N; h0 += held) {
            const int64_t hn = N - h0 < held ? N - h0 : held;
            if (e == 0 || N > held) {   // a set that fits is multiplied out once for all epochs
                const unsigned blocks = (unsigned)((hn + block - 1) / block);
                WideOrder *order = wide ? static_cast<WideOrder *>(c->oc_order_d) : nullptr;
                hipLaunchKernelGGL(wide ? online_columns_kernel<true> : online_columns_kernel<false>,
                                   dim3((unsigned)((hn + kSub - 1) / kSub), (unsigned)((G + kColGroups - 1) / kColGroups + (wide ? 1 : 0))),
                                   dim3(256), 0, s, hv + h0 * W, hn, W, c->last_word_mask, G, ld, c->oc_col_d, labels + h0, C, order);
                HDC_HIP(hipGetLastError());
                if (hn > 1 || wide) {
                    const int subs = (int)((std::min<int64_t>(hn, block) + kSub - 1) / kSub);
                    hipLaunchKernelGGL(wide ? online_gram_kernel<Products::kWide> : online_gram_kernel<Products::kTiles>,
                                       dim3((unsigned)(subs * (subs + 1) / 2 + (blocks > 1 ? (kTiles - subs * (subs + 1) / 2) + kSubs * kSubs : 0)), blocks),
                                       dim3(kGramWaves * kWave), 0, s, c->oc_col_d, ld, hn, D, G, block, c->oc_gram_d, order,
                                       c->oc_image_d, c->oc_pairs_d);
                }
                HDC_HIP(hipGetLastError());
            }
            rc = walk_held<BATCH>(c, labels + h0, hn, lr, batch, wide, acc, ld, &norm_at, s);
            if (rc != HDC_OK) return rc;
        }
    return HDC_OK;
}

int launch_online_chain(hdc_ctx_impl *c, const uint32_t *hv, const int32_t *labels, int64_t N, int32_t epochs,
                        float lr, int64_t batch, bool per_sample, float *acc, hipStream_t s) {
    if (online_spread_takes(c, N, lr, batch, per_sample))
        return per_sample ? launch_online_spread<false>(c, hv, labels, N, epochs, lr, 1, acc, s)
                          : launch_online_spread<true>(c, hv, labels, N, epochs, lr, (int)batch, acc, s);
    return per_sample ? walk_blocks<false>(c, hv, labels, N, epochs, lr, 1, acc, s)
                      : walk_blocks<true>(c, hv, labels, N, epochs, lr, (int)batch, acc, s);
}

}  // namespace hdc
