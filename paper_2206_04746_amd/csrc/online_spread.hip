// Online training of many samples, per sample and in batches: blocks of up to 2048 samples, the chain of a block spread
// over a workgroup per 16 of them (arXiv 2206.04746, Sec. III Eqs. 2-3, caption of Fig. 1; Sec. VI-D2 for batches).
//
// online_chain.hip tells how a block's chain is a triangular fixed point on the samples' scalar products with one
// another.  How many passes it takes hardly depends on the block's length: five or six settle 2048 samples as they do
// 256, because one sample moves the cosines of the others little (from rows of zeros 9 to 19, for 2 to 24 classes; with a third of
// the labels at random 8 to 11, from zeros 14 to 26; with all of them, where predictions are mostly wrong, 170 to 270 for 6 classes, 67
// for 24).  So a pass is spread over the chip and the block made long:
//   online_gram_kernel   once per call: <s_n, s_m> of all pairs of a block, in strips of 16 columns
//   row_dots_kernel      per block: <acc_c, s_m> against the rows as they stand
//   online_spread_kernel per block: cosines, predictions and weights of all samples
//   online_update_kernel per block: the updates, element by element in sample order, and the rows' squared norms
// 7352 samples, 6 classes, D = 10000, us, with blocks of 256 on one workgroup and now: three epochs 2003 and 775, one in
// batches of 64 879 and 450.  The rows come out as near the method in 64 bits: relative 2-norm 0.97e-7 to 1.39e-6 over ten models of
// 2 to 16 classes, D = 500 to 4000, rows of up to 1e6 to begin with, between 1.6 % nearer and 0.5 % farther than blocks of 256.
#include "online_lanes.h"

namespace hdc {

namespace {

constexpr int kOwn = kStripCols;          // samples of a workgroup: a lane to each in every row of 16 lanes
constexpr int kGroups = kSpan / kOwn;     // most workgroups of a block
constexpr int kDotSlices = 20;           // of the dot products, at most
constexpr int kWaves = 16, kThreads = kWaves * kWave;
constexpr int kHearing = 8, kHeard = kSpan / (kHearing * kWave);   // waves that wait for other workgroups' weights, words of a lane
constexpr int kLists = 4 * kWaves;        // a row of 16 lanes takes one list of sources
constexpr int kSteps = 36;                // most sources of a list: room for 2032 and the filling of 64 classes
constexpr int kRunGroup = 4;              // a class's sources are filled up to whole groups of these
constexpr int kListGroups = kSteps / kRunGroup;
constexpr int kNone = kSpan;              // a source that is none: its weight is zero
constexpr int kMaxClasses = 32;
constexpr int kRounds = 49, kManyRounds = 97;   // passes that the workgroups take together, at most, and one; the second with more than kWaves classes
__host__ __device__ constexpr int slots_of(int C) { return C <= kWaves ? kRounds : kManyRounds; }   // the last one for the end
constexpr int kSpinLimit = 1 << 24;       // loads of one word before a wait is given up (never: see wait_for)
// What such a word of a sample counts as: a weight that is no number, with no prediction and nothing changed; a squared norm's word of 0
// is no number as it is.  The rows say so then.
constexpr unsigned long long kLost = 0x7FC00000ull;
static_assert((kLost & 0x7FFFFFFFull) > 0x7F800000ull && kLost >> 32 == 0, "no number, and nothing beside it");
static_assert(kOwn * (kGroups - 1) + (kRunGroup - 1) * 2 * kMaxClasses <= kLists * kSteps, "room in the lists");

// ---- what workgroups tell one another ------------------------------------------------------------
// A slot of memory per pass; every word is written once, 0 says not yet.  A word carries its data, so that no order
// between words is asked for, and no fence.
//   [0, kSpan)           of a sample: w_y; above it bit 31: there, bit 9: its last word but for the last slot, bit 8: a weight
//                        of the workgroup has changed, bits 0 to 7: pred + 1
//   [kSpan, 2 kSpan)     w_p, bit 32: there (written only with a pred)
//   then [C][kGroups]    what a workgroup's samples add to a class's squared norm: the bits of it and one
//   and [C][kGroups]     the same up to the batch that runs on into the next workgroup (batches only)
__host__ __device__ constexpr int64_t slot_words(int C) { return 2 * kSpan + (int64_t)2 * C * kGroups; }
using Word = unsigned long long;

__device__ __forceinline__ void tell(Word *at, Word v) { __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ Word look(const Word *at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// A workgroup waits only for those that took their number before it.  They have begun, and what they wait for has, too:
// the wait ends however few workgroups fit the chip.
__device__ __forceinline__ Word wait_for(const Word *at) {
    Word v = look(at);
    for (int i = 0; !v && i < kSpinLimit; ++i) v = look(at);
    return v;
}
__device__ __forceinline__ Word norm_word(double v) { return (Word)__double_as_longlong(v) + 1; }
__device__ __forceinline__ double word_norm(Word v) { return __longlong_as_double((long long)(v - 1)); }

// The value of the lane before in the row of 16 lanes (its first: zero), and the sum up to a lane.
__device__ __forceinline__ double row_before(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x111, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x111, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_prefix(double v) {
    v = dpp_add<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    return dpp_add<0x118, 0xF>(v);
}
// The same sum of the four rows in every row: rows 0 and 1, 2 and 3 change places, then the halves.
__device__ __forceinline__ double sum_rows(double v) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
        const auto a = half ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = half ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
    }
    return v;
}
// Of all lanes, in every lane.
__device__ __forceinline__ double sum_lanes(double v) {
    v = row_prefix(v);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x15F, 0xF, 0xF, true);   // row_newbcast:15
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x15F, 0xF, 0xF, true);
    return sum_rows(__hiloint2double(hi, lo));
}

// A cosine; 0 for a row of zeros.  (Without a branch: each would keep the classes of a wave one after another.)
__device__ __forceinline__ double cosine_of(double dot, double nn, double inv_root_d) {
    double c = dot * refined_rsq(nn) * inv_root_d;
    asm volatile("" : "+v"(c));
    return nn <= 0.0 ? 0.0 : c;
}

// How many lanes before this one have the same key (0 to 63), of those that have any; which lanes do.
__device__ __forceinline__ int rank_of(int key, bool valid, uint64_t &same) {
    same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const uint64_t m = __ballot(key >> b & 1);
        same &= key >> b & 1 ? m : ~m;
    }
    return __popcll(same & ((1ull << (threadIdx.x & (kWave - 1))) - 1));
}

struct SpreadShared {
    int16_t strip[kSpan * kOwn];          // products with the samples before and its own (as halves): [sample][16]
    Word word[kSpan + 1];                 // what was last heard of a sample; [kNone]: zero
    double tail[kLists][kOwn];            // sums of a list's first class ...
    double head[2 * kMaxClasses][kOwn];   // ... and of the classes that begin inside a list
    double wrong_tail[kLists][kOwn];      // the same of the samples before for which a class was wrongly predicted
    double wrong_head[2 * kMaxClasses][kOwn];
    double cosine[kMaxClasses][kOwn];
    float heard_wp[kSpan];                // weights of classes wrongly predicted
    int8_t label[kSpan];                  // of the samples before, or -1
    uint2 named[kSpan];                   // these samples class after class (with the class from bit 16 on) and the weights
    uint16_t count[kSpan / kWave][2 * kMaxClasses];   // of 64 samples those of a class, then those of the 64s before
    int wrong_end[2 * kMaxClasses];       // of a class in named
    uint16_t src[kLists][kSteps];         // the lists: sources class after class
    uint8_t key[kLists * kListGroups + 8];// class of a group of sources
    int first_group[2 * kMaxClasses + 1]; // of a class
    int total[2 * kMaxClasses];           // sources of a class
    int front[2], wrong[2], flips[2];     // first workgroup that a weight of has changed; predictions that are wrong; those that have changed
    int parting[2];                       // whether a workgroup has gone on alone
    int own_changed, number, odd[kWaves], zero[kWaves];
    int2 own_class[kOwn];                 // its own samples: label, class wrongly predicted or -1
    double2 own_w[kOwn];                  // their weights, the second one negative
    double2 mine[kMaxClasses];            // what they add to the squared norms; up to the batch that runs on
    double start[kMaxClasses][kOwn], nrm[kMaxClasses];   // their dot products with the rows at the block's start; squared norms there
};
struct SortShared {                       // lies over tail and head
    uint16_t count[kSpan / kWave][2 * kMaxClasses];
};
static_assert(sizeof(SortShared) <= sizeof(double) * kOwn * (kLists + 2 * kMaxClasses), "");
static_assert(sizeof(SpreadShared) <= 160 * 1024, "LDS of a compute unit");
// a walk by samples: their records in what the passes sum, its panels' sums in the strip
static_assert(sizeof(OnlineWeight) * kSpan <= offsetof(SpreadShared, cosine) - offsetof(SpreadShared, word), "");
static_assert(sizeof(double) * kMaxClasses * kPanel <= sizeof(int16_t) * kSpan * kOwn, "");

struct StripProduct {
    static constexpr bool kPanels = true;
    const int16_t *strips;
    int odd;
    __device__ int operator()(int n, int m) const {
        return 2 * (int)strips[strip_start(m / kStripCols) + n * kStripCols + m % kStripCols] + odd;
    }
};

// acc[k] += w[k] of lane (16 j + u) x g[u], in every row of 16 lanes j, for I <= u < I + 4: CL sums side by side, or two for one.
template <int I, int CL>
__device__ __forceinline__ void add_own(double (&acc)[CL < 2 ? 2 : CL], const double (&w)[CL], const double *g) {
    if constexpr (CL == 1)
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc[0]), "+v"(acc[1]) : "v"(w[0]), "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
    else
#pragma unroll
        for (int k = 0; k < CL; k += 2)
            asm volatile("s_nop 1\n\t"
                         "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %1, %3, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %1, %3, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %0, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %1, %3, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %0, %2, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
                         "v_fmac_f64_dpp %1, %3, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
                         : "+v"(acc[k]), "+v"(acc[k + 1])
                         : "v"(w[k]), "v"(w[k + 1]), "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
}

// One wave finds the fixed point of a workgroup's samples by itself: a chain of dependent instructions, five to seven passes of about 900
// clocks where labels are at random, so nothing is read again in a pass that fits the registers (4000 samples of 6 classes, D = 2000, labels
// at random: 1604 us with LDS reads in every pass and products made after the last weights were heard, 1449 now).  Row q of lanes has classes q, q + 4 ... q + 4 CL - 4 and,
// for more classes than that, those 4 CL further on; what the samples before add to the dot products lies in tail and head (all
// of it; what counts in batches), the squared norms in wrong_tail and wrong_head.
template <int CL, int CHUNKS, bool BATCH>
__device__ __forceinline__ void settle_own(SpreadShared &s, const double (&product)[kOwn], int n0, int fb, int next_fb, int C, double dd, float lr,
                                           double inv_root_d) {
    const int lane = threadIdx.x & (kWave - 1), l = lane & (kOwn - 1), q = lane / kOwn;
    int2 of = s.own_class[l];
    double2 own = s.own_w[l];
    const int before_batch = fb - n0;   // (batches) own samples that count
    // What the samples before add: in registers for all passes, where there is room (a pass then stores nothing), else asked for when a
    // pass begins, or where it is used.
    constexpr bool kHold = CHUNKS == 1 && !BATCH, kAsk = CHUNKS == 1 && BATCH;
    double every_before[CL], counts_before[CL], norm[CL], norm_open[CL], grown[CL];
    auto load_before = [&](int h, int k) {
        const int at = min(4 * (CL * h + k) + q, C - 1);
        every_before[k] = s.tail[at][l];
        norm[k] = s.wrong_tail[at][0];
        if (BATCH) counts_before[k] = s.head[at][l], norm_open[k] = s.wrong_head[at][0];
    };
#pragma unroll
    for (int k = 0; kHold && k < CL; ++k) load_before(0, k);
    for (int pass = 0; pass < kOwn + 2; ++pass) {   // (16 settle them, one more finds nothing changed)
        double best = -4.0, cos_y = 0.0;
        int arg = kMaxClasses;
#pragma unroll
        for (int h = 0; h < CHUNKS; ++h) {
            double w[CL], every[CL < 2 ? 2 : CL] = {}, dot[CL < 2 ? 2 : CL] = {};
#pragma unroll
            for (int k = 0; kAsk && k < CL; ++k) load_before(0, k);
#pragma unroll
            for (int k = 0; k < CL; ++k) {
                const int c = 4 * (CL * h + k) + q;
                w[k] = c == of.x ? own.x : c == of.y ? own.y : 0.0;
            }
            each<4>([&](auto i_) {
                constexpr int i = 4 * decltype(i_)::value;
                add_own<i, CL>(every, w, product + i);
                if constexpr (BATCH) {
                    double counted[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) counted[u] = i + u < before_batch ? product[i + u] : 0.0;
                    add_own<i, CL>(dot, w, counted);
                }
            });
            if (CL == 1) every[0] += every[1], dot[0] += dot[1];
#pragma unroll
            for (int k = 0; k < CL; ++k) {
                const int c = 4 * (CL * h + k) + q;
                if (CHUNKS > 1) load_before(h, k);
                const double all = every[k] + every_before[k], counts = BATCH ? dot[k] + counts_before[k] : all;
                const double run = row_prefix(w[k] * fma(w[k], dd, 2.0 * all)), before = row_before(run);
                double nn = norm[k] + before;
                if (BATCH) {
                    const double at_fb = __shfl(before, kOwn * q + min(max(fb - n0, 0), kOwn - 1), kWave);
                    nn = fb >= n0 ? norm[k] + at_fb : norm_open[k];
                }
                if (kHold)
                    grown[k] = run;
                else
                    s.cosine[c][l] = run;   // (32 classes there)
                const double cs = cosine_of(counts, nn, inv_root_d);
                const bool better = (c < C) & (cs > best);
                best = better ? cs : best;
                arg = better ? c : arg;
                cos_y = c == of.x ? cs : cos_y;
            }
        }
        cos_y = sum_rows(cos_y);   // (of one row)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            auto swap = [&](uint32_t v) {
                return half ? __builtin_amdgcn_permlane32_swap(v, v, false, false) : __builtin_amdgcn_permlane16_swap(v, v, false, false);
            };
            const auto lo = swap((uint32_t)__double2loint(best)), hi = swap((uint32_t)__double2hiint(best)), at = swap((uint32_t)arg);
            const double a = __hiloint2double((int)hi[0], (int)lo[0]), b = __hiloint2double((int)hi[1], (int)lo[1]);
            const bool second = (b > a) | ((b == a) & (at[1] < at[0]));
            best = second ? b : a;
            arg = (int)(second ? at[1] : at[0]);
        }
        const bool wrong = (of.x >= 0) & (arg != of.x);
        const double wy = of.x >= 0 ? (double)(float)(1.0 - cos_y) : 0.0, wp = wrong ? -(double)(float)((double)lr * (1.0 - best)) : 0.0;
        const int pred = wrong ? arg : -1;
        const bool moved = __ballot(wy != own.x || wp != own.y || pred != of.y) != 0;
        own = make_double2(wy, wp);
        of.y = pred;
        if (!moved) break;
    }
    if constexpr (kHold) {
#pragma unroll
        for (int k = 0; k < CL; ++k) s.cosine[4 * k + q][l] = grown[k];
    }
    if (q == 0) {
        s.own_class[l] = of;
        s.own_w[l] = own;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < C)
        s.mine[lane] = make_double2(s.cosine[lane][kOwn - 1], BATCH && next_fb > n0 ? s.cosine[lane][min(next_fb - n0, kOwn) - 1] : 0.0);
}

// What bounds it: two hops to other workgroups a pass (0.9 to 1.2 us each) and between them the dependent instructions of
// one wave, 9 clocks each.  16 samples a workgroup, because a row of 16 lanes then holds one list's sources against all of them,
// and 2048 samples are half the chip's compute units, one workgroup each for the products in LDS.  6 classes, D = 10000: 136 us for a
// block from zero rows, 27 to 30 for one of settled rows, where eight blocks of 256 took 131 us.
// In batches 18 vector registers (48 with two classes a wave) are in scratch; settled blocks take 37 to 60 us there.
// Class c is wave (c + 8) % 16's: the first waves are busy with what they hear, the last one decides.
template <int CPW, bool BATCH>
__global__ __launch_bounds__(kThreads) void online_spread_kernel(const int16_t *__restrict__ strips, const double *__restrict__ part,
                                                                 int slices, int nb, int batch, const int32_t *__restrict__ labels,
                                                                 const double *__restrict__ normpart, int G, int C, int D, float lr,
                                                                 double inv_root_d, Word *__restrict__ slots, int *__restrict__ state,
                                                                 OnlineWeight *__restrict__ out) {
    extern __shared__ __align__(16) char shared[];
    SpreadShared &s = *reinterpret_cast<SpreadShared *>(shared);
    SortShared &sort = *reinterpret_cast<SortShared *>(&s.tail[0][0]);
    int tid = threadIdx.x, lane = tid & (kWave - 1), l = lane & (kOwn - 1), q = lane / kOwn;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int own_class = (wave + kHearing) % kWaves;   // and those 16 and more further on
    if (tid == 0) s.number = atomicAdd(state, 1);   // (in the order in which they begin: wait_for)
    int label[2];      // of samples tid and tid + kThreads
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int n = tid + u * kThreads;
        label[u] = labels[min(n, nb - 1)];
        label[u] = n < nb && label[u] >= 0 && label[u] < C ? label[u] : -1;
        s.label[n] = (int8_t)label[u];
    }
    double nrm[CPW];
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = min(own_class + k * kWaves, C - 1);
        double p[4], sum = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = normpart[(int64_t)c * G + min(i * kWave + lane, G - 1)];
#pragma unroll
        for (int i = 0; i < 4; ++i) sum += i * kWave + lane < G ? p[i] : 0.0;
        for (int g = 4 * kWave + lane; g < G; g += kWave) sum += normpart[(int64_t)c * G + g];
        nrm[k] = sum;
    }
    if (tid < 2) s.wrong[tid] = s.flips[tid] = s.parting[tid] = 0;
    for (int i = tid; i < (int)sizeof(sort.count) / 4; i += kThreads) reinterpret_cast<uint32_t *>(&sort.count[0][0])[i] = 0;
    for (int i = tid; i < kLists * kSteps / 2; i += kThreads) reinterpret_cast<uint32_t *>(&s.src[0][0])[i] = kNone | kNone << 16;
    for (int i = tid; i <= kSpan; i += kThreads) s.word[i] = 0;
    __syncthreads();
    const int group = __builtin_amdgcn_readfirstlane(s.number), n0 = group * kOwn;   // n0: samples before, too
    const int groups = (nb + kOwn - 1) / kOwn;
    const int odd = D & 1;
    auto whole = [&](int g) { return 2 * g + odd; };

    // ---- what does not change from pass to pass
    uint4 copy[kSpan * kOwn * 2 / 16 / kThreads];
    const uint4 *strip = reinterpret_cast<const uint4 *>(strips + strip_start(group));
    const int units = (n0 + kOwn) * kOwn * 2 / 16;
#pragma unroll
    for (int u = 0; u < kSpan * kOwn * 2 / 16 / kThreads; ++u) copy[u] = strip[min(tid + u * kThreads, units - 1)];
    int y = n0 + l < nb ? labels[n0 + l] : -1;   // of the sample of this lane
    y = y >= 0 && y < C ? y : -1;
    double start[CPW];
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const int c = min(own_class + k * kWaves, C - 1);
        double p[5], dot = 0.0;     // (kDotSlices at most, a quarter to a row of lanes)
#pragma unroll
        for (int i = 0; i < 5; ++i) p[i] = part[((int64_t)min(4 * i + q, slices - 1) * C + c) * kSpan + n0 + l];
#pragma unroll
        for (int i = 0; i < 5; ++i) dot += 4 * i + q < slices ? p[i] : 0.0;
        start[k] = sum_rows(dot);
        nrm[k] = sum_lanes(nrm[k]);
        if (own_class + k * kWaves < C) {
            s.start[own_class + k * kWaves][l] = start[k];
            s.nrm[own_class + k * kWaves] = nrm[k];
        }
    }
    {
        bool strange = false, zero = true;
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            strange |= !(nrm[k] < __builtin_inf());
            zero &= nrm[k] == 0.0;
        }
        if (lane == 0) {
            s.odd[wave] = strange;
            s.zero[wave] = zero;
        }
    }
    // The samples before, class by class (in batches those of the batch that runs into this workgroup's samples after the
    // others): numbers within a class by the ballots of 64 samples and a sum over those before.
    const int first_open = BATCH ? n0 / batch * batch : n0;   // first sample of that batch
    const int classes = BATCH ? 2 * C : C;
    int key[2], rank[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int n = tid + u * kThreads;
        const bool valid = n < n0 && label[u] >= 0;
        key[u] = valid ? label[u] + (BATCH && n >= first_open ? C : 0) : -1;
        uint64_t same;
        rank[u] = rank_of(key[u], valid, same);
        if (valid && rank[u] == 0) sort.count[wave + u * kWaves][key[u]] = (uint16_t)__popcll(same);
    }
    if (tid < kOwn) {
        s.own_class[tid] = make_int2(y, -1);
        s.own_w[tid] = make_double2(0.0, 0.0);
    }
    if (tid < 2) s.front[tid] = group;
#pragma unroll
    for (int u = 0; u < kSpan * kOwn * 2 / 16 / kThreads; ++u)
        if (tid + u * kThreads < units) reinterpret_cast<uint4 *>(s.strip)[tid + u * kThreads] = copy[u];
    __syncthreads();
    if (__builtin_expect(__ballot(lane < kWaves && s.odd[lane & (kWaves - 1)]) != 0, 0)) {   // rows that are not finite: the same everywhere
        if (group) return;
        __syncthreads();
        OnlineWeight *rec = reinterpret_cast<OnlineWeight *>(s.word);
        walk_block<CPW, BATCH>(StripProduct{strips, odd}, part, kSpan, slices, nb, batch, labels, normpart, nullptr, nullptr, G, C, D,
                               lr, inv_root_d, rec, &s.cosine[0][0], reinterpret_cast<double *>(s.strip));
        for (int n = tid; n < nb; n += kThreads) out[n] = rec[n];
        if (tid == 0) state[1] = 0;
        return;
    }
    const bool zero_model = __ballot(lane < kWaves && !s.zero[lane & (kWaves - 1)]) == 0;
    bool changed = false, parting = false; // (the deciding wave's) a weight, in this pass; this workgroup goes on alone
    const int decider = kWaves - 1;
    // Weights from the cosines.  (guess: labels count as predictions, where rows of zeros would say class 0 of every sample.
    // The passes end in the same place from any start.)
    auto decide = [&](bool guess) {
        const int2 of = s.own_class[l];
        const double2 w = s.own_w[l];
        const double cos_y = s.cosine[max(of.x, 0)][l];
        double best = -4.0;
        int arg = 0;
        for (int c0 = 0; c0 < C; c0 += 8) {   // eight at a time (the last one repeats: it cannot win twice)
            double v[8];
            int at[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = s.cosine[min(c0 + u, C - 1)][l];
                at[u] = c0 + u;
            }
#pragma unroll
            for (int step = 1; step < 8; step *= 2)
#pragma unroll
                for (int u = 0; u < 8; u += 2 * step) {
                    const bool other = v[u + step] > v[u];
                    v[u] = other ? v[u + step] : v[u];
                    at[u] = other ? at[u + step] : at[u];
                }
            const bool better = v[0] > best;
            best = better ? v[0] : best;
            arg = better ? at[0] : arg;
        }
        const bool wrong = (of.x >= 0) & (arg != of.x) & !guess;
        const double wy = of.x >= 0 ? (double)(float)(1.0 - cos_y) : 0.0, wp = wrong ? -(double)(float)((double)lr * (1.0 - best)) : 0.0;
        const int pred = wrong ? arg : -1;
        changed = __ballot(wy != w.x || wp != w.y || pred != of.y) != 0;
        if (lane < kOwn) {
            s.own_class[l] = make_int2(of.x, pred);
            s.own_w[l] = make_double2(wy, wp);
        }
        if (lane == 0) s.own_changed = changed;
    };
    auto tell_weights = [&](Word *slot) {
        const int pred = s.own_class[l].y;
        const double2 w = s.own_w[l];
        if (lane < kOwn) {
            if (pred >= 0) tell(slot + kSpan + n0 + l, 1ull << 32 | __float_as_uint((float)-w.y));
            tell(slot + n0 + l, 1ull << 63 | (Word)((changed ? 0x100 : 0) | (parting ? 0x200 : 0)) << 32 | (Word)(pred + 1) << 32 | __float_as_uint((float)w.x));
        }
    };
    const int64_t words = slot_words(C);
    // One wave takes long for its 16 samples with two classes a wave, and the more classes the sooner passes settle (24, labels at
    // random, 67 passes of 2048 samples; 6, 270).  4000 samples, D = 2000, us, one workgroup after another, by passes, blocks of 256:
    // 17 classes 2391, 2154, 1770; 24 2343, 1717, 1692, six tenths at random 2096, 1335, 1556; 32 2309, 1442, 1802.  In batches a workgroup
    // has no samples of its own to settle (24 classes, batches of 32, at random: 924, 1407, 1001).
    constexpr bool kPassesOnly = CPW == 2 && !BATCH;
    constexpr int kPasses = kPassesOnly ? kManyRounds : kRounds;
    // The first pass: no sample of the block counts yet.  Told before the lists are made, it is there when they are.
#pragma unroll
    for (int k = 0; k < CPW; ++k)
        if (own_class + k * kWaves < C && q == 0) s.cosine[own_class + k * kWaves][l] = cosine_of(start[k], nrm[k], inv_root_d);
    __syncthreads();
    if (wave == decider) {
        decide(zero_model);
        changed = true;
        if (lane == 0) s.own_changed = 1;
        tell_weights(slots);
    }

    for (int v = wave; v < classes; v += kWaves) {
        const int x = lane < kSpan / kWave ? sort.count[lane][v] : 0, sum = lane_sum(x);
        if (lane < kSpan / kWave) sort.count[lane][v] = (uint16_t)(sum - x);
        if (lane == kWave - 1) s.total[v] = sum;
    }
    __syncthreads();
    int all_groups;
    {
        const int g = lane < classes ? (s.total[lane] + kRunGroup - 1) / kRunGroup : 0, end = lane_sum(g);
        all_groups = __builtin_amdgcn_readlane(end, kWave - 1);
        if (wave == 0 && lane < classes) s.first_group[lane] = end - g;
        if (tid == 0) s.first_group[classes] = all_groups;
    }
    const int per = max(1, (all_groups + kLists - 1) / kLists);   // groups of a list
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (key[u] >= 0) {
            const int r = sort.count[wave + u * kWaves][key[u]] + rank[u], g = s.first_group[key[u]] + r / kRunGroup;
            s.src[g / per][g % per * kRunGroup + r % kRunGroup] = (uint16_t)(tid + u * kThreads);
            if (r % kRunGroup == 0) s.key[g] = (uint8_t)key[u];
        }
    __syncthreads();
    const int list = 4 * wave + q;
    int wsrc[(kSteps + 15) / 16];    // the samples whose weights this lane broadcasts
#pragma unroll
    for (int i = 0; i < (kSteps + 15) / 16; ++i) wsrc[i] = 16 * i + l < kSteps ? s.src[list][min(16 * i + l, kSteps - 1)] : kNone;
    constexpr int kFull = (CPW == 1 ? BATCH ? 2 : 3 : 1) * kRunGroup;   // products kept as fp64, the rest as fp32 (17 bits, to be widened in every pass): all of them would not fit the registers
    double kept[kFull];
    float half_kept[kSteps - kFull];
    each<kListGroups>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        if (g < per) {
            uint32_t n[2];
            __builtin_memcpy(n, &s.src[list][kRunGroup * g], 8);
#pragma unroll
            for (int u = 0; u < kRunGroup; ++u) {
                const int from = n[u >> 1] >> (16 * (u & 1)) & 0xFFFF;
                const int x = s.strip[min(from, kSpan - 1) * kOwn + l];
                const int product = from == kNone ? 0 : whole(x);
                if constexpr (kRunGroup * g < kFull)
                    kept[kRunGroup * g + u] = (double)product;
                else
                    half_kept[kRunGroup * g + u - kFull] = (float)product;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kRunGroup; ++u)
                if constexpr (kRunGroup * g < kFull)
                    kept[kRunGroup * g + u] = 0.0;
                else
                    half_kept[kRunGroup * g + u - kFull] = 0.0f;
        }
    });
    int dest = -1;   // lane g of a row: where its list's sum after group g goes, if a class ends there
    if (l < per && list * per + l < all_groups) {
        const int g = list * per + l, v = s.key[g];
        if (l == per - 1 || g + 1 == all_groups || s.key[g + 1] != v) dest = s.key[list * per] == v ? list : kLists + v;
    }
    const uint64_t any_dest = __ballot(dest >= 0);
    const uint32_t ends = (uint32_t)(any_dest | any_dest >> 16 | any_dest >> 32 | any_dest >> 48);   // groups after which a class ends in some row
    // A class's sum: head[class] if it begins inside a list, and the tails of the lists that begin with it.
    int from_list[CPW][BATCH ? 2 : 1], to_list[CPW][BATCH ? 2 : 1];
    bool begins[CPW][BATCH ? 2 : 1];
#pragma unroll
    for (int k = 0; k < CPW; ++k)
#pragma unroll
        for (int p = 0; p < (BATCH ? 2 : 1); ++p) {
            const int v = min(own_class + k * kWaves, C - 1) + p * C, a = s.first_group[v], b = s.first_group[v + 1];
            from_list[k][p] = __builtin_amdgcn_readfirstlane((a + per - 1) / per);
            to_list[k][p] = __builtin_amdgcn_readfirstlane((b + per - 1) / per);
            begins[k][p] = __builtin_amdgcn_readfirstlane(a % per != 0 && b > a);
        }
    const int fb = BATCH ? (n0 + l) / batch * batch : n0 + l;   // first sample that does not count for this lane's
    const int next_fb = BATCH ? (n0 + kOwn) / batch * batch : 0;   // start of the batch that runs on into the next workgroup
    const double dd = (double)D;

    // ---- passes, all workgroups together
    double grown[CPW][2] = {};             // of workgroups lane and lane + 64, as last heard
    double open[CPW] = {};                 // (batches) of the one the open batch begins in, up to there
    const int open_group = first_open / kOwn;
    const bool within = BATCH && first_open % kOwn != 0;   // the open batch begins inside that one's samples
    int wrong_per = 1;
    bool wrong_ones = false;
    int front = 0;                         // workgroups before this one are done: their weights have stopped changing
    auto wrong_key = [&](int n, int wrong) { return max(wrong, 0) + (BATCH && n >= first_open ? C : 0); };
    bool done = false;
    int r = 1;
    for (; r < kPasses; ++r) {
        asm volatile("" : "+v"(tid));   // (addresses are formed anew in a pass: kept over all, they would not fit the registers)
        lane = tid & (kWave - 1), l = lane & (kOwn - 1), q = lane / kOwn;
        Word *slot = slots + (r - 1) * words;
        int rank[kHeard];   // of the samples heard of: number within the class wrongly predicted, and that class
        if (wave < kHearing) {   // the weights of the samples before
            const int first = front * kOwn;
            Word v[kHeard], vp[kHeard];
            bool wanted[kHeard];
            int before[kHeard];
#pragma unroll
            for (int u = 0; u < kHeard; ++u) {
                const int n = tid + u * kHearing * kWave;
                const Word last = s.word[n];
                wanted[u] = n >= first && n < n0;
                v[u] = wanted[u] ? 0 : last;
                vp[u] = 0;
                before[u] = (int)(last >> 32 & 0xFF);
            }
            int tries = 0;
            for (; tries < kSpinLimit; ++tries) {
                bool missing = false;
#pragma unroll
                for (int u = 0; u < kHeard; ++u)
                    if (wanted[u] && !v[u]) {
                        v[u] = look(slot + tid + u * kHearing * kWave);
                        if (before[u]) vp[u] = look(slot + kSpan + tid + u * kHearing * kWave);   // (as a rule wrong again)
                    }
#pragma unroll
                for (int u = 0; u < kHeard; ++u) missing |= wanted[u] && !v[u];
                if (!__ballot(missing)) break;
            }
            if (__builtin_expect(tries == kSpinLimit, 0))
#pragma unroll
                for (int u = 0; u < kHeard; ++u)
                    if (!v[u]) v[u] = kLost;
            int told = group, flips = 0, wrong_here = 0;
            bool parts = false;
#pragma unroll
            for (int u = 0; u < kHeard; ++u) {
                const int n = tid + u * kHearing * kWave;
                const uint32_t hi = (uint32_t)(v[u] >> 32);
                s.count[wave + u * kHearing][lane] = 0;
                if (wanted[u]) s.word[n] = v[u];
                const uint64_t m = __ballot(wanted[u] && (hi & 0x100));
                if (m) told = min(told, ((wave + u * kHearing) * kWave + __builtin_ctzll(m)) / kOwn);
                const int wrong = (int)(hi & 0xFF) - 1;
                flips += __popcll(__ballot(wrong + 1 != before[u]));
                parts |= wanted[u] && (hi & 0x200);
                rank[u] = -1;
                if (const uint64_t any = __ballot(wrong >= 0)) {   // numbers of the samples a class was wrongly predicted for, by the ballots of 64
                    if (wanted[u] && wrong >= 0) {
                        if (!vp[u]) vp[u] = wait_for(slot + kSpan + n);
                        s.heard_wp[n] = __uint_as_float((uint32_t)(vp[u] ? vp[u] : kLost));
                    }
                    uint64_t same;
                    const int key = wrong_key(n, wrong), k = rank_of(key, wrong >= 0, same);
                    if (wrong >= 0 && k == 0) s.count[wave + u * kHearing][key] = (uint16_t)__popcll(same);
                    if (wrong >= 0) rank[u] = k << 8 | key;
                    wrong_here += __popcll(any);
                }
            }
            if (told < group && lane == 0) atomicMin(&s.front[r & 1], told);
            if (flips && lane == 0) atomicAdd(&s.flips[r & 1], flips);
            if (wrong_here && lane == 0) atomicAdd(&s.wrong[r & 1], wrong_here);
            if (parts) s.parting[r & 1] = 1;
        }
        __syncthreads();
        front = __builtin_amdgcn_readfirstlane(s.front[r & 1]);
        if (front == group && !s.own_changed) {
            done = true;
            break;
        }
        if (s.parting[r & 1]) break;
        // Where most predictions change at the second pass and most are wrong then, or half of them change at the third, a pass settles
        // few samples: the workgroups go on one after another (no passes tried: 1585 us; all of them first, 1685: 4000 samples of 6
        // classes, labels at random).  From rows that were trained on other labels, or that are none, most predictions change at
        // the second pass, because they are right then, and few at the third.  From zero rows of classes that are like one another
        // they change from the fourth pass on, and settle by the eighteenth: 110 us for the first 2048 samples, 510 one workgroup
        // after another.  They change among the earliest first, so that few samples before a workgroup say nothing (9 classes, 2197
        // samples, D = 2115: 310 us, and 775 where a workgroup after 256 samples asked at the fourth pass).
        parting = r + 1 == kPasses || (!kPassesOnly && ((r == 2 && 4 * s.flips[0] > 3 * n0 && 2 * s.wrong[0] > n0 && n0 >= 4 * kWave) ||
                                                        (r == 3 && 2 * s.flips[1] > n0 && n0 >= 8 * kWave)));
        wrong_ones = s.wrong[r & 1] != 0;
        if (wrong_ones)
            for (int v = wave; v < classes; v += kWaves) {
                const int x = lane < kSpan / kWave ? s.count[lane][v] : 0, sum = lane_sum(x);
                if (lane < kSpan / kWave) s.count[lane][v] = (uint16_t)(sum - x);
                if (lane == kWave - 1) s.wrong_end[v] = sum;
            }
        {
            double w[(kSteps + 15) / 16];
#pragma unroll
            for (int i = 0; i < (kSteps + 15) / 16; ++i) w[i] = (double)__uint_as_float((uint32_t)s.word[wsrc[i]]);
            double sum = 0.0;
            double *sums = &s.tail[0][l];   // (head follows tail)
            each<kListGroups>([&](auto g_) {
                constexpr int g = decltype(g_)::value;
                if (g < per) {
                    if constexpr (kRunGroup * g < kFull) {
                        add_rows<kRunGroup * g % 16, kRunGroup>(sum, w[kRunGroup * g / 16], kept + kRunGroup * g);
                    } else {
                        double x[kRunGroup];
#pragma unroll
                        for (int u = 0; u < kRunGroup; ++u) {
                            asm volatile("" : "+v"(half_kept[kRunGroup * g + u - kFull]));   // (not widened once and for all)
                            x[u] = (double)half_kept[kRunGroup * g + u - kFull];
                        }
                        add_rows<kRunGroup * g % 16, kRunGroup>(sum, w[kRunGroup * g / 16], x);
                    }
                    if (ends >> g & 1) {   // uniform
                        const int d = __builtin_amdgcn_update_dpp(0, dest, 0x150 + g, 0xF, 0xF, true);   // row_newbcast
                        if (d >= 0) {
                            sums[d * kOwn] = sum;
                            sum = 0.0;
                        }
                    }
                }
            });
        }
        __syncthreads();
        if (tid == 0) {
            s.front[(r + 1) & 1] = group;
            s.wrong[(r + 1) & 1] = s.flips[(r + 1) & 1] = 0;
        }
        if (wrong_ones) {   // listed class by class, then dealt to the rows of lanes in equal numbers, as the others are
            const int total = lane < classes ? s.wrong_end[lane] : 0, end = lane_sum(total);
            const int entries = __builtin_amdgcn_readlane(end, kWave - 1);
            wrong_per = (entries + kLists - 1) / kLists;
            if (wave < kHearing) {
#pragma unroll
                for (int u = 0; u < kHeard; ++u)
                    if (__ballot(rank[u] >= 0)) {
                        const int n = tid + u * kHearing * kWave, v = rank[u] & 0xFF, e0 = __shfl(end - total, v & (kWave - 1), kWave);
                        if (rank[u] >= 0)
                            s.named[e0 + s.count[wave + u * kHearing][v] + (rank[u] >> 8)] = make_uint2((uint32_t)(n | v << 16), __float_as_uint(s.heard_wp[n]));
                    }
            }
            __syncthreads();
            if (wave == 0 && lane < classes) s.wrong_end[lane] = end;
            const int e0 = list * wrong_per, e1 = min(e0 + wrong_per, entries);
            const int first = (int)(s.named[min(e0, kSpan - 1)].x >> 16);
            double sum = 0.0;
            for (int at = 0; at < wrong_per; at += kOwn) {   // 16 entries of a list: one to a lane of its row
                const int e = e0 + at + l;
                const uint2 x = s.named[min(e, kSpan - 1)];
                const int v = (int)(x.x >> 16), after = (int)(s.named[min(e + 1, kSpan - 1)].x >> 16);
                const int row = e < e1 ? (int)(x.x & 0xFFFF) * kOwn : 0;
                const double w = e < e1 ? -(double)__uint_as_float(x.y) : 0.0;
                const int goes = e < e1 && (e + 1 == e1 || after != v) ? v == first ? list : kLists + v : -1;
                const uint64_t m = __ballot(goes >= 0);
                const uint32_t stops = (uint32_t)(m | m >> 16 | m >> 32 | m >> 48);
                each<kOwn / 4>([&](auto i_) {
                    constexpr int i = 4 * decltype(i_)::value;
                    if (at + i < wrong_per) {
                        int16_t g[4];
                        each<4>([&](auto u_) {
                            constexpr int u = decltype(u_)::value;
                            g[u] = s.strip[__builtin_amdgcn_update_dpp(0, row, 0x150 + i + u, 0xF, 0xF, true) + l];   // row_newbcast
                        });
                        double x[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) x[u] = (double)whole(g[u]);
                        if (stops >> i & 15) each<4>([&](auto u_) {
                            constexpr int u = decltype(u_)::value;
                            add_rows<i + u, 1>(sum, w, x + u);
                            if (stops >> (i + u) & 1) {   // uniform
                                const int d = __builtin_amdgcn_update_dpp(0, goes, 0x150 + i + u, 0xF, 0xF, true);
                                if (d >= 0) {
                                    (&s.wrong_tail[0][l])[d * kOwn] = sum;   // (wrong_head follows)
                                    sum = 0.0;
                                }
                            }
                        });
                        else add_rows<i, 4>(sum, w, x);
                    }
                });
            }
            __syncthreads();
        }
        const uint32_t wrong_inverse = ((1u << 20) + wrong_per - 1) / wrong_per;   // (numbers up to 2100, divided by up to 32)
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = own_class + k * kWaves;
            if (c < C) {
                double old = 0.0, late = 0.0;   // from samples before; of those, from the open batch's
#pragma unroll
                for (int p = 0; p < (BATCH ? 2 : 1); ++p) {
                    const double head = s.head[c + p * C][l];
                    double t = begins[k][p] && q == 0 ? head : 0.0;
#pragma unroll 1
                    for (int i0 = from_list[k][p]; i0 < to_list[k][p]; i0 += 16) {
                        double v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = s.tail[min(i0 + 4 * u + q, kLists - 1)][l];
#pragma unroll
                        for (int u = 0; u < 4; ++u) t += i0 + 4 * u + q < to_list[k][p] ? v[u] : 0.0;
                    }
                    if (wrong_ones) {
                        const int v = c + p * C, e1 = s.wrong_end[v], e0 = v ? s.wrong_end[max(v - 1, 0)] : 0;
                        const int i0 = (int)((uint32_t)(e0 + wrong_per - 1) * wrong_inverse >> 20);   // first list that begins with the class
                        if (e1 > e0 && i0 * wrong_per != e0 && q == 0) t += s.wrong_head[v][l];
#pragma unroll 1
                        for (int i = i0 + q; i * wrong_per < e1; i += 4) t += s.wrong_tail[i][l];
                    }
                    (p ? late : old) = t;
                }
                double every = old + late, dot = old + (BATCH && fb <= n0 ? 0.0 : late);
#pragma unroll
                for (int u = 0; u < kOwn / 4; ++u) {   // its own samples, four to a row of lanes
                    const int n = 4 * q + u;
                    const int2 of = s.own_class[n];
                    const double2 w = s.own_w[n];
                    const double g = (double)whole(s.strip[(n0 + n) * kOwn + l]);
                    const double x = of.x == c ? w.x : of.y == c ? w.y : 0.0;
                    every = fma(x, n < l ? g : 0.0, every);
                    if (BATCH) dot = fma(x, n0 + n < fb ? g : 0.0, dot);
                }
                const double from_start = s.start[c][l];
                every = from_start + sum_rows(every);
                dot = BATCH ? from_start + sum_rows(dot) : every;
                const int2 of = s.own_class[l];
                const double2 w = s.own_w[l];
                const double x = of.x == c ? w.x : of.y == c ? w.y : 0.0;
                const double run = row_prefix(x * fma(x, dd, 2.0 * every));   // what the samples up to each add to the squared norm
                Word *norms = slot + 2 * kSpan + (int64_t)c * kGroups, *opens = norms + (int64_t)C * kGroups;
                const double run_open = BATCH && next_fb > n0 ? lane_f64(run, min(next_fb - n0, kOwn) - 1) : 0.0;
                if (lane == kOwn - 1) {
                    tell(norms + group, norm_word(run));
                    if (BATCH) tell(opens + group, norm_word(run_open));
                    s.mine[c] = make_double2(run, run_open);
                }
                Word v[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) v[u] = lane + u * kWave >= front && lane + u * kWave < group ? look(norms + lane + u * kWave) : 1;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (!v[u]) v[u] = wait_for(norms + lane + u * kWave);
                    if (lane + u * kWave >= front && lane + u * kWave < group) grown[k][u] = word_norm(v[u]);
                }
                if (within && open_group >= front && open_group < group) open[k] = word_norm(wait_for(opens + open_group));
                const double before = row_before(run), base = s.nrm[c] + sum_lanes(grown[k][0] + grown[k][1]);
                double nn = base + before;
                if (BATCH) {
                    const double until = (lane < open_group ? grown[k][0] : 0.0) + (lane + kWave < open_group ? grown[k][1] : 0.0);
                    const double at_open = s.nrm[c] + sum_lanes(until) + (within ? open[k] : 0.0);
                    const double at_fb = __shfl(before, min(max(fb - n0, 0), kOwn - 1), kWave);
                    nn = fb >= n0 ? base + at_fb : at_open;
                }
                const double cs = cosine_of(dot, nn, inv_root_d);
                if (q == 0) s.cosine[c][l] = cs;
            }
        }
        __syncthreads();
        if (wave == decider) {
            decide(false);
            if (r + 1 < kPasses) tell_weights(slots + r * words);
        }
        if (parting) break;
    }
    Word *slot = slots + (slots_of(C) - 1) * words;   // the last one: weights and squared norms for good
    if (done) {
        if (wave == decider) {
            changed = parting = false;
            tell_weights(slot);
        }
        if (wave == 0 && lane < C) {
            Word *norms = slot + 2 * kSpan + (int64_t)lane * kGroups;
            tell(norms + group, norm_word(s.mine[lane].x));
            if (BATCH) tell(norms + (int64_t)C * kGroups + group, norm_word(s.mine[lane].y));
        }
        if (wave == decider && lane < kOwn && n0 + l < nb)
            out[n0 + l] = OnlineWeight{s.own_class[l].x, s.own_class[l].y, (float)s.own_w[l].x, (float)-s.own_w[l].y};
        if (group == groups - 1 && tid == 0) state[1] = r;   // slots in use (no other workgroup takes more passes)
        return;
    }

    // ---- Where many predictions are wrong passes settle few samples each: the rest one workgroup after another, in
    // batches one batch after another.  What the samples before add is summed as it becomes known (a wave its classes, four
    // samples to a row of lanes); then one wave finds the fixed point of the 16 samples by itself.
    __syncthreads();
    const bool one_batch = BATCH && first_open + batch >= n0 + kOwn;   // its samples are all of the open batch: the others of it do not count for their cosines
    const int last = one_batch ? open_group + within : group;   // workgroups before this one do
    const int turn = (l + 4 * q) & (kOwn - 1);       // lanes 0 to 3 of a row: its four samples
    double old[CPW] = {}, late[CPW] = {};
    bool lost = false;   // a wait was given up
    auto add = [&](int j, double (&norm)[CPW], double (&norm_open)[CPW], bool ask_norm) {
        const int n = j * kOwn + turn;
        double p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = (double)whole(s.strip[(j * kOwn + 4 * q + u) * kOwn + l]);
        Word v = s.word[n];
        float wp = s.heard_wp[n];
        if (j >= front) {   // uniform
            const bool norms = ask_norm;
            Word vp = 0, vn[CPW] = {};
            v = 0;
            int tries = 0;
            for (; tries < kSpinLimit; ++tries) {   // all that is to come at once
                if (!v) v = look(slot + n);
                if (!vp) vp = look(slot + kSpan + n);
                bool missing = !v || (((uint32_t)(v >> 32) & 0xFF) && !vp);
#pragma unroll
                for (int k = 0; k < CPW; ++k) {
                    const int c = own_class + k * kWaves;
                    if (norms && c < C && !vn[k]) vn[k] = look(slot + 2 * kSpan + (int64_t)c * kGroups + j);
                }
#pragma unroll
                for (int k = 0; k < CPW; ++k) missing |= norms && own_class + k * kWaves < C && !vn[k];
                if (!__ballot(missing)) break;
                if (group - j > 8) __builtin_amdgcn_s_sleep(8);
            }
            lost |= tries == kSpinLimit;
            wp = __uint_as_float((uint32_t)vp);
#pragma unroll
            for (int k = 0; k < CPW; ++k)
                if (norms && own_class + k * kWaves < C) {
                    const double more = word_norm(vn[k]);
                    norm[k] += more;
                    if (j < open_group) norm_open[k] += more;
                }
        }
        const int pred = (int)(v >> 32 & 0xFF) - 1, label = s.label[n];
        const bool is_late = BATCH && n >= first_open;
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = own_class + k * kWaves;
            const double x = label == c ? (double)__uint_as_float((uint32_t)v) : pred == c ? -(double)wp : 0.0;
            add_rows<0, 4>(old[k], is_late ? 0.0 : x, p);
            if (BATCH) add_rows<0, 4>(late[k], is_late ? x : 0.0, p);
        }
    };
    if (own_class < C) {
        double norm[CPW], norm_open[CPW];
        const int known = min(front, open_group);
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const double start_norm = s.nrm[min(own_class + k * kWaves, C - 1)];
            norm[k] = start_norm + sum_lanes((lane < front ? grown[k][0] : 0.0) + (lane + kWave < front ? grown[k][1] : 0.0));
            norm_open[k] = start_norm + sum_lanes((lane < known ? grown[k][0] : 0.0) + (lane + kWave < known ? grown[k][1] : 0.0));
        }
        for (int j = 0; j < last; ++j) add(j, norm, norm_open, !one_batch || j < open_group);
        if (__builtin_expect(lost, 0))
#pragma unroll
            for (int k = 0; k < CPW; ++k) old[k] = __builtin_nan("");
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = own_class + k * kWaves;
            if (c < C) {
                if (within)
                    norm_open[k] += open_group < front ? open[k] : word_norm(wait_for(slot + 2 * kSpan + (int64_t)(C + c) * kGroups + open_group));
                const double from_start = s.start[c][l], all = from_start + sum_rows(old[k] + late[k]);
                const double counts = BATCH && fb <= n0 ? from_start + sum_rows(old[k]) : all;
                if (q == 0) {
                    s.tail[c][l] = all;          // (the sums of the passes are used up)
                    s.head[c][l] = counts;
                }
                if (lane == 0) {
                    s.wrong_tail[c][0] = norm[k];
                    s.wrong_head[c][0] = norm_open[k];
                }
            }
        }
    }
    // The settling wave's products of the 16 samples with one another, on their way while others wait for the last weights: it has
    // class 15, so none of its own with fewer.
    constexpr int kSettler = kWaves - 1 - kHearing;
    double product[kOwn] = {};
    if (wave == kSettler && !one_batch) {
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            const double g = (double)whole(s.strip[(n0 + u) * kOwn + l]);
            product[u] = u < l ? g : 0.0;
        }
    }
    __syncthreads();
    if (one_batch) {   // no sample of its own counts: cosines at once; then what it adds to the squared norms
        for (int c = wave; c < C; c += kWaves)
            if (q == 0) s.cosine[c][l] = cosine_of(s.head[c][l], s.wrong_head[c][0], inv_root_d);
        __syncthreads();
        if (wave == decider) {
            decide(false);
            changed = parting = false;
            tell_weights(slot);
            if (lane < kOwn && n0 + l < nb)
                out[n0 + l] = OnlineWeight{s.own_class[l].x, s.own_class[l].y, (float)s.own_w[l].x, (float)-s.own_w[l].y};
        }
        __syncthreads();
        if (own_class < C) {
            double unused[CPW];
            for (int j = last; j < group; ++j) add(j, unused, unused, false);
            if (__builtin_expect(lost, 0))
#pragma unroll
                for (int k = 0; k < CPW; ++k) old[k] = __builtin_nan("");
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                const int c = own_class + k * kWaves;
                if (c < C) {
                    double every = old[k] + late[k];
#pragma unroll
                    for (int u = 0; u < kOwn / 4; ++u) {
                        const int n = 4 * q + u;
                        const int2 of = s.own_class[n];
                        const double2 w = s.own_w[n];
                        const double g = (double)whole(s.strip[(n0 + n) * kOwn + l]);
                        every = fma(of.x == c ? w.x : of.y == c ? w.y : 0.0, n < l ? g : 0.0, every);
                    }
                    every = s.start[c][l] + sum_rows(every);
                    const int2 of = s.own_class[l];
                    const double2 w = s.own_w[l];
                    const double x = of.x == c ? w.x : of.y == c ? w.y : 0.0, run = row_prefix(x * fma(x, dd, 2.0 * every));
                    if (lane == kOwn - 1) {
                        Word *norms = slot + 2 * kSpan + (int64_t)c * kGroups;
                        tell(norms + group, norm_word(run));
                        tell(norms + (int64_t)C * kGroups + group, norm_word(next_fb > n0 ? run : 0.0));
                    }
                }
            }
        }
        if (group == groups - 1 && tid == 0) state[1] = kPasses;
        return;
    }
    if (wave != kSettler) return;
    if constexpr (CPW == 2) {
        settle_own<BATCH ? 2 : 4, BATCH ? 4 : 2, BATCH>(s, product, n0, fb, next_fb, C, dd, lr, inv_root_d);
    } else {
        if (C <= 4)
            settle_own<1, 1, BATCH>(s, product, n0, fb, next_fb, C, dd, lr, inv_root_d);
        else if (C <= 8)
            settle_own<2, 1, BATCH>(s, product, n0, fb, next_fb, C, dd, lr, inv_root_d);
        else
            settle_own<BATCH ? 2 : 4, BATCH ? 2 : 1, BATCH>(s, product, n0, fb, next_fb, C, dd, lr, inv_root_d);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int2 of = s.own_class[l];
    const double2 w = s.own_w[l];
    if (q == 0) {
        if (of.y >= 0) tell(slot + kSpan + n0 + l, 1ull << 32 | __float_as_uint((float)-w.y));
        tell(slot + n0 + l, 1ull << 63 | (Word)(of.y + 1) << 32 | __float_as_uint((float)w.x));
        if (n0 + l < nb) out[n0 + l] = OnlineWeight{of.x, of.y, (float)w.x, (float)-w.y};
    }
    if (lane < C) {
        Word *norms = slot + 2 * kSpan + (int64_t)lane * kGroups;
        tell(norms + group, norm_word(s.mine[lane].x));
        if (BATCH) tell(norms + (int64_t)C * kGroups + group, norm_word(s.mine[lane].y));
    }
    if (group == groups - 1 && lane == 0) state[1] = kPasses;
}

// ---- the rows ------------------------------------------------------------------------------------
// A block per group of 64 dimensions, class c is wave c % 16's.  A lane keeps one element of a row in a register and takes the
// updates that name its class in sample order, one fp32 add each (in batches an fp64 sum a batch and one rounding).
// The chain of additions is what bounds it, so all else is kept off it: the block lists the updates class after
// class (as the workgroups of the chain do the samples before), a wave takes 64 of them at a time, turns their
// 64 x 64 bits so that a lane has those of its dimension, and an update is three instructions, the last of which reads its weight from another
// lane and adds it: a shift, the sign put on 1.0, a multiply-add (exact: the product is +-weight).  The block clears its share of the slots, too.
struct UpdateShared {
    uint2 list[2 * kSpan];             // sample, weight: class after class
    uint16_t count[kSpan / kWave][kMaxClasses];
    int total[kMaxClasses];
};

// A 64 x 64 matrix of bits, row i in lane i's (lo, hi), turned: column i.
__device__ __forceinline__ void transpose_bits(uint32_t &lo, uint32_t &hi) {
    const int lane = threadIdx.x & (kWave - 1);
    {
        const auto h = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);   // rows 0 to 31; 32 to 63: of dimensions 0 to 31 in the lower lanes
        lo = h[0];
        hi = h[1];
    }
    const uint32_t pick16 = lane & 16 ? 0x07060302u : 0x05040100u, pick8 = lane & 8 ? 0x03070105u : 0x06020400u;
    uint32_t *const half[2] = {&lo, &hi};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t x = *half[i];
        const auto h = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = __builtin_amdgcn_perm(h[1], h[0], pick16);
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true);   // row_ror:8
        x = __builtin_amdgcn_perm(y, x, pick8);
        auto step = [&](uint32_t other, int width, uint32_t keep) {   // the lane that differs in bit `width`
            const bool up = lane & width;
            const uint32_t moved = up ? other >> width : other << width, mask = up ? ~keep : keep;
            x = (x & mask) | (moved & ~mask);
        };
        const int mirrored = __builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);           // row_half_mirror: lane ^ 7
        step((uint32_t)__builtin_amdgcn_update_dpp(0, mirrored, 0x1B, 0xF, 0xF, true), 4, 0x0F0F0F0Fu);   // quad_perm 3,2,1,0: lane ^ 3
        step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true), 2, 0x33333333u);     // quad_perm 2,3,0,1
        step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true), 1, 0x55555555u);     // quad_perm 1,0,3,2
        *half[i] = x;
    }
}

__device__ __forceinline__ uint32_t signed_one(uint32_t bits, uint32_t sign, uint32_t one) {
    return __builtin_amdgcn_bitop3_b32(bits, sign, one, 0xEA);   // bits & sign | one
}

// a += w of lane (16 j + I) x s, in every row of 16 lanes j.
template <int I>
__device__ __forceinline__ void add_update(float &a, float w, float s) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(a) : "v"(w), "v"(s), "n"(I));
}

// A workgroup per 64 dimensions, a wave per class, a lane per dimension.  What bounds it is the chain of additions to an element, in
// sample order: about 340 of them a class for 2048 samples of 6.  The samples' bits are transposed once (a word per lane is 32
// samples of its dimension), so that an addition is a sign of one instruction and a multiply-add that takes the weight from a lane of
// its row by DPP.  2048 samples, 6 classes, D = 10000: 10.9 us, and 16.3 in batches of 64 (fp64 sums, one rounding a batch);
// with a lane's bit and weight fetched for every addition 17.3 and 29.5.
template <bool BATCH>
__global__ __launch_bounds__(kThreads) void online_update_kernel(const uint64_t *__restrict__ col, int64_t ld, int nb, int batch,
                                                                 const OnlineWeight *__restrict__ recs, float *acc, int D, int C, int G,
                                                                 double *__restrict__ normpart, Word *__restrict__ slots, int *__restrict__ state) {
    __shared__ UpdateShared s;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), l = lane & 15, g = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    OnlineWeight r[2];   // of samples tid and tid + kThreads
#pragma unroll
    for (int u = 0; u < 2; ++u) r[u] = recs[min(tid + u * kThreads, nb - 1)];
    const int d = g * kWave + lane;
    float first = 0.0f;  // the element of the wave's first class
    if (d < D && wave < C) first = acc[(int64_t)wave * D + d];
    reinterpret_cast<uint32_t *>(&s.count[0][0])[tid & (kSpan / kWave * kMaxClasses / 2 - 1)] = 0;
    {
        const int64_t words = slot_words(C), last = (slots_of(C) - 1) * words, used = min(state[1] * words, last), end = last - used;   // and the last one
        for (int64_t i = (int64_t)blockIdx.x * kThreads + tid; i < used + words; i += (int64_t)gridDim.x * kThreads)
            slots[i < used ? i : i + end] = 0;
        if (blockIdx.x == 0 && tid == 0) state[0] = 0;
    }
    __syncthreads();
    // numbers within a class's list, of both classes a sample may name
    int rank[2][2], key[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const bool in = tid + u * kThreads < nb;
        key[u][0] = in && r[u].y >= 0 && r[u].w_y != 0.0f ? r[u].y : -1;
        key[u][1] = in && r[u].pred >= 0 && r[u].w_p != 0.0f ? r[u].pred : -1;
        uint64_t named[2] = {__ballot(key[u][0] >= 0), __ballot(key[u][1] >= 0)}, with[2][2] = {{named[0], named[1]}, {named[0], named[1]}};
#pragma unroll
        for (int b = 0; b < 5; ++b)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint64_t m = __ballot(key[u][j] >> b & 1);
#pragma unroll
                for (int i = 0; i < 2; ++i) with[i][j] &= key[u][i] >> b & 1 ? m : ~m;
            }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint64_t same = with[i][0] | with[i][1];   // samples that name the class
            rank[u][i] = __popcll(same & ((1ull << lane) - 1));
            if (key[u][i] >= 0 && rank[u][i] == 0) s.count[wave + u * kWaves][key[u][i]] = (uint16_t)__popcll(same);
        }
    }
    __syncthreads();
    for (int c = wave; c < C; c += kWaves) {
        const int x = lane < kSpan / kWave ? s.count[lane][c] : 0, sum = lane_sum(x);
        if (lane < kSpan / kWave) s.count[lane][c] = (uint16_t)(sum - x);
        if (lane == kWave - 1) s.total[c] = sum;
    }
    __syncthreads();
    const int total = lane < C ? s.total[lane] : 0, end = lane_sum(total);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int at = __shfl(end - total, max(key[u][i], 0), kWave);
            if (key[u][i] >= 0)
                s.list[at + s.count[wave + u * kWaves][key[u][i]] + rank[u][i]] =
                    make_uint2((uint32_t)(tid + u * kThreads), __float_as_uint(i ? -r[u].w_p : r[u].w_y));
        }
    __syncthreads();
    uint32_t sign = 0x80000000u, one = BATCH ? 0x3FF00000u : 0x3F800000u;   // 1.0's upper word, 1.0f
    asm volatile("" : "+v"(sign), "+v"(one));   // (in registers: an instruction takes one constant at most)
    const uint32_t inverse = ((1u << 20) + batch - 1) / batch;   // samples' batches: numbers below 2048, divided by up to 256 (right up to 512)
    for (int c = wave; c < C; c += kWaves) {
        const int entries = __builtin_amdgcn_readlane(total, c);
        const uint2 *list = s.list + __builtin_amdgcn_readlane(end, c) - entries;
        float a = c == wave ? first : d < D ? acc[(int64_t)c * D + d] : 0.0f;
        double delta = 0.0;
        uint64_t bits = 0;
        if (entries) bits = col[(int64_t)g * ld + list[min(lane, entries - 1)].x];
        for (int e0 = 0; e0 < entries; e0 += kWave) {
            uint32_t lo = ~(uint32_t)bits, hi = ~(uint32_t)(bits >> 32);   // set: subtract
            if (e0 + kWave < entries) bits = col[(int64_t)g * ld + list[min(e0 + kWave + lane, entries - 1)].x];
            float w[4];   // 16 entries in every row of lanes; past the end weight 0
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint2 x = list[min(e0 + 16 * i + l, entries - 1)];
                w[i] = e0 + 16 * i + l < entries ? __uint_as_float(x.y) : 0.0f;
            }
            uint64_t ends = 0;     // (batches) entries after which another batch begins
            if (BATCH) {
                const int e = min(e0 + lane, entries - 1);
                const uint32_t here = list[e].x * inverse >> 20, after = list[min(e + 1, entries - 1)].x * inverse >> 20;
                ends = __ballot(e0 + lane < entries && (e + 1 == entries || here != after));
            }
            transpose_bits(lo, hi);
            each<4>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
                if (e0 + 16 * i < entries) {   // uniform
                    const uint32_t m = i < 2 ? lo : hi;
                    if constexpr (BATCH) {
                        const double w64 = (double)w[i];
                        const uint32_t stops = (uint32_t)(ends >> (16 * i));
                        each<4>([&](auto j_) {
                            constexpr int j = 4 * decltype(j_)::value;
                            double x[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                x[u] = __hiloint2double((int)signed_one(m << (31 - (16 * (i & 1) + j + u)), sign, one), 0);
                            if (stops >> j & 15)
                                each<4>([&](auto u_) {
                                    constexpr int u = decltype(u_)::value;
                                    add_rows<j + u, 1>(delta, w64, x + u);
                                    if (stops >> (j + u) & 1) {   // uniform
                                        asm volatile("");         // (a branch: selects would be on every addition's way)
                                        a = (float)((double)a + delta);
                                        delta = 0.0;
                                    }
                                });
                            else
                                add_rows<j, 4>(delta, w64, x);
                        });
                    } else {
                        each<16>([&](auto u_) {
                            constexpr int u = decltype(u_)::value;
                            add_update<u>(a, w[i], __uint_as_float(signed_one(m << (31 - (16 * (i & 1) + u)), sign, one)));
                        });
                    }
                }
            });
        }
        double p = 0.0;
        if (d < D) {
            acc[(int64_t)c * D + d] = a;
            p = (double)a * (double)a;
        }
        p = lane_prefix(p);
        if (lane == kWave - 1) normpart[(int64_t)c * G + g] = p;
    }
}

constexpr float kTameSpread = 1e30f;   // a learning rate below which no weight overflows

int64_t held_spans(int G) { return std::max<int64_t>(1, std::min<int64_t>(8, held_samples(G) / kSpan)); }

template <int CPW, bool BATCH>
int launch_spread(hdc_ctx_impl *c, const int16_t *strips, int slices, int nb, int batch, const int32_t *labels, int G, float lr, hipStream_t s) {
    auto kern = online_spread_kernel<CPW, BATCH>;
    const int slot = (CPW - 1) * 2 + BATCH;
    if (!c->os_attr_set[slot]) {
        HDC_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SpreadShared)));
        c->os_attr_set[slot] = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((nb + kOwn - 1) / kOwn)), dim3(kThreads), sizeof(SpreadShared), s, strips, c->os_part_d, slices, nb, batch,
                       labels, c->ob_norm_d, G, c->p.C, c->p.D, lr, 1.0 / sqrt((double)c->p.D), (Word *)c->os_slots_d, c->os_state_d,
                       static_cast<OnlineWeight *>(c->os_rec_d));
    HDC_HIP(hipGetLastError());
    return HDC_OK;
}

}  // namespace

// What a call needs beside the blocks' scratch (reserve_online_chain).
int reserve_online_spread(hdc_ctx_impl *c) {
    if (c->os_ready || c->p.C > kMaxClasses) return HDC_OK;
    const int C = c->p.C, D = c->p.D, G = (D + kWave - 1) / kWave;
    const int slices = row_dots_slices(D, kDotSlices);
    const size_t slot_bytes = (size_t)slots_of(C) * slot_words(C) * sizeof(Word);
    struct { void **at; size_t bytes; } parts[] = {
        {(void **)&c->os_slots_d, slot_bytes + 256},
        {(void **)&c->os_strips_d, (size_t)held_spans(G) * kSpanProducts * sizeof(int16_t)},
        {(void **)&c->os_part_d, (size_t)slices * C * kSpan * sizeof(double)},
        {(void **)&c->os_rec_d, (size_t)kSpan * sizeof(OnlineWeight)},
    };
    size_t want = 0;
    for (const auto &p : parts) want += (p.bytes + 255) / 256 * 256;
    const int rc = grow(&c->os_mem_d, &c->os_mem_bytes, want);
    if (rc != HDC_OK) return rc;
    char *next = c->os_mem_d;
    for (const auto &p : parts) {
        *p.at = next;
        next += (p.bytes + 255) / 256 * 256;
    }
    c->os_state_d = reinterpret_cast<int *>(c->os_mem_d + slot_bytes);
    HDC_HIP(hipMemset(c->os_mem_d, 0, slot_bytes + 256));   // from here on the kernels leave the slots as they found them
    HDC_HIP(hipStreamSynchronize(nullptr));
    c->os_ready = true;
    return HDC_OK;
}

// Calls of more samples than a few blocks of 256 hold (batch 0: per sample).  A batch costs three launches of its own otherwise,
// about 14 us, and here a call about 100 us and each block 70, whatever the batch: so many batches it must have.  (Here against
// three launches a batch, us, D = 2000 and 3 classes: 2000 samples in 16 batches 170 and 204, in 11 178 and 148; 8000 in 32 378
// and 466; 4000 in 16 234 and 230; 1100 in 18, of 12 classes, 184 and 173.)  With more than 16 classes a wave takes two, and batches
// are those that fill a workgroup (1000 dimensions, 32 classes, 4100 samples in batches of 5: 2092 as before).
bool online_spread_pays(const hdc_ctx_impl *c, int64_t N, int64_t batch) {
    if (c->p.C > kMaxClasses || c->p.D > 65535 || N <= 1024) return false;
    if (batch == 0) return true;
    const bool few = c->p.C <= kWaves;
    return batch <= 256 && N >= (few ? 1280 : 1536) && N >= (8 + 5 * ((N + kSpan - 1) / kSpan)) * batch && (few || batch >= kOwn);
}

bool online_spread_takes(const hdc_ctx_impl *c, int64_t N, float lr, int64_t batch, bool per_sample) {
    return c->os_ready && online_spread_pays(c, N, per_sample ? 0 : batch) && fabsf(lr) < kTameSpread;
}

template <bool BATCH>
int launch_online_spread(hdc_ctx_impl *c, const uint32_t *hv, const int32_t *labels, int64_t N, int32_t epochs, float lr, int batch,
                         float *acc, hipStream_t s) {
    const int C = c->p.C, D = c->p.D, W = c->W, G = (D + kWave - 1) / kWave;
    int slices;
    ProfScope walk(c, HDC_K_ONLINE, s, !BATCH);   // a walk by samples as a whole; of batches each block's three steps
    ProfScope spread(c, HDC_K_ONLINE_SPREAD, s);
    int rc = launch_norm(c, acc, G, s);
    if (rc != HDC_OK) return rc;
    const int block = kSpan / batch * batch;   // whole batches
    const int64_t ld = held_samples(G), held = std::max<int64_t>(1, std::min<int64_t>(ld / block, held_spans(G))) * block;
    for (int32_t e = 0; e < epochs; ++e)
        for (int64_t h0 = 0; h0 < N; h0 += held) {
            const int64_t hn = N - h0 < held ? N - h0 : held;
            if (e == 0 || N > held) {   // a set that fits is multiplied out once for all epochs
                launch_columns(c, hv + h0 * W, hn, ld, s);
                HDC_HIP(hipGetLastError());
                launch_strips(c, hn, ld, block, c->os_strips_d, s);
                HDC_HIP(hipGetLastError());
            }
            for (int64_t b0 = 0; b0 < hn; b0 += block) {
                const int nb = (int)std::min<int64_t>(block, hn - b0);
                const uint64_t *col = c->oc_col_d + b0;
                {
                    ProfScope prof(c, HDC_K_ONLINE_FWD, s, BATCH);
                    rc = launch_row_dots(c, hv + (h0 + b0) * W, nb, acc, c->os_part_d, (int64_t)C * kSpan, 1, kSpan, nullptr, kDotSlices, &slices, s);
                }
                if (rc != HDC_OK) return rc;
                {
                    ProfScope prof(c, HDC_K_ONLINE, s, BATCH);
                    const int16_t *strips = c->os_strips_d + b0 / block * kSpanProducts;
                    rc = C <= kWaves ? launch_spread<1, BATCH>(c, strips, slices, nb, batch, labels + h0 + b0, G, lr, s)
                                     : launch_spread<2, BATCH>(c, strips, slices, nb, batch, labels + h0 + b0, G, lr, s);
                }
                if (rc != HDC_OK) return rc;
                {
                    ProfScope prof(c, HDC_K_ONLINE_BWD, s, BATCH);
                    hipLaunchKernelGGL(online_update_kernel<BATCH>, dim3((unsigned)G), dim3(kThreads), 0, s, col, ld, nb, batch,
                                       static_cast<const OnlineWeight *>(c->os_rec_d), acc, D, C, G, c->ob_norm_d, (Word *)c->os_slots_d,
                                       c->os_state_d);
                }
                HDC_HIP(hipGetLastError());
            }
        }
    return HDC_OK;
}
template int launch_online_spread<false>(hdc_ctx_impl *, const uint32_t *, const int32_t *, int64_t, int32_t, float, int, float *, hipStream_t);
template int launch_online_spread<true>(hdc_ctx_impl *, const uint32_t *, const int32_t *, int64_t, int32_t, float, int, float *, hipStream_t);

}  // namespace hdc
