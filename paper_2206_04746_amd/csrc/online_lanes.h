// Device functions that the block-wise online trainers share (online_chain.hip, online_spread.hip).
#pragma once

#include <algorithm>
#include <type_traits>

#include "hdc_internal.h"
#include "online_weight.h"

namespace hdc {

// f(0), f(1) ... f(N - 1) with the number as a type
template <int N, int I = 0, typename F>
__device__ __forceinline__ void each(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<N, I + 1>(f);
    }
}

// ---- lanes ------------------------------------------------------------------------------------------
__device__ __forceinline__ float lane_f32(float v, int i) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, ROWS == 0xF);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, ROWS == 0xF);
    return v + __hiloint2double(hi, lo);
}
// Inclusive sum over the lanes: four shifts within a row of 16, then the row totals.
__device__ __forceinline__ double lane_prefix(double v) {
    v = dpp_add<0x111, 0xF>(v);   // row_shr:1
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ double lane_f64(double v, int i) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i),
                            __builtin_amdgcn_readlane(__double2loint(v), i));
}
// The value of the lane before (lane 0: zero).
__device__ __forceinline__ double lane_before(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xF, 0xF, true);   // wave_shr:1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
// Sum over the lanes up to this one.
__device__ __forceinline__ int lane_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);    // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15, 31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}

// acc += w of lane (16 k + I) x g, in every row of 16 lanes k, for GR rows.  (Such a broadcast wants two wait states
// after a vector write of its operand; five after one of the execution mask by the vector unit, of which there is none.)
template <int I, int GR>
__device__ __forceinline__ void add_rows(double &acc, double w, const double *g) {
    if constexpr (GR == 4)
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %0, %1, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %0, %1, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %0, %1, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc) : "v"(w), "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
    else if constexpr (GR == 1)
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(w), "v"(g[0]), "n"(I));
    else
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%4 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %0, %1, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc) : "v"(w), "v"(g[0]), "v"(g[1]), "n"(I), "n"(I + 1));
}

// ---- the chain sample by sample -------------------------------------------------------------------
__device__ __forceinline__ double refined_rsq(double nn) {
    double r = __builtin_amdgcn_rsq(nn);
    r = r * fma(-0.5 * nn * r, r, 1.5);
    return r * fma(-0.5 * nn * r, r, 1.5);
}

// The samples of a block one after another: a wave's lanes deal the samples before among them for each of
// its classes, and the decision is taken class by class, as in the kernels that walk sample by sample
// (BATCH: as in the batched trainer, which passes over classes whose cosine is no number).  cosv: [C] in LDS.
// product(n, m): of samples n < m.  part: [slice][class][span].
// A longer block goes in panels of up to kPanel samples, whole batches: what the samples before a panel add to its dot products is summed
// at once, 64 samples of the panel side by side, and lies in `sums` ([C][kPanel] in LDS) with the products at the block's start.  2000
// samples, 6 classes, D = 1000: 10.2 ms where each sample is added to by all before it, 4.0 so, 3.6 in blocks of 256 (batches of 20: 11.0, 4.5, 3.7).
constexpr int kPanel = 256;

template <int CPW, bool BATCH, typename Product>
__device__ __noinline__ void walk_block(Product product, const double *__restrict__ part, int span, int slices, int nb, int batch,
                           const int32_t *__restrict__ labels, const double *__restrict__ normpart, const double *before,
                           double *grown, int G, int C, int D, float lr, double inv_root_d, OnlineWeight *rec, double *cosv,
                           double *sums = nullptr) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double nrm[CPW], frozen[CPW], at_start[CPW];   // squared norms now, where the batch began, where the block did
    for (int k = 0; k < CPW; ++k) {
        const int c = wave * CPW + k;
        double s = 0.0;
        for (int g = lane; g < G && c < C; g += kWave) s += normpart[(int64_t)c * G + g];
        nrm[k] = frozen[k] = lane_f64(lane_prefix(s), kWave - 1) + (before && c < C ? before[c] : 0.0);
        at_start[k] = nrm[k];
    }
    const int panel = Product::kPanels ? (BATCH ? kPanel / batch * batch : kPanel) : nb;
    int p0 = 0;   // first sample of the panel
    for (int m = 0; m < nb; ++m) {
        const int first = BATCH ? m / batch * batch : m;
        if (Product::kPanels && m % panel == 0) {
            p0 = m;
            __syncthreads();   // the record before is there
#pragma unroll 1
            for (int k = 0; k < CPW; ++k) {
                const int c = wave * CPW + k;
                if (c >= C) continue;
                double sum[kPanel / kWave] = {};   // of samples p0 + lane, + 64 ...
                int at[kPanel / kWave];
#pragma unroll
                for (int u = 0; u < kPanel / kWave; ++u) at[u] = min(p0 + u * kWave + lane, nb - 1);
                for (int i = 0; i < slices; ++i)
#pragma unroll
                    for (int u = 0; u < kPanel / kWave; ++u) sum[u] += part[((int64_t)i * C + c) * span + at[u]];
                for (int b0 = 0; b0 < p0; b0 += kWave) {
                    const OnlineWeight r = rec[min(b0 + lane, p0 - 1)];
                    const bool named = b0 + lane < p0 && (r.y == c || r.pred == c);
                    const float w = r.y == c ? r.w_y : -r.w_p;
                    for (uint64_t left = __ballot(named); left;) {
                        constexpr int kAtOnce = CPW == 1 && !BATCH ? 4 : 2;   // within the registers a call leaves free (past the last one: it again, of no weight)
                        float weight[kAtOnce];
                        int g[kAtOnce][kPanel / kWave];
#pragma unroll
                        for (int j = 0; j < kAtOnce; ++j) {
                            const int i = left ? __builtin_ctzll(left) : 0;
                            weight[j] = left ? lane_f32(w, i) : 0.0f;
                            left &= left - 1;
#pragma unroll
                            for (int u = 0; u < kPanel / kWave; ++u) g[j][u] = product(b0 + i, at[u]);
                        }
#pragma unroll
                        for (int j = 0; j < kAtOnce; ++j)
#pragma unroll
                            for (int u = 0; u < kPanel / kWave; ++u) sum[u] = fma((double)weight[j], (double)g[j][u], sum[u]);
                    }
                }
#pragma unroll
                for (int u = 0; u < kPanel / kWave; ++u) sums[c * kPanel + u * kWave + lane] = sum[u];
            }
        }
        int y = labels[m];
        y = y >= 0 && y < C ? y : -1;
        double all[CPW];
        __syncthreads();   // the record before is there, cosv has been read
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = wave * CPW + k;
            if (first == m) frozen[k] = nrm[k];
            if (c >= C) continue;
            double start = 0.0, old = 0.0, own = 0.0;
            if (Product::kPanels)
                start = sums[c * kPanel + m - p0];
            else
                for (int i = 0; i < slices; ++i) start += part[((int64_t)i * C + c) * span + m];
            for (int n = p0 + lane; n < m; n += kWave) {
                const OnlineWeight r = rec[n];
                const double g = (double)product(n, m);
                const double term = r.y == c ? (double)r.w_y * g : r.pred == c ? -(double)r.w_p * g : 0.0;
                (n < first ? old : own) += term;
            }
            const double dot = start + lane_f64(lane_prefix(old), kWave - 1);
            all[k] = dot + lane_f64(lane_prefix(own), kWave - 1);
            const double nn = frozen[k];
            if (lane == 0) cosv[c] = nn <= 0.0 ? 0.0 : dot * refined_rsq(nn) * inv_root_d;
        }
        __syncthreads();
        int pred = BATCH ? -1 : 0;
        double best = BATCH ? -2.0 : cosv[0];
        for (int c = BATCH ? 0 : 1; c < C; ++c) {
            const double v = cosv[c];
            if (v > best) {
                best = v;
                pred = c;
            }
        }
        OnlineWeight r = {y, -1, 0.0f, 0.0f};
        if (y >= 0) {
            r.w_y = (float)(1.0 - cosv[y]);
            if (pred >= 0 && pred != y) {
                r.pred = pred;
                r.w_p = (float)((double)lr * (1.0 - best));
            }
        }
        if (tid == 0) rec[m] = r;
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const int c = wave * CPW + k;
            const double w = r.y == c ? (double)r.w_y : r.pred == c ? -(double)r.w_p : 0.0;
            if (c < C && (r.y == c || r.pred == c)) nrm[k] += w * (2.0 * all[k] + w * (double)D);
        }
    }
    for (int k = 0; k < CPW && grown; ++k)
        if (lane == 0 && wave * CPW + k < C) grown[wave * CPW + k] = nrm[k] - at_start[k];
    __syncthreads();
}

}  // namespace hdc
