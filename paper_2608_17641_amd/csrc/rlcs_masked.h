// GAE with observation-skip masking (the planned extension of Section 9.3: the recurrence is
// carried across masked tokens, beta_t = 1) and optional whitening of the advantages.
//
// A masked step (an observation token) passes on both the running advantage A and the value W
// that the preceding unmasked step sees as its successor: the value of the next unmasked step.
//   unmasked, continuing:  A = r - V + gamma W' + gamma lambda A',   W = V;
//   unmasked, cut:         A = r - V + gamma * (0 | bv | boot),       W = V;
//   masked, continuing:    A = A', W = W';
//   masked, cut:           A = 0,  W = (0 | bv | boot);
// where a cut is a termination (successor 0), a truncation (its continuation bv_t) or the row's
// last step (the bootstrap), and A', W' are those of the step after. W does not depend on A, so the
// kernels run two scans of the pairs of Eq. 2 over the flat [N*T] array: W (a constant at every
// step but masked continuing ones, which are the identity), then, with W' known at every step, A.
// Each lane composes its K steps, a DPP wave scan composes lanes, LDS composes waves and carries
// chunks. (One scan of the triangular 2 x 2 maps of (A, W), five floats each, took one barrier
// less, but 45 vector operations a wave for its DPP steps instead of 24 and more at every
// composition; with eight waves on a SIMD these kernels are bound by vector operations.)
//
// Whitening: the scan kernel also reduces the advantages of the unmasked steps of each
// workgroup to fp64 sums (count, sum, sum of squares) and stores them as the workgroup's
// partial. A second kernel rewrites the advantages: each of its workgroups first adds up all
// partials itself, in one fixed order, so every workgroup derives the same mean and
// 1/sqrt(var + eps) (var the unbiased variance) and results are reproducible bit for bit.
// The kernel boundary orders the partials before their readers, so no atomics or fences are
// needed. With more than kDirectPartials partials a small kernel in between first adds them
// in blocks of kDirectPartials. fp64 sums of fp32 advantages lose accuracy in the variance only
// when |mean| / std approaches 1e6, far past what fp32 advantages resolve anyway.
#pragma once

#include <stddef.h>

#include "rlcs_kernels.h"

namespace rlcs {

// The state between two steps: the advantage, and the value of the next unmasked step.
struct AW {
    float A, W;
};

// fp64 sums of the advantages of the unmasked steps of one workgroup (or of a block of
// partials): count, sum, sum of squares.
struct alignas(32) Moments {
    double n, s1, s2, pad;
};

struct MaskedArgs {
    Args a;              // in[0] r, in[1] v, in[2] bv; term, trunc; row_value = boot;
                         // out0 adv, out1 ret (optional)
    const uint8_t* mask; // [N, T], nonzero = the step takes part; null = every step does
    // whitening only (workspace): one partial per workgroup
    Moments* partials;
};

constexpr int kDirectPartials = 4096;  // partials one normalize workgroup adds up itself

constexpr int kMaskedWaves = 16;  // most waves of a workgroup

// One lane's K consecutive steps of a chunk (lane l owns the (63-l)-th group of its wave's
// span: the carry flows from lane l-1 to lane l).
template <typename DT, int K, bool TR, bool HM>
struct MaskedChunk {
    static constexpr uint32_t kAll = (1u << K) - 1u;
    static constexpr int kWords = K * int(sizeof(DT)) / 4;
    float r[K], v[K];
    // What a cut step hands to the step before it (the other steps': not used). One value for the
    // continuation and the bootstrap: both kept to the second scan held the truncating kernels at 100
    // VGPRs instead of 90 (bfloat16) and cost 4 to 8 % (600 x 1024 5.6 -> 5.2 us).
    float end[K];
    uint32_t mk, cut, valid;  // steps that take part; cut steps; the lane's steps
    int64_t p0;
    // the maps of the scan at hand (of W, then of A): the steps', and lanes 0..lane composed
    float al[K], be[K];
    Pair incl;

    // Vector loads of the lane's K steps (16-byte aligned data, T >= K, all K steps inside the
    // array; `base` a row start at or before p0), every one issued before the first use; at most
    // one row edge. `in_range` selects the steps that are the lane's: all, or those of a ragged
    // end of the workgroup's range.
    __device__ __forceinline__ void load_full(const MaskedArgs& ma, const RowBase& base,
                                              uint32_t in_range) {
        const Args& a = ma.a;
        valid = in_range;
        const uint8_t* fallback = reinterpret_cast<const uint8_t*>(a.in[0]);
        uint32_t tw[(K + 3) / 4], rw[(K + 3) / 4], mw[(K + 3) / 4];
        if (TR) load_flag_words<K>(a.trunc, p0, rw);
        load_flag_words<K>(a.term ? a.term : fallback, p0, tw);
        if (HM) load_flag_words<K>(ma.mask, p0, mw);
        uint32_t wr[kWords], wv[kWords], wb[kWords];
        load_words<DT, K>(a.in[0], p0, wr);
        load_words<DT, K>(a.in[1], p0, wv);
        int64_t row, t;
        row_and_step(base, p0, a.T, a.inv_T, row, t);
        const int ke = (t + K - 1 >= a.T - 1) ? int(a.T - 1 - t) : -1;
        const float rv_raw = load_one<DT>(a.row_value ? a.row_value : a.in[0], min(row, a.N - 1));
        const uint32_t trunc = TR ? flag_mask<K>(rw) : 0u;
        if (TR && trunc) load_words<DT, K>(a.in[2], p0, wb);
        else {
#pragma unroll
            for (int i = 0; i < kWords; ++i) wb[i] = 0u;
        }
        unpack_words<DT, K>(wr, r);
        unpack_words<DT, K>(wv, v);
        unpack_words<DT, K>(wb, end);
        const uint32_t term = a.term ? flag_mask<K>(tw) : 0u;
        mk = HM ? flag_mask<K>(mw) : kAll;
        cut = term | trunc | (ke >= 0 ? (1u << ke) : 0u);
        const float rv = a.row_value ? rv_raw : 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) end[k] = bit(term, k) ? 0.f : (TR && bit(trunc, k) ? end[k] : (k == ke ? rv : 0.f));
    }

    // Steps of a chunk with steps outside [lo, hi): element-wise, masked.
    __device__ __forceinline__ void load_masked(const MaskedArgs& ma, const RowBase& base,
                                                int64_t lo, int64_t hi) {
        const Args& a = ma.a;
        valid = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (p0 + k >= lo && p0 + k < hi) valid |= 1u << k;
        uint32_t edge = 0;
        float B[K], bv[K];
#pragma unroll
        for (int k = 0; k < K; ++k) B[k] = 0.f;
        if (valid) {
            const int64_t first = p0 + __builtin_ctz(valid);
            int64_t row, t;
            row_and_step(base, first, a.T, a.inv_T, row, t);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (p0 + k < first || !bit(valid, k)) continue;
                if (t == a.T - 1) {
                    edge |= 1u << k;
                    if (a.row_value) B[k] = load_one<DT>(a.row_value, row);
                }
                if (++t == a.T) { t = 0; ++row; }
            }
        }
        const uint32_t term = a.term ? load_flags_masked<K>(a.term, p0, valid) : 0u;
        const uint32_t trunc = TR ? load_flags_masked<K>(a.trunc, p0, valid) : 0u;
        mk = HM ? load_flags_masked<K>(ma.mask, p0, valid) : valid;
        load_k<DT, K>(a.in[0], p0, valid, false, r);
        load_k<DT, K>(a.in[1], p0, valid, false, v);
        load_k<DT, K>(a.in[2], p0, valid & trunc, false, bv);
        cut = term | trunc | edge;
#pragma unroll
        for (int k = 0; k < K; ++k) end[k] = bit(term, k) ? 0.f : (TR && bit(trunc, k) ? bv[k] : B[k]);
    }

    // Composes the lane's steps (step 0 outermost) and scans the wave: the wave's map in lane 63.
    __device__ __forceinline__ Pair scan(int lane) {
        Pair agg{al[K - 1], be[K - 1]};
#pragma unroll
        for (int k = K - 2; k >= 0; --k) agg = compose(Pair{al[k], be[k]}, agg);
        incl = wave_scan_inclusive(agg, lane);
        return incl;
    }

    // First scan: W. `valid` steps only; the others are the identity.
    __device__ __forceinline__ Pair values(int lane) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool in = bit(mk, k), on = !bit(valid, k) || (!in && !bit(cut, k));
            al[k] = on ? 0.f : (in ? v[k] : end[k]);
            be[k] = on ? 1.f : 0.f;
        }
        return scan(lane);
    }
    // Second scan: A, given the W entering the wave's span. Returns W at the lane's first step in
    // `first`.
    __device__ __forceinline__ Pair advantages(const Params& P, float Ww, int lane, float& first) {
        float w = shift_up1(apply(incl, Ww), Ww);  // the W entering the lane
        const float gl = P.gamma * P.lambda;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            const bool in = bit(mk, k), c = bit(cut, k);
            const float next = fmaf(be[k], w, al[k]);
            const float a = fmaf(P.gamma, c ? end[k] : w, r[k] - v[k]);
            al[k] = (in && bit(valid, k)) ? a : 0.f;
            be[k] = bit(valid, k) ? (c ? 0.f : (in ? gl : 1.f)) : 1.f;
            w = next;
        }
        first = w;
        return scan(lane);
    }

    // Outputs given Aw, the advantage entering the wave's span; returns the advantage at the lane's
    // first step. Accumulates the advantages that take part into the sum and sum of squares (their
    // count is count_wave's). `full`: the lane's steps are vector-aligned (stored as vectors when
    // all of them are the lane's).
    float adv[K];  // the lane's advantages (kept for the fused whitening)
    // K = 8: the wave's LDS slot for whole-line stores. A wave whose lanes all store whole
    // vectors holds 512 consecutive outputs (lane l the group 63 - l of them).
    f32x4* oslot = nullptr;

    // Stores the lane's K outputs `v` to `out`: whole lines through the wave's slot when every
    // lane of the wave stores whole vectors (K = 8), else per lane.
    __device__ __forceinline__ void store(float* out, bool vstore, const float (&v)[K]) {
        if constexpr (K == 8) {
            if (__all(vstore)) {
                const int lane = threadIdx.x & (kWave - 1);
                const int g = kWave - 1 - lane;
                const int64_t base = p0 - int64_t(g) * K;
                store8_lines(out, base, base + kWave * K, g, lane, v, oslot);
                return;
            }
        }
        store_k<K>(out, p0, valid, vstore, v);
    }

    template <bool STATS, bool STORE = true>
    __device__ __forceinline__ float finish(const Args& a, float Aw, bool full, double& s1, double& s2) {
        float x = shift_up1(apply(incl, Aw), Aw);
#pragma unroll
        for (int k = K - 1; k >= 0; --k) {
            x = fmaf(be[k], x, al[k]);
            adv[k] = x;
            if (STATS) {
                const double d = double(bit(valid & mk, k) ? x : 0.f);
                s1 += d;
                s2 = fma(d, d, s2);
            }
        }
        if (STORE) {
            store(a.out0, full && valid == kAll, adv);
            store_returns(a, full);
        }
        return x;
    }

    // Steps of the wave that take part (the same in every lane).
    __device__ __forceinline__ int count_wave() const {
        int n = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) n += __popcll(__ballot(bit(valid & mk, k)));
        return n;
    }

    // The value targets, if asked for.
    __device__ __forceinline__ void store_returns(const Args& a, bool full) {
        if (!a.out1) return;
        float ret[K];
#pragma unroll
        for (int k = 0; k < K; ++k) ret[k] = adv[k] + v[k];
        store(a.out1, full && valid == kAll, ret);
    }
};

// Sum over the 64 lanes in fp64, in lane 63, in one fixed order: a DPP prefix sum inside each row
// of 16 lanes (both 32-bit halves moved by row shifts, zeros shifted in), then the row broadcasts
// of lanes 15 and 31 as in the scans. Against a shuffle butterfly (12 LDS-speed permutes per value)
// row shifts took whitened masked GAE 1024 x 2048 from 21.9 to 19.8 us.
template <int kCtrl, int kRows = 0xf>
__device__ __forceinline__ double dpp_move_f64(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u)), kCtrl, kRows, 0xf, false));
    const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), kCtrl, kRows, 0xf, false));
    return __longlong_as_double((uint64_t(hi) << 32) | lo);
}
__device__ __forceinline__ double read_lane_f64(double v, int lane) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), lane));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u >> 32)), lane));
    return __longlong_as_double((uint64_t(hi) << 32) | lo);
}
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_move_f64<kDppRowShr + 1>(x);
    x += dpp_move_f64<kDppRowShr + 2>(x);
    x += dpp_move_f64<kDppRowShr + 4>(x);
    x += dpp_move_f64<kDppRowShr + 8>(x);
    x += dpp_move_f64<kDppBcast15, 0xa>(x);
    x += dpp_move_f64<kDppBcast31, 0xc>(x);
    return x;
}

// Sum over the first 16 lanes, the same value in every lane (the other lanes' values are not used).
__device__ __forceinline__ double row_sum(double x) {
    x += dpp_move_f64<kDppRowShr + 1>(x);
    x += dpp_move_f64<kDppRowShr + 2>(x);
    x += dpp_move_f64<kDppRowShr + 4>(x);
    x += dpp_move_f64<kDppRowShr + 8>(x);
    return read_lane_f64(x, 15);
}

// Step 1 of one chunk [chunk_lo, chunk_hi) of a workgroup's range [lo, hi) (lane l of wave w
// owns the (63-l)-th group of K steps of the wave's span).
template <typename DT, int K, bool TR, bool HM>
__device__ __forceinline__ void masked_chunk_load(MaskedChunk<DT, K, TR, HM>& c, const MaskedArgs& ma,
                                                  const RowBase& base, int64_t lo, int64_t hi,
                                                  int64_t chunk_lo, int64_t chunk_hi, bool can_full,
                                                  int lane, int wave) {
    const Args& a = ma.a;
    c.p0 = chunk_lo + (int64_t(wave) * kWave + (kWave - 1 - lane)) * K;
    const bool full = can_full && chunk_lo >= lo && chunk_hi <= hi;
    if (full) {
        c.load_full(ma, base, MaskedChunk<DT, K, TR, HM>::kAll);
    } else if (can_full) {
        // lane by lane: vector loads wherever the lane's K steps lie inside the array (the
        // steps outside the range masked off), element-wise otherwise
        constexpr uint32_t kAll = MaskedChunk<DT, K, TR, HM>::kAll;
        const int64_t p = c.p0;
        if (p >= lo && p + K <= hi) {
            c.load_full(ma, base, kAll);
        } else if (p + K > lo && p < hi && p >= 0 && p + K <= a.N * a.T) {
            uint32_t m = kAll;
            RowBase b = base;
            if (p < lo) {
                m &= (kAll << uint32_t(lo - p)) & kAll;
                b = RowBase{base.pos - a.T, base.row - 1, base.t};  // the row before
            }
            if (p + K > hi) m &= kAll >> uint32_t(p + K - hi);
            c.load_full(ma, b, m);
        } else {
            c.load_masked(ma, base, lo, hi);
        }
    } else {
        c.load_masked(ma, base, lo, hi);
    }
}

// Rows kernel for masked GAE: workgroup g of W = blockDim / 64 waves owns rows [g*R, g*R + R) and
// walks them in chunks of E = W*64*K steps from the end. `wave_local`: every row lies within one wave's span, so no
// carry crosses waves.
template <typename DT, int K, bool VEC, bool TR, bool HM, bool STATS>
__global__ void __launch_bounds__(kMaskedWaves * kWave) masked_gae_kernel(MaskedArgs ma, int64_t rows_per_wg,
                                                                          int wave_local) {
    const Args& a = ma.a;
    const int W = blockDim.x / kWave;
    const int64_t E = int64_t(W) * kWave * K;
    __shared__ float s_m[4][kMaskedWaves];  // the waves' maps of W and of A
    __shared__ float s_cA, s_cW;
    __shared__ double s_stat[3][kMaskedWaves];
    extern __shared__ f32x4 s_out[];  // K = 8: 2 KB per wave
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t row_lo = int64_t(blockIdx.x) * rows_per_wg;
    const int64_t row_hi = min(row_lo + rows_per_wg, a.N);
    const int64_t lo = row_lo * a.T, hi = row_hi * a.T;
    const bool can_full = VEC && a.T >= K;
    const RowBase base{lo, row_lo, 0};
    AW carry{0.f, 0.f};
    int64_t n = 0;
    double s1 = 0.0, s2 = 0.0;
    int64_t chunk_hi = (hi + K - 1) / K * K;
    for (;;) {
        const int64_t chunk_lo = chunk_hi - E;
        MaskedChunk<DT, K, TR, HM> c;
        c.oslot = s_out + wave * 2 * kWave;
        masked_chunk_load(c, ma, base, lo, hi, chunk_lo, chunk_hi, can_full, lane, wave);
        AW in = carry;  // the state entering the wave's span
        const Pair mw = c.values(lane);
        if (!wave_local) {
            if (lane == kWave - 1) { s_m[0][wave] = mw.a; s_m[1][wave] = mw.b; }
            __syncthreads();
            in.W = apply(waves_in<true>(s_m[0], s_m[1], W, wave, lane), carry.W);
        }
        float w_first;
        const Pair mA = c.advantages(a.p, in.W, lane, w_first);
        if (!wave_local) {
            if (lane == kWave - 1) { s_m[2][wave] = mA.a; s_m[3][wave] = mA.b; }
            __syncthreads();
            in.A = apply(waves_in<true>(s_m[2], s_m[3], W, wave, lane), carry.A);
        }
        const float a_first = c.template finish<STATS>(a, in.A, can_full, s1, s2);
        if (STATS) n += c.count_wave();
        if (chunk_lo <= lo) break;
        // the next chunk (earlier in time) continues from the state at chunk_lo, held by lane
        // 63 of wave 0
        if (threadIdx.x == kWave - 1) { s_cA = a_first; s_cW = w_first; }
        __syncthreads();
        carry = AW{s_cA, s_cW};
        chunk_hi = chunk_lo;
    }
    if constexpr (STATS) {
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane == kWave - 1) { s_stat[0][wave] = double(n); s_stat[1][wave] = s1; s_stat[2][wave] = s2; }
        __syncthreads();
        if (threadIdx.x == 0) {
            Moments m{0.0, 0.0, 0.0, 0.0};
            for (int w = 0; w < W; ++w) { m.n += s_stat[0][w]; m.s1 += s_stat[1][w]; m.s2 += s_stat[2][w]; }
            ma.partials[blockIdx.x] = m;
        }
    }
}

// Sum of partials [lo, hi) over a workgroup of kNormThreads threads, in one fixed order
// (thread-serial over a stride of kNormThreads, a butterfly within each wave, then the waves in
// order), returned to every thread. Every thread of the workgroup must call it.
constexpr int kNormThreads = 256;

__device__ __forceinline__ Moments sum_partials(const Moments* part, int64_t lo, int64_t hi) {
    __shared__ double s_sum[3][kNormThreads / kWave];
    double n = 0.0, s1 = 0.0, s2 = 0.0;
    constexpr int kBatch = 4;  // partials per thread in flight
    for (int64_t g0 = lo + threadIdx.x; g0 < hi; g0 += int64_t(kBatch) * kNormThreads) {
        Moments m[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t g = g0 + int64_t(u) * kNormThreads;
            m[u] = g < hi ? part[g] : Moments{0.0, 0.0, 0.0, 0.0};
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) { n += m[u].n; s1 += m[u].s1; s2 += m[u].s2; }
    }
    n = wave_sum(n);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) { s_sum[0][wave] = n; s_sum[1][wave] = s1; s_sum[2][wave] = s2; }
    __syncthreads();
    Moments t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kNormThreads / kWave; ++w) { t.n += s_sum[0][w]; t.s1 += s_sum[1][w]; t.s2 += s_sum[2][w]; }
    return t;
}

// Second-level partials: workgroup j adds partials [j * kDirectPartials, (j + 1) * kDirectPartials).
__global__ void __launch_bounds__(kNormThreads) masked_sum_partials_kernel(const Moments* part,
                                                                           int64_t G, Moments* out) {
    const int64_t lo = int64_t(blockIdx.x) * kDirectPartials;
    const Moments t = sum_partials(part, lo, min(lo + kDirectPartials, G));
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// adv <- (adv - mean) * rstd over all `total` elements, mean and rstd from the sum of the G
// partials. Each thread rewrites kNormVec 16-byte vectors (strided by the workgroup size, so
// that a wave's accesses are contiguous), its loads issued before the partials are added up;
// workgroup 0 also does the elements past the last vector and stores {mean, rstd} to `stats`.
// The element-wise form is for advantages not 16-byte aligned.
constexpr int kNormVec = 4;

__device__ __forceinline__ void whitening(const Moments* part, int64_t G, float eps, double* stats,
                                          float& mean, float& rstd) {
    const Moments t = sum_partials(part, 0, G);
    const double m = t.n > 0.0 ? t.s1 / t.n : 0.0;
    const double var = t.n > 1.0 ? fmax(t.s2 - t.s1 * m, 0.0) / (t.n - 1.0) : 0.0;
    const double r = 1.0 / sqrt(var + double(eps));
    if (blockIdx.x == 0 && threadIdx.x == 0) { stats[0] = m; stats[1] = r; }
    mean = float(m);
    rstd = float(r);
}

__global__ void __launch_bounds__(kNormThreads) masked_normalize_kernel(float* adv, int64_t total,
                                                                        const Moments* part,
                                                                        int64_t G, float eps,
                                                                        double* stats, int vec) {
    float mean, rstd;
    const int64_t base = int64_t(blockIdx.x) * kNormThreads * kNormVec + threadIdx.x;
    if (vec) {
        f32x4* p = reinterpret_cast<f32x4*>(adv);
        const int64_t nv = total / 4;
        f32x4 x[kNormVec];
#pragma unroll
        for (int u = 0; u < kNormVec; ++u) {
            const int64_t i = base + int64_t(u) * kNormThreads;
            if (i < nv) x[u] = __builtin_nontemporal_load(p + i);
        }
        whitening(part, G, eps, stats, mean, rstd);
#pragma unroll
        for (int u = 0; u < kNormVec; ++u) {
            const int64_t i = base + int64_t(u) * kNormThreads;
            if (i < nv) __builtin_nontemporal_store((x[u] - mean) * rstd, p + i);
        }
        if (blockIdx.x == 0 && threadIdx.x < total - nv * 4) {
            const int64_t i = nv * 4 + threadIdx.x;
            adv[i] = (adv[i] - mean) * rstd;
        }
    } else {
        // the same 4 * kNormVec * kNormThreads elements per workgroup, one at a time
        const int64_t first = int64_t(blockIdx.x) * kNormThreads * kNormVec * 4 + threadIdx.x;
        float x[4 * kNormVec];
#pragma unroll
        for (int u = 0; u < 4 * kNormVec; ++u) {
            const int64_t i = first + int64_t(u) * kNormThreads;
            if (i < total) x[u] = adv[i];
        }
        whitening(part, G, eps, stats, mean, rstd);
#pragma unroll
        for (int u = 0; u < 4 * kNormVec; ++u) {
            const int64_t i = first + int64_t(u) * kNormThreads;
            if (i < total) adv[i] = (x[u] - mean) * rstd;
        }
    }
}

// ---------------------------------------------------------------- whitening in one pass
// When every workgroup of a whitened call is resident on the GPU at once and holds one chunk,
// the call runs as one kernel: each workgroup computes its advantages, keeps them in registers
// and publishes its fp64 moments; workgroup 0 adds them all up (one record per lane and turn) into
// the mean and 1/sqrt(var + eps) and publishes them in kStatsCopies copies; every other
// workgroup waits for its copy; then each whitens its advantages and stores them, once. Two round
// trips through memory follow the last moments; the value targets are stored behind the moments,
// where they fill that wait (stored before, they held the moments up). The sums run in one fixed
// order, so results are reproducible bit for bit. No atomic read-modify-write is on that way
// (a counter that every workgroup increments serializes them, about 17 ns each). A waiting
// workgroup polls one record with one lane, with pauses that grow, so
// that the waiting workgroups do not flood memory while others still stream their data (every
// workgroup polling every record it needs slowed whole calls several times over).
//
// No wait needs the whole grid resident, which the host can ask of an idle GPU only: two such calls
// on two streams may each hold a part of it. A workgroup other than 0 that has polled kWaitPolls
// times (some 0.1 ms) stores its advantages as they are and leaves, which makes room for those
// still to start; workgroup 0 alone waits on, and whitens what the others left behind once it has
// the statistics. Who whitens is settled by exchanges on two words:
//   a leaver puts kLeft in its hand word behind its stores and counts itself in the call's word;
//   workgroup 0, with the statistics out, closes the call's word (its tag, no leavers) and, if it
//     held leavers, puts kClosed in every hand word: those that held kLeft are its own to whiten;
//   a leaver that finds the call closed takes its hand back: it whitens for itself unless it finds
//     kClosed there in place of its kLeft.
// A call that nobody leaves pays one atomic of workgroup 0 (kClosed in every hand word each time
// took 1024 x 2048 float32 from 12.0 to 12.5 us).
//
// With 32 waves on a CU the vector operations count: whitened 1024 x 2048 float32 took 594 a wave
// and 14.1 us with the triangular scan, 444 and 12.0 us now (two pair scans, counts by ballots,
// sums by row broadcasts, returns behind the moments); 64 x 4096 10.1 -> 8.3, 4096 x 256 10.4 -> 9.0.
//
// Workspace of the whitening (zero-filled once before its first use; every call leaves it
// ready for the next):
//   [0, 16)    mean and 1/sqrt(var + eps) of the last call, two doubles (for the caller);
//   [16, 24)   generation: the number of one-pass calls made on the workspace (mod 2^31);
//              workgroup 0 advances it once every moment of its call is in, hence after every
//              workgroup of the call has read it;
//   [24, 32)   the call's word: the tag of the last call that closed << 32 | leavers since;
//   kMaskedFusedOff: one tagged moments record (six words) per workgroup, kFusedMaxGroups;
//   kMaskedStatsOff: kStatsCopies copies of the tagged statistics record (four words), one per
//              128-byte line;
//   kMaskedTwoPassOff: the partials of the two-pass form (Moments, 32 bytes each), whose last
//              word is workgroup g's hand in the one-pass form: kLeft, kClosed or kTaken with its
//              call's tag (the two-pass form leaves 0 there, which no tag equals).
// A tagged word holds a 32-bit half of a double in its low half and the tag 2*gen + 1 of its
// call in the high half; a reader takes a double only when both of its words carry the
// current tag, so no word of another call (or of the two-pass partials, which live apart)
// passes for a current one. Workgroup 0's polls are bounded as well (about a second); on
// exhaustion the statistics are NaN.
constexpr int64_t kFusedMaxGroups = 1024;
constexpr int kStatsCopies = 64;
constexpr size_t kMaskedGenOff = 16;
constexpr size_t kMaskedCloseOff = 24;
constexpr size_t kMaskedFusedOff = 64;
constexpr size_t kMaskedStatsOff = (kMaskedFusedOff + 48 * size_t(kFusedMaxGroups) + 127) / 128 * 128;
constexpr size_t kMaskedTwoPassOff = kMaskedStatsOff + 128 * size_t(kStatsCopies);
constexpr uint32_t kWaitPolls = 256;
constexpr uint64_t kLeft = uint64_t(1) << 32, kClosed = uint64_t(2) << 32, kTaken = uint64_t(3) << 32;

__device__ __forceinline__ uint64_t* hand_word(char* ws, int64_t g) {
    return reinterpret_cast<uint64_t*>(ws + kMaskedTwoPassOff + sizeof(Moments) * size_t(g) + offsetof(Moments, pad));
}
// Puts `v` there and says what was there before. Relaxed: whoever leaves has fenced its stores, and
// workgroup 0 fences where it finds that someone has (a fence writes back or drops cache lines).
__device__ __forceinline__ uint64_t exchange(uint64_t* word, uint64_t v) {
    return __hip_atomic_exchange(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One lane of a workgroup whose advantages are stored and fenced: whether workgroup 0 whitens them.
__device__ __forceinline__ bool leave(char* ws, int64_t g, uint32_t tag) {
    uint64_t* hand = hand_word(ws, g);
    if (exchange(hand, kLeft | tag) == (kClosed | tag)) return false;
    const uint64_t old = __hip_atomic_fetch_add(reinterpret_cast<uint64_t*>(ws + kMaskedCloseOff), uint64_t(1),
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return uint32_t(old >> 32) != tag || exchange(hand, kTaken | tag) == (kClosed | tag);
}

__device__ __forceinline__ void put_tagged(uint64_t* w, double v, uint32_t tag) {
    const uint64_t u = uint64_t(__double_as_longlong(v));
    st_relaxed(w, uint64_t(tag) << 32 | (u & 0xffffffffu));
    st_relaxed(w + 1, uint64_t(tag) << 32 | (u >> 32));
}

// Doubles v[0 .. M) from the tagged words w[0 .. 2M) once every word carries `tag`: all words
// are loaded at once and reloaded until they do, after a pause that doubles from `pause`
// to about 500 cycles. False, and NaN, after `most` rounds.
template <int M>
__device__ __forceinline__ bool get_tagged(const uint64_t* w, uint32_t tag, double (&v)[M], int pause, uint32_t most) {
    uint64_t x[2 * M];
#pragma unroll
    for (int i = 0; i < 2 * M; ++i) x[i] = ld_relaxed(w + i);
    for (uint32_t polls = 0;; ++polls) {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < 2 * M; ++i) ok = ok && uint32_t(x[i] >> 32) == tag;
        if (ok) break;
        if (polls >= most) {
#pragma unroll
            for (int i = 0; i < M; ++i) v[i] = __builtin_nan("");
            return false;
        }
        for (int i = 0; i < pause; ++i) __builtin_amdgcn_s_sleep(2);
        pause = min(2 * pause, 4);
        // every word again, all loads in flight together: a word that already carried the tag
        // carries it still (each word of a record is written once per call)
#pragma unroll
        for (int i = 0; i < 2 * M; ++i) x[i] = ld_relaxed(w + i);
    }
#pragma unroll
    for (int i = 0; i < M; ++i)
        v[i] = __longlong_as_double(int64_t((x[2 * i + 1] << 32) | (x[2 * i] & 0xffffffffu)));
    return true;
}

// Workgroup 0 of a call that some of the G - 1 others have left: takes their hands and whitens the
// advantages of those that left (R rows of T steps each, N rows in all). Every lane takes part.
__device__ __forceinline__ void whiten_left(char* ws, uint32_t tag, int64_t G, float* adv, int64_t R, int64_t N,
                                            int64_t T, float mean, float rstd) {
    __shared__ uint64_t s_left[kMaskedWaves];
    const int W = blockDim.x / kWave;
    for (int64_t g0 = 0; g0 < G; g0 += blockDim.x) {
        const int64_t g = g0 + threadIdx.x;
        const bool left = g > 0 && g < G && exchange(hand_word(ws, g), kClosed | tag) == (kLeft | tag);
        const uint64_t mask = __ballot(left);
        if ((threadIdx.x & (kWave - 1)) == 0) s_left[threadIdx.x / kWave] = mask;
        __syncthreads();
        __threadfence();
        for (int w = 0; w < W; ++w) {
            for (uint64_t m = s_left[w]; m; m &= m - 1) {
                const int64_t row = (g0 + w * kWave + __builtin_ctzll(m)) * R;
                const int64_t end = min(row + R, N) * T;
                for (int64_t p = row * T + threadIdx.x; p < end; p += blockDim.x) adv[p] = (adv[p] - mean) * rstd;
            }
        }
        __syncthreads();  // s_left has been read
    }
}

// One-pass whitened masked GAE: workgroup g of the G <= kFusedMaxGroups owns rows [g*R, g*R + R),
// which fit in one chunk. `ws`: the whitening workspace; `wait`: polls before a workgroup leaves.
template <typename DT, int K, bool VEC, bool TR, bool HM>
__global__ void __launch_bounds__(kMaskedWaves * kWave) masked_gae_fused_kernel(MaskedArgs ma, int64_t rows_per_wg,
                                                                                int wave_local, float eps,
                                                                                char* ws, uint32_t wait) {
    const Args& a = ma.a;
    const int W = blockDim.x / kWave;
    const int64_t E = int64_t(W) * kWave * K;
    __shared__ float s_m[4][kMaskedWaves];  // the waves' maps of W and of A
    __shared__ double s_stat[3][kMaskedWaves];
    __shared__ uint32_t s_tag;
    __shared__ bool s_have;  // the workgroup has the statistics
    __shared__ uint32_t s_leavers;
    __shared__ float s_mean, s_rstd;
    extern __shared__ f32x4 s_out[];  // K = 8: 2 KB per wave
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t G = gridDim.x, g = blockIdx.x;
    const int64_t row_lo = g * rows_per_wg;
    const int64_t row_hi = min(row_lo + rows_per_wg, a.N);
    const int64_t lo = row_lo * a.T, hi = row_hi * a.T;
    const bool can_full = VEC && a.T >= K;
    const RowBase base{lo, row_lo, 0};
    const int64_t chunk_hi = (hi + K - 1) / K * K;
    const int64_t chunk_lo = chunk_hi - E;  // <= lo: the rows fit in one chunk
    uint64_t* gen_word = reinterpret_cast<uint64_t*>(ws + kMaskedGenOff);
    uint64_t* rec = reinterpret_cast<uint64_t*>(ws + kMaskedFusedOff);
    uint64_t* stats_rec = reinterpret_cast<uint64_t*>(ws + kMaskedStatsOff);
    // the generation cannot move before this workgroup's moments are in
    if (threadIdx.x == 0) s_tag = 2u * (uint32_t(ld_relaxed(gen_word)) & 0x7fffffffu) + 1u;

    MaskedChunk<DT, K, TR, HM> c;
    c.oslot = s_out + wave * 2 * kWave;
    masked_chunk_load(c, ma, base, lo, hi, chunk_lo, chunk_hi, can_full, lane, wave);
    AW in{0.f, 0.f};
    const Pair mw = c.values(lane);
    if (!wave_local) {
        if (lane == kWave - 1) { s_m[0][wave] = mw.a; s_m[1][wave] = mw.b; }
        __syncthreads();
        in.W = waves_in<true>(s_m[0], s_m[1], W, wave, lane).a;
    }
    float w_first;
    const Pair mA = c.advantages(a.p, in.W, lane, w_first);
    if (!wave_local) {
        if (lane == kWave - 1) { s_m[2][wave] = mA.a; s_m[3][wave] = mA.b; }
        __syncthreads();
        in.A = waves_in<true>(s_m[2], s_m[3], W, wave, lane).a;
    }
    double s1 = 0.0, s2 = 0.0;
    c.template finish<true, false>(a, in.A, can_full, s1, s2);

    // this workgroup's moments, summed by wave 0: lane w takes wave w's
    const int n = c.count_wave();
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == kWave - 1) { s_stat[0][wave] = double(n); s_stat[1][wave] = s1; s_stat[2][wave] = s2; }
    __syncthreads();
    const uint32_t tag = s_tag;
    double v[3] = {0.0, 0.0, 0.0};
    if (wave == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = row_sum(lane < W ? s_stat[q][lane] : 0.0);
        if (g != 0 && lane < 6) {  // lane i: word i of the record
            const double x = lane < 2 ? v[0] : lane < 4 ? v[1] : v[2];
            const uint64_t u = uint64_t(__double_as_longlong(x));
            st_relaxed(rec + 6 * g + lane, uint64_t(tag) << 32 | ((lane & 1) ? u >> 32 : u & 0xffffffffu));
        }
    }
    // the value targets go out behind the moments, while the statistics are on their way
    c.store_returns(a, can_full);
    auto wait_stats = [&](uint32_t most) {  // one lane
        double m[2];
        s_have = get_tagged<2>(stats_rec + 16 * (g % kStatsCopies), tag, m, 2, most);
        s_mean = float(m[0]);
        s_rstd = float(m[1]);
    };
    if (g != 0) {
        if (threadIdx.x == 0) wait_stats(wait);
    } else {
        // workgroup 0: every workgroup's moments (its own from above), in turns of one per lane
        if (threadIdx.x != 0) { v[0] = v[1] = v[2] = 0.0; }
        for (int64_t i = threadIdx.x; i < G; i += blockDim.x) {
            if (i == 0) continue;
            double m[3];
            get_tagged<3>(rec + 6 * i, tag, m, 1, kMaxPolls);
#pragma unroll
            for (int q = 0; q < 3; ++q) v[q] += m[q];
        }
        __syncthreads();  // wave 0 has read s_stat
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = wave_sum(v[q]);
        if (lane == kWave - 1) { s_stat[0][wave] = v[0]; s_stat[1][wave] = v[1]; s_stat[2][wave] = v[2]; }
        __syncthreads();
        if (wave == 0) {
            Moments t;
            t.n = row_sum(lane < W ? s_stat[0][lane] : 0.0);
            t.s1 = row_sum(lane < W ? s_stat[1][lane] : 0.0);
            t.s2 = row_sum(lane < W ? s_stat[2][lane] : 0.0);
            const double m = t.n > 0.0 ? t.s1 / t.n : 0.0;
            const double var = t.n > 1.0 ? fmax(t.s2 - t.s1 * m, 0.0) / (t.n - 1.0) : 0.0;
            const double r = 1.0 / sqrt(var + double(eps));
            uint64_t* copy = stats_rec + 16 * lane;  // one 128-byte line per copy
            put_tagged(copy, m, tag);
            put_tagged(copy + 2, r, tag);
            if (lane == 0) {
                // every moment of the call is in, so every workgroup has read the generation
                double* stats = reinterpret_cast<double*>(ws);
                stats[0] = m;
                stats[1] = r;
                st_relaxed(gen_word, uint64_t(((tag - 1u) / 2u + 1u) & 0x7fffffffu));
                s_have = true;
                s_mean = float(m);
                s_rstd = float(r);
            }
        }
    }
    __syncthreads();
    const bool full = can_full && c.valid == MaskedChunk<DT, K, TR, HM>::kAll;
    if (!s_have) {  // waited long enough: the rest is workgroup 0's, unless it has closed
        c.store(a.out0, full, c.adv);
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0 && !leave(ws, g, tag)) wait_stats(kMaxPolls);
        __syncthreads();
        if (!s_have) return;
    }
    const float mean = s_mean, rstd = s_rstd;
    uint64_t closed = 0;
    if (g == 0 && G > 1 && threadIdx.x == 0)
        closed = exchange(reinterpret_cast<uint64_t*>(ws + kMaskedCloseOff), uint64_t(tag) << 32);
    float y[K];
#pragma unroll
    for (int k = 0; k < K; ++k) y[k] = (c.adv[k] - mean) * rstd;
    c.store(a.out0, full, y);
    if (g != 0 || G == 1) return;
    if (threadIdx.x == 0) s_leavers = uint32_t(closed);
    __syncthreads();
    if (s_leavers) whiten_left(ws, tag, G, a.out0, rows_per_wg, a.N, a.T, mean, rstd);
}

}  // namespace rlcs
