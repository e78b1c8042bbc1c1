// Whole-column walks with four adjacent columns to a lane: time-major buffers of many columns, and
// vector traces of a multiple of four features (geometry and flags as in rlcs_columns.h).
//
// Bound by memory: a lane's loads are 16 bytes (float32) or 8 (bfloat16) of data and 4 of flags
// per step, a quarter of the instructions of one column per lane. LC lanes side by side cover a
// block of 4 * LC columns; the 64 / LC lane groups of a wave and then the W waves of a workgroup
// take consecutive spans of K steps. Per chunk of W * (64 / LC) * K steps: the lane's four serial
// maps, a shuffle scan over the lane groups, an LDS composition over the waves, the carry to the
// next chunk through LDS; the next chunk's loads go out before this one's are used. No
// workspace, no look-back. Vectors start at any column (unaligned accesses); where the columns
// are not a multiple of four the last lane's vector is moved back onto the last four columns
// and it stores only its own, so nothing outside the grid of (n, t) is touched.
//
// Loads are ordinary ones: blocks share lines of flags (and of data where rows do not start on a
// line), which non-temporal loads fetch once per block (64 x 1024 x 256 vector traces 31.2 us
// against 23.2, time-major GAE 768 x 9762 45.7 against 37.7). Stores are non-temporal (plain:
// time-major GAE 256 x 8192 10.2 us against 8.7).
#pragma once

#include "rlcs.h"
#include "rlcs_columns.h"

namespace rlcs {

constexpr int kCvV = 4;         // columns per lane
constexpr int kCvMaxWaves = 8;  // waves per workgroup at most

// Four adjacent elements at any address.
template <typename DT>
__device__ __forceinline__ void load_any4(const DT* p, uint32_t (&w)[sizeof(DT)]) {
    if constexpr (sizeof(DT) == 4) {
        const u32x4 u = *reinterpret_cast<const u32x4_any*>(p);
        w[0] = u.x; w[1] = u.y; w[2] = u.z; w[3] = u.w;
    } else {
        const u32x2 u = *reinterpret_cast<const u32x2_any*>(p);
        w[0] = u.x; w[1] = u.y;
    }
}

// Element v (a constant) of a vector's words.
template <typename DT>
__device__ __forceinline__ float vec_elem(const uint32_t (&w)[sizeof(DT)], int v) {
    return word_elem<DT>(w[sizeof(DT) == 4 ? v : v >> 1], v);
}

// The maps of a lane's four columns. VB distinct factors: four where each column has flags of its
// own, one where a step's flags are shared by every column.
template <int VB>
struct Map4 {
    float a[kCvV], b[VB];
    __device__ __forceinline__ static Map4 identity() {
        Map4 m;
#pragma unroll
        for (int v = 0; v < kCvV; ++v) m.a[v] = 0.f;
#pragma unroll
        for (int v = 0; v < VB; ++v) m.b[v] = 1.f;
        return m;
    }
    __device__ __forceinline__ float factor(int v) const { return b[VB == 1 ? 0 : v]; }
};

template <int VB>
__device__ __forceinline__ Map4<VB> compose(const Map4<VB>& outer, const Map4<VB>& inner) {
    Map4<VB> m;
#pragma unroll
    for (int v = 0; v < kCvV; ++v) m.a[v] = fmaf(outer.factor(v), inner.a[v], outer.a[v]);
#pragma unroll
    for (int v = 0; v < VB; ++v) m.b[v] = outer.b[v] * inner.b[v];
    return m;
}

// FCOL: flags laid out like the data. Grid: one workgroup per block of 4 * LC columns.
template <class Op, typename DT, int K, int LC, bool TR, bool FCOL>
__global__ void __launch_bounds__(kCvMaxWaves * kWave) cols_vec_kernel(Args a, ColGeom g, int64_t blocks) {
    constexpr bool kBack = Op::kBackward;
    constexpr int V = kCvV, NS = Op::kSlots, G = kWave / LC, VB = FCOL ? V : 1;
    constexpr int NB = Op::kNbr > 0 ? Op::kNbr : 1;
    constexpr int kTS = TR ? Op::kTruncSlot : -1;
    typedef Map4<VB> M;
    __shared__ f32x4 s_a[kCvMaxWaves][LC];
    __shared__ float s_b[kCvMaxWaves][LC][VB];
    __shared__ f32x4 s_carry[LC];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave), W = blockDim.x / kWave;
    const int cl = lane % LC, grp = lane / LC;
    // the lane's columns [c0, c0 + V), of which it owns those from j0 on
    const int64_t j0 = (narrow_group(blockIdx.x, blocks) * LC + cl) * V;
    const bool active = j0 < g.J;
    const int64_t c0 = min(j0, g.J - V);
    const int skip = active ? int(j0 - c0) : V;
    int64_t base = c0, fbase = c0;
    if constexpr (!FCOL) {
        const int64_t b = c0 / g.C;
        base = b * g.bstride + (c0 - b * g.C);
        fbase = b * g.fbstride;
    }
    const int64_t T = a.T, st = g.st, L = int64_t(W) * G * K;
    const int64_t P = (T + L - 1) / L;
    const uint8_t* fallback = reinterpret_cast<const uint8_t*>(a.in[0]);
    const uint8_t* term_p = a.term ? a.term : fallback;  // what it reads is dropped without one
    auto load_flags = [&](const uint8_t* f, int64_t t) -> uint32_t {
        if constexpr (FCOL) return *reinterpret_cast<const flags4_any*>(f + fbase + t * st);
        else return f[fbase + t * g.fst];
    };
    f32x4 carry = {0.f, 0.f, 0.f, 0.f};

    // a chunk's loads, all from clamped steps of the column (continuations apart: only where a step
    // is truncated, once its flags are in)
    struct Raw {
        uint32_t tw[K], rw[K], w[NS][K][sizeof(DT)], nw[NB][sizeof(DT)], rvw[sizeof(DT)];
        uint32_t ptw, prw;
    };
    auto start_of = [&](int64_t i) { return (kBack ? P - 1 - i : i) * L + int64_t(wave * G + grp) * K; };
    auto issue = [&](int64_t i, Raw& x) {
        const int64_t t0 = start_of(i);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t t = min(t0 + k, T - 1);
            x.rw[k] = TR ? load_flags(a.trunc, t) : 0u;
            x.tw[k] = load_flags(term_p, t);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (Op::slot_used(s, TR) && s != kTS)
                    load_any4(static_cast<const DT*>(a.in[s]) + base + min(t0 + k, T - 1) * st, x.w[s][k]);
        }
        if constexpr (kBack) {
            if constexpr (Op::kNbr > 0) {
                const int64_t t = min(t0 + K, T - 1);
#pragma unroll
                for (int n = 0; n < Op::kNbr; ++n)
                    load_any4(static_cast<const DT*>(a.in[Op::nbr_slot(n)]) + base + t * st, x.nw[n]);
            }
            if (Op::kRowValue && a.row_value && i == 0) load_any4(static_cast<const DT*>(a.row_value) + c0, x.rvw);
        } else if constexpr (Op::kNbr > 0) {
            const int64_t t = min(max(t0 - 1, int64_t(0)), T - 1);
            x.ptw = load_flags(term_p, t);
            x.prw = TR ? load_flags(a.trunc, t) : 0u;
        }
    };
    Raw raw;
    issue(0, raw);
    for (int64_t i = 0; i < P; ++i) {
        const int64_t t0 = start_of(i);
        // the next chunk's loads go out before this one's are used
        Raw next;
        if (i + 1 < P) issue(i + 1, next);
        __builtin_amdgcn_sched_barrier(0);
        auto& w = raw.w;
        auto& rw = raw.rw;
        auto& tw = raw.tw;
        uint32_t valid = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (t0 + k < T) valid |= 1u << k;
        uint32_t edge = 0;
        if (kBack) {
            if (t0 < T && t0 + K >= T) edge = 1u << int(T - 1 - t0);
        } else if (t0 == 0) {
            edge = 1u;
        }
        if (!a.term) {
#pragma unroll
            for (int k = 0; k < K; ++k) tw[k] = 0u;
            raw.ptw = 0u;
        }
        if constexpr (kTS >= 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
#pragma unroll
                for (unsigned i2 = 0; i2 < sizeof(DT); ++i2) w[kTS][k][i2] = 0u;
                if (rw[k] && bit(valid, k)) load_any4(static_cast<const DT*>(a.in[kTS]) + base + (t0 + k) * st, w[kTS][k]);
            }
        }
        // per column: Table 1's coefficients and the serial composition of the lane's steps
        float al[V][K], be[V][K], nb[V][NB], B[V][K];
        uint32_t term[V], trunc[V];
        auto inputs = [&](int v, float (&d)[NS][K]) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
#pragma unroll
                for (int k = 0; k < K; ++k) d[s][k] = Op::slot_used(s, TR) ? vec_elem<DT>(w[s][k], v) : 0.f;
            }
        };
        M m;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            term[v] = trunc[v] = 0u;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t byte = FCOL ? 0xffu << (8 * v) : 0xffu;
                if (tw[k] & byte) term[v] |= 1u << k;
                if (TR && (rw[k] & byte)) trunc[v] |= 1u << k;
                B[v][k] = bit(edge, k) ? (a.row_value ? vec_elem<DT>(raw.rvw, v) : 0.f) : 0.f;
            }
            term[v] &= valid;
            trunc[v] &= valid;
            nb[v][0] = 0.f;
            if constexpr (kBack) {
                if constexpr (Op::kNbr > 0) {
                    float nv[Op::kNbrRaw];
#pragma unroll
                    for (int n = 0; n < Op::kNbr; ++n) nv[n] = vec_elem<DT>(raw.nw[n], v);
                    Op::nbr_fix(a, nv, nb[v]);
                }
            } else if constexpr (Op::kNbr > 0) {
                nb[v][0] = t0 > 0 && ((raw.ptw | raw.prw) & (FCOL ? 0xffu << (8 * v) : 0xffu)) ? 1.f : 0.f;
            }
            float d[NS][K];
            inputs(v, d);
            Op::template build<K, TR>(a.p, d, term[v], trunc[v], edge, B[v], nb[v], al[v], be[v]);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (!bit(valid, k)) { al[v][k] = 0.f; be[v][k] = 1.f; }
            Pair agg = Pair{al[v][kBack ? K - 1 : 0], be[v][kBack ? K - 1 : 0]};
#pragma unroll
            for (int k = 1; k < K; ++k)
                agg = compose(Pair{al[v][kBack ? K - 1 - k : k], be[v][kBack ? K - 1 - k : k]}, agg);
            m.a[v] = agg.a;
            if (v < VB) m.b[v] = agg.b;
        }
        // lane groups of the wave: inclusive scan from the carry-source side, then the
        // composition of the groups on this group's carry-source side
        auto from = [&](const M& x, int src) {
            M y;
#pragma unroll
            for (int v = 0; v < V; ++v) y.a[v] = __shfl(x.a[v], src);
#pragma unroll
            for (int v = 0; v < VB; ++v) y.b[v] = __shfl(x.b[v], src);
            return y;
        };
        M in = M::identity();
        if constexpr (G > 1) {
#pragma unroll
            for (int dg = 1; dg < G; dg <<= 1) {
                const M o = from(m, kBack ? lane + dg * LC : lane - dg * LC);
                if (kBack ? (grp + dg < G) : (grp >= dg)) m = compose(m, o);
            }
            const M o = from(m, kBack ? lane + LC : lane - LC);
            if (kBack ? (grp + 1 < G) : (grp > 0)) in = o;
        }
        // the waves, then the value entering the chunk
        if (W > 1) {
            if (grp == (kBack ? 0 : G - 1)) {
                s_a[wave][cl] = f32x4{m.a[0], m.a[1], m.a[2], m.a[3]};
#pragma unroll
                for (int v = 0; v < VB; ++v) s_b[wave][cl][v] = m.b[v];
            }
            __syncthreads();
            float x[V] = {carry.x, carry.y, carry.z, carry.w};
            for (int j = kBack ? W - 1 : 0; j != wave; j += kBack ? -1 : 1) {
                const f32x4 wa = s_a[j][cl];
#pragma unroll
                for (int v = 0; v < V; ++v) x[v] = fmaf(s_b[j][cl][VB == 1 ? 0 : v], x[v], wa[v]);
            }
            carry = f32x4{x[0], x[1], x[2], x[3]};
        }
        float out_edge[V];
        f32x4 o0v[K], o1v[K];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float X = fmaf(in.factor(v), carry[v], in.a[v]);
            float A[K], d[NS][K], o0[K], o1[K];
            float x = X;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = kBack ? K - 1 - k : k;
                A[q] = fmaf(be[v][q], x, al[v][q]);
                x = A[q];
            }
            out_edge[v] = x;
            inputs(v, d);
            Op::template finish<K, TR>(a.p, d, term[v], trunc[v], edge, B[v], nb[v], A, X, o0, o1);
#pragma unroll
            for (int k = 0; k < K; ++k) { o0v[k][v] = o0[k]; o1v[k][v] = o1[k]; }
        }
        auto store = [&](float* out, const f32x4 (&o)[K]) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!bit(valid, k)) continue;
                float* p = out + base + (t0 + k) * st;
                if (skip == 0) {
                    store4_any(p, o[k]);
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (v >= skip) p[v] = o[k][v];
                }
            }
        };
        store(a.out0, o0v);
        if (a.out1) store(a.out1, o1v);
        if (i + 1 == P) break;
        if (wave == (kBack ? 0 : W - 1) && grp == (kBack ? 0 : G - 1))
            s_carry[cl] = f32x4{out_edge[0], out_edge[1], out_edge[2], out_edge[3]};
        __syncthreads();
        carry = s_carry[cl];
        raw = next;
    }
}

// Launches for one policy (instantiated one translation unit per policy or two, since the kernels
// are large): lc = 4, 8, 16 or 32; 8 or 16 for vector traces.
constexpr int kCvK = 4;  // steps per lane

template <class Op>
bool colvec_launch(const Args& a, const ColGeom& g, rlcs_dtype dtype, bool tr, int lc, hipStream_t s);

namespace cv {

template <class Op, typename DT, bool TR, bool FCOL, int LC>
void launch(const Args& a, const ColGeom& g, hipStream_t s) {
    constexpr int steps = kWave / LC * kCvK;  // per wave
    const int64_t blocks = (g.J + LC * kCvV - 1) / (LC * kCvV);
    const int64_t need = (a.T + steps - 1) / steps;
    // no more waves than share the chunks evenly: 160 steps of LC = 16 in two chunks of five waves, not
    // eight and two (V-Trace 160 x 65536 float32 64.6 -> 62.6 us, 160 x 60001 75.4 -> 68.7). Not where
    // vector traces have three blocks or more per CU: 325 x 150 x 200 bfloat16 16.8 against 18.7 (with two,
    // 165 x 150 x 200 12.1 -> 10.2)
    const int64_t chunks = FCOL || blocks < 768 ? (need + kCvMaxWaves - 1) / kCvMaxWaves : 1;
    const int64_t even = (need + chunks - 1) / chunks;
    const unsigned W = unsigned(even < kCvMaxWaves ? even : kCvMaxWaves);
    hipLaunchKernelGGL((cols_vec_kernel<Op, DT, kCvK, LC, TR, FCOL>), dim3(unsigned(blocks)), dim3(W * kWave),
                       0, s, a, g, blocks);
}

template <class Op, typename DT, bool TR, bool FCOL>
void launch_lc(const Args& a, const ColGeom& g, int lc, hipStream_t s) {
    if (lc == 4) launch<Op, DT, TR, FCOL, 4>(a, g, s);
    else if (lc == 8) launch<Op, DT, TR, FCOL, 8>(a, g, s);
    else if (lc == 16) launch<Op, DT, TR, FCOL, 16>(a, g, s);
    else launch<Op, DT, TR, FCOL, 32>(a, g, s);
}

// Vector traces (flags shared by a step's columns) run the eligibility-trace policy only.
template <class Op, typename DT, bool TR>
void launch_flags(const Args& a, const ColGeom& g, int lc, hipStream_t s) {
    if constexpr (std::is_same<Op, ForwardOp<true, false>>::value) {
        if (!g.fcol) {
            if (lc == 8) launch<Op, DT, TR, false, 8>(a, g, s);
            else launch<Op, DT, TR, false, 16>(a, g, s);
            return;
        }
    }
    launch_lc<Op, DT, TR, true>(a, g, lc, s);
}

}  // namespace cv

#define RLCS_COLVEC(OP)                                                                              \
    template <>                                                                                      \
    bool colvec_launch<OP>(const Args& a, const ColGeom& g, rlcs_dtype dtype, bool tr, int lc,       \
                           hipStream_t s) {                                                          \
        if (dtype == RLCS_BF16) {                                                                    \
            if (tr) cv::launch_flags<OP, bf16_t, true>(a, g, lc, s);                                 \
            else cv::launch_flags<OP, bf16_t, false>(a, g, lc, s);                                   \
        } else {                                                                                     \
            if (tr) cv::launch_flags<OP, float, true>(a, g, lc, s);                                  \
            else cv::launch_flags<OP, float, false>(a, g, lc, s);                                    \
        }                                                                                            \
        return hipGetLastError() == hipSuccess;                                                      \
    }

}  // namespace rlcs
