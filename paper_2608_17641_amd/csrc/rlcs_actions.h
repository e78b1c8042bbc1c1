// Full-form Retrace (Sections 3.3.3 and 7.3): the per-step terms E_pi Q(s_t), Q(s_t, a_t) and
// rho_t = pi(a_t|s_t) / mu_t are reduced from [N, T, A] Q-values and target probabilities and
// scanned in the same kernel.
//
// Bound by the bytes of Q and pi (8A of the 26 + 8A bytes of a float32 step). A wave owns
// 64 * K consecutive steps and reduces them straight from registers: L lanes (a power of two,
// 64 at most) take one step, each lane one vector of V = 4 consecutive actions per load, so one
// load instruction of the wave covers 64 / L consecutive steps, whose rows of A actions are
// contiguous in memory (a round). The next rounds' loads are out while a batch of rounds is
// reduced; sums over a step's lanes run by DPP. Rows start on any element, so the vectors are
// unaligned (a lane past its row's last action drops what it read; the last vector of the
// tensors is moved back to stay inside them), which costs nothing where A is a multiple of V
// and a line crossing or two otherwise. The terms of each step pass through LDS (12 bytes per
// step) to the lane that scans it.
//
// Two rounds in flight while two are reduced (kActBatch): four and four held 105 VGPRs, four
// waves per SIMD, and ran 4096 x 256 x 18 float32 in 36.7 us instead of 33.1, 1024 x 256 x 256 in
// 102.5 instead of 95.2. bfloat16 vectors of eight actions (16 bytes) were slower than of four:
// 4096 x 256 x 18 27.4 us against 22.3, 4096 x 300 x 7 20.8 against 17.7.
#pragma once

#include "rlcs_kernels.h"

namespace rlcs {

constexpr int kActV = 4;      // actions per lane and load
constexpr int kActBatch = 2;  // rounds in flight while as many are reduced
constexpr int kActMaxWaves = 16;

// LDS of a workgroup of W waves, K steps per lane: three terms per step (one step past the
// chunk, rounded up).
template <int K>
inline size_t action_lds(int W) { return size_t(3) * size_t(W * kWave * K + 4) * sizeof(float); }

template <int kCtrl>
__device__ __forceinline__ float dpp_add(float v) { return v + dpp_move<kCtrl>(0.f, v); }

// Sum over each group of L consecutive lanes (L a power of two), in every lane of it.
template <int L>
__device__ __forceinline__ float group_sum(float v) {
    if (L > 1) v = dpp_add<0xb1>(v);   // quad_perm [1,0,3,2]
    if (L > 2) v = dpp_add<0x4e>(v);   // quad_perm [2,3,0,1]
    if (L > 4) v = dpp_add<0x141>(v);  // row_half_mirror: the other quad of eight
    if (L > 8) v = dpp_add<0x140>(v);  // row_mirror: the other half of sixteen
    if (L > 16) v += __shfl_xor(v, 16);
    if (L > 32) v += __shfl_xor(v, 32);
    return v;
}

// Raw words of four consecutive elements at any element address.
template <typename DT, bool NT>
__device__ __forceinline__ void load_any4(const DT* p, uint32_t (&w)[sizeof(DT)]) {
    if constexpr (sizeof(DT) == 4) {
        const auto* v = reinterpret_cast<const u32x4_any*>(p);
        const u32x4 u = NT ? __builtin_nontemporal_load(v) : *v;
        w[0] = u.x; w[1] = u.y; w[2] = u.z; w[3] = u.w;
    } else {
        const auto* v = reinterpret_cast<const u32x2_any*>(p);
        const u32x2 u = NT ? __builtin_nontemporal_load(v) : *v;
        w[0] = u.x; w[1] = u.y;
    }
}

// A lane's K steps (1 or 4) of an input from step p0 on, as raw words: one vector load where they
// all lie in the array (`whole`), else the steps of `mask`.
template <typename DT, int K>
__device__ __forceinline__ void load_steps(const void* base, int64_t p0, uint32_t mask, bool whole,
                                           uint32_t (&w)[sizeof(DT)]) {
    const DT* x = static_cast<const DT*>(base);
    if constexpr (K == 1) {
        if (mask) put_element(w, 0, x[p0]);
    } else if (whole) {
        if (mask) load_any4<DT, false>(x + p0, w);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (bit(mask, k)) put_element(w, k, x[p0 + k]);
    }
}
template <int K>
__device__ __forceinline__ void load_step_flags(const uint8_t* base, int64_t p0, uint32_t mask,
                                                bool whole, uint32_t& w) {
    if constexpr (K == 1) {
        if (mask) w = base[p0];
    } else if (whole) {
        if (mask) w = *reinterpret_cast<const flags4_any*>(base + p0);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (bit(mask, k)) w |= uint32_t(base[p0 + k]) << (8 * k);
    }
}

// One round of a wave: 64 / L steps, one vector of Q and one of pi per lane.
template <typename DT>
struct ActionRound {
    uint32_t q[sizeof(DT)], p[sizeof(DT)];
};

// Element `at` of a vector's words (any element where `at` is past the last).
template <typename DT>
__device__ __forceinline__ float vector_element(const uint32_t (&w)[sizeof(DT)], uint32_t at) {
    if constexpr (sizeof(DT) == 4) {
        const uint32_t lo = (at & 1u) ? w[1] : w[0], hi = (at & 1u) ? w[3] : w[2];
        return __uint_as_float((at & 2u) ? hi : lo);
    } else {
        const uint32_t w0 = w[0], w1 = w[1];  // selected as values: a select of addresses would
        const uint32_t u = (at & 2u) ? w1 : w0;  // put the vector into private memory
        return __uint_as_float((at & 1u) ? (u & 0xffff0000u) : (u << 16));
    }
}

// The rounds of one wave: steps [s_lo, s_lo + n_steps) of the [steps, A] tensors, into the LDS
// slots from `slot0` on: s_act holds each step's taken action (as bits), replaced by
// Q(s_t, a_t); s_eq and s_pa receive E_pi Q(s_t) and pi(a_t|s_t). Steps whose action lies outside
// [0, A) keep their s_act and s_pa. TAIL: some round reaches the last V elements of the tensors
// or past them, so vectors are moved back; otherwise no address needs a bound.
// `then` runs once the first rounds' loads are out; it puts the taken actions into s_act.
template <typename DT, int L, bool NT, bool TAIL, class ThenFn>
__device__ __forceinline__ void reduce_actions(const DT* Q, const DT* Pi, int64_t A, int64_t elements,
                                               int64_t s_lo, int n_steps, int lane, float* s_act,
                                               float* s_eq, float* s_pa, ThenFn&& then) {
    constexpr int V = kActV;
    constexpr int spr = kWave / L;  // steps per round
    const int fg = lane & (L - 1), sub = lane / L;
    const uint32_t lane_row = L < kWave ? uint32_t(sub) * uint32_t(A) : 0u;  // L < 64: A <= 128
    const int64_t C = L == kWave ? (A + kWave * V - 1) / (kWave * V) : 1;    // rounds per step
    const int64_t rounds = int64_t((n_steps + spr - 1) / spr) * C;

    // loads: the round's first element (uniform), and the actions of its steps left from there
    int64_t e_load = s_lo * A, left_load = A;
    auto load_round = [&](ActionRound<DT>& x) {
        // a lane past its row's actions reads its row's first vector of the round, a lane past
        // the range the rows after it
        const uint32_t off = lane_row + (fg * V < left_load ? uint32_t(fg * V) : 0u);
        if constexpr (TAIL) {
            const int64_t e = min(e_load + off, elements - V);  // negative below V elements in all
            if (elements >= V) {
                load_any4<DT, NT>(Q + e, x.q);
                load_any4<DT, NT>(Pi + e, x.p);
            } else {
                x = ActionRound<DT>{};
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    put_element(x.q, u, e + u >= 0 ? Q[e + u] : DT{});
                    put_element(x.p, u, e + u >= 0 ? Pi[e + u] : DT{});
                }
            }
        } else {
            load_any4<DT, NT>(Q + e_load + off, x.q);
            load_any4<DT, NT>(Pi + e_load + off, x.p);
        }
        if (L == kWave && left_load > kWave * V) {
            e_load += kWave * V;
            left_load -= kWave * V;
        } else {
            e_load += spr * A - (A - left_load);
            left_load = A;
        }
    };
    int s_red = 0;  // the first step of the round to reduce
    int64_t e_red = s_lo * A, left_red = A;
    float esum = 0.f;
    uint32_t taken = 0;
    auto reduce_round = [&](const ActionRound<DT>& x) {
        const bool live = s_red + sub < n_steps;
        const int slot = s_red + sub;  // slots past n_steps are read, not written
        if (L < kWave || left_red == A) {
            taken = __float_as_uint(s_act[live ? slot : 0]);
            esum = 0.f;
        }
        // the lane's n actions; the taken one is its `at`-th if at < n
        const uint32_t n = fg * V < left_red ? uint32_t(min(left_red - fg * V, int64_t(V))) : 0u;
        const uint32_t at = taken - uint32_t(A - left_red) - uint32_t(fg * V);
        int sh = 0;  // the vector was moved back by this much
        if constexpr (TAIL)
            sh = int(max(e_red + int64_t(lane_row + uint32_t(fg * V)) - (elements - V), int64_t(0)));
        float qv[V], pv[V];
        unpack_words<DT, V>(x.q, qv);
        unpack_words<DT, V>(x.p, pv);
        float qa = 0.f, pa = 0.f;
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const uint32_t k = uint32_t(u - sh);
            esum = k < n ? fmaf(pv[u], qv[u], esum) : esum;
            if constexpr (TAIL) {
                qa = k == at ? qv[u] : qa;
                pa = k == at ? pv[u] : pa;
            }
        }
        if constexpr (!TAIL) {
            qa = vector_element<DT>(x.q, at);
            pa = vector_element<DT>(x.p, at);
        }
        if (live && at < n) {
            s_act[slot] = qa;
            s_pa[slot] = pa;
        }
        if (L == kWave && left_red > kWave * V) {
            e_red += kWave * V;
            left_red -= kWave * V;
            return;
        }
        const float sum = group_sum<L>(esum);
        if (live && fg == 0) s_eq[slot] = sum;
        e_red += spr * A - (A - left_red);
        left_red = A;
        s_red += spr;
    };
    ActionRound<DT> x[kActBatch], y[kActBatch];
#pragma unroll
    for (int u = 0; u < kActBatch; ++u)
        if (u < rounds) load_round(x[u]);
    then();
    wave_lds_sync();
    for (int64_t i = 0; i < rounds; i += 2 * kActBatch) {
#pragma unroll
        for (int u = 0; u < kActBatch; ++u)
            if (i + kActBatch + u < rounds) load_round(y[u]);
#pragma unroll
        for (int u = 0; u < kActBatch; ++u)
            if (i + u < rounds) reduce_round(x[u]);
#pragma unroll
        for (int u = 0; u < kActBatch; ++u)
            if (i + 2 * kActBatch + u < rounds) load_round(x[u]);
#pragma unroll
        for (int u = 0; u < kActBatch; ++u)
            if (i + kActBatch + u < rounds) reduce_round(y[u]);
    }
}

// Workgroup g owns rows [g * R, g * R + R), R * T <= E = W * 64 * K steps, or one longer row
// walked in chunks of E steps from its end. L: lanes per step, the fewest (a power of two, 64 at
// most) that hold its A actions a vector to a lane. NT: Q and pi by non-temporal loads. Grid:
// ceil(N / R) workgroups of W waves.
template <typename DT, bool TR, int L, int K, bool NT>
__global__ void __launch_bounds__(kActMaxWaves * kWave) action_rows_kernel(Args a, int64_t R) {
    using Op = RetraceFullOp;
    constexpr int kSpan = kWave * K;  // steps per wave
    extern __shared__ __align__(16) float s_terms[];
    __shared__ float s_a[kActMaxWaves], s_b[kActMaxWaves];
    __shared__ float s_carry;
    const int W = int(blockDim.x) / kWave;
    const int E = W * kSpan, stride = E + 4;
    float* s_act = s_terms;               // the taken action, then Q(s_t, a_t)
    float* s_eq = s_terms + stride;       // E_pi Q(s_t)
    float* s_pa = s_terms + 2 * stride;   // pi(a_t|s_t)
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);  // uniform
    const int64_t T = a.T, A = a.A, steps = a.N * T, elements = steps * A;
    const int64_t row_lo = int64_t(blockIdx.x) * R;
    const int64_t lo = row_lo * T, hi = min(row_lo + R, a.N) * T;
    const RowBase base{lo, row_lo, 0};
    const int q0 = wave * kSpan + lane_group<true>(lane) * K;  // the lane's steps in the chunk

    float carry = 0.f;
    for (int64_t chunk_lo = hi - E;; chunk_lo -= E) {
        // the lane's own steps [p0, p0 + K); lane 0 also takes mu of the step past its own (in
        // the next wave, or the chunk before)
        const int64_t p0 = chunk_lo + q0;
        uint32_t valid = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (p0 + k >= lo && p0 + k < hi) valid |= 1u << k;
        const bool whole = p0 >= 0 && p0 + K <= steps;
        uint32_t tw[1] = {0u}, rw[1] = {0u};
        uint32_t r_w[sizeof(DT)] = {}, mu_w[sizeof(DT)] = {}, bv_w[sizeof(DT)] = {};
        uint32_t act_w[4] = {0u, 0u, 0u, 0u};
        if (TR) load_step_flags<K>(a.trunc, p0, valid, whole, rw[0]);
        load_steps<float, K>(a.actions, p0, valid, whole, act_w);
        if (a.term) load_step_flags<K>(a.term, p0, valid, whole, tw[0]);
        load_steps<DT, K>(a.in[3], p0, valid, whole, mu_w);
        load_steps<DT, K>(a.in[0], p0, valid, whole, r_w);
        float mu_next = 1.f;
        if (lane == 0 && bit(valid, K - 1) && p0 + K < hi) mu_next = load_one<DT>(a.in[3], p0 + K);
        // row edges and bootstraps of the lane's steps
        int64_t row = 0, t = 0;
        const int64_t p_first = max(p0, lo);
        if (valid) row_and_step(base, p_first, T, a.inv_T, row, t);
        uint32_t edge = 0;
        float B[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            B[k] = 0.f;
            if (p0 + k < p_first) continue;
            if (bit(valid, k) && t == T - 1) {
                edge |= 1u << k;
                if (a.row_value) B[k] = load_one<DT>(a.row_value, row);
            }
            if (++t == T) { t = 0; ++row; }
        }
        // while the first rounds' loads are in flight: the continuations, where a step is
        // truncated, and the taken actions to LDS
        uint32_t trunc = 0;
        auto then = [&]() {
            if (TR) {
                trunc = flag_mask<4>(rw) & valid;
                if (trunc) load_steps<DT, K>(a.in[4], p0, trunc, whole, bv_w);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                s_act[q0 + k] = __uint_as_float(act_w[k]);
                s_pa[q0 + k] = 0.f;  // stays so where the action lies outside the axis
            }
        };
        const int64_t ws = chunk_lo + int64_t(wave) * kSpan;
        const int64_t s_lo = max(ws, lo);
        const int n_steps = int(max(min(ws + kSpan, hi) - s_lo, int64_t(0)));
        const int slot0 = int(s_lo - chunk_lo);
        if (n_steps > 0) {
            const DT* Q = static_cast<const DT*>(a.in[1]);
            const DT* Pi = static_cast<const DT*>(a.in[2]);
            if ((s_lo + kSpan + 1) * A + kActV > elements)
                reduce_actions<DT, L, NT, true>(Q, Pi, A, elements, s_lo, n_steps, lane, s_act + slot0,
                                            s_eq + slot0, s_pa + slot0, then);
            else
                reduce_actions<DT, L, NT, false>(Q, Pi, A, elements, s_lo, n_steps, lane, s_act + slot0,
                                             s_eq + slot0, s_pa + slot0, then);
        }
        __syncthreads();

        // the scan: Table 1's coefficients from the reduced terms
        float d[Op::kSlots][K], nb[Op::kNbr];
        {
            float r[4], mu[4], bv[4];
            unpack_words<DT, 4>(r_w, r);
            unpack_words<DT, 4>(mu_w, mu);
            unpack_words<DT, 4>(bv_w, bv);
            bool bad = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const bool ok = bit(valid, k);
                const bool in = ok && act_w[k] < uint64_t(A);  // negative: above any A
                bad = bad || (ok && !in);
                d[0][k] = r[k];
                d[1][k] = in ? s_act[q0 + k] : 0.f;
                d[2][k] = ok ? s_eq[q0 + k] : 0.f;
                d[3][k] = ok ? s_pa[q0 + k] / mu[k] : 0.f;
                d[4][k] = bv[k];
            }
            if (bad && a.ws) report_bad_action(a.ws);  // the step takes Q and pi as 0
        }
        const uint32_t term = flag_mask<4>(tw) & valid;
        nb[0] = shift_up1(d[2][0], 0.f);
        nb[1] = shift_up1(Op::trace(a.p, d[3][0]), 0.f);
        if (lane == 0) {
            nb[0] = s_eq[q0 + K];
            nb[1] = Op::trace(a.p, s_pa[q0 + K] / mu_next);
        }
        float al[K], be[K];
        Op::template build<K, TR>(a.p, d, term, trunc, edge, B, nb, al, be);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (!bit(valid, k)) { al[k] = 0.f; be[k] = 1.f; }
        Pair agg = Pair{al[K - 1], be[K - 1]};
#pragma unroll
        for (int k = K - 2; k >= 0; --k) agg = compose(Pair{al[k], be[k]}, agg);
        const Pair incl = wave_scan_inclusive(agg, lane);
        Pair win = identity_pair();
        if (W > 1) {
            if (lane == kWave - 1) { s_a[wave] = incl.a; s_b[wave] = incl.b; }
            __syncthreads();
            win = waves_in<true>(s_a, s_b, W, wave, lane);
        }
        const float Xw = apply(win, carry);
        const float X = shift_up1(apply(incl, Xw), Xw);
        float An[K], o0[K], o1[K];
        float nxt = X;
#pragma unroll
        for (int k = K - 1; k >= 0; --k) { An[k] = fmaf(be[k], nxt, al[k]); nxt = An[k]; }
        Op::template finish<K, TR>(a.p, d, term, trunc, edge, B, nb, An, X, o0, o1);
        if constexpr (K == 1) {
            if (valid) {
                __builtin_nontemporal_store(o0[0], a.out0 + p0);
                if (a.out1) __builtin_nontemporal_store(o1[0], a.out1 + p0);
            }
        } else if (valid == (1u << K) - 1u) {
            store4_any(a.out0 + p0, f32x4{o0[0], o0[1], o0[2], o0[3]});
            if (a.out1) store4_any(a.out1 + p0, f32x4{o1[0], o1[1], o1[2], o1[3]});
        } else if (valid) {
            store_k<K>(a.out0, p0, valid, false, o0);
            if (a.out1) store_k<K>(a.out1, p0, valid, false, o1);
        }
        if (chunk_lo <= lo) break;
        // the next chunk (earlier in time) continues from the state at chunk_lo (lane 63 of wave
        // 0) and finds this chunk's first step as the one past its own
        const float eq_first = s_eq[0], pa_first = s_pa[0];
        if (threadIdx.x == kWave - 1) s_carry = An[0];
        __syncthreads();
        carry = s_carry;
        if (threadIdx.x == 0) { s_eq[E] = eq_first; s_pa[E] = pa_first; }
    }
}

}  // namespace rlcs
