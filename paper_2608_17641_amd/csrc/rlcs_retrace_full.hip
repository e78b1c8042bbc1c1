// Retrace(lambda) entry point over the action axis (Table 1; Sections 3.3.3 and 7.3).
#include "rlcs_actions.h"
#include "rlcs_dispatch.h"

using namespace rlcs;
using namespace rlcs::host;

namespace {

// Q and pi of more than this many bytes are read by non-temporal loads. The caller's last
// writes or reads of smaller ones may still be in the 256 MB Infinity Cache, where ordinary
// loads find them faster; larger ones stream from HBM, where the hint pays. Three input sets in
// turn, float32, ordinary against non-temporal: 32 MB (4001 x 201 x 5) 13.8 against 15.3 us,
// 59 MB (4096 x 256 x 7) 16.0 against 17.5; 100 MB (x 12) 26.1 against 23.6, 134 MB
// (16384 x 256 x 4) 49.9 against 45.0, 151 MB (4096 x 256 x 18) 35.3 against 33.1, 537 MB (x 64)
// 101 against 92; bfloat16 with K = 1, 134 MB (511 x 1024 x 64) 37.0 against 33.4, 96 MB (500 x 1000 x
// 48) 32.9 against 30.4, 84 MB (2000 x 256 x 41) 31.5 against 30.6.
constexpr int64_t kActCachedBytes = int64_t(80) << 20;

// Calls of few actions (few bytes per step) scan K = 4 steps per lane, 256 per wave, from this
// many steps on: their waves of 64 steps hold too little to fill memory's latency (float32:
// 4096 x 256 x 4 11.8 us against 13.3 with K = 1, x 2 9.4 against 11.0; bfloat16 x 18 22.3 against
// 25.8, x 64 50.2 against 52.2). With more a wave of 256 steps is a long chain of rounds and
// K = 1 wins (float32 4096 x 256 x 12 23.6 us against 27.0, x 18 33.1 against 37.8), as it does in
// small calls (200 x 1024 x 4 5.6 against 6.8, 64 x 1024 x 18 8.6 against 17.0).
constexpr int64_t kActFourSteps = int64_t(1) << 19;
template <typename DT>
constexpr int kActFourLanes = sizeof(DT) == 4 ? 2 : 16;

// Long rows (sixteen waves or more) of at least this many environments take workgroups of eight
// waves, two to a CU, each of which reads while the other scans (512 x 4096 x 4 27.8 -> 24.6 us,
// 512 x 4096 x 18 74.7 -> 66.5); fewer rows keep sixteen (64 x 1024 x 18 8.4 us against 11.3).
constexpr int64_t kActTwoPerCu = 512;

template <typename DT, int L, int K, bool NT>
rlcs_status launch_actions(const Args& a, hipStream_t s) {
    constexpr int64_t span = kWave * K;  // steps per wave
    const int64_t T = a.T;
    // rows of up to one wave's span: as many whole rows as it holds; longer ones: one per
    // workgroup, as many waves as it needs (kActMaxWaves, then chunk by chunk)
    const int64_t R = T <= span ? span / T : 1;
    const int64_t need = (T + span - 1) / span;
    const int most = a.N >= kActTwoPerCu && need >= kActMaxWaves ? kActMaxWaves / 2 : kActMaxWaves;
    const int W = int(need < most ? need : most);
    const int64_t groups = (a.N + R - 1) / R;
    if (groups > INT32_MAX) return RLCS_ERR_INVALID_ARG;
    const dim3 grid(static_cast<unsigned>(groups)), block(unsigned(W * kWave));
    if (a.trunc)
        hipLaunchKernelGGL((action_rows_kernel<DT, true, L, K, NT>), grid, block, action_lds<K>(W), s, a, R);
    else
        hipLaunchKernelGGL((action_rows_kernel<DT, false, L, K, NT>), grid, block, action_lds<K>(W), s, a, R);
    return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
}

template <typename DT>
rlcs_status run_actions(const Args& a, hipStream_t s) {
    const bool nt = a.N * a.T > kActCachedBytes / (2 * int64_t(sizeof(DT))) / a.A;
    const bool four = a.N * a.T >= kActFourSteps || a.T > kActMaxWaves * kWave;
    const int64_t vectors = (a.A + kActV - 1) / kActV;
    auto go = [&](auto lanes) -> rlcs_status {
        constexpr int L = decltype(lanes)::value;
        if constexpr (L <= kActFourLanes<DT>) {
            if constexpr (sizeof(DT) == 2) {  // (so few steps of float32 are never above the limit)
                if (!four && nt) return launch_actions<DT, L, 1, true>(a, s);
            }
            if (!four) return launch_actions<DT, L, 1, false>(a, s);
            return nt ? launch_actions<DT, L, 4, true>(a, s) : launch_actions<DT, L, 4, false>(a, s);
        } else {
            return nt ? launch_actions<DT, L, 1, true>(a, s) : launch_actions<DT, L, 1, false>(a, s);
        }
    };
    if (vectors <= 1) return go(std::integral_constant<int, 1>{});
    if (vectors <= 2) return go(std::integral_constant<int, 2>{});
    if (vectors <= 4) return go(std::integral_constant<int, 4>{});
    if (vectors <= 8) return go(std::integral_constant<int, 8>{});
    if (vectors <= 16) return go(std::integral_constant<int, 16>{});
    if (vectors <= 32) return go(std::integral_constant<int, 32>{});
    return go(std::integral_constant<int, 64>{});
}

}  // namespace

extern "C" {

rlcs_status rlcs_retrace_full(const void* r, const void* q, const void* pi,
                              const int32_t* actions, const void* mu, const uint8_t* term,
                              const uint8_t* trunc, const void* bv, const void* boot,
                              float* delta, float* q_ret, int64_t N, int64_t T, int64_t A,
                              float gamma, float lambda, float c_bar, rlcs_dtype dtype,
                              void* ws, size_t ws_bytes, rlcs_stream_t stream) {
    rlcs_status st = check_common(N, T, dtype, {r, q, pi, mu, bv, boot}, {delta, q_ret});
    if (st != RLCS_OK) return st;
    if (!unit_interval(gamma) || !unit_interval(lambda) || !positive(c_bar)) return RLCS_ERR_INVALID_ARG;
    if (A < 1 || A > INT32_MAX) return RLCS_ERR_INVALID_ARG;
    if (N == 0 || T == 0) return RLCS_OK;
    if (N * T > INT64_MAX / A) return RLCS_ERR_INVALID_ARG;
    if (!r || !q || !pi || !actions || !mu || !delta || (trunc && !bv)) return RLCS_ERR_INVALID_ARG;
    if (!aligned(actions, 4)) return RLCS_ERR_INVALID_ARG;
    Args a = make_args(N, T, gamma, lambda, 1.f, c_bar);
    a.in[0] = r; a.in[1] = q; a.in[2] = pi; a.in[3] = mu; a.in[4] = bv;
    a.actions = actions; a.A = A;
    a.term = term; a.trunc = trunc; a.row_value = boot;
    a.out0 = delta; a.out1 = q_ret;
    // a workspace, if given, receives the out-of-range-action report in its error word
    a.ws = (ws && ws_bytes >= sizeof(WsHeader) && aligned(ws, 64)) ? ws : nullptr;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    return dtype == RLCS_BF16 ? run_actions<bf16_t>(a, s) : run_actions<float>(a, s);
}

}  // extern "C"
