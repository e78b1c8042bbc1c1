// Host-side pieces shared by the entry points: argument checks (all before any HIP call),
// the choice of kernel variant, and the launches. Each entry point lives in its own
// translation unit so that the library's kernels compile in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <climits>
#include <cstdint>
#include <initializer_list>
#include <type_traits>

#include "rlcs.h"
#include "rlcs_kernels.h"

namespace rlcs {
namespace host {

// Workgroups of `kernel` (with `threads` lanes) that the current device holds at once, or 0.
template <class Kernel>
int64_t resident_groups(Kernel kernel, int threads, size_t lds = 0) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds) != hipSuccess) return 0;
    return int64_t(cus) * per_cu;
}

// Waves per workgroup: 4 for rows of up to 4*64*K steps (several rows per workgroup), 16 for
// longer rows (one row, or a 16*64*K-step tile of one, per workgroup).
constexpr int kSmallWaves = 4;
constexpr int kLargeWaves = 16;
// Wave-rows calls of float32 GAE with truncation take workgroups of four waves (each wave still
// on its own) from 2^18 to 2^20 steps (1024 to 4096 waves), one wave per workgroup otherwise.
// Measured (C harness, cold, one-wave against four-wave workgroups): 4096 x 256 5.21 -> 4.78 us,
// 8192 x 128 5.20 -> 4.85, 16384 x 64 5.23 -> 4.91, 4096 x 128 3.55 -> 3.49, 2048 x 256 3.53 ->
// 3.49, 1024 x 256 3.00 -> 2.92; with fewer waves the four-wave grid leaves CUs idle (512 x 256
// 2.57 -> 2.59, 4096 x 32 2.59 -> 2.70); above 2^20 steps four waves lose 4-8 % (6144 x 256 6.17
// -> 6.68, 16384 x 256 14.6 -> 15.3), and so they do without truncation (4096 x 256 4.29 ->
// 4.46), for bfloat16 (16384 x 64 4.69 -> 4.92) and for V-Trace (4096 x 256 6.03 -> 6.16). Two
// waves per workgroup lost everywhere, eight gained less than four.
constexpr int64_t kWaveRowsQuadMinSteps = int64_t(1) << 18;
constexpr int64_t kWaveRowsQuadSteps = int64_t(1) << 20;
template <class Op, typename DT, bool TR> struct WaveRowsQuads : std::false_type {};
template <> struct WaveRowsQuads<GaeOp, float, true> : std::true_type {};

// Steps per lane: one 16-byte vector of each input.
template <typename DT> struct Width;
template <> struct Width<float> { static constexpr int K = 4; };
template <> struct Width<bf16_t> { static constexpr int K = 8; };

// Smallest tile of the split-row variant (float32, 4 waves), which sizes the workspace.
constexpr int64_t kMinTile = int64_t(kSmallWaves) * kWave * Width<float>::K;

// Rows longer than one large workgroup's chunk are split across workgroups (a workspace given,
// T a multiple of K) when there are fewer than kSplitBelowRows of them. With more rows, or
// shorter ones, whole-row workgroups are faster: a tile waiting for its neighbours' maps costs
// more than the idle CUs (timed: 64 x 4096 fp32 GAE 3.9 us whole-row, 5.2 us split; 512 x 8192
// the same either way; 16 x 16384 bf16 9.2 us whole-row, 6.4 us split).
constexpr int64_t kSplitBelowRows = 256;
// Split rows use 4-wave tiles, or 16-wave tiles when a row would have more than this many
// 4-wave ones (all tiles of a row draw their tickets from one word).
constexpr int64_t kMaxSmallTilesPerRow = 64;

// Longest supported row (the kernels keep offsets within a row range in 32 bits).
constexpr int64_t kMaxT = int64_t(1) << 30;

// Kernel-variant override of the calling thread (rlcs_testing_set_variant, a test-only entry
// point); defined in rlcs_common.hip.
extern thread_local int g_variant;
extern thread_local int g_whitening_wait;  // rlcs_testing_set_whitening_wait; -1: as ever

inline bool aligned(const void* p, size_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; }
inline bool unit_interval(float x) { return x >= 0.f && x <= 1.f; }  // false for NaN
inline bool positive(float x) { return x > 0.f; }                     // false for NaN, true for +inf

inline size_t dtype_size(rlcs_dtype d) { return d == RLCS_BF16 ? 2 : 4; }

// Common checks of sizes, dtype and the element alignment of every given pointer.
inline rlcs_status check_common(int64_t N, int64_t T, rlcs_dtype dtype,
                         std::initializer_list<const void*> data, std::initializer_list<const void*> outs) {
    if (N < 0 || T < 0) return RLCS_ERR_INVALID_ARG;
    if (dtype != RLCS_F32 && dtype != RLCS_BF16) return RLCS_ERR_DTYPE;
    if (T > kMaxT || (T > 0 && N > INT64_MAX / T)) return RLCS_ERR_INVALID_ARG;
    const size_t es = dtype_size(dtype);
    for (const void* p : data)
        if (p && !aligned(p, es)) return RLCS_ERR_INVALID_ARG;
    for (const void* p : outs)
        if (p && !aligned(p, 4)) return RLCS_ERR_INVALID_ARG;
    return RLCS_OK;
}

// How one call is run.
struct Plan {
    bool split;           // tiles kernel (rows split across workgroups) vs rows kernel
    int waves;            // waves per workgroup
    int64_t tiles_per_row;  // tiles kernel: tiles of each row (grid = N * tiles_per_row)
    int64_t rows_per_wg;  // rows kernel: rows per workgroup
    bool pad;             // rows kernel, vector path: lanes outside the range or in row gaps skip
    int wave_rows_log2T;  // >= 0: wave_rows_kernel (rows tile a wave exactly; T = 2^log2T)
    int flat_R;           // > 0: flat_rows_kernel with this many whole rows per workgroup
    int flat_W;           // its waves per workgroup (4, or 16 for float32 rows)
    uint32_t flat_magic;  // ceil(2^flat_shift(flat_W) / T): a lane's row by multiply-shift
    int ragged_R;         // > 0: ragged_rows_kernel with this many whole rows per workgroup
    int ragged_W;         // its waves per workgroup
    int ragged_grid;      // its lanes' first step is a multiple of this
    uint32_t ragged_magic;
};

// The ragged rows kernel's plan for rows of T steps, K <= T <= kRaggedWaves * 64 * K: as many
// whole rows as fit four waves, or one longer row on as many waves as it needs; the lanes start on
// the coarsest of a 128-byte line of inputs, a 16-byte vector and a step that leaves them room
// (a range of R * T steps starts up to `grid` - gcd(R * T, grid) steps past one). More rows to a
// workgroup gain more than the alignment: GAE 9001 x 201 float32 8.5 us with five rows from any
// step against 9.3 with four from a line, 9001 x 401 bfloat16 12.6 against 13.9.
inline void plan_ragged(Plan& p, int64_t T, int64_t K) {
    const int64_t span = int64_t(kWave) * K, four = kSmallWaves * span;
    const int64_t R = T < four ? four / T : 1;
    const int64_t most = R > 1 ? four : kRaggedWaves * span;
    for (const int64_t grid : {8 * K, K, int64_t(1)}) {
        int64_t g = grid, b = R * T % grid;
        while (b) { const int64_t r = g % b; g = b; b = r; }
        const int64_t steps = R * T + grid - g;
        if (steps > most) continue;
        p.ragged_R = int(R);
        p.ragged_W = int((steps + span - 1) / span);
        p.ragged_grid = int(grid);
        p.ragged_magic = R > 1 ? uint32_t(((int64_t(1) << flat_shift(4)) + T - 1) / T) : 0u;
        return;
    }
}

template <class Op, typename DT, bool VEC, bool TR, int W, bool PAD = false>
void launch_w(const Args& a, const Plan& p, hipStream_t stream) {
    constexpr int K = Width<DT>::K;
    const dim3 block(W * kWave);
    if (p.split) {
        hipLaunchKernelGGL((tiles_kernel<Op, DT, K, W, VEC, TR>),
                           dim3(unsigned(a.N * p.tiles_per_row)), block, 0, stream, a,
                           p.tiles_per_row);
        return;
    }
    const int64_t groups = (a.N + p.rows_per_wg - 1) / p.rows_per_wg;
    hipLaunchKernelGGL((rows_kernel<Op, DT, K, W, VEC, TR, PAD>), dim3(unsigned(groups)), block,
                       0, stream, a, p.rows_per_wg);
}

template <class Op, typename DT, bool VEC, bool TR>
rlcs_status launch(const Args& a, const Plan& p, hipStream_t stream) {
    if (p.ragged_R > 0) {
        constexpr int K = Width<DT>::K;
        hipLaunchKernelGGL((ragged_rows_kernel<Op, DT, K, TR, false>), dim3(unsigned((a.N + p.ragged_R - 1) / p.ragged_R)),
                           dim3(unsigned(p.ragged_W * kWave)), K == 8 ? p.ragged_W * 2048 : 0, stream, a,
                           p.ragged_R, p.ragged_magic, p.ragged_grid);
        return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
    }
    if constexpr (VEC) {
        if (p.flat_R > 0) {
            const dim3 grid(unsigned((a.N + p.flat_R - 1) / p.flat_R));
            if constexpr (sizeof(DT) == 4) {
                if (p.flat_W == kLargeWaves) {
                    hipLaunchKernelGGL((flat_rows_kernel<Op, DT, Width<DT>::K, TR, kLargeWaves>), grid,
                                       dim3(kLargeWaves * kWave), 0, stream, a, p.flat_R, p.flat_magic);
                    return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
                }
            }
            hipLaunchKernelGGL((flat_rows_kernel<Op, DT, Width<DT>::K, TR, kSmallWaves>), grid,
                               dim3(kSmallWaves * kWave), 0, stream, a, p.flat_R, p.flat_magic);
            return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
        }
        if (p.wave_rows_log2T >= 0) {
            constexpr int64_t span = int64_t(kWave) * Width<DT>::K;
            const int64_t waves = (a.N * a.T + span - 1) / span;
            if constexpr (WaveRowsQuads<Op, DT, TR>::value) {
                if (a.N * a.T >= kWaveRowsQuadMinSteps && a.N * a.T <= kWaveRowsQuadSteps) {
                    hipLaunchKernelGGL((wave_rows_kernel<Op, DT, Width<DT>::K, TR, 4>),
                                       dim3(unsigned((waves + 3) / 4)), dim3(4 * kWave), 0, stream, a,
                                       p.wave_rows_log2T);
                    return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
                }
            }
            hipLaunchKernelGGL((wave_rows_kernel<Op, DT, Width<DT>::K, TR>), dim3(unsigned(waves)),
                               dim3(kWave), 0, stream, a, p.wave_rows_log2T);
            return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
        }
    }
    if constexpr (VEC) {
        if (p.pad && !p.split) {
            if (p.waves == kSmallWaves) launch_w<Op, DT, true, TR, kSmallWaves, true>(a, p, stream);
            else launch_w<Op, DT, true, TR, kLargeWaves, true>(a, p, stream);
            return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
        }
    }
    if (p.waves == kSmallWaves) launch_w<Op, DT, VEC, TR, kSmallWaves>(a, p, stream);
    else launch_w<Op, DT, VEC, TR, kLargeWaves>(a, p, stream);
    return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
}

template <class Op, typename DT>
rlcs_status dispatch_dt(Args& a, bool has_trunc, void* ws, size_t ws_bytes, hipStream_t stream) {
    constexpr int K = Width<DT>::K;
    constexpr int64_t E_small = int64_t(kSmallWaves) * kWave * K;
    constexpr int64_t E_large = int64_t(kLargeWaves) * kWave * K;
    const int64_t N = a.N, T = a.T;

    // Vector path: 16-byte data and output vectors, K-byte flag vectors.
    bool vec = true;
    for (int s = 0; s < Op::kSlots; ++s)
        if (Op::slot_used(s, has_trunc) && !aligned(a.in[s], 16)) vec = false;
    if (!aligned(a.out0, 16) || (a.out1 && !aligned(a.out1, 16))) vec = false;
    if (Op::kFlags && ((a.term && !aligned(a.term, K)) || (has_trunc && !aligned(a.trunc, K)))) vec = false;

    Plan p{};
    // Split rows: 4-wave tiles unless a row would have too many of them.
    const int64_t P_small = (T + E_small - 1) / E_small;
    const bool small_tiles = P_small <= kMaxSmallTilesPerRow;
    p.tiles_per_row = small_tiles ? P_small : (T + E_large - 1) / E_large;
    const bool slots_ok = N <= kWsSlots;  // one draw slot per row
    const size_t ws_need = slots_ok ? kWsRecordsOffset + size_t(N * p.tiles_per_row) * kWsRecordBytes
                                    : kWsRecordsOffset;
    const bool ws_ok = ws && ws_bytes >= ws_need && aligned(ws, 64);
    const int forced = g_variant;
    if (forced == 2) {
        if (!ws_ok) return RLCS_ERR_WORKSPACE;
        p.split = slots_ok;  // more rows than draw slots: whole rows
    } else if (forced == 1) {
        p.split = false;
    } else {
        p.split = ws_ok && slots_ok && T % K == 0 && T > E_large && N < kSplitBelowRows;
    }
    if (p.split) p.waves = small_tiles ? kSmallWaves : kLargeWaves;
    else if (T > E_small) p.waves = kLargeWaves;
    else p.waves = kSmallWaves;
    p.wave_rows_log2T = -1;
    p.flat_R = 0;
    p.flat_W = kSmallWaves;
    // Dense rows up to one sixteen-wave chunk (float32) or one wave (bfloat16), except powers of
    // two that tile a wave: the flat rows kernel. Measured against
    // the rows kernel (C harness, cold): GAE 4096x192 fp32 5.05 -> 4.62 us, 4096x252 5.97 -> 5.22,
    // 4096x500 10.04 -> 8.68, 4096x1000 16.59 -> 15.48, 4096x1024 16.13 -> 15.54; bf16 16384x200
    // 12.83 -> 11.14, 16384x504 24.98 -> 23.16; longer bf16 rows were within 2.5 % either way
    // (16384x1000 45.4 -> 44.2, 16384x2048 82.3 -> 83.4) and keep the rows kernel.
    // Rows whose length is not a multiple of K take it as well when a workgroup's rows can start
    // and end on vector boundaries (R a multiple of K / gcd(T, K), N*T a multiple of K).
    // float32 rows up to one sixteen-wave chunk (4096 steps) take it too, in sixteen-wave
    // ranges where four waves hold none, in place of one sixteen-wave rows-kernel workgroup per
    // row (same protocol, GAE): 4096x2000 36.2 -> 29.9 us, 2048x3000 32.7 -> 24.7, 1024x4096
    // 19.6 -> 17.1, 4096x1500 33.0 -> 24.7, 2048x2048 19.7 -> 17.0, 8192x1100 44.1 -> 34.0;
    // 64x4096 even (4.45 -> 4.43).
    const int64_t flat_max = sizeof(DT) == 4 ? E_large : int64_t(kWave) * K;
    if (!p.split && vec && T > K && T <= flat_max && (N * T) % K == 0 &&
        !((T & (T - 1)) == 0 && T <= int64_t(kWave) * K)) {
        int64_t gcd = K, b = T % K;
        while (b) { const int64_t r = gcd % b; gcd = b; b = r; }
        const int64_t step = K / gcd;  // rows per vector-aligned range
        int64_t R = E_small / T / step * step;
        int W = kSmallWaves;
        // float32 rows too long for `step` of them in four waves (more than 1024 steps, or more
        // than 256 that are not a multiple of K): sixteen waves hold 4096 steps
        if (R == 0 && sizeof(DT) == 4) {
            R = E_large / T / step * step;
            W = kLargeWaves;
        }
        const int64_t magic = ((int64_t(1) << flat_shift(W)) + T - 1) / T;
        if (R > 0 && (int64_t(W) * kWave * K - 1) * magic < (int64_t(1) << 32)) {
            p.flat_R = int(R);
            p.flat_W = W;
            p.flat_magic = uint32_t(magic);
            if ((N + R - 1) / R > INT32_MAX) return RLCS_ERR_INVALID_ARG;
        }
    }
    if (!p.split && vec && T >= K && T <= int64_t(kWave) * K && (T & (T - 1)) == 0) {
        // rows tile a wave exactly: the wave-rows kernel
        if ((N * T + int64_t(kWave) * K - 1) / (int64_t(kWave) * K) > INT32_MAX) return RLCS_ERR_INVALID_ARG;
        int l = 0;
        while ((int64_t(1) << l) < T) ++l;
        p.wave_rows_log2T = l;
    }
    // Other rows of up to sixteen waves run on the ragged rows kernel, except rows that fill a
    // four-wave chunk of the rows kernel exactly (aligned arrays; bfloat16 rows of 1024 and 2048
    // steps: eligibility traces 16384 x 1024 23.3 us there against 26.0, GAE 16384 x 2048 85.5
    // against 86.9). Measured against the rows kernel, which they took before, lane by lane or
    // one sixteen-wave workgroup per row: V-Trace 4096 x 2001 float32 43.6 -> 33.8 us, GAE 4096 x
    // 4095 106 -> 60, TD(lambda) 5001 x 3001 78.8 -> 43.4, GAE 9001 x 15 4.5 -> 3.5; bfloat16
    // V-Trace 8192 x 3001 113 -> 73, 8192 x 4096 122 -> 98, 8192 x 1500 44.2 -> 38.2, GAE 4096 x
    // 8192 98 -> 90, 16384 x 1000 46.1 -> 44.9, 300 x 4000 8.2 -> 8.0.
    if (!p.split && p.flat_R == 0 && p.wave_rows_log2T < 0 && T >= K && T <= E_large &&
        (!vec || T % K || E_small % T)) {
        plan_ragged(p, T, K);
        if (p.ragged_R > 0 && (N + p.ragged_R - 1) / p.ragged_R > INT32_MAX) return RLCS_ERR_INVALID_ARG;
    }
    if (p.split) {
        if (N * p.tiles_per_row > INT32_MAX) return RLCS_ERR_INVALID_ARG;
        a.ws = ws;
    } else {
        const int64_t E = int64_t(p.waves) * kWave * K;
        // Whole rows per workgroup: as many as fit in one chunk (at least one). When T is not
        // a multiple of K a row range may start mid-vector, costing up to K-1 extra slots.
        const int64_t slack = (T % K == 0) ? 0 : K - 1;
        p.rows_per_wg = (T <= E - slack) ? (E - slack) / T : 1;
        if ((N + p.rows_per_wg - 1) / p.rows_per_wg > INT32_MAX) return RLCS_ERR_INVALID_ARG;
        // When a workgroup's rows do not fill its chunks exactly, every chunk still takes the
        // vector path lane by lane: only the lanes at the ragged ends of the workgroup's range
        // go element-wise.
        p.pad = vec && T >= K && (T % K != 0 || (p.rows_per_wg * T) % E != 0);
    }

    if constexpr (Op::kFlags) {
        if (has_trunc) {
            return vec ? launch<Op, DT, true, true>(a, p, stream)
                       : launch<Op, DT, false, true>(a, p, stream);
        }
    }
    return vec ? launch<Op, DT, true, false>(a, p, stream)
               : launch<Op, DT, false, false>(a, p, stream);
}

template <class Op>
rlcs_status dispatch(Args& a, rlcs_dtype dtype, bool has_trunc, void* ws, size_t ws_bytes,
                     rlcs_stream_t stream) {
    if (a.N == 0 || a.T == 0) return RLCS_OK;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (dtype == RLCS_BF16) return dispatch_dt<Op, bf16_t>(a, has_trunc, ws, ws_bytes, s);
    return dispatch_dt<Op, float>(a, has_trunc, ws, ws_bytes, s);
}

// Rows with a row stride (period) above T, whole rows per workgroup: the ragged rows kernel where one
// workgroup holds a row, except as below; otherwise the rows kernel over the positions
// n * period + t (the steps t >= T of each period are skipped), vector loads and stores where a lane's
// steps allow when the arrays are aligned, else element-wise.
template <class Op>
rlcs_status dispatch_strided_rows(Args& a, int64_t period, rlcs_dtype dtype, bool has_trunc,
                                  rlcs_stream_t stream) {
    if (a.N == 0 || a.T == 0) return RLCS_OK;
    if (period > kMaxT) return RLCS_ERR_INVALID_ARG;
    a.period = period;
    a.inv_period = 1.f / float(period);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    auto run = [&](auto dt_tag) -> rlcs_status {
        using DT = decltype(dt_tag);
        constexpr int K = Width<DT>::K;
        // Whole vectors throughout: T >= K, data and outputs 16-byte aligned, flags K-byte aligned.
        bool vec = a.T >= K;
        for (int i = 0; i < Op::kSlots; ++i)
            if (Op::slot_used(i, has_trunc) && !aligned(a.in[i], 16)) vec = false;
        if (!aligned(a.out0, 16) || (a.out1 && !aligned(a.out1, 16))) vec = false;
        if (Op::kFlags && ((a.term && !aligned(a.term, K)) || (has_trunc && !aligned(a.trunc, K)))) vec = false;
        const int64_t E_small = int64_t(kSmallWaves) * kWave * K;
        // Rows of one vector to sixteen waves: each row's lanes from its own first step on. As many
        // rows as four waves hold, or one on as many waves as it needs. Against the lane-by-lane
        // rows kernel: V-Trace bfloat16 13064 x 64 (stride 68) 14.5 -> 6.1 us, eligibility traces
        // 32523 x 907 (911) 124 -> 49, GAE float32 5038 x 483 (491) 17.7 -> 11.1.
        // Not bfloat16 rows of whole aligned vectors (32 to 2048 steps) that do not tile a wave of 128
        // steps or more: the rows kernel's one load per vector is faster there (V-Trace 8192 x 200
        // (256) 6.9 us against 8.8, GAE 6000 x 768 (832) 14.0 against 15.5, 2500 x 2000 (2048) 14.6
        // against 15.9, eligibility traces 9.1 against 10.6), while 8192 x 512 (576) 13.2 us and
        // 16000 x 128 (192) 8.4 gain from 13.7 and 9.3 here.
        const int64_t LR = (a.T + K - 1) / K;
        const bool whole = vec && sizeof(DT) == 2 && a.T % K == 0 && period % K == 0 && a.T >= 32 &&
                           a.T <= E_small && (a.T < 128 || kWave * K % a.T != 0);
        if (g_variant == 0 && !whole && a.T >= K && LR <= kRaggedWaves * kWave) {
            const int64_t R = LR <= kSmallWaves * kWave ? kSmallWaves * kWave / LR : 1;
            const int64_t groups = (a.N + R - 1) / R;
            if (groups > INT32_MAX) return RLCS_ERR_INVALID_ARG;
            const uint32_t magic = R > 1 ? uint32_t(((int64_t(1) << flat_shift(4)) + LR - 1) / LR) : 0u;
            const dim3 grid(static_cast<unsigned>(groups)), block(unsigned((R * LR + kWave - 1) / kWave * kWave));
            if (Op::kFlags && has_trunc)
                hipLaunchKernelGGL((ragged_rows_kernel<Op, DT, K, true, true>), grid, block, 0, s, a, int(R), magic, int(LR));
            else
                hipLaunchKernelGGL((ragged_rows_kernel<Op, DT, K, false, true>), grid, block, 0, s, a, int(R), magic, int(LR));
            return hipGetLastError() == hipSuccess ? RLCS_OK : RLCS_ERR_LAUNCH;
        }
        Plan p{};
        p.split = false;
        p.waves = (a.T <= E_small) ? kSmallWaves : kLargeWaves;
        const int64_t E = int64_t(p.waves) * kWave * K;
        const int64_t slack = (period % K == 0) ? 0 : K - 1;
        // as many rows as fit in one chunk: the last one's gap is not part of the range
        p.rows_per_wg = (a.T <= E - slack) ? (E - slack - a.T) / period + 1 : 1;
        if ((a.N + p.rows_per_wg - 1) / p.rows_per_wg > INT32_MAX) return RLCS_ERR_INVALID_ARG;
        p.wave_rows_log2T = -1;
        p.flat_R = 0;
        p.flat_W = kSmallWaves;
        // Vector path, lane by lane (lanes whose steps reach into a gap or past the range go
        // element-wise).
        p.pad = vec;
        auto go = [&](auto tr_tag) -> rlcs_status {
            constexpr bool TR = decltype(tr_tag)::value;
            return vec ? launch<Op, DT, true, TR>(a, p, s) : launch<Op, DT, false, TR>(a, p, s);
        };
        if constexpr (Op::kFlags) {
            if (has_trunc) return go(std::true_type{});
        }
        return go(std::false_type{});
    };
    if (dtype == RLCS_BF16) return run(bf16_t{});
    return run(float{});
}

inline Args make_args(int64_t N, int64_t T, float gamma, float lambda, float rho_bar, float c_bar) {
    Args a{};
    a.N = N;
    a.T = T;
    a.inv_T = T > 0 ? 1.f / float(T) : 0.f;
    a.period = T;
    a.inv_period = a.inv_T;
    a.p = Params{gamma, lambda, rho_bar, c_bar};
    return a;
}


}  // namespace host
}  // namespace rlcs
