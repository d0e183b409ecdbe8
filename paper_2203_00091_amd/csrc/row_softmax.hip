// Stage 2 of the DFSS forward pass: softmax over the kept scores of each row, in place
// (arXiv 2203.00091, Sec. 3.1; max-subtracted form of App. A.1.3).  The row is read
// once into registers, reduced with cross-lane shuffles, and written once -- the
// register-cached variant App. A.1.3 describes.  The dense baseline runs the same kernel
// on full rows.
#include "dfss_device.hpp"
#include "dfss_kernels.hpp"

namespace dfss {

namespace {

constexpr int NT = 256;

// A team of TPR lanes owns a row; lane t holds the 16-byte chunks t, t+TPR, ... (NCH of them).  Bound by the stream, read once and
// written once (24 heads x 4096 x 4096, 806 MB: 5.6 TB/s cold, 6.9 right after stage 1, whose output is partly still in the last-level
// cache); a team has RPT rows, all of their loads in flight before the first is used.
// F32: the row holds fp32 values (the 4-byte mode), else bfloat16.
template <int TPR, int NCH, bool F32, int RPT>
__global__ __launch_bounds__(NT) void k_row_softmax(uint32_t *__restrict__ x, long rows, int cols) {
    constexpr int EPC = F32 ? 4 : 8;    // elements per 16-byte chunk
    constexpr int TEAMS = NT / TPR;
    const int tid = threadIdx.x;
    const long row0 = (long)blockIdx.x * (TEAMS * RPT) + tid / TPR;   // rows row0, row0 + TEAMS, ...
    const int t = tid % TPR;
    const int chunks = cols / EPC;

    u32x4 raw[RPT][NCH];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const u32x4 *p = reinterpret_cast<const u32x4 *>(x) + (row0 + j * TEAMS) * (long)chunks;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = t + i * TPR;
            if (row0 + j * TEAMS < rows && c < chunks) raw[j][i] = p[c];
        }
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const bool live = row0 + j * TEAMS < rows;
        u32x4 *p = reinterpret_cast<u32x4 *>(x) + (row0 + j * TEAMS) * (long)chunks;
        float v[NCH][EPC];
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = t + i * TPR;
            if (live && c < chunks) {
                const u32x4 u = raw[j][i];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (F32) {
                        v[i][e] = __uint_as_float(u[e]);   // (by value: a bit cast applied to the element lvalue itself reads element 0)
                    } else {
                        v[i][2 * e] = bf16_lo_to_f32(u[e]);
                        v[i][2 * e + 1] = bf16_hi_to_f32(u[e]);
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < EPC; ++e) v[i][e] = -INFINITY;
            }
#pragma unroll
            for (int e = 0; e < EPC; ++e) m = fmaxf(m, v[i][e]);
        }
        m = wave_xor_max(m, TPR);
        if (!live) m = 0.f;

        constexpr float kLog2e = 1.4426950408889634f;
        const float mb = m * kLog2e;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NCH; ++i)
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                v[i][e] = __builtin_amdgcn_exp2f(v[i][e] * kLog2e - mb);  // exp(x - max); padding lanes give exp2(-inf) = 0
                s += v[i][e];
            }
        s = wave_xor_sum(s, TPR);
        const float inv = 1.0f / s;

#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = t + i * TPR;
            if (live && c < chunks) {
                u32x4 u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (F32) u[e] = __float_as_uint(v[i][e] * inv);
                    else u[e] = pack_bf16x2(v[i][2 * e] * inv, v[i][2 * e + 1] * inv);
                }
                p[c] = u;
            }
        }
    }
}

template <int TPR, int NCH, bool F32, int RPT = 1>
hipError_t launch(void *x, long rows, int cols, hipStream_t st) {
    const int rpw = NT / TPR * RPT;
    const unsigned grid = (unsigned)((rows + rpw - 1) / rpw);
    hipLaunchKernelGGL((k_row_softmax<TPR, NCH, F32, RPT>), dim3(grid), dim3(NT), 0, st, (uint32_t *)x, rows, cols);
    return hipGetLastError();
}

template <bool F32>
hipError_t dispatch(void *x, long rows, int cols, hipStream_t st) {
    const int chunks = cols / (F32 ? 4 : 8);
    // two rows per team where a row is one load per lane (98304 rows x 256 17.4 -> 16.5 us, 24576 x 512 8.8 -> 8.3; four rows
    // 17.7, and two where a row is two loads 74.2 -> 77.4: fewer waves)
    constexpr int R = F32 ? 1 : 2;
    if (chunks <= 8) return launch<8, 1, F32, R>(x, rows, cols, st);
    if (chunks <= 16) return launch<16, 1, F32, R>(x, rows, cols, st);
    if (chunks <= 32) return launch<32, 1, F32, R>(x, rows, cols, st);
    if (chunks <= 64) return launch<64, 1, F32, R>(x, rows, cols, st);
    if (chunks <= 128) return launch<64, 2, F32>(x, rows, cols, st);
    if (chunks <= 256) return launch<64, 4, F32>(x, rows, cols, st);
    if (chunks <= 512) return launch<64, 8, F32>(x, rows, cols, st);
    if (chunks <= 1024) return launch<64, 16, F32>(x, rows, cols, st);
    if constexpr (F32)
        if (chunks <= 2048) return launch<64, 32, F32>(x, rows, cols, st);
    return hipErrorInvalidValue;  // rows longer than 8192 elements: rejected by the caller
}

}  // namespace

hipError_t launch_row_softmax(void *x, long rows, int cols, hipStream_t st) {
    return dispatch<false>(x, rows, cols, st);
}
hipError_t launch_row_softmax_f32(void *x, long rows, int cols, hipStream_t st) {
    return dispatch<true>(x, rows, cols, st);
}

}  // namespace dfss
