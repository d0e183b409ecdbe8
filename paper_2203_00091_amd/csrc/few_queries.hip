// Whole DFSS forward pass in one kernel for calls with few query tiles (see fused_attention.hip for the method and the
// operand layouts: arXiv 2203.00091, Sec. 3.1 stages, Sec. 3.4 pruning on the accumulators, App. A.1.3 softmax).
//
// One new query against a cache of keys, a short prompt, a single short sequence: K and V are read for at most a few query
// tiles, and the kernels that give a workgroup 64 or 128 queries leave most compute units idle while each of their
// workgroups walks over the keys alone.  Here a workgroup owns 16 queries and its waves share the KEYS: wave w takes every
// NW-th 64-key block, on its own, and the partial results are merged through LDS at the end.  What bounds it is the rate at
// which a compute unit can pull K and V, so all of the design goes into bytes in flight:
//   K     16 bytes per lane straight from global memory in the layout of the matrix operand (nobody shares it: no LDS),
//         one block ahead, in registers
//   V     by asynchronous copies, one block ahead, into LDS that belongs to the wave (the transposing read needs LDS)
// No barrier before the merge: a wave waits for its own copies only.
// Measured: a round of one block per wave (128 KiB per workgroup) takes 2.3 us whether 12 or 96 workgroups run, 57 GB/s per
// compute unit; 1024 heads x 1 query x 4096 keys 177 us (6 TB/s).  96 heads x 1 x 4096, warm: 47.9 us with 64-query
// workgroups, 21.1 us here (from memory 28.4; shared between two workgroups each, below, 19.6 and 24.1).
#include <math.h>

#include <type_traits>

#include "block_list.hpp"
#include "dfss_device.hpp"
#include "dfss_kernels.hpp"

namespace dfss {

namespace {

constexpr int KB = 64;    // keys per block
constexpr float kTau = 8.0f;
constexpr float kLog2e = 1.4426950408889634f;

enum { MODE_2TO4 = 0, MODE_1TO2 = 1 };

// Any Lq; Lk a multiple of 4 (the absent keys of a partial last block are copies of the last key whose scores become -inf;
// absent queries are computed on a copy of the last one and not stored).
// BIAS: key_bias fp32 [BH / H][Lk], as in k_fused; blocks whose keys are all masked are skipped.
// SPLIT (no key bias): `splits` workgroups share the keys of a query tile; each writes its partial result (reference, row sums,
// unnormalised O, fp32) to `part` [item][split][16 x (D + 2)] and k_few_merge forms O.
template <int D, int MODE, int NW, bool PRESCALE, bool BIAS, bool SPLIT>
__global__ __launch_bounds__(64 * NW) void k_few(const __bf16 *__restrict__ Q, const __bf16 *__restrict__ K,
                                                 const __bf16 *__restrict__ V, const float *__restrict__ key_bias, int H,
                                                 int Lq, int Lk, float scale, uint16_t *__restrict__ O,
                                                 int splits, float *__restrict__ part) {
    constexpr int CPR = D / 8;          // 16-byte chunks per row
    constexpr int TILE = KB * CPR;      // chunks per V block
    constexpr int LPT = TILE / 64;      // asynchronous copies per lane and V block
    constexpr int STEPS = D / 32;       // MFMA k-steps of Q K^T
    constexpr int DS = D / 16;          // 16-column tiles of O
    constexpr int NF = 4 * DS + 5;      // floats per lane of a partial result
    __shared__ u32x4 Vs[NW * 2 * TILE];
    static_assert(NW * NF * 64 * 4 <= NW * 2 * TILE * 16, "the partial results fit into the V buffers");

    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l = threadIdx.x & 63, li = l & 15, kb = l >> 4;
    const unsigned qtiles = (Lq + 15) / 16;
    const unsigned share = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned item = SPLIT ? share / (unsigned)splits : share;
    const int sp = SPLIT ? share % (unsigned)splits : 0;
    const int q0 = (item % qtiles) * 16, bh = item / qtiles;
    static_assert(!SPLIT || !BIAS, "shared keys: no key bias");
    const int first = __builtin_amdgcn_readfirstlane(sp * NW + w), stride = SPLIT ? NW * splits : NW;   // this wave's blocks
    const int nblocks = (Lk + KB - 1) / KB;

    // V block: row = key, chunk c at row * CPR + (c ^ tr_row_swizzle(row))
    int v_row[LPT], v_chunk[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * 64 + l;
        v_row[i] = p / CPR;
        v_chunk[i] = ((p % CPR) ^ tr_row_swizzle<CPR>(v_row[i])) * 8;
    }
    const uint32_t lds_v = lds_address(&Vs[w * 2 * TILE]);
    const uint64_t v_base = uniform_address(V + (size_t)bh * Lk * D);
    const __bf16 *const Kh = K + (size_t)bh * Lk * D;
    const float *const brow = BIAS ? key_bias + (size_t)(bh / H) * Lk : nullptr;

    // What a wave holds of a block in registers.  MFMA row i of tile t is key 16 (i / 4) + 4 t + i % 4 (as in k_fused), so
    // that lane (query li, kb) ends up with the scores of keys 16 kb .. +15.
    struct Block {
        u32x4 k[STEPS][4];
        f32x4 bias[BIAS ? 4 : 1];
    };
    auto load_block = [&](int jb, auto parity, Block &b) {
        const int last = Lk - 1 - jb * KB;   // the block's last real key (KB - 1 or more: all are)
        const uint64_t vs = v_base + (uint64_t)jb * (KB * D * 2);
#pragma unroll
        for (int i = 0; i < LPT; ++i)
            async_copy16(vs, 2u * ((v_row[i] < last ? v_row[i] : last) * D + v_chunk[i]), lds_v + 16u * (decltype(parity)::value * TILE + i * 64));
        const __bf16 *const ks = Kh + (size_t)jb * (KB * D);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int key = 16 * (li >> 2) + 4 * t + (li & 3);
            const __bf16 *const row = ks + (key < last ? key : last) * D + 8 * kb;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) b.k[s][t] = *reinterpret_cast<const u32x4 *>(row + 32 * s);
            if constexpr (BIAS) {   // (Lk is a multiple of 4: four keys exist together)
                const int k4 = 16 * kb + 4 * t;
                b.bias[t] = *reinterpret_cast<const f32x4 *>(brow + jb * KB + (k4 < last ? k4 : last - 3));
            }
        }
    };

    BlockList<BIAS, true> blocks;
    if constexpr (BIAS) {
        blocks.init(true, brow, false, nullptr, 0, 0, 16, 0, Lq, Lk, nblocks, l);
        for (int i = 0; i < first; ++i) blocks.take();
    }
    int next_plain = first;
    auto take = [&]() -> int {
        if constexpr (BIAS) {
            const int j = blocks.take();
            for (int i = 1; i < stride; ++i) blocks.take();
            return __builtin_amdgcn_readfirstlane(j);
        } else {
            const int j = next_plain;
            next_plain += stride;
            return j;
        }
    };

    Block b0, b1;
    int jb = take(), jn = take();
    if (jb < nblocks) load_block(jb, std::integral_constant<int, 0>{}, b0);

    // Q operand: lane (column li, chunk kb) of step s holds Q[q][32 s + 8 kb .. +7]
    bf16x8 bq[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const int qrow = q0 + li < Lq ? q0 + li : Lq - 1;
        const u32x4 raw = *reinterpret_cast<const u32x4 *>(Q + ((size_t)bh * Lq + qrow) * D + 32 * s + 8 * kb);
        if constexpr (PRESCALE) {
            u32x4 sc;
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[e] = pack_bf16x2(bf16_lo_to_f32(raw[e]) * scale, bf16_hi_to_f32(raw[e]) * scale);
            bq[s] = __builtin_bit_cast(bf16x8, sc);
        } else {
            bq[s] = __builtin_bit_cast(bf16x8, raw);
        }
    }

    float m_ref = -1.0e30f;   // reference of the query in column li (the same in its four lanes)
    f32x4 acc_o[DS], acc_l = {0.f, 0.f, 0.f, 0.f};   // O and row sums, rows 4 kb + r
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) acc_o[ds] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t one2 = 0x3F803F80u;  // two bfloat16 ones
    const bf16x8 ones8 = __builtin_bit_cast(bf16x8, u32x4{one2, one2, one2, one2});
    const int tr_row = li >> 2, tr_sub = (li >> 1) & 1, tr_byte = 8 * (li & 1);

    auto block = [&](auto parity, const Block &b, Block &after) {
        constexpr int buf = decltype(parity)::value;
        // This block is in, and the LDS reads of the block before it (whose buffer the next copies overwrite) are done.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        asm volatile("" ::: "memory");
        if (jn < nblocks) load_block(jn, std::integral_constant<int, buf ^ 1>{}, after);

        // acc[t][r] = s(query li, key 64 jb + 16 kb + 4 t + r)
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (BIAS && PRESCALE) acc[t] = b.bias[t];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) acc[t] = mfma16(__builtin_bit_cast(bf16x8, b.k[s][t]), bq[s], acc[t]);
            if constexpr (!PRESCALE) {
                acc[t] = acc[t] * scale;
                if constexpr (BIAS) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[t][r] = add_unfused(acc[t][r], b.bias[t][r]);
                }
            }
        }
        if (jb * KB + KB > Lk) {   // the block that the keys end in
            const int left = Lk - jb * KB - 16 * kb;   // real keys from this lane's first one on (a multiple of 4)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * t >= left) acc[t] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        }

        float kept[8];
        uint32_t idx = 0;
        float m_blk = -3.0e38f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float lo, hi;
            uint32_t code;
            if constexpr (MODE == MODE_2TO4) select_2of4(acc[t][0], acc[t][1], acc[t][2], acc[t][3], 4 * t, lo, hi, code);
            else select_1of2(acc[t][0], acc[t][1], acc[t][2], acc[t][3], 4 * t, lo, hi, code);
            kept[2 * t] = lo;
            kept[2 * t + 1] = hi;
            idx |= code;
            m_blk = fmaxf(fmaxf(m_blk, lo), hi);
        }
        if (__any(m_blk > m_ref + kTau)) {   // raise the reference where the block outgrew it (rare after the first one)
            m_blk = fmaxf(m_blk, __shfl_xor(m_blk, 16, 64));
            m_blk = fmaxf(m_blk, __shfl_xor(m_blk, 32, 64));
            const float m_new = m_blk > m_ref + kTau ? m_blk : m_ref;
            const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * kLog2e);
            m_ref = m_new;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float a_r = __shfl(alpha, 4 * kb + r, 64);
                acc_l[r] *= a_r;
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) acc_o[ds][r] *= a_r;
            }
        }
        const float mb = m_ref * kLog2e;
        u32x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            pk[e] = pack_bf16x2(__builtin_amdgcn_exp2f(__builtin_fmaf(kept[2 * e], kLog2e, -mb)),
                                __builtin_amdgcn_exp2f(__builtin_fmaf(kept[2 * e + 1], kLog2e, -mb)));
        const bf16x8 a = __builtin_bit_cast(bf16x8, pk);
        const char *vbase = reinterpret_cast<const char *>(&Vs[(2 * w + buf) * TILE]);
        auto tr = [&](int key0, int ds) {
            const int row = key0 + tr_row;
            const int chunk = (2 * ds + tr_sub) ^ tr_row_swizzle<CPR>(row);
            return lds_read_tr16(vbase + (row * CPR + chunk) * 16 + tr_byte);
        };
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            const s16x4 t0 = tr(8 * kb, ds), t1 = tr(8 * kb + 4, ds), t2 = tr(32 + 8 * kb, ds), t3 = tr(36 + 8 * kb, ds);
            const s16x8 lo = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
            const s16x8 hi = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
            const bf16x16 bv = __builtin_bit_cast(
                bf16x16, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15));
            acc_o[ds] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a, bv, acc_o[ds], (int)idx, 0, 0);
        }
        acc_l = mfma16(a, ones8, acc_l);   // (against ones the positions do not matter: dense instruction)
        jb = jn;
        jn = take();
    };
    while (jb < nblocks) {
        block(std::integral_constant<int, 0>{}, b0, b1);
        if (jb >= nblocks) break;
        block(std::integral_constant<int, 1>{}, b1, b0);
    }

    // Merge: value f of lane l of wave g at float f * 64 + l of the wave's slot; wave w forms the 16-column tiles w,
    // w + NW, ... of O.  (No copy is in flight: a wave waits for its last block.)
    __syncthreads();   // every wave is done with its V buffers
    float *const slots = reinterpret_cast<float *>(Vs);
    {
        float *const mine = slots + w * (NF * 64) + l;
        mine[0] = m_ref;
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(1 + r) * 64] = acc_l[r];
#pragma unroll
        for (int ds = 0; ds < DS; ++ds)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(5 + 4 * ds + r) * 64] = acc_o[ds][r];
    }
    __syncthreads();
#pragma unroll
    for (int d0 = 0; d0 < DS; d0 += NW) {
        const int ds = d0 + w;
        if (ds >= DS) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * kb + r;
            if (q0 + row >= Lq) continue;
            float m = -1.0e30f;
#pragma unroll
            for (int g = 0; g < NW; ++g) m = fmaxf(m, slots[g * (NF * 64) + row]);
            float sum = 0.f, o = 0.f;
#pragma unroll
            for (int g = 0; g < NW; ++g) {
                const float f = __builtin_amdgcn_exp2f((slots[g * (NF * 64) + row] - m) * kLog2e);
                sum += f * slots[g * (NF * 64) + (1 + r) * 64 + l];
                o += f * slots[g * (NF * 64) + (5 + 4 * ds + r) * 64 + l];
            }
            if constexpr (SPLIT) {
                float *const P = part + ((size_t)item * splits + sp) * (16 * (D + 2));
                if (ds == 0 && li == 0) P[row] = m, P[16 + row] = sum;
                P[32 + row * D + 16 * ds + li] = o;
                continue;
            }
            O[((size_t)bh * Lq + q0 + row) * D + 16 * ds + li] = (uint16_t)(pack_bf16x2(o * __builtin_amdgcn_rcpf(sum), 0.f) & 0xFFFFu);
        }
    }
}

// O of the query tiles whose keys `splits` workgroups shared, in a fixed order.  One workgroup per tile; a thread forms 8
// columns of a row.
template <int D>
__global__ __launch_bounds__(2 * D) void k_few_merge(const float *__restrict__ part, int splits, int Lq, uint16_t *__restrict__ O) {
    const unsigned qtiles = (Lq + 15) / 16;
    const int q0 = (blockIdx.x % qtiles) * 16, bh = blockIdx.x / qtiles;
    const int row = threadIdx.x / (D / 8), c = (threadIdx.x % (D / 8)) * 8;
    if (q0 + row >= Lq) return;
    const float *const P = part + (size_t)blockIdx.x * splits * (16 * (D + 2));
    float m = -1.0e30f;
    for (int sp = 0; sp < splits; ++sp) m = fmaxf(m, P[sp * (16 * (D + 2)) + row]);
    float sum = 0.f;
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
    for (int sp = 0; sp < splits; ++sp) {
        const float *const S = P + sp * (16 * (D + 2));
        const float f = __builtin_amdgcn_exp2f((S[row] - m) * kLog2e);
        const f32x4 *const src = reinterpret_cast<const f32x4 *>(S + 32 + row * D + c);
        sum += f * S[16 + row];
        a0 += src[0] * f;
        a1 += src[1] * f;
    }
    const float inv = __builtin_amdgcn_rcpf(sum);
    a0 *= inv, a1 *= inv;
    *reinterpret_cast<u32x4 *>(O + ((size_t)bh * Lq + q0 + row) * D + c) = u32x4{
        pack_bf16x2(a0[0], a0[1]), pack_bf16x2(a0[2], a0[3]), pack_bf16x2(a1[0], a1[1]), pack_bf16x2(a1[2], a1[3])};
}

constexpr int waves_of(int d) { return d == 64 ? 8 : 4; }

template <int D, int MODE, int NW, bool SPLIT>
hipError_t launch_few(const void *Q, const void *K, const void *V, const float *key_bias, int H, int BH, int Lq, int Lk,
                      float scale, void *O, int splits, float *part, hipStream_t st) {
    const unsigned tiles = (unsigned)((long)BH * ((Lq + 15) / 16));
#define DFSS_LAUNCH(PRE, BB)                                                                                             \
    hipLaunchKernelGGL((k_few<D, MODE, NW, PRE, BB, SPLIT>), dim3(tiles * splits), dim3(64 * NW), 0, st,                 \
                       (const __bf16 *)Q, (const __bf16 *)K, (const __bf16 *)V, key_bias, H, Lq, Lk, scale, (uint16_t *)O, \
                       splits, part)
    const bool pre = is_pow2(scale);
    if constexpr (SPLIT) {   // (no key bias: see few_queries_splits)
        if (pre) DFSS_LAUNCH(true, false); else DFSS_LAUNCH(false, false);
    } else if (pre) {
        if (key_bias) DFSS_LAUNCH(true, true); else DFSS_LAUNCH(true, false);
    } else {
        if (key_bias) DFSS_LAUNCH(false, true); else DFSS_LAUNCH(false, false);
    }
#undef DFSS_LAUNCH
    if (SPLIT) hipLaunchKernelGGL(k_few_merge<D>, dim3(tiles), dim3(2 * D), 0, st, part, splits, Lq, (uint16_t *)O);
    return hipGetLastError();
}

template <bool SPLIT>
hipError_t launch_any(const void *Q, const void *K, const void *V, const float *key_bias, int H, int BH, int Lq, int Lk, int d,
                      int mode, float scale, void *O, int splits, float *part, hipStream_t st) {
    // Tiles that do not fit the chip at once: two waves per workgroup, so that several workgroups share a compute unit and one
    // starts while another merges (1 query, 2 against 8 waves, d = 64: 768 heads x 592 keys 19.0 and 27.0 us -- the 64-query
    // kernel 24.7 --, 384 x 260 6.3 and 8.3, 1024 x 4096 177 and 179).
    const bool many = !SPLIT && (long)BH * ((Lq + 15) / 16) > 256;
#define DFSS_FEW(DD, MM)                                                                                                     \
    (many ? launch_few<DD, MM, 2, false>(Q, K, V, key_bias, H, BH, Lq, Lk, scale, O, 1, nullptr, st)                          \
          : launch_few<DD, MM, waves_of(DD), SPLIT>(Q, K, V, key_bias, H, BH, Lq, Lk, scale, O, splits, part, st))
    if (d == 64) return mode == 0 ? DFSS_FEW(64, MODE_2TO4) : DFSS_FEW(64, MODE_1TO2);
    return mode == 0 ? DFSS_FEW(128, MODE_2TO4) : DFSS_FEW(128, MODE_1TO2);
#undef DFSS_FEW
}

}  // namespace

// mode 0 or 1; any Lq, Lk a multiple of 4; key_bias may be null.
hipError_t launch_fused_attention_few(const void *Q, const void *K, const void *V, const float *key_bias, int H, int BH,
                                      int Lq, int Lk, int d, int mode, float scale, void *O, hipStream_t st) {
    return launch_any<false>(Q, K, V, key_bias, H, BH, Lq, Lk, d, mode, scale, O, 1, nullptr, st);
}

// Workgroups per query tile where a workspace lets several share its keys.  1 query, d = 64, us, alone and shared, the merge
// kernel included, K and V warm: 12 heads x 4096 keys 20.5 and 11.6, 12 x 3072 16.3 and 11.2, 64 x 3072 16.5 and 14.0, 96 x
// 4096 21.2 and 19.6; d = 128: 12 x 1536 16.8 and 11.5, 96 x 4096 41.1 and 34.4.  The line at 104 tiles (which share in
// twos): with the fewest keys that share, warm, it breaks even at 98 .. 104 (d = 64, 3072 keys: 98 heads 16.8 and 16.7, 104
// 16.9 and 17.3, 112 17.0 and 18.1; d = 128, 1536 keys: 104 18.3 and 18.0, 112 18.5 and 18.7), with 8192 at 112 and beyond.
// Cold, as in a model of many layers, it pays up to 128 tiles (4096 keys: 96 heads 28.4 and 24.1, 104 28.7 and 25.7, 128
// 29.6 and 29.2).  Not with a key bias: each workgroup would scan the whole bias row first (half of 4096 keys masked, 12
// heads: 16.5 and 18.1).
int few_queries_splits(int BH, int Lq, int Lk, int d) {
    const long tiles = (long)BH * ((Lq + 15) / 16);
    const int nblocks = (Lk + KB - 1) / KB, nw = waves_of(d);
    long n = 256 / tiles;                        // all workgroups on the chip at once, one per compute unit
    if (n > nblocks / (2 * nw)) n = nblocks / (2 * nw);   // at least two blocks per wave
    return tiles > 104 || nblocks < 6 * nw || n < 2 ? 1 : (int)n;
}

size_t few_queries_workspace_bytes(int BH, int Lq, int Lk, int d) {
    const int n = few_queries_splits(BH, Lq, Lk, d);
    return n == 1 ? 0 : (size_t)BH * ((Lq + 15) / 16) * n * 16 * (d + 2) * sizeof(float);
}

// The same with a workspace of few_queries_workspace_bytes (not 0).
hipError_t launch_fused_attention_few_split(const void *Q, const void *K, const void *V, int BH, int Lq, int Lk, int d, int mode,
                                            float scale, void *O, void *part, hipStream_t st) {
    return launch_any<true>(Q, K, V, nullptr, 1, BH, Lq, Lk, d, mode, scale, O, few_queries_splits(BH, Lq, Lk, d),
                            (float *)part, st);
}

}  // namespace dfss
