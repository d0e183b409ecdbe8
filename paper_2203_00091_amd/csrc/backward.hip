// Backward pass of DFSS attention through the fixed selection of the forward pass.
//
// The paper finetunes with DFSS attention (arXiv 2203.00091, Sec. 5.1) but describes no backward
// kernel; the selection is treated as a constant of the step, so with P the softmax weights of the
// kept entries (Sec. 3.1) and dO the upstream gradient:
//     dV = P^T dO,   dP = (dO V^T) at the kept positions,   delta_i = dO_i . O_i,
//     dS = P .* (dP - delta),   dQ = scale dS K,   dK = scale dS^T Q.
//
//   k_backward_dq      dQ, and -delta for the other one; walks the keys, layout of the one-kernel forward pass
//   k_backward_dkv     dV and dK in one pass over the queries
//   k_backward_merge   gradients from the sums of workgroups that shared keys or queries
//   k_spmm_t           out = A^T X for a compressed A (the public transposed product).  The contraction
//                      runs over queries, across which the N:M structure does not run, so the tile
//                      of A is expanded to dense bfloat16 in LDS and both operands are read with the
//                      transposing LDS read.
#include <type_traits>

#include "dfss_device.hpp"
#include "dfss_kernels.hpp"

namespace dfss {

namespace {

constexpr int NT = 256;   // 4 waves
constexpr int KB = 128;   // keys per block

// ------------------------------------------------------------------------------------------------
// out[bh][key][c] = sum_q A[bh][q][key] X[bh][q][c]
// A: kept values bf16 [BH, Lq, Lk/2] + metadata in the library's order; X: bf16 [BH, Lq, D].
// One workgroup owns 128 keys of one head (wave w: keys 32 w .. 32 w + 31, all D columns) and walks
// over the queries 64 at a time.
// ------------------------------------------------------------------------------------------------
// UNP: X holds LqR <= Lq rows per head and out LkR <= Lk rows, while A and meta have the layout of the padded lengths
// Lq (a multiple of 64) and Lk (of 128).  The rows LqR .. Lq - 1 of A hold meaningless entries: they are expanded to
// zeros; the places of the absent rows of a partial last X tile take its last real row; keys past LkR are not stored.
template <int D, bool UNP>
__global__ __launch_bounds__(NT, 2) void k_spmm_t(const uint32_t *__restrict__ A, const uint32_t *__restrict__ meta,
                                                  const __bf16 *__restrict__ X, int Lq, int Lk, int LqR, int LkR,
                                                  uint16_t *__restrict__ out) {
    constexpr int QB = 64;              // queries per step
    constexpr int CPR = D / 8;          // 16-byte chunks per X row
    constexpr int XT = QB * CPR;        // chunks per X tile
    constexpr int LPT = XT / NT;        // asynchronous copies per thread per tile
    constexpr int DS = D / 16;          // 16-column output tiles
    constexpr int AROW = 2 * KB + 16;   // bytes per row of the expanded A tile (padded; three workgroups fit a CU at D = 64)
    __shared__ u32x4 Xs[2][XT];
    __shared__ __attribute__((aligned(16))) char Ad[2][QB * AROW];

    const int tid = threadIdx.x;
    const int w = tid >> 6, l = tid & 63, li = l & 15, g = l >> 4;

    const unsigned kblocks = Lk / KB;
    const unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int jblk = item % kblocks;
    const int bh = item / kblocks;
    const int nq = Lq / QB;

    // X tile in LDS: row = query, chunk c at row * CPR + (c ^ tr_row_swizzle(row))
    const __bf16 *Xh = X + (size_t)bh * LqR * D;
    int src_off[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * NT + tid;
        const int row = p / CPR, c = (p % CPR) ^ tr_row_swizzle<CPR>(row);
        src_off[i] = row * D + c * 8;
    }
    const uint32_t lds_x = lds_address(&Xs[0][w * 64]);
    auto issue_x = [&](int qb, int buf) {
        const __bf16 *src = Xh + (size_t)qb * QB * D;
        const int real = LqR - qb * QB;   // real rows from this tile's first one on
        if (UNP && real < QB) {
#pragma unroll
            for (int i = 0; i < LPT; ++i) {
                const int p = i * NT + tid;
                const int row = p / CPR, c = (p % CPR) ^ tr_row_swizzle<CPR>(row);
                async_copy16(src, 2u * ((row < real ? row : real - 1) * D + c * 8), lds_x + 16u * (buf * XT + i * NT));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LPT; ++i) async_copy16(src, 2u * src_off[i], lds_x + 16u * (buf * XT + i * NT));
    };

    // A tile: thread (query aq, chunk ac) expands the 32 keys 128 jblk + 32 ac .. +31 of its query
    const int aq = tid >> 2, ac = tid & 3;
    const int meta_slot = ((ac & 1) << 1) | (ac >> 1);
    struct ARaw {
        u32x4 v0, v1;      // 16 kept values
        uint32_t word;     // their 8 position codes
    };
    auto load_a = [&](int qb) {
        ARaw r;
        const int q = qb * QB + aq;
        const u32x4 *pr = reinterpret_cast<const u32x4 *>(A + ((size_t)bh * Lq + q) * (size_t)(Lk / 4)) + jblk * 8 + ac * 2;
        r.v0 = pr[0];
        r.v1 = pr[1];
        r.word = meta[((((size_t)bh * (Lq / 16) + (q >> 4)) * kblocks + jblk) * 16 + (q & 15)) * 4 + meta_slot];
        return r;
    };
    auto expand_a = [&](const ARaw &r, int buf, int qb) {
        u32x4 *dst = reinterpret_cast<u32x4 *>(&Ad[buf][aq * AROW + ac * 64]);
        if (UNP && qb * QB + aq >= LqR) {   // a row past the end: it takes no part in the sums
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i] = u32x4{0u, 0u, 0u, 0u};
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {       // 8 keys = 2 groups per 16 bytes
            u32x4 o;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int grp = 2 * i + h;
                const uint32_t kept = grp < 4 ? r.v0[grp] : r.v1[grp - 4];
                const uint32_t lo = kept & 0xFFFFu, hi = kept >> 16;
                const uint32_t code = (r.word >> (4 * grp)) & 0xFu;
                const uint32_t plo = code & 3u, phi = code >> 2;
                const uint32_t k0 = plo == 0 ? lo : 0u;
                const uint32_t k1 = plo == 1 ? lo : (phi == 1 ? hi : 0u);
                const uint32_t k2 = plo == 2 ? lo : (phi == 2 ? hi : 0u);
                const uint32_t k3 = phi == 3 ? hi : 0u;
                o[2 * h] = k0 | (k1 << 16);
                o[2 * h + 1] = k2 | (k3 << 16);
            }
            dst[i] = o;
        }
    };

    f32x4 acc[2][DS];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < DS; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // transposing reads: lane li of a 16-lane group addresses element [row0 + li/4][col0 + 4 (li%4)]
    const int tr_row = li >> 2;
    const int tr_sub = (li >> 1) & 1, tr_byte = 8 * (li & 1);

    // One step = 64 queries.  The compressed operand is loaded two steps ahead into registers (r0 for
    // even steps, r1 for odd ones: fixed names, so no register is copied while its load is in flight),
    // the X tile one step ahead into the other LDS buffer.
    auto step = [&](int qb, ARaw &r) {
        const int buf = qb & 1;
        expand_a(r, buf, qb);
        // X(qb) must have landed; the three loads of A(qb + 1), issued after its copy, may stay in flight
        if (qb >= 1 && qb + 1 < nq) wait_async_copies_keep<3>();
        else wait_async_copies();
        __syncthreads();       // both tiles are complete; the other buffers are free
        if (qb + 1 < nq) issue_x(qb + 1, buf ^ 1);
        if (qb + 2 < nq) r = load_a(qb + 2);
        const char *abase = &Ad[buf][0];
        const char *xbase = reinterpret_cast<const char *>(&Xs[buf][0]);
        auto tr_a = [&](int q0, int col0) {
            return lds_read_tr16(abase + (q0 + tr_row) * AROW + (col0 + 4 * (li & 3)) * 2);
        };
        auto tr_x = [&](int q0, int nt) {
            const int row = q0 + tr_row;
            const int chunk = (2 * nt + tr_sub) ^ tr_row_swizzle<CPR>(row);
            return lds_read_tr16(xbase + (row * CPR + chunk) * 16 + tr_byte);
        };
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {     // 32 queries per MFMA step; lane group g takes queries 8 g .. 8 g + 7
            const int q0 = 32 * ks + 8 * g;
            bf16x8 a[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const s16x4 t0 = tr_a(q0, 32 * w + 16 * mt), t1 = tr_a(q0 + 4, 32 * w + 16 * mt);
                a[mt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
            for (int nt = 0; nt < DS; ++nt) {
                const s16x4 t0 = tr_x(q0, nt), t1 = tr_x(q0 + 4, nt);
                const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) acc[mt][nt] = mfma16(a[mt], b, acc[mt][nt]);
            }
        }
    };

    issue_x(0, 0);
    ARaw r0 = load_a(0), r1 = r0;
    if (nq > 1) r1 = load_a(1);
    for (int qb = 0; qb < nq; qb += 2) {
        step(qb, r0);
        if (qb + 1 < nq) step(qb + 1, r1);
    }

    // acc[mt][nt][r] = out[key 128 jblk + 32 w + 16 mt + 4 g + r][16 nt + li]
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int krow = jblk * KB + 32 * w + 16 * mt + 4 * g + r;
            if (UNP && krow >= LkR) continue;
            const size_t key = (size_t)bh * LkR + krow;
#pragma unroll
            for (int nt = 0; nt < DS; ++nt)
                out[key * D + 16 * nt + li] = (uint16_t)(pack_bf16x2(acc[mt][nt][r], 0.f) & 0xFFFFu);
        }
}

// ------------------------------------------------------------------------------------------------
// The gradients.  dS is formed twice, once per direction of the sums it enters, and never written: the kept weights and
// the metadata are read twice (2 x 1.125 B per score) instead of P twice, dS' written and read once, the metadata three
// times (4.4 B), and the product that dS' costs a second time runs on the matrix unit.  The whole call, warm, before (dS'
// written, one transposed product each for dV and dK) and with that, 4096 x 4096 with 24 heads: 518 -> 298 us; 512 x 512 with
// 192 heads: 71 -> 51 us; d = 128, 2048 x 2048 with 64 heads: 500 -> 354 us.  (Now 283, 49 and 353: see where the weights come from.)
// ------------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Bit `pos` of w in every bit, and x where the bits of such a mask are set, else y: one instruction each.  (The empty
// statement hides where the mask comes from: the pair otherwise becomes a mask, a comparison and a select.  The values
// themselves stay out of assembly: the compiler has to see who reads the result of a matrix instruction.)
__device__ __forceinline__ uint32_t spread_bit(uint32_t w, int pos) {
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)w, pos, 1);
    asm("" : "+v"(m));
    return m;
}
__device__ __forceinline__ float choose(uint32_t m, float x, float y) {
    return __uint_as_float((m & __float_as_uint(x)) | (~m & __float_as_uint(y)));
}

// dQ = scale * dS K with dS = P .* (dO V^T - delta) at the kept positions, delta_q = dO_q . O_q; and -delta, fp32
// [BH][Lq], for the kernel below.
// The layout is that of the one-kernel forward pass (fused_attention32.hip) with dO in the place of Q, V in the place of
// K and K in the place of V: a wave owns 32 queries, keys sit on the rows of the first product, so that a lane ends up
// with dP of 16 consecutive keys of one query and finds its 8 kept weights in 16 consecutive bytes of P, their position
// codes in 16 bits of the metadata; the 8 dS values ARE the compressed operand of the sparse instruction, the codes its
// index.  The first product starts from -delta (delta belongs to the lane's query), so dP - delta needs no instruction.
// UNP: dO, O, dQ hold LqR <= Lq rows per head and V, K LkR <= Lk keys, while P and meta have the layout of the padded
// lengths Lq (a multiple of 64) and Lk (of 128).  Rows past LqR are computed on a copy of the last one and not stored; the
// places of absent keys in a partial last block take the block's last key (their weights are 0).  Blocks that hold no real
// key are not visited.
// SPLIT: `splits` workgroups share the keys of a query tile, each a run of pairs of blocks; their sums, unscaled fp32, go to
// `part` [split][head and query][D], and k_backward_merge forms dQ.
// (Second number of the bounds: waves per SIMD.  At d = 128 it is what registers (four waves) and LDS (two) allow.  At d = 64
// that would be three; the two-wave form asks for six, which the compiler reports as out of reach, because the order of
// instructions that it arrives at on the way is the faster one: 1 - 2 % on small grids, 4 - 6 % on unpadded lengths against
// three (12 heads x 100 x 1000 20.9 and 22.0 us; 24 x 1024 x 1024 level).)
// PACED: the workgroups of a compute unit keep level (Pace).
template <int D, int NW, bool UNP, bool SPLIT, bool PACED>
__global__ __launch_bounds__(64 * NW, D == 128 ? NW / 2 : NW == 4 ? 3 : 6) void k_backward_dq(
    const __bf16 *__restrict__ dO, const __bf16 *__restrict__ V, const __bf16 *__restrict__ O,
    const uint32_t *__restrict__ P, const uint32_t *__restrict__ meta, const __bf16 *__restrict__ K, int Lq, int Lk,
    int LqR, int LkR, float scale, uint16_t *__restrict__ dQ, float *__restrict__ neg_delta, int splits,
    float *__restrict__ part) {
    constexpr int THREADS = 64 * NW;
    constexpr int KEYS = 64;                 // keys per block: two 32-key tiles
    constexpr int CPR = D / 8;               // 16-byte chunks per row
    constexpr int TILE = KEYS * CPR;         // chunks per V (or K) block
    constexpr int LPT = TILE / THREADS;      // asynchronous copies per thread, block and operand
    constexpr int STEPS = D / 16;
    constexpr int DT = D / 32;
    constexpr bool EARLY = D == 128 && (NW == 4 || SPLIT);   // operands are read ahead
    constexpr int TQ = 32 * NW;
    __shared__ u32x4 Vs[2][TILE], Kr[2][TILE], Ps[NW][32 * 8];

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, lj = l & 31, h = l >> 5;
    const unsigned qtiles = (Lq + TQ - 1) / TQ;
    const unsigned share = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned item = SPLIT ? share / (unsigned)splits : share;
    const int sp = SPLIT ? share % (unsigned)splits : 0;
    const int qt = item % qtiles, bh = item / qtiles;
    const int q0 = qt * TQ + w * 32;
    const int nblocks = (LkR + KEYS - 1) / KEYS;

    // V block: row slot 32 t + 8 g + 4 h' + x holds key 32 t + 16 h' + 4 g + x, chunk c at slot * CPR + (c ^ operand_row_swizzle)
    // K block: row = key, chunk c at row * CPR + (c ^ tr32_swizzle(row))
    int v_key[LPT], v_chunk[LPT], k_key[LPT], k_chunk[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * THREADS + tid, slot = p / CPR;
        v_key[i] = (slot & 32) | (((slot >> 2) & 1) << 4) | (((slot >> 3) & 3) << 2) | (slot & 3);
        v_chunk[i] = ((p % CPR) ^ operand_row_swizzle<CPR, 32>(slot)) * 8;
        k_key[i] = slot;
        k_chunk[i] = ((p % CPR) ^ tr32_swizzle<CPR>(slot)) * 8;
    }
    const uint32_t lds_v = lds_address(&Vs[0][w * 64]), lds_k = lds_address(&Kr[0][w * 64]);
    const uint64_t v_base = uniform_address(V + (size_t)bh * LkR * D), k_base = uniform_address(K + (size_t)bh * LkR * D);
    auto issue_block = [&](int jb, int buf) {
        const uint64_t vs = v_base + (uint64_t)jb * (KEYS * D * 2), ks = k_base + (uint64_t)jb * (KEYS * D * 2);
        const int last = UNP ? LkR - jb * KEYS - 1 : KEYS - 1;   // the block's last real key
#pragma unroll
        for (int i = 0; i < LPT; ++i)
            async_copy16(vs, 2u * ((UNP && v_key[i] > last ? last : v_key[i]) * D + v_chunk[i]), lds_v + 16u * (buf * TILE + i * THREADS));
#pragma unroll
        for (int i = 0; i < LPT; ++i)
            async_copy16(ks, 2u * ((UNP && k_key[i] > last ? last : k_key[i]) * D + k_chunk[i]), lds_k + 16u * (buf * TILE + i * THREADS));
    };
    // Blocks go in pairs (the last pair may be a single block).  The workgroups start at different pairs and wrap around (rows
    // of P are a power of two apart for the usual lengths; workgroups in step would read the same few memory channels),
    // four neighbours at the same one: they share K and V blocks in the L2 (512 x 512, 192 heads 28.1 -> 26.5 us against
    // one by one; 4096 x 4096, 24 heads 140 -> 137 us; d = 128, 64 heads x 2048 152.6 -> 150 us).
    const int npairs = (nblocks + 1) / 2;
    const int rot = __builtin_amdgcn_readfirstlane(SPLIT ? npairs * sp / splits : (int)((item / 4) % (unsigned)npairs));
    const int visits = SPLIT ? __builtin_amdgcn_readfirstlane(npairs * (sp + 1) / splits) - rot : npairs;   // (splits <= npairs)
    issue_block(2 * rot, 0);

    // Weights and codes of the wave's queries for a pair of blocks (128 keys: a whole line of P per row), asked for one pair
    // ahead.  The weights go through LDS, whole lines at a time: loaded by the lane that needs them, one row per lane, an instruction
    // takes 64 address cycles instead of 16, and the address unit was busy 70 % of the time (4096 x 4096, 24 heads: whole
    // backward pass 296 -> 284 us; d = 128, 64 heads x 2048 362 -> 351; 512 x 512, 192 heads 53.1 -> 50.7; small grids level).
    // Row r, chunk c (keys 16 c .. +15) at r * 8 + (c ^ operand_row_swizzle(r)); copy i brings rows 8 i .. +7, for which the
    // pattern is that of copy i % 2.  (Waves past the last query read the last 32 rows.)
    const int pq0 = q0 < Lq ? q0 : Lq - 32;
    const uint64_t p_base = uniform_address(P + ((size_t)bh * Lq + pq0) * (size_t)(Lk / 4));
    const uint32_t p_off = (uint32_t)(l >> 3) * (uint32_t)Lk + 16u * ((l & 7) ^ operand_row_swizzle<8, 32>(l >> 3));
    const uint32_t lds_p = lds_address(&Ps[w][0]);
    const u32x4 *const m_row = reinterpret_cast<const u32x4 *>(meta) + ((size_t)bh * (Lq / 16) + ((pq0 + lj) >> 4)) * (Lk / KB) * 16 + (lj & 15);
    constexpr int KEPT_LOADS = 5;
    auto load_kept = [&](int pair) {   // returns the codes: slot 2 t + i the word of 32 keys 64 i + 32 t .. +31 of the pair
#pragma unroll
        for (int i = 0; i < 4; ++i)
            async_copy16(p_base + (uint64_t)pair * 128u + (uint64_t)(8 * i) * (uint64_t)Lk, i & 1 ? p_off ^ 64u : p_off, lds_p + 16u * 64 * i);
        return m_row[(size_t)pair * 16];
    };
    struct Kept {   // v[2 i + t] = keys 64 i + 32 t + 16 h .. +15 of the pair
        u32x4 v[4], codes;
    };
    u32x4 next_codes = load_kept(rot);

    bf16x8 bq[STEPS];
    float nd = 0.f;   // -delta of query lj
    const int qrow = q0 + lj < LqR ? q0 + lj : LqR - 1;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const size_t off = ((size_t)bh * LqR + qrow) * D + 16 * s + 8 * h;
        const u32x4 g = *reinterpret_cast<const u32x4 *>(dO + off), o = *reinterpret_cast<const u32x4 *>(O + off);
        bq[s] = __builtin_bit_cast(bf16x8, g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            nd -= bf16_lo_to_f32(g[e]) * bf16_lo_to_f32(o[e]) + bf16_hi_to_f32(g[e]) * bf16_hi_to_f32(o[e]);
    }
    nd += __shfl_xor(nd, 32, kWave);
    if (h == 0 && q0 + lj < Lq && (!SPLIT || sp == 0)) neg_delta[(size_t)bh * Lq + q0 + lj] = nd;
    f32x16 start;
#pragma unroll
    for (int r = 0; r < 16; ++r) start[r] = nd;

    f32x16 acc_q[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_q[dt][r] = 0.f;

    const int s16 = l & 15;
    const int tr_row = s16 >> 2, tr_sub = (s16 >> 1) & 1, tr_byte = 8 * (s16 & 1), tr_xor = tr32_swizzle<CPR>(tr_row);
    const int tr_colgrp = (l >> 4) & 1;

    // one block; buf: its LDS buffer and its place in the pair
    auto block = [&](auto parity, const Kept &cur) {
        constexpr int buf = decltype(parity)::value;
        const char *kbase = reinterpret_cast<const char *>(&Kr[buf][0]);
        auto tr = [&](int key0, int dt) {
            return lds_read_tr16(kbase + ((key0 + tr_row) * CPR + ((4 * dt + 2 * tr_colgrp + tr_sub) ^ tr_xor)) * 16 + tr_byte);
        };
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // acc[4 g + x] = dO[q] . V[key] - delta_q, key 64 jb + 32 t + 16 h + 4 g + x
            f32x16 acc;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const bf16x8 av = __builtin_bit_cast(
                    bf16x8, Vs[buf][(32 * t + lj) * CPR + ((2 * s + h) ^ operand_row_swizzle<CPR, 32>(lj))]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bq[s], s == 0 ? start : acc, 0, 0, 0);
            }
            const uint32_t codes = cur.codes[2 * t + buf] >> (16 * h);
            const u32x4 kept = cur.v[2 * buf + t];
            u32x4 ds;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // codes p_lo | p_hi << 2 with p_lo in 0 .. 2, p_hi in 1 .. 3
                const uint32_t b0 = spread_bit(codes, 4 * g), b1 = spread_bit(codes, 4 * g + 1);
                const uint32_t b2 = spread_bit(codes, 4 * g + 2), b3 = spread_bit(codes, 4 * g + 3);
                const float lo = choose(b1, acc[4 * g + 2], choose(b0, acc[4 * g + 1], acc[4 * g]));
                const float hi = choose(b3, choose(b2, acc[4 * g + 3], acc[4 * g + 2]), acc[4 * g + 1]);
                ds[g] = pack_bf16x2(bf16_lo_to_f32(kept[g]) * lo, bf16_hi_to_f32(kept[g]) * hi);
            }
            const bf16x8 a = __builtin_bit_cast(bf16x8, ds);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const int k0 = 32 * t + 8 * h;
                const s16x4 t0 = tr(k0, dt), t1 = tr(k0 + 4, dt), t2 = tr(k0 + 16, dt), t3 = tr(k0 + 20, dt);
                const s16x8 lo = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
                const s16x8 hi = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
                const bf16x16 b = __builtin_bit_cast(
                    bf16x16, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15));
                acc_q[dt] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a, b, acc_q[dt], (int)codes, 0, 0);
            }
            // (d = 128, four waves: whole pass 24 x 4096 x 4096 502 -> 500 us, 64 x 2048 level; two waves, 20 x 1500 x 1500 76.8 and 77.3, but with
            // shared keys 5 x 2240 x 2240 68.7 -> 66.2, 2 x 2368 x 636 34.3 -> 33.3; d = 64, three waves per SIMD, 3 % slower)
            if constexpr (EARLY) {
                read_ahead<STEPS, 1, 2, 0>();
                read_ahead<DT, 4, 2, 0>();
            }
        }
    };
    int pair = rot;
    Pace<PACED> pace(visits);
    for (int it = 0; it < visits; ++it) {
        pace.at(visits - it);
        const bool single = 2 * pair + 1 >= nblocks, last = it + 1 == visits;
        const int after = pair + 1 == npairs ? 0 : pair + 1;
        wait_async_copies();   // the pair's first block and its weights are in
        __syncthreads();
        if (!single) issue_block(2 * pair + 1, 1);
        Kept cur;
        cur.codes = next_codes;
#pragma unroll
        for (int i = 0; i < 4; ++i) cur.v[i] = Ps[w][lj * 8 + ((2 * i + h) ^ operand_row_swizzle<8, 32>(lj))];
        // The weights have to be in registers before their place is given to the next ones.  Two waves, on grids where a SIMD has one:
        // behind the first block, whose products hide that wait (d = 128 whole pass, 20 x 1100 x 1100 61.8 -> 60.0 us, 16 x 2000 x 2000
        // 103 -> 99; d = 64, 24 x 1024 x 1024 35.5 -> 35.0).  Right away with four waves (24 x 4096 x 4096 274, behind it 278) and, together with
        // the reads in order, where keys are shared at d = 128.
        auto ask = [&]() {
            asm volatile("" : "+v"(cur.v[0]), "+v"(cur.v[1]), "+v"(cur.v[2]), "+v"(cur.v[3]) : : "memory");
            if (!last) next_codes = load_kept(after);
        };
        if constexpr (NW == 4 || EARLY) ask();
        block(std::integral_constant<int, 0>{}, cur);
        if constexpr (!(NW == 4 || EARLY)) ask();
        if (single) {   // (the other buffer is free: everybody is past its use)
            __syncthreads();
            if (!last) issue_block(2 * after, 0);
        } else {
            // the second block is in; the weights of the next pair, issued after it, stay in flight
            if (!last) wait_async_copies_keep<KEPT_LOADS>();
            else wait_async_copies();
            __syncthreads();
            if (!last) issue_block(2 * after, 0);
            block(std::integral_constant<int, 1>{}, cur);
        }
        pair = after;
    }

    // acc_q[dt][r] = dQ[q][32 dt + lj] / scale, q = q0 + 8 (r / 4) + 4 h + r % 4
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int q = q0 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (q >= LqR) continue;
        const size_t row = (size_t)bh * LqR + q;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if constexpr (SPLIT) part[((size_t)sp * (gridDim.x / splits / qtiles * LqR) + row) * D + 32 * dt + lj] = acc_q[dt][r];
            else dQ[row * D + 32 * dt + lj] = (uint16_t)(pack_bf16x2(acc_q[dt][r] * scale, 0.f) & 0xFFFFu);
        }
    }
}

// Gradients from the sums of workgroups that shared them, added in a fixed order: out = scale (part[0] + part[1] + ...), n values
// (a multiple of 8) each, consecutive parts `stride` apart.  A thread forms 8 consecutive values; the jobs follow one another.
struct MergeJob {
    const float *part;
    uint16_t *out;
    size_t n, stride;
    int splits;
    float scale;
};
struct MergeJobs {
    MergeJob job[3];
};
__global__ __launch_bounds__(NT) void k_backward_merge(MergeJobs jobs) {
    size_t i = 8 * ((size_t)blockIdx.x * NT + threadIdx.x);
    MergeJob j = jobs.job[0];
    if (i >= j.n) {
        i -= j.n;
        j = jobs.job[1];
        if (i >= j.n) {
            i -= j.n;
            j = jobs.job[2];
            if (i >= j.n) return;
        }
    }
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll 4
    for (int sp = 0; sp < j.splits; ++sp) {
        const f32x4 *const src = reinterpret_cast<const f32x4 *>(j.part + sp * j.stride + i);
        a += src[0];
        b += src[1];
    }
    a *= j.scale, b *= j.scale;
    *reinterpret_cast<u32x4 *>(j.out + i) = u32x4{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
}

// Sixteen zeros made on the spot (as a constant they are kept in sixteen registers of their own and copied from there)
__device__ __forceinline__ f32x16 fresh_zeros() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        uint64_t p = 0;
        asm volatile("" : "+v"(p));
        z[r] = __uint_as_float((uint32_t)p), z[r + 1] = __uint_as_float((uint32_t)(p >> 32));
    }
    return z;
}

// Expands the kept weights of 32 queries x 32 keys (see k_backward_dkv) where some are infinite or NaN: times the identity
// such a weight would spread over its whole row (0 x infinity).  They are taken out, marked (1: NaN, 2: infinity, 3: -infinity),
// expanded on their own and put back where they belong.
__device__ __forceinline__ f32x16 expand_non_finite(u32x4 kept, bf16x16 eye, uint32_t codes) {
    u32x4 marks;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t clean = 0u, mark = 0u;
#pragma unroll
        for (int h = 0; h < 32; h += 16) {
            const uint32_t w = (kept[e] >> h) & 0xFFFFu;
            const bool bad = (w & 0x7F80u) == 0x7F80u;
            clean |= bad ? 0u : w << h;
            mark |= (!bad ? 0u : (w & 0x7Fu) ? 0x3F80u : (w & 0x8000u) ? 0x4040u : 0x4000u) << h;   // bfloat16 1, 3, 2
        }
        kept[e] = clean;
        marks[e] = mark;
    }
    f32x16 x = fresh_zeros();
    x = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, marks), eye, x, (int)codes, 0, 0);
    uint32_t kinds = 0u;   // two bits per register
#pragma unroll
    for (int r = 0; r < 16; ++r) kinds |= (uint32_t)(int)x[r] << (2 * r);
    x = fresh_zeros();
    x = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, kept), eye, x, (int)codes, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint32_t k = (kinds >> (2 * r)) & 3u;
        const uint32_t v = k == 1u ? 0x7FC00000u : k == 2u ? 0x7F800000u : 0xFF800000u;
        x[r] = __uint_as_float(k ? v : __float_as_uint(x[r]));
    }
    return x;
}

// dV = P^T dO and dK = scale * dS^T Q in one pass over the queries; a workgroup owns 128 keys of a head, a wave 32 of them.
// Both sums contract over the queries, across which the N:M structure does not run, so a wave needs P (and dP) with a KEY
// in every lane and the queries along the registers.  The matrix unit does that transposition: the compressed weights
// of 32 queries x 32 keys times the identity (one sparse instruction, operand and index as stored) is the dense tile in
// the accumulator layout -- column = key, registers = queries, exact in fp32 -- with no vector instruction per element.
// dP - delta arrives in the same layout from the dense product of dO (rows) with V (columns, in registers for the whole
// kernel), started from -delta of the rows; dS is one multiplication per element.  Rounded to bfloat16 both tiles are the A
// operands (row = key) of the two products, contraction index 8 m' + 4 h + x of step m = register order, against dO
// and Q from the transposing LDS read in the same order.
// 13 matrix instructions of 32 cycles per 32 x 32 tile at d = 64 (25 at d = 128) keep the matrix unit busy 61 % of the time
// (4096 x 4096, 24 heads, 148 us; the vector unit 34 %; d = 128, 64 heads x 2048, 196 us: 54 and 21 %).  The rest is waiting: one
// wait for the copies and one barrier per block, with P, which comes from memory, asked for one block ahead.
// SPLIT: `splits` workgroups share the queries of a key tile, a run of blocks each; their sums, unscaled fp32, go to `part`
// [split][dV, dK][head and key][D], and k_backward_merge forms dV and dK.
// UNP as above; the rows LqR .. Lq - 1 of P, whatever they hold, count as zeros.
// What is infinite or NaN has to stay at the kept places, but the two products are formed at every place: a row of V that no
// query kept, a row of dO, a weight that is infinite or NaN meets zeros there, and 0 times it is NaN.  Such a NaN always
// reaches the sums.  A workgroup without a NaN in its sums is done; another one starts again, CAREFUL: non-finite weights are
// expanded apart, and dS is formed by the multiplication in which 0 times anything is 0.
// w: the wave.  Result, the same in every thread of the workgroup: start again.
template <int D>
struct DkvPlace {   // the kernel's LDS in 16-byte units (an access is one of a few lane offsets plus a constant);
                    // every place but the V operand twice, BUF apart
    static constexpr int QB = D == 64 ? 64 : 32;    // queries per block (d = 128: so that two workgroups share a compute unit)
    static constexpr int XT = QB * (D / 8);         // chunks per dO (or Q) block
    static constexpr int PT = QB * 8;               // chunks per block of kept weights (128 keys = 128 bytes per row)
    static constexpr bool V_LDS = D == 128;         // the V operand: in LDS where registers are short (read back for every tile)
    static constexpr int AT_G = 0, AT_Q = XT, AT_P = 2 * XT, AT_M = AT_P + PT, AT_D = AT_M + QB, BUF = AT_D + QB / 4, AT_V = 2 * BUF;
    static constexpr int SIZE = AT_V + (V_LDS ? KB * (D / 8) : 0);
};
template <int D, bool UNP, bool CAREFUL, bool SPLIT, bool PACED>
__device__ __forceinline__ bool dkv_pass(
    u32x4 *Smem, const int w, const uint32_t *__restrict__ P, const uint32_t *__restrict__ meta, const __bf16 *__restrict__ dO,
    const __bf16 *__restrict__ Q, const __bf16 *__restrict__ V, const float *__restrict__ neg_delta, int Lq, int Lk,
    int LqR, int LkR, float scale, uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, int splits, float *__restrict__ part) {
    using L = DkvPlace<D>;
    constexpr int QB = L::QB, XT = L::XT, PT = L::PT, AT_G = L::AT_G, AT_Q = L::AT_Q, AT_P = L::AT_P, AT_M = L::AT_M, AT_D = L::AT_D;
    constexpr int BUF = L::BUF, AT_V = L::AT_V;
    constexpr bool V_LDS = L::V_LDS;
    constexpr int CPR = D / 8;
    constexpr int LPT = XT / NT;
    constexpr int STEPS = D / 16;
    constexpr int DT = D / 32;
    static_assert(XT % NT == 0 && PT % NT == 0, "every thread copies the same number of chunks");

    // (the lane number is asked for again in a second pass, so that nothing derived from it is kept through the first one)
    int tid = threadIdx.x;
    if constexpr (CAREFUL) {
        tid = __lane_id();
        asm volatile("" : "+v"(tid));
        tid += 64 * w;
    }
    const int l = tid & 63, lj = l & 31, h = l >> 5;
    const unsigned kblocks = Lk / KB;
    const unsigned share = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned item = SPLIT ? share / (unsigned)splits : share;
    const int sp = SPLIT ? share % (unsigned)splits : 0;
    const int jblk = item % kblocks, bh = item / kblocks;
    const int all = (LqR + QB - 1) / QB;   // blocks of queries: this workgroup takes nq of them from qb0 on (splits <= all)
    const int qb0 = SPLIT ? __builtin_amdgcn_readfirstlane(all * sp / splits) : 0;
    const int nq = SPLIT ? __builtin_amdgcn_readfirstlane(all * (sp + 1) / splits) - qb0 : all;

    // dO and Q blocks: row = query, chunk c at row * CPR + (c ^ both_ways_swizzle(row)); kept weights: row = query, chunk c
    // at row * 8 + (c ^ operand_row_swizzle(row)); metadata: 16 bytes per row
    int x_row[LPT], x_chunk[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * NT + tid;
        x_row[i] = p / CPR;
        x_chunk[i] = ((p % CPR) ^ both_ways_swizzle<CPR>(x_row[i])) * 8;
    }
    const uint32_t lds = lds_address(Smem), lds_w = lds + 16u * 64 * w;
    const uint64_t g_base = uniform_address(dO + (size_t)bh * LqR * D), q_base = uniform_address(Q + (size_t)bh * LqR * D);
    const uint64_t p_base = uniform_address(P + ((size_t)bh * Lq * (size_t)(Lk / 4) + (size_t)jblk * 32));
    const uint64_t m_base = uniform_address(meta + ((size_t)bh * (Lq / 16) * kblocks + jblk) * 64);
    const uint64_t d_base = uniform_address(neg_delta + (size_t)bh * Lq);
    const uint32_t p_off = (uint32_t)(tid >> 3) * (uint32_t)Lk + 16u * ((tid & 7) ^ operand_row_swizzle<8, 32>(tid >> 3));
    auto issue_block = [&](int qb, int buf) {
        const uint64_t gs = g_base + (uint64_t)qb * (QB * D * 2), qs = q_base + (uint64_t)qb * (QB * D * 2);
        const int last = UNP ? LqR - qb * QB - 1 : QB - 1;   // the block's last real row
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const uint32_t off = 2u * ((UNP && x_row[i] > last ? last : x_row[i]) * D + x_chunk[i]);
            async_copy16(gs, off, lds_w + 16u * (buf * BUF + AT_G + i * NT));
            async_copy16(qs, off, lds_w + 16u * (buf * BUF + AT_Q + i * NT));
        }
        // (32 rows further: the swizzle takes row bits 1 .. 3, which do not move)
#pragma unroll
        for (int i = 0; i < PT / NT; ++i)
            async_copy16(p_base + ((uint64_t)qb * QB + 32 * i) * (uint64_t)Lk, p_off, lds_w + 16u * (buf * BUF + AT_P + i * NT));
        if (w == 0) {
            if (l < QB)
                async_copy16(m_base + (uint64_t)qb * (QB / 16) * kblocks * 256u, (uint32_t)(l >> 4) * kblocks * 256u + 16u * (l & 15),
                             lds + 16u * (buf * BUF + AT_M));
        } else if (w == 1) {
            if (l < QB / 4) async_copy16(d_base + (uint64_t)qb * (QB * 4), 16u * l, lds + 16u * (buf * BUF + AT_D));
        }
    };
    issue_block(qb0, 0);

    // V operand: column = key lj of this wave, k = 16 s + 8 h .. +7
    bf16x8 bv[V_LDS ? 1 : STEPS];
    {
        const int real = UNP ? LkR - jblk * KB : KB;   // real keys of this workgroup
        const __bf16 *const v_rows = V + ((size_t)bh * LkR + (size_t)jblk * KB) * D;
        if constexpr (V_LDS) {   // row = key, chunk c at row * CPR + (c ^ operand_row_swizzle(row))
#pragma unroll
            for (int i = 0; i < KB * CPR / NT; ++i) {
                const int p = i * NT + tid, row = p / CPR;
                async_copy16(v_rows, 2u * ((UNP && row >= real ? real - 1 : row) * D + ((p % CPR) ^ operand_row_swizzle<CPR, 32>(row)) * 8),
                             lds_w + 16u * (AT_V + i * NT));
            }
        } else {
            const int row = UNP && 32 * w + lj >= real ? real - 1 : 32 * w + lj;
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                bv[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(v_rows + row * D + 16 * s + 8 * h));
        }
    }
    // the identity as B operand of the sparse instruction: lane (column lj, h) holds keys 8 h .. +7 and 16 + 8 h .. +7
    bf16x16 eye;
    {
        s16x16 e16;
#pragma unroll
        for (int e = 0; e < 16; ++e) e16[e] = (e < 8 ? 8 * h + e : 8 + 8 * h + e) == lj ? (short)0x3F80 : (short)0;
        eye = __builtin_bit_cast(bf16x16, e16);
    }

    f32x16 acc_v[DT], acc_k[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_v[dt][r] = 0.f, acc_k[dt][r] = 0.f;

    // Lane offsets (bytes).  Operand read of dO (and of V): row lj, chunk 2 s + h.  Transposing read of dO and Q: rows
    // row0 + 4 h + 8 j + tr_row (j = 0, 1; row0 a multiple of 16: it does not move the swizzle), columns 32 dt .. +31.
    const int s16 = l & 15;
    const int tr_row = s16 >> 2, tr_chunk = 2 * ((l >> 4) & 1) + ((s16 >> 1) & 1), tr_byte = 8 * (s16 & 1);
    int op_off[STEPS], v_off[V_LDS ? STEPS : 1], tr_off[2][DT];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        op_off[s] = 16 * (lj * CPR + ((2 * s + h) ^ both_ways_swizzle<CPR>(lj)));
        if constexpr (V_LDS) v_off[s] = 16 * (AT_V + (32 * w + lj) * CPR + ((2 * s + h) ^ operand_row_swizzle<CPR, 32>(lj)));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const int row = 4 * h + 8 * j + tr_row;
            tr_off[j][dt] = 16 * (row * CPR + ((4 * dt + tr_chunk) ^ both_ways_swizzle<CPR>(row))) + tr_byte;
        }
    const int p_lane = 16 * (lj * 8 + ((2 * w + h) ^ operand_row_swizzle<8, 32>(lj)));
    const int m_lane = 16 * lj + 4 * (((w & 1) << 1) | (w >> 1));   // the word of 32-key chunk w in a row's 16 bytes
    const int d_lane = 16 * h;
    const char *const smem = reinterpret_cast<const char *>(Smem);
    auto read16 = [&](int lane_off, int at) { return *reinterpret_cast<const u32x4 *>(smem + lane_off + 16 * at); };

    auto block = [&](auto parity, int qb) {
        constexpr int buf = decltype(parity)::value;
        wait_async_copies();
        __syncthreads();
        if (qb + 1 < qb0 + nq) issue_block(qb + 1, buf ^ 1);
#pragma unroll
        for (int qt = 0; qt < QB / 32; ++qt) {
            constexpr int B0 = buf * BUF;
            u32x4 kept = read16(p_lane, B0 + AT_P + 32 * 8 * qt);
            if (UNP && qb * QB + 32 * qt + lj >= LqR) kept = u32x4{0u, 0u, 0u, 0u};
            const uint32_t codes = *reinterpret_cast<const uint32_t *>(smem + m_lane + 16 * (B0 + AT_M + 32 * qt)) >> (16 * h);
            f32x16 dp, pd;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 nd = __builtin_bit_cast(f32x4, read16(d_lane, B0 + AT_D + 8 * qt + 2 * g));   // rows 32 qt + 8 g + 4 h .. +3
#pragma unroll
                for (int x = 0; x < 4; ++x) dp[4 * g + x] = nd[x];
            }
            if constexpr (CAREFUL) {
                pd = expand_non_finite(kept, eye, codes);
            } else {
                pd = fresh_zeros();
                pd = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8, kept), eye, pd, (int)codes, 0, 0);
            }
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const bf16x8 ag = __builtin_bit_cast(bf16x8, read16(op_off[s], B0 + AT_G + 32 * CPR * qt));
                bf16x8 b;
                if constexpr (V_LDS) b = __builtin_bit_cast(bf16x8, read16(v_off[s], 0));
                else b = bv[s];
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ag, b, dp, 0, 0, 0);
            }
            // register r: query 32 qt + 8 (r / 4) + 4 h + r % 4, key lj
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                u32x4 pw, sw;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 8 * m + 2 * e;
                    pw[e] = pack_bf16x2(pd[r], pd[r + 1]);
                    if constexpr (CAREFUL) sw[e] = pack_bf16x2(mul_or_zero(pd[r], dp[r]), mul_or_zero(pd[r + 1], dp[r + 1]));
                    else sw[e] = pack_bf16x2(pd[r] * dp[r], pd[r + 1] * dp[r + 1]);
                }
                const bf16x8 ap = __builtin_bit_cast(bf16x8, pw), as = __builtin_bit_cast(bf16x8, sw);
                auto tr = [&](int at, int dt) {
                    const int rows = 16 * (B0 + at + CPR * (32 * qt + 16 * m));
                    const s16x4 t0 = lds_read_tr16(smem + tr_off[0][dt] + rows), t1 = lds_read_tr16(smem + tr_off[1][dt] + rows);
                    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7));
                };
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    acc_v[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap, tr(AT_G, dt), acc_v[dt], 0, 0, 0);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    acc_k[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as, tr(AT_Q, dt), acc_k[dt], 0, 0, 0);
            }
            // (unpadded lengths at d = 64, whole pass: 24 heads x 1000 41.6 -> 37.3 us, x 4000 288 -> 281.  With the tile multiples the
            // order that the compiler finds is as fast, at d = 128 it is the faster one by 2 - 13 %.)
            if constexpr (UNP && !CAREFUL && D == 64) read_ahead<4 * DT, 2, 2, 0>();
        }
    };
    Pace<PACED> pace(nq);
    for (int i = 0; i < nq; i += 2) {
        pace.at(nq - i);
        block(std::integral_constant<int, 0>{}, qb0 + i);
        if (i + 1 < nq) block(std::integral_constant<int, 1>{}, qb0 + i + 1);
    }

    // acc[dt][r]: key 8 (r / 4) + 4 (lane / 32) + r % 4 of the wave's 32, column 32 dt + lane % 32
    auto store = [&]() {
        const int lane = __lane_id();   // (asked for again: a register less through the loop)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = jblk * KB + 32 * w + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (UNP && key >= LkR) continue;
            if constexpr (SPLIT) {   // [split][dV, dK][head and key][D]; the 64-bit part of the address is the same in every lane
                const size_t n = (size_t)(gridDim.x / splits / kblocks) * LkR * D;
                float *const pv = part + 2 * sp * n + (size_t)bh * LkR * D;
                const uint32_t to = (uint32_t)key * D + (lane & 31);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) pv[to + 32 * dt] = acc_v[dt][r], pv[n + to + 32 * dt] = acc_k[dt][r];
                continue;
            }
            const size_t at = ((size_t)bh * LkR + key) * D + (lane & 31);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                dV[at + 32 * dt] = (uint16_t)(pack_bf16x2(acc_v[dt][r], 0.f) & 0xFFFFu);
                dK[at + 32 * dt] = (uint16_t)(pack_bf16x2(acc_k[dt][r] * scale, 0.f) & 0xFFFFu);
            }
        }
    };
    if constexpr (CAREFUL) {
        store();
        return false;
    } else {
        // Did some sum become NaN?  A NaN in the row of a key fills the whole row, so one column of each tile tells; their total
        // is NaN with it (or infinite).  The care in every pass would cost 5 - 18 % on small grids.  The waves agree through LDS,
        // at a place of the buffer that the last block did not use, while the stores of the ones without a NaN are on their way.
        f32x4 total = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r & 3] += acc_v[0][r], total[r & 3] += acc_k[0][r];
        uint32_t t = __float_as_uint((total[0] + total[1]) + (total[2] + total[3]));
        asm("" : "+v"(t));   // (as a number, under the flags of this library, it could not be NaN)
        uint32_t *const flags = reinterpret_cast<uint32_t *>(Smem + (((nq - 1) & 1) ? 0 : BUF));
        const bool mine = __any((t & 0x7F800000u) == 0x7F800000u);
        if (__lane_id() == 0) flags[w] = mine ? 1u : 0u;
        if (__builtin_expect(!mine, 1)) store();
        __syncthreads();
        const uint32_t any = flags[0] | flags[1] | flags[2] | flags[3];
        if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)any) == 0, 1)) return false;
        __syncthreads();   // everybody has read the flags; the buffers are free
        return true;
    }
}

template <int D, bool UNP, bool SPLIT, bool PACED>
__global__ __launch_bounds__(NT, D == 64 ? 3 : 2) void k_backward_dkv(
    const uint32_t *__restrict__ P, const uint32_t *__restrict__ meta, const __bf16 *__restrict__ dO,
    const __bf16 *__restrict__ Q, const __bf16 *__restrict__ V, const float *__restrict__ neg_delta, int Lq, int Lk,
    int LqR, int LkR, float scale, uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, int splits, float *__restrict__ part) {
    __shared__ u32x4 Smem[DkvPlace<D>::SIZE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (dkv_pass<D, UNP, false, SPLIT, PACED>(Smem, w, P, meta, dO, Q, V, neg_delta, Lq, Lk, LqR, LkR, scale, dK, dV, splits, part))
        dkv_pass<D, UNP, true, SPLIT, false>(Smem, w, P, meta, dO, Q, V, neg_delta, Lq, Lk, LqR, LkR, scale, dK, dV, splits, part);
}

}  // namespace

hipError_t launch_spmm_t(const void *vals, const void *meta, const void *X, int BH, int Lq, int Lk, int LqR, int LkR,
                         int d, void *out, hipStream_t st) {
    const unsigned grid = (unsigned)((long)BH * (Lk / KB));
    const bool unp = LqR != Lq || LkR != Lk;
#define DFSS_LAUNCH(DD, UU)                                                                                        \
    hipLaunchKernelGGL((k_spmm_t<DD, UU>), dim3(grid), dim3(NT), 0, st, (const uint32_t *)vals, (const uint32_t *)meta, \
                       (const __bf16 *)X, Lq, Lk, LqR, LkR, (uint16_t *)out)
    if (d == 64) {
        if (unp) DFSS_LAUNCH(64, true); else DFSS_LAUNCH(64, false);
    } else {
        if (unp) DFSS_LAUNCH(128, true); else DFSS_LAUNCH(128, false);
    }
#undef DFSS_LAUNCH
    return hipGetLastError();
}

namespace {

size_t align256(size_t x) { return (x + 255) / 256 * 256; }
size_t delta_bytes(int BH, int Lq) { return align256((size_t)BH * Lq * sizeof(float)); }
size_t dq_sum_bytes(int n, int BH, int LqR, int d) { return n == 1 ? 0 : align256((size_t)n * BH * LqR * d * sizeof(float)); }
size_t dkv_sum_bytes(int n, int BH, int LkR, int d) { return n == 1 ? 0 : align256((size_t)n * 2 * BH * LkR * d * sizeof(float)); }

// How many workgroups share the keys of a query tile (dQ) and the queries of a key tile (dV and dK); 1: none.  A tile is walked at
// the pace of one workgroup, and a small grid leaves most of the chip idle; sharing costs the sums, written and read in fp32,
// and the kernel that adds them.  The counts -- the powers of two and, for the keys, two pairs of blocks each -- are those with the least of
//     us per step x steps / count x (1 + slope (workgroups / chip - 1) beyond a full chip) + sums, at 5 TB/s + 4 us for that kernel,
//     the first part at least what it takes to read K and V (Q and dO), at 6 TB/s
// (a larger count has to save a tenth; without the lower bound d = 128, 64 heads x 64 x 4096 82 us, with it 76), as long as the workgroups
// are all resident at once; beyond that a further round begins (d = 128, 3 heads x 3072 x 1536: 56 us with it, 50 without; d = 64, 16 x
// 1536 x 8192 180 and 166; 96 x 256 x 8192 253 and 236).
// Shared where it gains 2 us or more and the two kernels take longer than their launches (one head x 512 x 512, d = 64: 19.2 us, with a
// third launch 22.1).  At d = 128, where the keys weigh more, sooner (one head x 64 x 512 18.5 -> 16.5 us, x 768 23.0 -> 16.9, 48 x 64 x 512
// 20.6 -> 20.1; 64 x 64 x 512 21.3, shared 21.8.  On the GPU: where call after call is launched by the host, the first of these takes 18.8 and 20.6.)
// Measured alone: a step of dQ, 128 keys, 1.4 us at d = 64 and 2.2 at d = 128, the chip full with 512 workgroups of two waves (1024 and 512
// are resident); a step of dV and dK, 64 queries, 0.9 and 1.56 us, full with 256 of four (768 and 512).
// The whole pass, before (keys shared at d = 128 up to 128 tiles) and now, us: d = 64, one head x 4096 x 4096 102 -> 34, 4 x 4096 103
// -> 68, 4 x 2048 55 -> 33, 4 x 1024 31 -> 23, 4 x 4096 x 512 66 -> 26; d = 128, one head x 4096 122 -> 48, 4 x 4096 171 -> 109, 4 x
// 2048 76 -> 47; left alone, rightly: 12 x 1024 (31.4; shared by two 32.0), 24 x 512 (19.4; 25.5), 48 x 512 at d = 128 (33.9; 46.3).
// (12 x 2048 x 2048, d = 64, would gain: 61.5, shared by two 57.4.)
// room: bytes there are for the sums; the counts are those whose sums fit, and if they do not fit together, those of the part that gains more.
struct Sharing {
    int dq, dkv;
};
float shared_us(float step, int steps, int n, float fill, float slope, double sum_bytes, double read_bytes) {
    const float work = step * (float)steps / (float)n * (fill * n > 1.f ? 1.f + slope * (fill * n - 1.f) : 1.f), read = (float)(read_bytes / 6.0e6);
    return (n > 1 && work < read ? read : work) + (n > 1 ? (float)(n * sum_bytes / 5.0e6) : 0.f);
}
Sharing sharing(int BH, int Lq, int Lk, int LqR, int LkR, int d, size_t room = SIZE_MAX) {
    const float kGain = d == 64 ? 6.f : 3.f, kHost = d == 64 ? 16.f : 10.f;
    const int pairs = (LkR + KB - 1) / KB, steps = (LqR + 63) / 64;
    const long wg_q = (long)BH * (Lq / 64), wg_k = (long)BH * (Lk / KB);
    const long resident_q = d == 64 ? 1024 : 512, resident_k = d == 64 ? 768 : 512;
    const float step_q = d == 64 ? 1.4f : 2.2f, step_k = d == 64 ? 0.9f : 1.56f;
    const double bytes_q = 8. * BH * LqR * d, bytes_k = 16. * BH * LkR * d;   // sums, written and read
    const double read_q = 4. * BH * LkR * d, read_k = 4. * BH * LqR * d;
    Sharing s = {1, 1};
    const float alone_q = shared_us(step_q, pairs, 1, wg_q / 512.f, 0.f, 0., 0.), alone_k = shared_us(step_k, steps, 1, wg_k / 256.f, 0.f, 0., 0.);
    float best_q = alone_q, best_k = alone_k;
    const int most = pairs / 2 < 32 ? pairs / 2 : 32;
    for (int n = 2; n <= most && wg_q < 512 && n * wg_q <= resident_q && dq_sum_bytes(n, BH, LqR, d) <= room; n = n < most && 2 * n > most ? most : 2 * n) {   // (128-query workgroups do not share)
        const float us = shared_us(step_q, pairs, n, wg_q / 512.f, d == 64 ? 0.35f : 1.f, bytes_q, read_q);
        if (us < 0.9f * best_q) best_q = us, s.dq = n;
    }
    for (int n = 2; n <= 16 && n <= steps / 4 && wg_k <= 256 && n * wg_k <= resident_k && dkv_sum_bytes(n, BH, LkR, d) <= room; n *= 2) {
        const float us = shared_us(step_k, steps, n, wg_k / 256.f, 0.35f, bytes_k, read_k);
        if (us < 0.92f * best_k) best_k = us, s.dkv = n;
    }
    float gain_q = alone_q - best_q, gain_k = alone_k - best_k;
    if (dkv_sum_bytes(s.dkv, BH, LkR, d) > room - dq_sum_bytes(s.dq, BH, LqR, d)) {
        if (gain_q < gain_k) s.dq = 1, gain_q = 0.f;
        else s.dkv = 1, gain_k = 0.f;
    }
    // the kernel that adds is paid once
    if (alone_q + alone_k < kHost || gain_q + gain_k < kGain) return {1, 1};
    if (gain_q < 1.f) s.dq = 1;
    if (gain_k < 1.f) s.dkv = 1;
    return s;
}

}  // namespace

// The row terms -delta, fp32 [BH][Lq] (the least that the pass needs), then the sums of the workgroups that share keys (dQ) and of
// those that share queries (dV and dK).
size_t backward_workspace_least(int BH, int Lq) { return delta_bytes(BH, Lq); }
size_t backward_workspace_bytes(int BH, int Lq, int Lk, int LqR, int LkR, int d) {
    const Sharing s = sharing(BH, Lq, Lk, LqR, LkR, d);
    return delta_bytes(BH, Lq) + dq_sum_bytes(s.dq, BH, LqR, d) + dkv_sum_bytes(s.dkv, BH, LkR, d);
}

// P, meta: as kept from the forward pass.  ws: backward_workspace_least or more; keys and queries are shared as far as the sums fit
// (the whole is less for a large grid than for a small one, and a workspace made for the largest shape has to do for all).
hipError_t launch_backward(const void *dO, const void *Q, const void *K, const void *V, const void *O, const void *P,
                           const void *meta, int BH, int Lq, int Lk, int LqR, int LkR, int d, float scale, void *ws,
                           size_t ws_bytes, void *dQ, void *dK, void *dV, hipStream_t st) {
    const bool unp = LqR != Lq || LkR != Lk;
    const Sharing s = sharing(BH, Lq, Lk, LqR, LkR, d, ws_bytes - delta_bytes(BH, Lq));
    float *const neg_delta = (float *)ws, *const part_q = (float *)((char *)ws + delta_bytes(BH, Lq));
    float *const part_kv = (float *)((char *)part_q + dq_sum_bytes(s.dq, BH, LqR, d));
    const int splits = s.dq, splits_kv = s.dkv;
    // 128-query workgroups where they fill the chip (three per compute unit at d = 64, two at d = 128), else 64-query ones
    const bool four = (long)BH * ((Lq + 127) / 128) >= 512;
    const unsigned grid_q = (unsigned)((long)BH * (four ? (Lq + 127) / 128 : Lq / 64)) * splits;
    const unsigned grid_k = (unsigned)((long)BH * (Lk / KB)) * splits_kv;
    // Workgroups that keep level; not those that share: at the rate of one wave per SIMD it costs 1 - 3 %.  Two to a compute unit: also
    // where the last round has more than one for each (whole pass without and with, 49 x 2048 x 2048 306 and 295, 100 x 1024 x 1024 165 and
    // 161, 26 x 4096 x 4096 584 and 565; one for each, 96 x 1024 x 1024, 147 and 156).  Three: 80 x 2048 x 2048, two thirds full, 259 and 270.
    auto level = [](unsigned grid, unsigned per_cu, int walked) {
        return keep_level(grid, per_cu, walked, per_cu == 2 ? 4 : 6, per_cu == 2 ? 512 : 1024) && !(per_cu == 2 && grid > 512 && grid % 512 == 256);
    };
    const bool level_q = splits == 1 && level(grid_q, d == 128 ? 2 : four ? 3 : 4, Lk);
    const bool level_k = splits_kv == 1 && level(grid_k, d == 128 ? 2 : 3, Lq);
#define DFSS_DQ(DD, NW, UU, SS, LL)                                                                                      \
    hipLaunchKernelGGL((k_backward_dq<DD, NW, UU, SS, LL>), dim3(grid_q), dim3(64 * NW), 0, st, (const __bf16 *)dO,          \
                       (const __bf16 *)V, (const __bf16 *)O, (const uint32_t *)P, (const uint32_t *)meta,               \
                       (const __bf16 *)K, Lq, Lk, LqR, LkR, scale, (uint16_t *)dQ, neg_delta, splits, part_q)
#define DFSS_DKV(DD, UU, SS, LL)                                                                                         \
    hipLaunchKernelGGL((k_backward_dkv<DD, UU, SS, LL>), dim3(grid_k), dim3(NT), 0, st, (const uint32_t *)P,                 \
                       (const uint32_t *)meta, (const __bf16 *)dO, (const __bf16 *)Q, (const __bf16 *)V, neg_delta, Lq, Lk, \
                       LqR, LkR, scale, (uint16_t *)dK, (uint16_t *)dV, splits_kv, part_kv)
#define DFSS_BOTH(DD, UU)                                                \
    do {                                                                 \
        if (four && level_q) DFSS_DQ(DD, 4, UU, false, true);            \
        else if (four) DFSS_DQ(DD, 4, UU, false, false);                 \
        else if (level_q) DFSS_DQ(DD, 2, UU, false, true);               \
        else if (splits == 1) DFSS_DQ(DD, 2, UU, false, false);          \
        else DFSS_DQ(DD, 2, UU, true, false);                            \
        if (level_k) DFSS_DKV(DD, UU, false, true);                      \
        else if (splits_kv == 1) DFSS_DKV(DD, UU, false, false);         \
        else DFSS_DKV(DD, UU, true, false);                              \
    } while (0)
    if (d == 64) {
        if (unp) DFSS_BOTH(64, true); else DFSS_BOTH(64, false);
    } else {
        if (unp) DFSS_BOTH(128, true); else DFSS_BOTH(128, false);
    }
#undef DFSS_BOTH
#undef DFSS_DKV
#undef DFSS_DQ
    if (splits > 1 || splits_kv > 1) {
        const size_t nq = splits > 1 ? (size_t)BH * LqR * d : 0, nk = splits_kv > 1 ? (size_t)BH * LkR * d : 0;
        const MergeJobs jobs = {{{part_q, (uint16_t *)dQ, nq, nq, splits, scale},
                                 {part_kv, (uint16_t *)dV, nk, 2 * nk, splits_kv, 1.f},
                                 {part_kv + nk, (uint16_t *)dK, nk, 2 * nk, splits_kv, scale}}};
        const size_t threads = (nq + 2 * nk) / 8;
        hipLaunchKernelGGL(k_backward_merge, dim3((unsigned)((threads + NT - 1) / NT)), dim3(NT), 0, st, jobs);
    }
    return hipGetLastError();
}

}  // namespace dfss
