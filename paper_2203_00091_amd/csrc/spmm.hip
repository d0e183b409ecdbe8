// Stage 3 of the DFSS forward pass: O = A_sparse V with the 2:4-compressed attention
// weights (arXiv 2203.00091, Sec. 3.1), on the gfx950 structured-sparse matrix
// instruction v_smfmac_f32_16x16x64_bf16.  Per 128-key block a lane loads the 32 bytes of
// kept weights and the 32-bit metadata word that the same lane of stage 1 stored; the two
// halves of the word are the index operands of two instructions (selected with ABID), so
// nothing is decoded or shuffled.  1:2 pruning is stored with the same codes and runs
// through the same kernel.  The dense variant (P V of Eq. 1, for the baseline) shares the
// V staging and uses v_mfma_f32_16x16x32_bf16.
//
// k_spmm: compressed weights; k_av: compressed SCORES (SOFTMAX: two-kernel forward pass) or dense weights.
//
// The product on scores takes the kept SCORES of stage 1 instead of weights and applies the softmax
// on the way (Sec. 3.1; the max-subtracted form of App. A.1.3 with a running reference m in the place of the
// maximum): the scores of a block become exp(s - m) in registers before they enter the matrix instruction,
// the accumulators are rescaled when a block exceeds m by more than a threshold, the row sums come from the
// matrix unit too (an all-ones operand), and the result is divided by the sum at the end.  It replaces the separate softmax kernel (one read and one write of all kept values)
// in the two-kernel forward pass.
//
// V blocks (128 keys x d) are copied global -> LDS by the direct-to-LDS load, double
// buffered, row-major with an XOR swizzle of the 16-byte chunks; the B operand (keys along
// the contraction, one d-column per lane) comes from the transposing LDS read.
//
// Which keys an instruction contracts over is free as long as A and B agree.  Sparse
// instruction h (0/1) of a block takes, for its 16-wide contraction chunk c, the keys
// 32c + 16h .. +15 of the block -- the 16 keys whose kept weights lane group c holds in
// half h of its 32 bytes.
#include <cstdlib>
#include <type_traits>

#include "dfss_device.hpp"
#include "dfss_kernels.hpp"

namespace dfss {

namespace {

constexpr int NT = 256;   // 4 waves
constexpr int KB = 128;   // keys per block

// UNPADDED: V holds LkR <= Lk keys per head and O LqR <= Lq rows, while P and meta have the layout of the padded
// lengths Lq (a multiple of 64) and Lk (of 128).  The weights of the absent keys are 0 (their scores were -inf); their
// places in a partial last block of V are filled with the block's last real key, and rows past LqR are not stored.
// SPARSE: compressed scores, turned into weights on the way; else dense weights.
// PACED (compressed scores): the workgroups of a compute unit keep level (Pace).
template <int D, bool SPARSE, int RB, bool UNPADDED = false, bool PACED = false>
__global__ __launch_bounds__(NT, 2) void k_av(const uint32_t *__restrict__ P, const uint32_t *__restrict__ meta,
                                              const __bf16 *__restrict__ V, int Lq, int Lk, int LqR, int LkR,
                                              uint16_t *__restrict__ O) {
    constexpr int CPR = D / 8;          // 16-byte chunks per V row
    constexpr int TILE = KB * CPR;      // chunks per V block
    constexpr int LPT = TILE / NT;      // direct-to-LDS loads per thread per block
    constexpr int DS = D / 16;          // 16-column output tiles
    constexpr int TQ = 64 * RB;         // queries per workgroup
    constexpr bool SOFTMAX = SPARSE;
    __shared__ u32x4 Vs[2][TILE];

    const int tid = threadIdx.x;
    const int w = tid >> 6, l = tid & 63, li = l & 15, kb = l >> 4;

    const unsigned qtiles = Lq / TQ;
    const unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int qt = item % qtiles;
    const int bh = item / qtiles;
    const int rb0 = (qt * TQ >> 4) + w * RB;   // first 16-row block of this wave
    const int nblocks = Lk / KB;
    const int meta_slot = ((kb & 1) << 1) | (kb >> 1);   // where the word of 32-key chunk kb sits in a row's 16 bytes

    // LDS position p (16-byte units) = row * CPR + (c ^ v_swizzle(row)) holds chunk c of key `row`.  With rows of 256 bytes
    // two lanes meet in a pair of banks this way; tr_row_swizzle avoids that, but its patterns differ between the four reads
    // of an operand and between h = 0 and 1, and the addresses cost more (4 heads x 64 x 8192: 53.8 against 60.2 us, 4 x
    // 512 x 512 6.1 and 6.6; on dense weights no difference).
    auto v_swizzle = [](int row) { return CPR == 16 ? (row & 3) << 1 : tr_row_swizzle<CPR>(row); };
    const __bf16 *Vh = V + (size_t)bh * LkR * D;
    int src_off[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * NT + tid;
        const int row = p / CPR, c = (p % CPR) ^ v_swizzle(row);
        src_off[i] = row * D + c * 8;
    }
    const uint32_t lds_v = lds_address(&Vs[0][w * 64]);   // this wave's 1 KB slice of copy 0, buffer 0
    auto issue_block = [&](int jb, int buf) {
        const __bf16 *src = Vh + (size_t)jb * KB * D;
        const int real = LkR - jb * KB;   // real keys from this block's first one on
        if (UNPADDED && real < KB) {
#pragma unroll
            for (int i = 0; i < LPT; ++i) {
                const int p = i * NT + tid;
                const int row = p / CPR, c = (p % CPR) ^ v_swizzle(row);
                async_copy16(src, 2u * ((row < real ? row : real - 1) * D + c * 8), lds_v + 16u * (buf * TILE + i * NT));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LPT; ++i) async_copy16(src, 2u * src_off[i], lds_v + 16u * (buf * TILE + i * NT));
    };

    // A operand of one block
    struct AFrag {
        u32x4 v[SPARSE ? 2 : 4];
        uint32_t idx;
    };
    auto load_a = [&](int jb, AFrag (&a)[RB]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const size_t row = (size_t)bh * Lq + (size_t)(rb0 + rb) * 16 + li;
            if constexpr (SPARSE) {
                // kept weights of keys 128 jb + 32 kb .. +31: 16 of them, 32 bytes
                const u32x4 *pr = reinterpret_cast<const u32x4 *>(P + row * (size_t)(Lk / 4)) + jb * 8 + kb * 2;
                a[rb].v[0] = pr[0];
                a[rb].v[1] = pr[1];
                a[rb].idx = meta[((((size_t)bh * (Lq / 16) + rb0 + rb) * nblocks + jb) * 16 + li) * 4 + meta_slot];
            } else {
                // dense weights: MFMA m takes keys 128 jb + 32 m + 8 kb .. +7
                const u32x4 *pr = reinterpret_cast<const u32x4 *>(P + row * (size_t)(Lk / 2)) + jb * 16 + kb;
#pragma unroll
                for (int m = 0; m < 4; ++m) a[rb].v[m] = pr[4 * m];
                a[rb].idx = 0;
            }
        }
    };

    f32x4 acc[RB][DS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) acc[rb][ds] = f32x4{0.f, 0.f, 0.f, 0.f};

    // transposing read: lane li of a 16-lane group addresses V[key0 + li/4][col0 + 4*(li%4)]
    const int tr_row = li >> 2;
    const int tr_sub = (li >> 1) & 1;      // which 16-byte chunk of the 32-byte column group
    const int tr_byte = 8 * (li & 1);

    // SOFTMAX: reference value of row li of each row block (the same in the four lane groups kb of a row)
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr float kTau = 8.0f;   // the running reference of a row is raised when a score exceeds it by more than this
    float m_run[RB];
    f32x4 acc_l[RB];               // row sums, rows 4 kb + r (from the matrix unit: an all-ones B operand)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) m_run[rb] = -INFINITY, acc_l[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t one2 = 0x3F803F80u;   // two bfloat16 ones
    const bf16x8 ones8 = __builtin_bit_cast(bf16x8, u32x4{one2, one2, one2, one2});

    // SOFTMAX: turns the kept scores of one block into exp(s - m) in place, m = the row's reference value: the largest
    // score seen when it was last set.  It is raised (and the accumulators, which hold the blocks before, rescaled)
    // only when a score exceeds it by more than kTau, so weights stay below e^kTau and the common block needs no
    // cross-lane traffic; softmax does not depend on m (App. A.1.3 subtracts the row maximum for the same reason).
    auto softmax_block = [&](AFrag (&a)[RB]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            float x[16];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[2 * e] = bf16_lo_to_f32(a[rb].v[0][e]);
                x[2 * e + 1] = bf16_hi_to_f32(a[rb].v[0][e]);
                x[8 + 2 * e] = bf16_lo_to_f32(a[rb].v[1][e]);
                x[8 + 2 * e + 1] = bf16_hi_to_f32(a[rb].v[1][e]);
            }
            float bm = fmaxf(x[0], x[1]);
#pragma unroll
            for (int e = 2; e < 16; e += 2) bm = fmaxf(fmaxf(x[e], x[e + 1]), bm);   // this lane's 16 scores
            // (m_run = -inf, the start: any finite score is above -inf + kTau = -inf)
            if (__builtin_amdgcn_ballot_w64(bm > m_run[rb] + kTau) != 0) {   // rare after the first blocks
                bm = fmaxf(bm, __shfl_xor(bm, 16, kWave));
                bm = fmaxf(bm, __shfl_xor(bm, 32, kWave));   // maximum of row li over the block's 64 kept scores
                const bool up = bm > m_run[rb] + kTau;       // (the same in the four lanes of a row)
                // (a row still at -inf gets the factor 0: its sums are 0 anyway)
                const float f = up ? __builtin_amdgcn_exp2f((m_run[rb] - bm) * kLog2e) : 1.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float fr = __shfl(f, 4 * kb + r, kWave);   // accumulator row 4 kb + r
                    acc_l[rb][r] *= fr;
#pragma unroll
                    for (int ds = 0; ds < DS; ++ds) acc[rb][ds][r] *= fr;
                }
                if (up) m_run[rb] = bm;
            }
            // a row whose keys so far are all masked (-inf): subtract 0, its weights are exp(-inf) = 0
            const float mb = m_run[rb] == -INFINITY ? 0.f : m_run[rb] * kLog2e;
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], kLog2e, -mb));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[rb].v[0][e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
                a[rb].v[1][e] = pack_bf16x2(x[8 + 2 * e], x[8 + 2 * e + 1]);
            }
        }
    };

    // The A operand is loaded two blocks ahead: block jb + 1 is in registers while block jb is multiplied, so that the
    // softmax of block jb + 1 runs on the vector unit under the matrix instructions of block jb.
    // Order of the blocks: workgroup g starts at block g mod nblocks and wraps around (neither the product nor the
    // softmax with its running reference depends on the order).  The rows of P are a power of two apart for the usual
    // lengths, so that workgroups marching from block 0 in step would all read the same few memory channels at a time.
    const int rot = __builtin_amdgcn_readfirstlane((int)(item % (unsigned)nblocks));
    auto blk = [&](int it) { return it + rot < nblocks ? it + rot : it + rot - nblocks; };
    issue_block(blk(0), 0);
    AFrag a_cur[RB], a_nxt[RB], a_far[RB];
    load_a(blk(0), a_cur);
    if (nblocks > 1) load_a(blk(1), a_nxt);
    if constexpr (SOFTMAX) softmax_block(a_cur);

    Pace<PACED> pace(nblocks);
    for (int jb = 0; jb < nblocks; ++jb) {   // jb: place in the order
        pace.at(nblocks - jb);
        const int buf = jb & 1;
        wait_async_copies();  // vmcnt(0): this block's V copies and the A loads of the next block are in
        __syncthreads();
        if (jb + 1 < nblocks) issue_block(blk(jb + 1), buf ^ 1);
        if (jb + 2 < nblocks) load_a(blk(jb + 2), a_far);
        const char *vbase = reinterpret_cast<const char *>(&Vs[buf][0]);
        auto tr = [&](int key0, int ds) {
            const int row = key0 + tr_row;
            const int chunk = (2 * ds + tr_sub) ^ v_swizzle(row);
            return lds_read_tr16(vbase + (row * CPR + chunk) * 16 + tr_byte);
        };
        if constexpr (SPARSE) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k0 = 32 * (kb >> 1) + 16 * h + 8 * (kb & 1);
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) {
                    const s16x4 t0 = tr(k0, ds), t1 = tr(k0 + 4, ds), t2 = tr(64 + k0, ds), t3 = tr(64 + k0 + 4, ds);
                    const s16x8 lo = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
                    const s16x8 hi = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
                    const bf16x16 b = __builtin_bit_cast(
                        bf16x16, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15));
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const bf16x8 a = __builtin_bit_cast(bf16x8, a_cur[rb].v[h]);
                        if (h == 0)
                            acc[rb][ds] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a, b, acc[rb][ds],
                                                                                    (int)a_cur[rb].idx, 0, 0);
                        else
                            acc[rb][ds] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(a, b, acc[rb][ds],
                                                                                    (int)a_cur[rb].idx, 0, 1);
                    }
                }
                if constexpr (SOFTMAX) {   // row sums of the (rounded) weights
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const bf16x8 a = __builtin_bit_cast(bf16x8, a_cur[rb].v[h]);
                        // (against ones the positions do not matter: the dense instruction, 32 "keys" per row)
                        acc_l[rb] = mfma16(a, ones8, acc_l[rb]);
                    }
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int k0 = 32 * m + 8 * kb;
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) {
                    const s16x4 t0 = tr(k0, ds), t1 = tr(k0 + 4, ds);
                    const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb][ds] = mfma16(__builtin_bit_cast(bf16x8, a_cur[rb].v[m]), b, acc[rb][ds]);
                }
            }
        }
        if (jb + 1 < nblocks) {
            if constexpr (SOFTMAX) softmax_block(a_nxt);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) a_cur[rb] = a_nxt[rb], a_nxt[rb] = a_far[rb];
        }
    }

    // acc[rb][ds][r] = O[q][16 ds + li], q = 16 (rb0 + rb) + 4 kb + r
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int qrow = (rb0 + rb) * 16 + 4 * kb + r;
            if (UNPADDED && qrow >= LqR) continue;
            const size_t q = (size_t)bh * LqR + qrow;
            const float ir = SOFTMAX ? 1.0f / acc_l[rb][r] : 1.f;   // (the sum of row 4 kb + r, in every column)
#pragma unroll
            for (int ds = 0; ds < DS; ++ds)
                O[q * D + 16 * ds + li] = (uint16_t)(pack_bf16x2(SOFTMAX ? acc[rb][ds][r] * ir : acc[rb][ds][r], 0.f) & 0xFFFFu);
        }
    }
}

// O = A_sparse V from compressed weights.  Bound by the stream of kept weights (1.125 bytes per score, read once): little
// arithmetic per byte, so what counts is that the loads cost few cycles and that enough of them are in flight.
// The weights of a wave's rows come by asynchronous copies, whole 128-byte lines, into LDS of the wave's own; there every lane
// picks up its row.  Loaded by the lane that needs them, one row per lane, an instruction takes 64 address cycles instead
// of 16, and the address unit was busy 75 % of the time (4096 x 4096, 24 heads).  As soon as a block's weights are in registers the
// copies of the block PD further on are issued into their place.  Before (register loads; pairs of blocks where the weights
// exceed the cache) and now, us, the call over and over: d = 64, 24 heads x 4096 x 4096 100 -> 89 (403 MB of weights, 5.1 TB/s with
// the codes), 24 x 4000 x 4000 118 -> 89, 24 x 1024 x 1024 9.4 -> 7.5, 192 x 512 x 512 15.6 -> 13.7; d = 128, 64 x 2048 x 2048 87.6 ->
// 83.3, 24 x 2048 x 2048 39.0 -> 27.1, 64 x 512 x 512 9.9 -> 8.5.
// V comes out of the L2 for every workgroup, one block ahead.  The workgroups start at different blocks and wrap around: the
// rows of P are a power of two apart for the usual lengths, and workgroups in step would read the same few memory
// channels at a time.  At d = 64 four neighbours start together and share V blocks; at d = 128 every one starts on its own.
// (Two blocks of weights ahead at d = 64 on such grids: 102 us instead of 89, as two workgroups per compute unit are left of three; a wave
// of its own for V, 64 keys at a time, in front of two blocks of weights: 111.)
// VB: V buffers, one if there is one block of keys.
// PACED: the workgroups of a compute unit keep level (Pace).
template <int D, int RB, int NW, int PD, bool UNPADDED, int VB = 2, bool PACED = true>
__global__ __launch_bounds__(64 * NW, D == 128 ? 2 : VB == 1 ? 5 : NW == 8 ? 4 : 3) void k_spmm(
    const uint32_t *__restrict__ P, const uint32_t *__restrict__ meta, const __bf16 *__restrict__ V, int Lq, int Lk, int LqR, int LkR,
    uint16_t *__restrict__ O) {
    constexpr int THREADS = 64 * NW;
    constexpr int CPR = D / 8;              // 16-byte chunks per V row
    constexpr int TILE = KB * CPR;          // chunks per V block
    constexpr int LPT = TILE / THREADS;     // copies per thread and V block
    constexpr int DS = D / 16;              // 16-column output tiles
    constexpr int TQ = 16 * RB * NW;        // queries per workgroup
    constexpr int PT = 16 * RB * 8;         // chunks of a wave's kept weights of one block (128 bytes per row)
    constexpr int PL = PT / 64;             // copies per thread for them
    constexpr bool CODES_LDS = PD > 1;      // (with one block in flight every wait is for everything, and the codes come in registers)
    constexpr int CT = CODES_LDS ? 16 * RB : 0;   // chunks of their codes
    __shared__ u32x4 Vs[VB][TILE], Ps[NW][PD][PT + CT];

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15, kb = l >> 4;

    const unsigned qtiles = (Lq + TQ - 1) / TQ;
    const unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int qt = item % qtiles;
    const int bh = item / qtiles;
    const int rb0 = (qt * TQ >> 4) + w * RB;   // first 16-row block of this wave
    const int rbp = rb0 * 16 < Lq ? rb0 : Lq / 16 - RB;   // (a wave past the last query reads the last rows and stores nothing)
    const int nblocks = Lk / KB;
    const int meta_slot = ((kb & 1) << 1) | (kb >> 1);   // where the word of 32-key chunk kb sits in a row's 16 bytes

    // LDS position p (16-byte units) = row * CPR + (c ^ v_swizzle(row)) holds chunk c of key `row` (the pattern of k_av)
    auto v_swizzle = [](int row) { return CPR == 16 ? (row & 3) << 1 : tr_row_swizzle<CPR>(row); };
    int v_row[LPT], v_chunk[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int p = i * THREADS + tid;
        v_row[i] = p / CPR;
        v_chunk[i] = ((p % CPR) ^ v_swizzle(v_row[i])) * 8;
    }
    const uint32_t lds_v = lds_address(&Vs[0][w * 64]);   // this wave's 1 KB slice of copy 0, buffer 0
    const uint32_t lds_p = lds_address(&Ps[w][0][0]);
    const uint64_t v_base = uniform_address(V + (size_t)bh * LkR * D);
    auto issue_v = [&](int jb, int buf) {
        const uint64_t src = v_base + (uint64_t)jb * (KB * D * 2);
        const int last = UNPADDED ? LkR - jb * KB - 1 : KB - 1;   // the block's last real key
#pragma unroll
        for (int i = 0; i < LPT; ++i)
            async_copy16(src, 2u * ((UNPADDED && v_row[i] > last ? last : v_row[i]) * D + v_chunk[i]), lds_v + 16u * (buf * TILE + i * THREADS));
    };
    // The wave's kept weights of a block: row r, chunk c (keys 16 c .. +15) at r * 8 + (c ^ ((r >> 1) & 7)); copy i brings rows
    // 8 i .. +7, for which the pattern is that of copy i % 2.  (Two lanes meet in every group of banks of the reads below; so do lane
    // groups of V's at d = 128: conflicts in 17 and 50 % of the LDS cycles.  LDS does not bound the kernel: with chunk c at ((c >> 1) | (c & 1) << 2) ^
    // (r & 7), free of conflicts, 23 shapes were level at d = 64 and up to 2.5 % slower at d = 128 (8 x 2048 x 2048 16.3 and 16.7 us), with V by
    // tr_row_swizzle in addition up to 4.7 % (64 x 512 x 512 8.5 and 8.8).)
    const uint64_t p_base = uniform_address(P + ((size_t)bh * Lq + (size_t)rbp * 16) * (size_t)(Lk / 4));
    const uint32_t p_off = (uint32_t)(l >> 3) * (uint32_t)Lk + 16u * ((l & 7) ^ (l >> 4));
    const uint32_t *const m_row = meta + (((size_t)bh * (Lq / 16) + rbp) * nblocks * 16 + li) * 4 + meta_slot;
    const uint64_t c_base = uniform_address(meta + (((size_t)bh * (Lq / 16) + rbp) * nblocks * 16) * 4);
    constexpr int P_LOADS = PL + 1;         // (CODES_LDS)
    uint32_t codes[RB];
    auto issue_p = [&](int jb, int buf) {
        const uint64_t src = p_base + (uint64_t)jb * 128u;
#pragma unroll
        for (int i = 0; i < PL; ++i)
            async_copy16(src + (uint64_t)(8 * i) * (uint64_t)Lk, i & 1 ? p_off ^ 64u : p_off, lds_p + 16u * (buf * (PT + CT) + i * 64));
        if constexpr (CODES_LDS) {
            if (l < 16 * RB)
                async_copy16(c_base + (uint64_t)jb * 256u, (uint32_t)(l >> 4) * nblocks * 256u + 16u * (l & 15), lds_p + 16u * (buf * (PT + CT) + PT));
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) codes[rb] = m_row[((size_t)rb * nblocks + jb) * 64];
        }
    };

    const int rot = __builtin_amdgcn_readfirstlane((int)((D == 64 ? item / 4 : item) % (unsigned)nblocks));
    auto blk = [&](int it) { return it + rot < nblocks ? it + rot : it + rot - nblocks; };
    issue_v(blk(0), 0);
    issue_p(blk(0), 0);
    if (PD == 2 && nblocks > 1) issue_p(blk(1), 1);

    f32x4 acc[RB][DS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) acc[rb][ds] = f32x4{0.f, 0.f, 0.f, 0.f};

    // transposing read: lane li of a 16-lane group addresses V[key0 + li/4][col0 + 4*(li%4)]
    const int tr_row = li >> 2, tr_sub = (li >> 1) & 1, tr_byte = 8 * (li & 1);

    // block `it` in the order of visits; buf: its V buffer
    auto block = [&](auto parity, int it) {
        constexpr int buf = decltype(parity)::value;
        constexpr int pb = PD == 2 ? buf : 0;
        // V and the weights of this block are in (PD = 2: the weights of the next one, issued after this V, stay in flight)
        if (PD == 2 && it + 1 < nblocks) wait_async_copies_keep<P_LOADS>();
        else wait_async_copies();
        __syncthreads();
        u32x4 a[RB][2];
        uint32_t idx[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if constexpr (CODES_LDS) idx[rb] = reinterpret_cast<const uint32_t *>(&Ps[w][pb][PT + 16 * rb + li])[meta_slot];
            else idx[rb] = codes[rb];
#pragma unroll
            for (int h = 0; h < 2; ++h) a[rb][h] = Ps[w][pb][(16 * rb + li) * 8 + ((2 * kb + h) ^ ((li >> 1) & 7))];
        }
        if (VB == 2 && it + 1 < nblocks) issue_v(blk(it + 1), buf ^ 1);
        // (the weights have to be in registers before their place is given to the next ones)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) asm volatile("" : "+v"(a[rb][0]), "+v"(a[rb][1]), "+v"(idx[rb]) : : "memory");
        if (it + PD < nblocks) issue_p(blk(it + PD), pb);
        const char *vbase = reinterpret_cast<const char *>(&Vs[buf][0]);
        auto tr = [&](int key0, int ds) {
            const int row = key0 + tr_row;
            return lds_read_tr16(vbase + (row * CPR + ((2 * ds + tr_sub) ^ v_swizzle(row))) * 16 + tr_byte);
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k0 = 32 * (kb >> 1) + 16 * h + 8 * (kb & 1);
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) {
                const s16x4 t0 = tr(k0, ds), t1 = tr(k0 + 4, ds), t2 = tr(64 + k0, ds), t3 = tr(64 + k0 + 4, ds);
                const s16x8 lo = __builtin_shufflevector(t0, t1, 0, 1, 2, 3, 4, 5, 6, 7);
                const s16x8 hi = __builtin_shufflevector(t2, t3, 0, 1, 2, 3, 4, 5, 6, 7);
                const bf16x16 b = __builtin_bit_cast(
                    bf16x16, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const bf16x8 x = __builtin_bit_cast(bf16x8, a[rb][h]);
                    if (h == 0) acc[rb][ds] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(x, b, acc[rb][ds], (int)idx[rb], 0, 0);
                    else acc[rb][ds] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(x, b, acc[rb][ds], (int)idx[rb], 0, 1);
                }
            }
        }
    };
    Pace<PACED> pace(nblocks);
    for (int it = 0; it < nblocks; it += 2) {
        pace.at(nblocks - it);
        block(std::integral_constant<int, 0>{}, it);
        if constexpr (VB == 1) break;
        else if (it + 1 < nblocks) block(std::integral_constant<int, 1>{}, it + 1);
    }

    // acc[rb][ds][r] = O[q][16 ds + li], q = 16 (rb0 + rb) + 4 kb + r
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int qrow = (rb0 + rb) * 16 + 4 * kb + r;
            if (qrow >= LqR) continue;
            const size_t q = (size_t)bh * LqR + qrow;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds)
                O[q * D + 16 * ds + li] = (uint16_t)(pack_bf16x2(acc[rb][ds][r], 0.f) & 0xFFFFu);
        }
}

template <bool SPARSE>
hipError_t launch_av(const void *P, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d,
                  void *O, hipStream_t st) {
    if (LqR != Lq || LkR != Lk) {   // unpadded lengths: 64-query workgroups (Lq is a multiple of 64)
        const unsigned grid = (unsigned)((long)BH * (Lq / 64));
        const bool paced = SPARSE && keep_level(grid, d == 64 ? 4 : 2, Lk);
#define DFSS_LAUNCH(DD, PP)                                                                                         \
    hipLaunchKernelGGL((k_av<DD, SPARSE, 1, true, SPARSE && PP>), dim3(grid), dim3(NT), 0, st, (const uint32_t *)P, \
                       (const uint32_t *)meta, (const __bf16 *)V, Lq, Lk, LqR, LkR, (uint16_t *)O)
        if (d == 64) {
            if (paced) DFSS_LAUNCH(64, true); else DFSS_LAUNCH(64, false);
        } else {
            if (paced) DFSS_LAUNCH(128, true); else DFSS_LAUNCH(128, false);
        }
#undef DFSS_LAUNCH
        return hipGetLastError();
    }
    // two row blocks per wave when that still leaves two workgroups per compute unit (measured:
    // from there on the larger tile wins, below it the finer grid does)
    bool rb2 = (Lq % 128 == 0) && ((long)BH * (Lq / 128) >= 512);
    const unsigned grid = (unsigned)((long)BH * (Lq / (rb2 ? 128 : 64)));
    const bool paced = SPARSE && keep_level(grid, d == 128 ? 2 : rb2 ? 3 : 5, Lk);
#define DFSS_LAUNCH_P(DD, RR, PP)                                                                             \
    hipLaunchKernelGGL((k_av<DD, SPARSE, RR, false, SPARSE && PP>), dim3(grid), dim3(NT), 0, st, (const uint32_t *)P, \
                       (const uint32_t *)meta, (const __bf16 *)V, Lq, Lk, Lq, Lk, (uint16_t *)O)
#define DFSS_LAUNCH(DD, RR)                    \
    do {                                       \
        if (paced) DFSS_LAUNCH_P(DD, RR, true); \
        else DFSS_LAUNCH_P(DD, RR, false);     \
    } while (0)
    if (d == 64) {
        if (rb2) DFSS_LAUNCH(64, 2); else DFSS_LAUNCH(64, 1);
    } else {
        if (rb2) DFSS_LAUNCH(128, 2); else DFSS_LAUNCH(128, 1);
    }
#undef DFSS_LAUNCH_P
#undef DFSS_LAUNCH
    return hipGetLastError();
}

// The product on kept weights.  Queries per workgroup, measured over 40 shapes (us):
//   64 where 128-query workgroups would not fill the chip.  d = 64, three of those per compute unit at most: up to 511 of them
//     (384 of them, 24 heads x 2048 x 2048: 19.8 against 19.9; 256, 32 x 1024 x 1024: 9.2 against 10.3; 768 of them, 24 x
//     4096 x 4096: 120 against 89).  d = 128: up to 256 workgroups of 64 queries (12 x 1024 x 1024 9.7 against 11.2; with 384, 48 x
//     512 x 512 8.2 against 7.9)
//   256, eight waves, at d = 64 where 128-query workgroups would be more than the three per compute unit that fit and the larger
//     ones all fit at once (64 x 2048 x 2048 59.5 against 76.1, 224 x 512 x 512 16.1 against 16.9, 80 x 2048 x 2048, too many, 96.7
//     against 88.7, 512 x 256 x 256 13.6 against 13.1)
//   256 at d = 128 on long sequences: V is read half as often and there is room for two blocks of weights in
//     flight; from a workgroup per compute unit on (32 x 2048 x 2048 31.0 against 33.5, 64 x 2048 x 2048 83.3 against 88.0; 24 x
//     2048 x 2048 28.1 against 27.1) and 16 blocks of keys on (64 x 1024 x 1024 20.9 against 19.7)
// A larger tile only if not more than an eighth is added to the queries.
// d = 64, one workgroup of 64 queries per compute unit, weights that exceed the L2s (8 x 4 MB) and so come from further away: two
//   blocks of them in flight, for which there is room (4 x 4096 x 4096 21.7 -> 18.1 us, 8 x 2048 x 2048 12.4 -> 10.7; 6 x 2048 x 2048, 24 MB, level; 16 x
//   1024 x 1024, 16 MB, 6.5 against 6.6)
hipError_t launch_sparse(const void *P, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d,
                         void *O, hipStream_t st) {
    const bool unp = LqR != Lq || LkR != Lk;
    auto tiles = [&](int tq) { return (Lq + tq - 1) / tq; };
    auto fits = [&](int tq) { return 8 * (tiles(tq) * tq - Lq) <= Lq; };
    int tq = 64;
    if (fits(128) && (d == 64 ? (long)BH * tiles(128) >= 512 : (long)BH * tiles(64) > 256)) tq = 128;
    if (fits(256) && (d == 64 ? Lk >= 512 && (long)BH * tiles(128) > 768 && (long)BH * tiles(256) <= 512 : Lk >= 2048 && (long)BH * tiles(256) >= 256))
        tq = 256;
    const unsigned grid = (unsigned)((long)BH * tiles(tq));
    // Workgroups keep level where there are more of them than compute units (us, without and with: d = 64 24 x 2048 x 2048 20.9 and 19.6, 24 x
    // 4096 x 4096 92.0 and 89.3; d = 128 96 x 512 x 512 12.0 and 11.3, 64 x 1024 x 1024 20.2 and 19.6; 192 x 512 x 512 13.6 and 13.9, the other way).
    // Up to one per compute unit they only lose by it (2 x 4096 x 4096 17.4 and 17.7, d = 128 4 x 4096 x 4096 28.5 and 28.9, 12 x 1024 x 1024 9.4 and 9.5).
    const bool alone = grid <= 256;
#define DFSS_LAUNCH(DD, RR, WW, PP, VV, LL)                                                                           \
    do {                                                                                                              \
        if (unp)                                                                                                      \
            hipLaunchKernelGGL((k_spmm<DD, RR, WW, PP, true, VV, LL>), dim3(grid), dim3(64 * WW), 0, st, (const uint32_t *)P, \
                               (const uint32_t *)meta, (const __bf16 *)V, Lq, Lk, LqR, LkR, (uint16_t *)O);           \
        else                                                                                                          \
            hipLaunchKernelGGL((k_spmm<DD, RR, WW, PP, false, VV, LL>), dim3(grid), dim3(64 * WW), 0, st, (const uint32_t *)P, \
                               (const uint32_t *)meta, (const __bf16 *)V, Lq, Lk, LqR, LkR, (uint16_t *)O);           \
    } while (0)
    if (d == 64) {
        if (tq == 64 && alone && (long)BH * Lq * Lk >= (1l << 25)) DFSS_LAUNCH(64, 1, 4, 2, 2, false);
        else if (tq == 64 && alone) DFSS_LAUNCH(64, 1, 4, 1, 2, false);
        else if (tq == 64) DFSS_LAUNCH(64, 1, 4, 1, 2, true);
        else if (tq == 256) DFSS_LAUNCH(64, 2, 8, 1, 2, true);
        else if (Lk == KB) DFSS_LAUNCH(64, 2, 4, 1, 1, true);   // more workgroups at a time (1024 heads x 128 x 128 10.4 -> 9.7 us)
        else DFSS_LAUNCH(64, 2, 4, 1, 2, true);
    } else {
        if (tq == 64 && alone) DFSS_LAUNCH(128, 1, 4, 1, 2, false);
        else if (tq == 64) DFSS_LAUNCH(128, 1, 4, 1, 2, true);
        else if (tq == 128) DFSS_LAUNCH(128, 2, 4, 1, 2, true);
        else DFSS_LAUNCH(128, 2, 8, 2, 2, true);
    }
#undef DFSS_LAUNCH
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spmm(const void *vals, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d,
                       void *O, hipStream_t st) {
    return launch_sparse(vals, meta, V, BH, Lq, Lk, LqR, LkR, d, O, st);
}

hipError_t launch_softmax_spmm(const void *scores, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR,
                               int LkR, int d, void *O, hipStream_t st) {
    return launch_av<true>(scores, meta, V, BH, Lq, Lk, LqR, LkR, d, O, st);
}

hipError_t launch_dense_av(const void *P, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d, void *O,
                           hipStream_t st) {
    return launch_av<false>(P, nullptr, V, BH, Lq, Lk, LqR, LkR, d, O, st);
}

}  // namespace dfss
