// fp32-throughout variants of the two operations (for fp32 inputs), on the fp32 matrix instructions (gfx950):
//   out = softmax(q k^T * sm_scale) v + g * L2Norm(q) S             paper Eq. (2), (3), (5), (6)
//   S  <- gate * S + sum_i L2Norm(k_i)^T v_i                        paper Eq. (3), Eq. (4)
// v_mfma_f32_32x32x2_f32 and 16x16x4_f32 multiply and accumulate in fp32, so no step has reduced precision; exponentials are
// v_exp_f32 on arguments rounded once, with the rounding of the scale's factor made good (`pow2_diff`).
#include "arl2_device.h"

#include <math.h>

namespace arl2 {
namespace {

typedef __attribute__((address_space(3))) void lds_void;

// ---- readout ---------------------------------------------------------------------------------------
// Bound by the fp32 matrix rate (a 32 x 32 x 2 step takes 64 cycles for one dword per lane of each operand, so
// LDS and L2 have time to spare) and by the vector work, which never runs beside it on a SIMD.  One workgroup owns 32 or
// 16 (QW) query rows of one (stream, head); its four wavefronts share the rows and take every fourth block of 32 keys, each
// with a running maximum, row sum and O of its own that are merged at the end.  Keys are split inside the workgroup because
// fp32 problems have few rows: wavefronts without the split leave most SIMDs of the chip empty.  Tiles of 16 rows serve what
// is left beyond a multiple of one 32-row tile per CU (`launch_fwd_f32`).
//   S^T[key][q] = K Q^T    A = K rows from LDS, 16 bytes (four steps) per read;  B = q in registers
//   O^T[d][q]  += V^T P^T  A = V straight from global memory (a step reads row pieces of 4 QW bytes);
//                          B = the accumulator registers of S^T as they are: with lanes in 64 / QW groups gr, register r of
//                          a group is key (256 / QW) (r / 4) + 4 gr + r % 4, and that key's row of V is what the lane loads.
// A wavefront's K block travels straight from global memory to its own 32 rows of LDS (no registers, no barrier:
// nobody else reads it), requested while the second product of the block before it runs.  The rows are not padded
// (the direct load writes 16 bytes per lane in lane order); instead the lane at chunk j of row r loads chunk
// j ^ r, so that the rows a fragment read touches lie on different banks.
// The products of a row with a key or with the state are summed in several chains that are added at the end: one chain of
// D products is the larger error of the two that an output has (relative to 64 bits, two chains for the state: 2.14e-7 ->
// 1.57e-7 at D = 128; logits of +-20, chains of 16 products at D = 128 and two chains at D = 64: 1.11e-6 -> 4.4e-7 and
// 8.1e-7 -> 5.2e-7; a vector-ALU kernel with 16 lanes per row has 2.09e-7, 7.8e-7 and 7.9e-7).
// Measured, 12 heads x 128, 1560 tokens (15.7 GFLOP, 102 us at the 154 TFLOP/s that a large fp32 matrix product
// reaches): 156 us; 193 us with tiles of 32 rows only (588 of them: a third tile on 76 of the 256 CUs) and the library's
// expf (12 instructions per logit, 3 now); 7160 us on the vector ALU, 16 lanes per query row and two passes over the keys.
// 4 heads x 128, 500 tokens: 18 us, 30 us with 64 tiles of 32 rows; 2 heads x 64, 64 tokens: 7.2 us and 8.7 us.
// Error against 64 bits as with expf (1.57e-7 at usual logits, both), lower where logits are large at D = 64.
template <int D, int QW>
struct F32Cfg {
    static constexpr int NW = 4;                     // wavefronts = key groups
    static constexpr int NG = 64 / QW;               // lane groups: the contraction steps of one matrix instruction
    static constexpr int FPT = 4 * NG;               // features (or keys) that the groups hold four of each
    static constexpr int KT = D / FPT;               // 16-byte pieces of a row per lane
    static constexpr int NQ = 32 / FPT;              // quads of keys of a block per lane: it holds 4 NQ logits
    static constexpr int DB = D / QW;                // QW-feature blocks
    static constexpr int RPB = QW * QW / 64;         // accumulator registers of a block
    static constexpr int BPW = DB > NW ? DB / NW : 1;   // blocks of the output that a wavefront finishes
    static constexpr int KBUF = 32 * D * 4;          // bytes of a K block
    static constexpr int SMEM = NW * KBUF;           // also holds the four wavefronts' O
    static_assert(NW * DB * RPB * 64 * 4 <= SMEM, "the partial outputs pass through the K blocks");
};

template <int N>
__device__ __forceinline__ float group_sum(float x)
{
    if constexpr (N == 4) x += __shfl_xor(x, 16, kWave);
    return xhalf_sum(x);
}
template <int N>
__device__ __forceinline__ float group_max(float x)
{
    if constexpr (N == 4) x = fmaxf(x, __shfl_xor(x, 16, kWave));
    return xhalf_max(x);
}
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// exp of a difference of scaled logits d <= 0, which comes in powers of two: `err` is by how much of itself the scale's factor
// sm_scale log2(e) falls short (never zero or negative, so that -inf stays -inf).
__device__ __forceinline__ float pow2_diff(float d, float err) { return __builtin_amdgcn_exp2f(fmaf(d, err, d)); }

// Query rows q0 .. q0 + QW - 1 of (stream, head) bh.  x2: sm_scale log2(e) rounded towards zero, and what it falls short.
template <int D, int QW>
__device__ __forceinline__ void fwd_f32_tile(const FwdArgs &a, f32x2 x2, int bh, int q0, unsigned char *smem, float (*ml)[2][32])
{
    using C = F32Cfg<D, QW>;
    typedef float acc_t __attribute__((ext_vector_type(C::RPB)));
    constexpr int KT = C::KT, DB = C::DB, NW = C::NW, NG = C::NG, FPT = C::FPT, KBUF = C::KBUF;
    constexpr int NS = QW == 32 ? 1 : 2;      // accumulator blocks of S^T: 32 or 2 x 16 keys
    constexpr int CPR = D / 4;                // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;             // rows per direct load

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, gr = lane / QW, c = lane % QW;
    const int H = a.H, Lq = a.Lq, Lkv = a.Lkv;
    const int h = bh % H, b = bh / H;
    const int row = q0 + c;
    const bool valid = row < Lq;
    const uint32_t tok = (uint32_t)H * D * 4;                       // bytes of one token, all heads
    const size_t row_off = (((size_t)b * Lq + (valid ? row : q0)) * H + h) * D;
    const float *kg = (const float *)a.k + ((size_t)b * Lkv * H + h) * D;
    const float *vg = (const float *)a.v + ((size_t)b * Lkv * H + h) * D;

    // B operand of S^T: lane (row c, gr) holds features FPT t + 4 gr + 0..3 of its row
    f32x4 q[KT];
    auto load_q = [&](const float *src) {
        f32x4 ss = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            q[t] = *(const f32x4 *)(src + row_off + FPT * t + 4 * gr);
#pragma unroll
            for (int j = 0; j < 4; ++j) ss[j] = fmaf(q[t][j], q[t][j], ss[j]);
        }
        return group_sum<NG>((ss[0] + ss[1]) + (ss[2] + ss[3]));
    };
    float qss = load_q((const float *)a.q);

    // Buffer descriptors are rebuilt per block from 64-bit bases, so that 32-bit offsets only span 32 rows; rows past
    // the last key read as zero.
    const int nblk = (Lkv + 31) / 32;
    auto rsrc_of = [&](const float *base, int blk) {
        const int rows = Lkv - 32 * blk < 32 ? Lkv - 32 * blk : 32;
        return make_rsrc((const char *)base + (size_t)blk * 32 * tok, (uint32_t)(rows - 1) * tok + 4 * D);
    };
    unsigned char *kbuf = smem + wave * KBUF;
    auto fetch_k = [&](int blk) {
        const __amdgpu_buffer_rsrc_t r = rsrc_of(kg, blk);
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int kr = RPI * i + lane / CPR;
            const uint32_t off = (uint32_t)kr * tok + 16 * ((lane % CPR) ^ (kr % CPR));
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)(kbuf + 1024 * i), 16, (int)off, 0, 0, 0);
        }
    };
    // A operand of S^T: features FPT t + 4 gr + 0..3 of key 16 kb + c (QW = 16) or c
    auto k_piece = [&](int kb, int t) -> f32x4 {
        const int kr = 16 * kb + c;
        return *(const f32x4 *)(kbuf + kr * (D * 4) + 16 * ((NG * t + gr) ^ (kr % CPR)));
    };
    float vr[2][4][DB];                       // V rows of four logits, current and next
    uint32_t v_off;                           // of this lane in the block's first row: 4 gr tokens and 4 c bytes
    auto fetch_v = [&](__amdgpu_buffer_rsrc_t r, auto quad_) {
        constexpr int quad = decltype(quad_)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                vr[quad & 1][j][db] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(r, v_off + (uint32_t)(FPT * quad + j) * tok + 4 * QW * db, 0, 0));
    };

    acc_t o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = acc_t(0.f);
    // running maximum of the scaled logits, in powers of two (finite also while every logit was -inf); this lane's share of
    // the row sum
    float m = -FLT_MAX, l = 0.f;

    if (wave < nblk) fetch_k(wave);
#pragma unroll 1
    for (int blk = wave; blk < nblk; blk += NW) {
        const __amdgpu_buffer_rsrc_t v_rsrc = rsrc_of(vg, blk);
        v_off = 4 * gr * tok + 4 * c;
        asm volatile("" : "+v"(v_off));       // (one offset and not sixteen kept over the loop)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // the K block has landed
        fetch_v(v_rsrc, std::integral_constant<int, 0>{});
        acc_t sa[NS];
        if constexpr (D == 64 && QW == 32) {                        // even and odd steps
            acc_t s0 = acc_t(0.f), s1 = acc_t(0.f);
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const f32x4 ka = k_piece(0, t);
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    s0 = mfma_f32(ka[j], q[t][j], s0);
                    s1 = mfma_f32(ka[j + 1], q[t][j + 1], s1);
                }
            }
            sa[0] = s0 + s1;
        } else {                                                    // sixteen products from zero, added up while the next sixteen run
            constexpr int TPC = 4 / NG;                             // pieces per chain
            acc_t sum1[NS];
            static_for<0, KT / TPC + 1>([&](auto g_) {
                constexpr int g = decltype(g_)::value;
                acc_t done[NS];
                if constexpr (g > 0)
                    static_for<0, NS>([&](auto kb_) { done[decltype(kb_)::value] = sum1[decltype(kb_)::value]; });
                if constexpr (g < KT / TPC) {
                    static_for<0, NS>([&](auto kb_) { sum1[decltype(kb_)::value] = acc_t(0.f); });
                    static_for<TPC * g, TPC * g + TPC>([&](auto t_) {
                        constexpr int t = decltype(t_)::value;
                        f32x4 ka[NS];
                        static_for<0, NS>([&](auto kb_) { ka[decltype(kb_)::value] = k_piece(decltype(kb_)::value, t); });
                        static_for<0, 4 * NS>([&](auto j_) {
                            constexpr int j = decltype(j_)::value / NS, kb = decltype(j_)::value % NS;
                            sum1[kb] = mfma_f32(ka[kb][j], q[t][j], sum1[kb]);
                        });
                    });
                }
                if constexpr (g > 0)
                    static_for<0, NS>([&](auto kb_) {
                        constexpr int kb = decltype(kb_)::value;
                        if constexpr (g == 1) sa[kb] = done[kb];
                        else sa[kb] += done[kb];
                        asm volatile("" : "+v"(sa[kb]));            // (otherwise all sums are kept and added at the end)
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the K block has been read: it may be overwritten
        if (blk + NW < nblk) fetch_k(blk + NW);

        // logit i of a lane is key FPT (i / 4) + 4 gr + i % 4 of the block
        constexpr int NL = 4 * C::NQ;
        float s[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) s[i] = sa[i / C::RPB][i % C::RPB];
        if (32 * blk + 32 > Lkv) {                                  // keys past the end (last block only)
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (32 * blk + FPT * (i >> 2) + 4 * gr + (i & 3) >= Lkv) s[i] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < NL; ++i) mx = fmaxf(mx, s[i]);
        const float m_new = fmaxf(m, group_max<NG>(mx) * x2[0]);
        if (__any(m_new > m)) {
            const float alpha = pow2_diff(m - m_new, x2[1]);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            s[i] = pow2_diff(fmaf(s[i], x2[0], -m), x2[1]);
            l += s[i];
        }
        static_for<0, C::NQ>([&](auto quad_) {
            constexpr int quad = decltype(quad_)::value;
            if constexpr (quad < C::NQ - 1) fetch_v(v_rsrc, std::integral_constant<int, quad + 1>{});
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] = mfma_f32(vr[quad & 1][j][db], s[4 * quad + j], o[db]);
        });
    }

    // ---- merge the four shares: everything relative to the largest maximum
    l = group_sum<NG>(l);
    if (gr == 0) {
        ml[wave][0][c] = m;
        ml[wave][1][c] = l;
    }
    __syncthreads();                                                // also: no K block is read any more
    float m_all = ml[0][0][c];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, ml[w][0][c]);
    float l_all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l_all = fmaf(ml[w][1][c], pow2_diff(ml[w][0][c] - m_all, x2[1]), l_all);
    const float f = pow2_diff(m - m_all, x2[1]);
    float *ox = (float *)smem;                                      // [wavefront][feature block][register][lane]
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < C::RPB; ++r) ox[((wave * DB + db) * C::RPB + r) * 64 + lane] = o[db][r] * f;
    __syncthreads();
    // from here on a wavefront owns BPW blocks of output features
    if (wave * C::BPW >= DB) return;
    if (a.S != nullptr && a.q_lin != nullptr) qss = load_q((const float *)a.q_lin);   // the linear branch's own query (Eq. (3))
    const float rq = 1.0f / sqrtf(qss + a.l2_eps);
    const size_t gtok = (size_t)b * Lq + (valid ? row : q0);
    const size_t gi = a.g_per_token ? gtok : gtok * H + h;
#pragma unroll
    for (int ob = 0; ob < C::BPW; ++ob) {
        const int blk = wave * C::BPW + ob;
        acc_t out;
#pragma unroll
        for (int r = 0; r < C::RPB; ++r) {
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += ox[((w * DB + blk) * C::RPB + r) * 64 + lane];
            out[r] = sum / l_all;
        }
        if (a.S != nullptr) {
            const float *Sg = a.S + (size_t)bh * D * D + QW * blk + c;
            acc_t inter = acc_t(0.f), inter1 = acc_t(0.f);          // even and odd steps
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    inter = mfma_f32(Sg[(FPT * t + 4 * gr + j) * D], q[t][j], inter);
                    inter1 = mfma_f32(Sg[(FPT * t + 4 * gr + j + 1) * D], q[t][j + 1], inter1);
                }
            inter += inter1;
#pragma unroll
            for (int r = 0; r < C::RPB; ++r) {
                float g = 1.0f;                  // headwise or per-token gate, or one gate per output feature
                if (a.g != nullptr) {
                    const size_t ge = a.g_per_element ? gi * D + QW * blk + FPT * (r >> 2) + 4 * gr + (r & 3) : gi;
                    g = a.g_is_bf16 ? (float)((const bf16_t *)a.g)[ge] : ((const float *)a.g)[ge];
                }
                out[r] = fmaf(g, inter[r] * rq, out[r]);
            }
        }
        if (valid) {
            float *og = (float *)a.out + row_off + QW * blk + 4 * gr;
#pragma unroll
            for (int p = 0; p < C::RPB / 4; ++p)
                *(f32x4 *)(og + FPT * p) = f32x4{out[4 * p], out[4 * p + 1], out[4 * p + 2], out[4 * p + 3]};
        }
    }
}

// n_rb 32-row tiles per head, n_tiles in all; the first n_whole are served whole, the others as two tiles of 16 rows.
template <int D>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(FwdArgs a, int n_rb, int n_tiles, int n_whole, float scale_log2, float scale_err)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[F32Cfg<D, 32>::SMEM];
    __shared__ float ml[F32Cfg<D, 32>::NW][2][32];   // maximum and row sum of each wavefront's share, per query row
    int id = blockIdx.x, half = -1;
    if (id >= n_whole) {
        half = (id - n_whole) / (n_tiles - n_whole);
        id = n_whole + (id - n_whole) % (n_tiles - n_whole);
    }
    const int work = xcd_contiguous_id(id, n_tiles);                // the row blocks of a head share an XCD's L2
    const int bh = work / n_rb, q0 = (work % n_rb) * 32;
    const f32x2 x2 = {scale_log2, scale_err};
    if (half < 0) fwd_f32_tile<D, 32>(a, x2, bh, q0, smem, ml);
    else if (q0 + 16 * half < a.Lq) fwd_f32_tile<D, 16>(a, x2, bh, q0 + 16 * half, smem, ml);
}

// ---- commit ----------------------------------------------------------------------------------------
// One workgroup owns a BLK x BLK block of one head's state; its eight wavefronts take every eighth group of 16
// tokens and their sums are added, in order, through LDS.  Both operands of a step (two tokens) are read straight
// from global memory: a lane's feature of the token, 128 contiguous bytes per half-wave.  The rows of a group are
// also read whole for their norms, which scale the value operand; everything a group needs is requested one group
// ahead.  Re-reading the rows per block costs L2 traffic only, and needs neither a pass of its own for the norms nor
// partial sums in memory.
// Measured, 12 heads x 128, 1560 tokens (19 MB): 16 us; one thread per state element walking all tokens, after a
// kernel for the norms, took 572 + 19 us.  2 heads x 64, 64 tokens: 3.7 us against 9.5 + 6.7 us.
template <int D, int BLK>
__global__ __launch_bounds__(512, 2) void commit_f32_kernel(CommitArgs a)
{
    constexpr int NB = BLK / 32;              // 32-wide blocks per side
    constexpr int NBK = D / BLK;              // workgroups per side of a state
    constexpr int NW = 8;
    constexpr int TG = 16;                    // tokens per group
    constexpr int NRM = D / 16;               // 16-byte pieces of a row per lane: four lanes share a row
    __shared__ float red[NW][NB * NB * 16][64];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hh = lane >> 5, c = lane & 31;
    const int H = a.H, L = a.L;
    const int work = xcd_contiguous_id(blockIdx.x, gridDim.x);      // the blocks of a head share an XCD's L2
    const int bh = work / (NBK * NBK), d0 = (work / NBK) % NBK * BLK, e0 = work % NBK * BLK;
    const int h = bh % H, b = bh / H;
    const uint32_t tok = (uint32_t)H * D * 4;
    const float *kg = (const float *)a.k + ((size_t)b * L * H + h) * D;
    const float *vg = (const float *)a.v + ((size_t)b * L * H + h) * D;
    const int ngrp = (L + TG - 1) / TG;

    u32x4 nrm[NRM];
    float kr[TG / 2][NB], vr[TG / 2][NB];
    // descriptors per group, from 64-bit bases (see the readout); a group past the end reads zeros
    auto rsrc_of = [&](const float *base, int grp) {
        const int rows = L - TG * grp < TG ? L - TG * grp : TG;
        return make_rsrc((const char *)base + (size_t)(rows > 0 ? grp : 0) * TG * tok, rows > 0 ? (uint32_t)(rows - 1) * tok + 4 * D : 0u);
    };
    auto fetch = [&](int grp) {
        const __amdgpu_buffer_rsrc_t k_rsrc = rsrc_of(kg, grp), v_rsrc = rsrc_of(vg, grp);
#pragma unroll
        for (int i = 0; i < NRM; ++i)
            nrm[i] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, (uint32_t)(lane >> 2) * tok + 64 * i + 16 * (lane & 3), 0, 0);
#pragma unroll
        for (int t = 0; t < TG / 2; ++t)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const uint32_t off = (uint32_t)(2 * t + hh) * tok + 4 * c + 128 * i;
                kr[t][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(k_rsrc, off + 4 * d0, 0, 0));
                vr[t][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(v_rsrc, off + 4 * e0, 0, 0));
            }
    };
    f32x16 acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    fetch(wave);
#pragma unroll 1
    for (int grp = wave; grp < ngrp; grp += NW) {
        float ss = 0.f;                       // lanes 4 i .. 4 i + 3: token i of the group
#pragma unroll
        for (int i = 0; i < NRM; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = __uint_as_float(nrm[i][j]);
                ss = fmaf(x, x, ss);
            }
        ss += dpp_peek<0xB1>(ss);             // quad_perm [1,0,3,2]
        ss += dpp_peek<0x4E>(ss);             // quad_perm [2,3,0,1]
        const float rn = 1.0f / sqrtf(ss + a.l2_eps);
        float ka[TG / 2][NB], vb[TG / 2][NB];
#pragma unroll
        for (int t = 0; t < TG / 2; ++t) {
            const float r = __shfl(rn, 4 * (2 * t + hh), kWave);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                ka[t][i] = kr[t][i];
                vb[t][i] = vr[t][i] * r;
            }
        }
        fetch(grp + NW);                      // past the end: zeros, unused
#pragma unroll
        for (int t = 0; t < TG / 2; ++t)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[t][i], vb[t][j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[wave][(i * NB + j) * 16 + r][lane] = acc[i][j][r];
    __syncthreads();
    const float gate = a.gate[bh];
#pragma unroll
    for (int x = tid; x < NB * NB * 16 * 64; x += 512) {
        const int ln = x & 63, reg = x >> 6, r = reg & 15, blk = reg >> 4;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += red[w][reg][ln];
        const int d = d0 + 32 * (blk / NB) + 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), e = e0 + 32 * (blk % NB) + (ln & 31);
        float *Sp = a.S + ((size_t)bh * D + d) * D + e;
        *Sp = fmaf(gate, *Sp, sum);
    }
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs &a, hipStream_t stream)
{
    const int n_rb = (a.Lq + 31) / 32;
    const long long n_tiles = (long long)n_rb * a.B * a.H;
    if (n_tiles <= 0 || n_tiles > 0x3fffffffLL) return hipErrorInvalidValue;
    // Tiles beyond a multiple of one per CU are served by two workgroups of 16 rows each while those find a CU of their own:
    // they take half as long.  12 heads x 128, 1560 tokens (588 tiles, 76 beyond) 156 us, 4 heads, 500 tokens (64 tiles) 18 and
    // 30 us, 192 heads, 100 tokens (768 tiles, all whole) 37 us; with more than half of the CUs taken nothing would be shorter.
    const int rest = (int)(n_tiles % kNumCu);
    const bool halve = rest > 0 && 2 * rest <= kNumCu;
    const int n_whole = (int)n_tiles - (halve ? rest : 0);
    const double c = (double)a.sm_scale * 1.4426950408889634;
    float scale_log2 = (float)c;
    if (fabs((double)scale_log2) > fabs(c)) scale_log2 = nextafterf(scale_log2, 0.f);
    const float scale_err = fmaxf((float)((c - (double)scale_log2) / (double)scale_log2), FLT_MIN);
    const dim3 grid((unsigned)(2 * n_tiles - n_whole)), block(256);
    if (a.D == 64) return launch_kernel(fwd_f32_kernel<64>, grid, block, stream, a, n_rb, (int)n_tiles, n_whole, scale_log2, scale_err);
    if (a.D == 128) return launch_kernel(fwd_f32_kernel<128>, grid, block, stream, a, n_rb, (int)n_tiles, n_whole, scale_log2, scale_err);
    return hipErrorInvalidValue;
}

hipError_t launch_commit_f32(const CommitArgs &a, hipStream_t stream)
{
    // 32 x 32 blocks until they fill the chip several times over, then 64 x 64 ones (half the operand reads)
    const long long heads = (long long)a.B * a.H;
    const bool big = heads * (a.D / 32) * (a.D / 32) >= 4 * kNumCu;
    const long long nwg = heads * (a.D / (big ? 64 : 32)) * (a.D / (big ? 64 : 32));
    if (nwg <= 0 || nwg > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg), block(512);
    if (a.D == 64) return big ? launch_kernel(commit_f32_kernel<64, 64>, grid, block, stream, a) : launch_kernel(commit_f32_kernel<64, 32>, grid, block, stream, a);
    if (a.D == 128) return big ? launch_kernel(commit_f32_kernel<128, 64>, grid, block, stream, a) : launch_kernel(commit_f32_kernel<128, 32>, grid, block, stream, a);
    return hipErrorInvalidValue;
}

}  // namespace arl2
