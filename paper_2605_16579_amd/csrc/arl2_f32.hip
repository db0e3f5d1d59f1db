// The two operations for fp32 inputs, on gfx950:
//   out = softmax(q k^T * sm_scale) v + g * L2Norm(q) S             paper Eq. (2), (3), (5), (6)
//   S  <- gate * S + sum_i L2Norm(k_i)^T v_i                        paper Eq. (3), Eq. (4)
// The readout has two kernels.  One is on the fp32 matrix instructions, v_mfma_f32_32x32x2_f32 and 16x16x4_f32, which multiply and
// accumulate in fp32.  The other takes every fp32 operand as a sum of two halves (23 bits) and three products of the 16 times
// faster half-precision matrix instructions, which accumulate in fp32; it serves launches that fill the chip, and hands the tiles
// whose values two halves do not stand for to the code of the first (`fwd_f32_half_tile`, `halves_pay`).  In both, exponentials are
// v_exp_f32 on arguments rounded once, with the rounding of the scale's factor made good (`pow2_diff`).  The commit is on the fp32
// matrix instructions.
#include "arl2_device.h"

#include <math.h>

namespace arl2 {
namespace {

typedef __attribute__((address_space(3))) void lds_void;

// ---- readout, fp32 matrix instructions ---------------------------------------------------------------
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

// Query rows q0 .. q0 + QW - 1, those before row_end stored, of (stream, head) bh, by the four wavefronts of threads tid 0 .. 255.  x2: sm_scale log2(e) rounded towards zero, and what it falls short.
template <int D, int QW, bool SHORT_CHAINS = false>
__device__ __forceinline__ void fwd_f32_tile(const FwdArgs &a, f32x2 x2, int bh, int q0, int row_end, int tid, unsigned char *smem, float (*ml)[2][32])
{
    using C = F32Cfg<D, QW>;
    typedef float acc_t __attribute__((ext_vector_type(C::RPB)));
    constexpr int KT = C::KT, DB = C::DB, NW = C::NW, NG = C::NG, FPT = C::FPT, KBUF = C::KBUF;
    constexpr int NS = QW == 32 ? 1 : 2;      // accumulator blocks of S^T: 32 or 2 x 16 keys
    constexpr int CPR = D / 4;                // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;             // rows per direct load

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, gr = lane / QW, c = lane % QW;
    const int H = a.H, Lq = a.Lq, Lkv = a.Lkv;
    const int h = bh % H, b = bh / H;
    const int row = q0 + c;
    const bool valid = row < row_end;
    const uint32_t tok = (uint32_t)H * D * 4;                       // bytes of one token, all heads
    const size_t row_off = (((size_t)b * Lq + (valid ? row : Lq - 1)) * H + h) * D;
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
        if constexpr (D == 64 && QW == 32 && !SHORT_CHAINS) {       // even and odd steps
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
    const size_t gtok = (size_t)b * Lq + (valid ? row : Lq - 1);
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
    if (half < 0) fwd_f32_tile<D, 32>(a, x2, bh, q0, a.Lq, threadIdx.x, smem, ml);
    else if (q0 + 16 * half < a.Lq) fwd_f32_tile<D, 16>(a, x2, bh, q0 + 16 * half, a.Lq, threadIdx.x, smem, ml);
}

// ---- readout, sums of two halves ---------------------------------------------------------------------
// x s = hi + lo, s a power of two, hi = half(x s), lo = half(x s - hi): 23 of the 24 bits of an fp32 value (all of every second one's).
// A product a b is a.hi b.hi + a.hi b.lo + a.lo b.hi; a.lo b.lo, 2^-24 of it, is left out.  The half-precision matrix
// instructions multiply exactly and round an fp32 sum once per 8 or 16 products, the fp32 ones once per product, so the results are
// closer to 64 bits than with fp32 products, from 33 keys on (`halves_pay`) and whatever the size of the logits.  Relative 2-norm errors, fp32 products
// and this: with a state 1.57e-7 and 1.23e-7 at D = 128, 1.21e-7 and 1.13e-7 at D = 64; softmax alone, D = 128: 33 keys 1.67e-7 and 1.57e-7, 777 keys
// 3.0e-7 and 2.0e-7, logits four times as large 4.8e-7 and 4.0e-7, queries and keys along one direction with logits of 45 2.5e-6 and 2.4e-6 (with one
// chain of products over all 128 features 1.75e-7, 2.2e-7, 5.2e-7 and 3.1e-6).  The scales keep lo parts normal numbers: query rows
// have one each, the keys of a tile one from the largest of its first 128, with room for 64 times as large ones, each feature of the
// values, which is an output of its own, one from its largest among those keys, with room for 128 times as large ones, probabilities 2^15.
// What has no such parts is found out and done again on the fp32 instructions, by the same workgroup: infinities, NaN and values beyond the
// room (they end in a sum that is not finite); rows whose output is so small beside the scales that what lo lacks would show (`fits`);
// features whose values fall far below their scale for a few blocks (`look_for_lost`); and queries so large against the keys' scale that
// what the smallest parts of keys lack, 2^-35 of the largest, would show in logits (`kLargest`).  Single values of a feature among others are
// exact to 2^-34 of its largest among the first 128 keys.
//
// A workgroup owns 64 (or 32) query rows: two row groups of QW rows x four key groups, one wavefront each.  In an iteration a
// key group takes a block of 32 keys; its two wavefronts bring half of the block each from memory into registers and, as halves,
// into LDS, where both read all of it:
//   S^T[key][q] = K Q^T    A = K rows from LDS;  B = Q rows from LDS
//   O^T[d][q]  += V^T P^T  A = V through the transposing LDS read;  B = P from the accumulator registers of S^T
// An iteration has two halves between barriers: the products of S^T for the next block beside the softmax of this one and its
// values' way to LDS, then those of O^T beside the keys' way.  Each is 24 products per wavefront, in steps of three with one load's worth
// of splitting.
//
// What bounds it: the vector work (about 520 instructions per wavefront and iteration, half of them the splitting) and the
// fragments from LDS, which a SIMD does in turn, and the products, which run beside them only in part: 6400 cycles per iteration
// for 2 x 1536 of products.  v_fma_mixlo / mixhi_f16 take 8 cycles on a SIMD, the conversion of a pair and v_fma_mix_f32 4
// each, hence the separate steps of `put`.  Three bf16 parts (all 24 bits, six products, 32 cycles to split a pair against 20) were
// 30 % slower.  Measured per pass with a state, against fp32 products: 12 heads x 128, 1560 tokens 99 us, 162 us; 8 x 24 x 128, 777 tokens 359
// and 631 us; 2 x 16 x 64, 1560 tokens 125 and 181 us.  Of these a scale per feature of the values with the search for lost bits takes 2 %
// (64 heads x 128, 100 tokens 0.7 of 12.0 us) and the second chain of S^T 0.5 %.
template <int D, int QW>
struct F32HalfCfg {
    static constexpr int NKG = 4, NRG = 2, NW = NKG * NRG;   // key groups, row groups, wavefronts
    static constexpr int BM = NRG * QW;              // query rows per workgroup
    static constexpr int NG = 64 / QW;               // lane groups: each holds 8 features (or keys) of a contraction step
    static constexpr int KS = D / (8 * NG);          // steps of K Q^T
    static constexpr int NS = 32 / QW;               // QW-key blocks of S^T
    static constexpr int RPB = QW * QW / 64;         // accumulator registers of a QW x QW block
    static constexpr int FPT = 4 * NG;               // rows of a block that the lane groups hold four of each
    static constexpr int NL = QW / 2;                // logits per lane of a 32-key block
    static constexpr int NU = NL / 8;                // steps of V^T P^T
    static constexpr int DB = D / QW;                // QW-feature blocks of O^T
    static constexpr int NR = DB * RPB / NKG;        // registers of O that a wavefront finishes
    static constexpr int OB = NR > RPB ? NR / RPB : 1;   // blocks that they lie in
    static constexpr int CPR = D / 4;                // 16-byte chunks per row of fp32
    static constexpr int RPI = 64 / CPR;             // rows per load of a wavefront
    static constexpr int NLD = 16 / RPI;             // loads of half a block
    static constexpr int PART = 32 * D * 2;          // bytes of one part of a block of keys or values
    static constexpr int QPART = QW * D * 2;         // of a row group's rows
    static constexpr int V_OFF = NKG * 2 * PART, Q_OFF = 2 * V_OFF;
    static constexpr int SMEM = Q_OFF + NRG * 2 * QPART;
    static constexpr int OX = DB * RPB * 64 * 4;     // a wavefront's O
    static_assert(NW * OX <= Q_OFF, "the partial outputs pass through the blocks");
    static_assert(SMEM <= 160 * 1024, "more LDS than a CU has");
};

// The pairs of values that lanes l and l ^ 32 (l and l ^ 16) hold.
__device__ __forceinline__ f32x2 swap32(float x)
{
    const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
    return f32x2{__uint_as_float(y[0]), __uint_as_float(y[1])};
}
__device__ __forceinline__ f32x2 swap16(float x)
{
    const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false));
    return f32x2{__uint_as_float(y[0]), __uint_as_float(y[1])};
}
template <int N>
__device__ __forceinline__ float swap_sum(float x)
{
    if constexpr (N == 4) {
        const f32x2 y = swap16(x);
        x = y[0] + y[1];
    }
    const f32x2 y = swap32(x);
    return y[0] + y[1];
}
template <int N>
__device__ __forceinline__ float swap_max(float x)
{
    if constexpr (N == 4) {
        const f32x2 y = swap16(x);
        x = fmaxf(y[0], y[1]);
    }
    const f32x2 y = swap32(x);
    return fmaxf(y[0], y[1]);
}
// Over 16 or 32 consecutive lanes.
template <int N>
__device__ __forceinline__ float row_sum(float x)
{
    x = lane_group_sum<16>(x);
    if constexpr (N == 32) {
        const f32x2 y = swap16(x);
        x = y[0] + y[1];
    }
    return x;
}
template <int N>
__device__ __forceinline__ float row_max(float x)
{
    x = fmaxf(x, dpp_peek<0xB1>(x));
    x = fmaxf(x, dpp_peek<0x4E>(x));
    x = fmaxf(x, dpp_peek<0x141>(x));
    x = fmaxf(x, dpp_peek<0x140>(x));
    if constexpr (N == 32) {
        const f32x2 y = swap16(x);
        x = fmaxf(y[0], y[1]);
    }
    return x;
}

// ---- fp32 values as sums of two halves
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x16 mfma_f16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
constexpr float kPScale = 32768.f;            // probabilities are split times this, the most that halves have room for
// Largest key element times longest query, as a logit in powers of two, up to which tiles stay on halves: what lo parts of the keys lack adds 2^-35
// of that to a logit, here 2^-27.  (It says nothing about the logits, which the keys behind the first 128 may take further: these
// lack in proportion to their own size.)
constexpr float kLargest = 256.f;
struct Parts {
    u32x4 hi, lo;             // eight halves each
};
__device__ __forceinline__ uint32_t pack_f16(float x0, float x1)
{
    const f16x2 h = {(_Float16)x0, (_Float16)x1};
    uint32_t b = __builtin_bit_cast(uint32_t, h);
    asm("" : "+v"(b));
    return b;
}
// x s minus the half in the lower (upper) half of h.  (Left to itself the compiler joins this with the conversion that
// follows, in an instruction that takes twice as long as the two.)
__device__ __forceinline__ float rest_lo(float x, float s, uint32_t h)
{
    float r = fmaf(x, s, -(float)__builtin_bit_cast(f16x2, h)[0]);
    asm("" : "+v"(r));
    return r;
}
__device__ __forceinline__ float rest_hi(float x, float s, uint32_t h)
{
    float r = fmaf(x, s, -(float)__builtin_bit_cast(f16x2, h)[1]);
    asm("" : "+v"(r));
    return r;
}
template <class F>
__device__ __forceinline__ Parts split8(F &&x, float s)
{
    Parts r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        r.hi[p] = pack_f16(x(2 * p) * s, x(2 * p + 1) * s);
        r.lo[p] = pack_f16(rest_lo(x(2 * p), s, r.hi[p]), rest_hi(x(2 * p + 1), s, r.hi[p]));
    }
    return r;
}
// The power of two that takes `most` (>= 0) to 2^e .. 2^(e + 1), or 2^126 where that is less, and its inverse.  2^126 for zero: what the
// scale is for is zero throughout, or ends in a sum that is not finite.
__device__ __forceinline__ f32x2 scale_to(float most, int e)
{
    int x = (int)(__float_as_uint(most) >> 23);                      // biased exponent
    x = x < 127 + e - 126 ? 127 + e - 126 : x > 250 ? 250 : x;       // both powers are normal numbers
    return f32x2{__uint_as_float((uint32_t)(254 + e - x) << 23), __uint_as_float((uint32_t)(x - e) << 23)};
}
// Query rows q0 .. q0 + 2 QW - 1 of (stream, head) bh.  x2: sm_scale log2(e) rounded towards zero, and what it falls short.
// Returns false, with nothing written, where the halves do not stand for the values.
template <int D, int QW>
__device__ __forceinline__ bool fwd_f32_half_tile(const FwdArgs &a, f32x2 x2, int bh, int q0, unsigned char *smem)
{
    using C = F32HalfCfg<D, QW>;
    typedef float acc_t __attribute__((ext_vector_type(C::RPB)));
    constexpr int KS = C::KS, DB = C::DB, NG = C::NG, FPT = C::FPT, NS = C::NS, NL = C::NL, NU = C::NU, NKG = C::NKG, NLD = C::NLD;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, gr = lane / QW, c = lane % QW;
    const int kg = wave % NKG, rg = wave / NKG;
    const int H = a.H, Lq = a.Lq, Lkv = a.Lkv;
    const int h = bh % H, b = bh / H;
    const uint32_t tok = (uint32_t)H * D * 4;                       // bytes of one token, all heads
    const float *kgl = (const float *)a.k + ((size_t)b * Lkv * H + h) * D;
    const float *vgl = (const float *)a.v + ((size_t)b * Lkv * H + h) * D;

    // Blocks of 32 keys; iteration `it` takes 4 it + kg.  The two row groups of a key group move half of a block each: whole rows
    // into registers, and as halves into LDS.  Buffer descriptors are rebuilt per block from 64-bit bases, so that 32-bit
    // offsets only span 32 rows; rows past the last key, and blocks past the last one, read as zero.
    const int nblk = (Lkv + 31) / 32, nit = (nblk + NKG - 1) / NKG;
    const int row0 = 16 * rg + lane / C::CPR, col = lane % C::CPR;  // the lane's row of load 0, its four features
    uint32_t src0 = (uint32_t)row0 * tok + 16 * col;
    auto rsrc_of = [&](const float *base, int it) {
        const int blk = NKG * it + kg;
        const int rows = blk >= nblk ? 0 : Lkv - 32 * blk < 32 ? Lkv - 32 * blk : 32;
        return make_rsrc((const char *)base + (size_t)(rows > 0 ? blk : 0) * 32 * tok, rows > 0 ? (uint32_t)(rows - 1) * tok + 4 * D : 0);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t r, int i) -> f32x4 {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, src0 + C::RPI * i * tok, 0, 0));
    };
    // Rows of 2 D bytes, whose 16-byte chunks x are exchanged so that fragment reads find 64 different banks:
    //   keys, D = 128:   x ^ row % 16;          D = 64: x ^ row / 2 % 8
    //   values, D = 128: x ^ 4 (row % 4) ^ 2 (row / 4 % 2);  D = 64: x ^ 4 (row / 2 % 2) ^ 2 (row / 4 % 2)
    auto k_chunk = [](int r) { return D == 128 ? r & 15 : (r >> 1) & 7; };
    auto v_chunk = [](int r) { return (D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1)) ^ (2 * ((r >> 2) & 1)); };
    // Offsets of the lane's piece of load 0; that of load i lies i RPI rows further, its chunk exchanged by the constants below.
    float k_scale = 1.f;
    f32x4 v_scale;
    uint32_t k_put = kg * 2 * C::PART + row0 * (2 * D) + 16 * ((col >> 1) ^ k_chunk(row0)) + 8 * (col & 1);
    uint32_t v_put = C::V_OFF + kg * 2 * C::PART + row0 * (2 * D) + 16 * ((col >> 1) ^ v_chunk(row0)) + 8 * (col & 1);
    uint32_t hi[2];
    float rest[4];
    // Thirds of four values' way from registers to LDS; their lo parts `part` bytes behind the hi ones.
    auto put = [&](auto third_, const f32x4 &x, f32x4 s, uint32_t off, auto part_) {
        constexpr int third = decltype(third_)::value, PART = decltype(part_)::value;
        if constexpr (third == 0) {
            hi[0] = pack_f16(x[0] * s[0], x[1] * s[1]);
            hi[1] = pack_f16(x[2] * s[2], x[3] * s[3]);
        } else if constexpr (third == 1) {
            rest[0] = rest_lo(x[0], s[0], hi[0]);
            rest[1] = rest_hi(x[1], s[1], hi[0]);
            rest[2] = rest_lo(x[2], s[2], hi[1]);
            rest[3] = rest_hi(x[3], s[3], hi[1]);
        } else {
            unsigned char *p = smem + off;
            *(u32x2 *)p = u32x2{hi[0], hi[1]};
            *(u32x2 *)(p + PART) = u32x2{pack_f16(rest[0], rest[1]), pack_f16(rest[2], rest[3])};
        }
    };
    const std::integral_constant<int, C::PART> kv_part{};
    auto put_k = [&](auto third_, auto i_, const f32x4 &x) {
        constexpr int i = decltype(i_)::value;
        put(third_, x, f32x4(k_scale), (k_put ^ (16 * 2 * i)) + C::RPI * i * (2 * D), kv_part);
    };
    auto put_v = [&](auto third_, auto i_, const f32x4 &x) {
        constexpr int i = decltype(i_)::value;
        put(third_, x, v_scale, (v_put ^ (16 * (D == 128 ? 8 * (i & 1) ^ (i & 2) : 2 * (i & 1)))) + C::RPI * i * (2 * D), kv_part);
    };
    // The largest value that a lane sees of each of its features in two rows of a block each (no NaN; of all the wavefront's rows in the first
    // block), and whether over three blocks and more, or the first, all of it was below 1/4, 2^-10 of what the scale was taken from, and not zero.
    float seen[4];
    uint64_t lost = 0;
    auto look = [&](const f32x4 &x, const f32x4 &y) {
#pragma unroll
        for (int e = 0; e < 4; ++e) asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(seen[e]) : "v"(x[e]), "v"(y[e]));
    };
    auto look_for_lost = [&]() {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lost |= __ballot(seen[e] > 0.f) & __ballot(seen[e] * v_scale[e] < 0.25f);
            seen[e] = 0.f;
        }
    };
    // B operand of S^T: lane (row c, gr) takes features 8 (NG t + gr) + 0..7 of its row, scaled by a power of two of its own, as
    // halves from LDS rows like those of the keys.  Every wavefront moves an eighth of the rows.
    constexpr int QRW = C::BM / C::NW, NQL = QRW / C::RPI;          // rows and loads per wavefront
    f32x4 qraw[NQL];
    auto fetch_q = [&](const float *src, int ln) {
#pragma unroll
        for (int i = 0; i < NQL; ++i) {
            const int r = q0 + QRW * wave + C::RPI * i + ln / C::CPR;
            qraw[i] = *(const f32x4 *)(src + (((size_t)b * Lq + (r < Lq ? r : Lq - 1)) * H + h) * D + 4 * (ln % C::CPR));
        }
    };
    // info: [row][1 / scale, sum of squares]
    auto put_q = [&](float *info, int ln) {
        const int cq = ln % C::CPR;
#pragma unroll
        for (int i = 0; i < NQL; ++i) {
            const f32x4 x = qraw[i];
            const int r = QRW * wave + C::RPI * i + ln / C::CPR, rr = r % QW;
            const float ss = row_sum<C::CPR>(fmaf(x[0], x[0], x[1] * x[1]) + fmaf(x[2], x[2], x[3] * x[3]));
            const f32x2 s = scale_to(row_max<C::CPR>(fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])))), 12);
            static_for<0, 3>([&](auto third_) {
                put(third_, x, f32x4(s[0]), C::Q_OFF + (r / QW) * 2 * C::QPART + rr * (2 * D) + 16 * ((cq >> 1) ^ k_chunk(rr)) + 8 * (cq & 1), std::integral_constant<int, C::QPART>{});
            });
            if (cq == 0) *(f32x2 *)(info + 2 * r) = f32x2{s[1], ss};
        }
    };
    // Offsets of the lane's fragments of step 0.
    const uint32_t frag_off = c * (2 * D) + 16 * (gr ^ k_chunk(c));
    uint32_t q_off = C::Q_OFF + rg * 2 * C::QPART + frag_off, k_off = kg * 2 * C::PART + frag_off;
    auto q_frag = [&](int t) -> Parts {
        const unsigned char *p = smem + (q_off ^ (16 * NG * t));
        return Parts{*(const u32x4 *)p, *(const u32x4 *)(p + C::QPART)};
    };
    // A operand of S^T: eight features of key QW kb + c
    auto k_frag = [&](int kb, int t) -> Parts {
        const unsigned char *p = smem + (k_off ^ (16 * NG * t)) + QW * kb * (2 * D);
        return Parts{*(const u32x4 *)p, *(const u32x4 *)(p + C::PART)};
    };
    // A operand of O^T, block db, step u: keys 16 u + 4 gr + 0..3 and + 8 (QW = 16: + 16) of feature QW db + c
    const int v_row = ((lane & 15) >> 2) + 4 * gr;
    uint32_t v_off = C::V_OFF + kg * 2 * C::PART + v_row * (2 * D) + ((QW == 32 ? 32 * ((lane >> 4) & 1) : 0) ^ (16 * v_chunk(v_row))) + 8 * (lane & 3);
    auto v_frag = [&](int u, int db) -> Parts {
        const unsigned char *p = smem + (v_off ^ (2 * QW * db)) + 16 * u * (2 * D);
        return Parts{__builtin_bit_cast(u32x4, lds_read_tr_pair(p, FPT * 2 * D)), __builtin_bit_cast(u32x4, lds_read_tr_pair(p + C::PART, FPT * 2 * D))};
    };

    // ---- the first blocks, and with them the scale of the keys
    f32x4 raw[NLD], k0[NLD];
    {
        const __amdgpu_buffer_rsrc_t r = rsrc_of(kgl, 0);
#pragma unroll
        for (int i = 0; i < NLD; ++i) k0[i] = load(r, i);
    }
    fetch_q((const float *)a.q, lane);
    {
        const __amdgpu_buffer_rsrc_t r = rsrc_of(vgl, 0);
#pragma unroll
        for (int i = 0; i < NLD; ++i) raw[i] = load(r, i);
    }
    float *ml = (float *)(smem + C::V_OFF), *info = ml + C::NW, *most = info + 2 * C::BM;     // most: of every feature of the first values
    if (tid < D) most[tid] = 0.f;
    put_q(info, lane);
    {
        float km = 0.f;
#pragma unroll
        for (int i = 0; i < NLD; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) km = fmaxf(km, fabsf(k0[i][e]));
        km = swap_max<2>(row_max<32>(km));
        if (lane == 0) ml[wave] = km;
    }
    lds_barrier();
    float sc, q_inv = info[2 * (QW * rg + c)], qss = info[2 * (QW * rg + c) + 1];
    {
        float km = 0.f;
#pragma unroll
        for (int w = 0; w < C::NW; ++w) km = fmaxf(km, ml[w]);
        const f32x2 ks = scale_to(km, 9);
        k_scale = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(ks[0])));
        float qmost = 0.f;
#pragma unroll
        for (int r = 0; r < C::BM; r += 32) qmost = fmaxf(qmost, info[2 * (r + (lane & 31)) + 1]);
        qmost = row_max<32>(qmost);
        if (__builtin_amdgcn_readfirstlane(!(km * sqrtf(qmost) * x2[0] < kLargest))) {
            lds_barrier();
            return false;
        }
        sc = fmaxf(x2[0] * (q_inv * ks[1]), FLT_MIN);               // (not zero: keys past the end have a logit of -inf)
    }
    static_for<0, NLD>([&](auto i_) { static_for<0, 3>([&](auto third_) { put_k(third_, i_, k0[decltype(i_)::value]); }); });
    {
        const __amdgpu_buffer_rsrc_t r = rsrc_of(kgl, 1);
#pragma unroll
        for (int i = 0; i < NLD; ++i) k0[i] = load(r, i);
    }
    lds_barrier();

    acc_t o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = acc_t(0.f);
    // running maximum of the scaled logits, in powers of two (finite also while every logit was -inf); this lane's share of
    // the row sum
    float m = -FLT_MAX, l = 0.f;

    float s[NL];                              // logits of the block whose softmax is next
    acc_t sm[NS], sa[2][NS];                  // those of the block after it: products with a lo part, products of hi parts over half of the features each
    Parts pp[NU];                             // its probabilities
    // S^T of a block (S), beside the softmax of the block before it and its values on their way to LDS (P).
    auto products = [&](auto s_, auto p_, __amdgpu_buffer_rsrc_t next) {
        constexpr bool S = decltype(s_)::value, P = decltype(p_)::value;
        constexpr int N = KS * NS;                                  // step n: key block n % NS, features n / NS
        constexpr int NP = NL / 2;                                  // pairs of logits
        static_assert(N == NLD, "a load per step");
        Parts kf[2], qf[2];
        float ls[2] = {0.f, 0.f};
        if constexpr (S) {
            static_for<0, NS>([&](auto kb_) {
                constexpr int kb = decltype(kb_)::value;
                sm[kb] = sa[0][kb] = sa[1][kb] = acc_t(0.f);
            });
            kf[0] = k_frag(0, 0);
            qf[0] = q_frag(0);
        }
        static_for<0, N>([&](auto n_) {
            constexpr int n = decltype(n_)::value, kb = n % NS, t = n / NS;
            if constexpr (S && n + 1 < N) kf[(n + 1) & 1] = k_frag((n + 1) % NS, (n + 1) / NS);
            if constexpr (S && n + 1 < N && (n + 1) / NS != t) qf[(t + 1) & 1] = q_frag(t + 1);
            const Parts &k = kf[n & 1], &q = qf[t & 1];
            static_for<0, 3>([&](auto third_) {
                constexpr int third = decltype(third_)::value;
                if constexpr (S) {
                    if constexpr (third == 0) sm[kb] = mfma_f16(k.hi, q.lo, sm[kb]);
                    if constexpr (third == 1) sm[kb] = mfma_f16(k.lo, q.hi, sm[kb]);
                    if constexpr (third == 2) sa[2 * t / KS][kb] = mfma_f16(k.hi, q.hi, sa[2 * t / KS][kb]);
                }
                if constexpr (P) {
                    static_for<n * NP / N, (n + 1) * NP / N>([&](auto pair_) {
                        constexpr int i = 2 * decltype(pair_)::value;
                        if constexpr (third == 0) {
                            s[i] = fmaf(s[i], sc, -m);
                            s[i + 1] = fmaf(s[i + 1], sc, -m);
                            s[i] = fmaf(s[i], x2[1], s[i]);
                            s[i + 1] = fmaf(s[i + 1], x2[1], s[i + 1]);
                            s[i] = __builtin_amdgcn_exp2f(s[i]);
                        } else if constexpr (third == 1) {
                            s[i + 1] = __builtin_amdgcn_exp2f(s[i + 1]);
                            ls[0] += s[i];
                            ls[1] += s[i + 1];
                        } else {
                            const uint32_t hh = pack_f16(s[i] * kPScale, s[i + 1] * kPScale);
                            pp[i / 8].hi[i % 8 / 2] = hh;
                            pp[i / 8].lo[i % 8 / 2] = pack_f16(rest_lo(s[i], kPScale, hh), rest_hi(s[i + 1], kPScale, hh));
                        }
                    });
                    put_v(third_, n_, raw[n]);
                    if constexpr (third == 1 && n == 0) look(raw[0], raw[1]);
                    if constexpr (third == 2) raw[n] = load(next, n);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        l += ls[0] + ls[1];
    };
    // The logits out of the accumulators; logit i of a lane is key FPT (i / 4) + 4 gr + i % 4 of the block.
    auto logits = [&](int blk) {
#pragma unroll
        for (int i = 0; i < NL; ++i) s[i] = sm[i / C::RPB][i % C::RPB] + sa[0][i / C::RPB][i % C::RPB] + sa[1][i / C::RPB][i % C::RPB];
        if (__builtin_expect(32 * blk + 32 > Lkv, 0)) {             // keys past the end
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (32 * blk + FPT * (i >> 2) + 4 * gr + (i & 3) >= Lkv) s[i] = -INFINITY;
        }
    };
    auto new_max = [&]() -> float {
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < NL; ++i) mx = fmaxf(mx, s[i]);
        return fmaxf(m, swap_max<NG>(mx) * sc);
    };
    // O^T of the block, beside the next block's logits and keys on their way to LDS (MORE).
    float m_new;
    auto values = [&](auto more_, int blk, __amdgpu_buffer_rsrc_t next) {
        constexpr bool MORE = decltype(more_)::value;
        constexpr int N = NU * DB;                                  // step n: block n / NU, keys n % NU
        static_assert(N == NLD, "a load per step");
        Parts vf[2];
        vf[0] = v_frag(0, 0);
        acc_t t[2];
        static_for<0, N>([&](auto n_) {
            constexpr int n = decltype(n_)::value, u = n % NU, db = n / NU;
            if constexpr (n + 1 < N) vf[(n + 1) & 1] = v_frag((n + 1) % NU, (n + 1) / NU);
            const Parts &v = vf[n & 1];
            if constexpr (u == 0) t[db & 1] = acc_t(0.f);
            static_for<0, 3>([&](auto third_) {
                constexpr int third = decltype(third_)::value;
                if constexpr (third == 0) t[db & 1] = mfma_f16(v.hi, pp[u].lo, t[db & 1]);
                if constexpr (third == 1) t[db & 1] = mfma_f16(v.lo, pp[u].hi, t[db & 1]);
                if constexpr (third == 2) t[db & 1] = mfma_f16(v.hi, pp[u].hi, t[db & 1]);
                if constexpr (MORE) {
                    if constexpr (n == 0 && third == 1) logits(blk + NKG);
                    if constexpr (n == 1 && third == 1) m_new = new_max();
                    put_k(third_, n_, raw[n]);
                    if constexpr (third == 2) raw[n] = load(next, n);
                }
                if constexpr (u == NU - 1 && third == 1 && db > 0) o[db - 1] += t[(db - 1) & 1];
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        o[DB - 1] += t[(DB - 1) & 1];
    };
    const std::true_type yes{};
    const std::false_type no{};
    products(yes, no, rsrc_of(kgl, 0));
    logits(kg);
    m = new_max();
    // the scales of the values' features
    uint64_t zeros;                           // bit i: features 4 i .. 4 i + 3 are zero
    {
        f32x4 vm = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NLD; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) vm[e] = fmaxf(vm[e], fabsf(raw[i][e]));
#pragma unroll
        for (int e = 0; e < 4; ++e) vm[e] = swap_max<C::RPI>(vm[e]);
        if (lane < C::CPR)
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicMax((unsigned *)(most + 4 * col + e), __float_as_uint(vm[e]));     // (in the order of what is not negative)
#pragma unroll
        for (int e = 0; e < 4; ++e) seen[e] = 32 * kg + 16 * rg + 16 <= Lkv ? vm[e] : INFINITY;         // (a few keys alone may be small by chance)
        lds_barrier();                                              // the first keys have been read
        vm = *(const f32x4 *)(most + 4 * col);
#pragma unroll
        for (int e = 0; e < 4; ++e) v_scale[e] = scale_to(vm[e], 8)[0];
        zeros = __ballot(vm[0] == 0.f && vm[1] == 0.f && vm[2] == 0.f && vm[3] == 0.f);
    }
    static_for<0, NLD>([&](auto i_) { static_for<0, 3>([&](auto third_) { put_k(third_, i_, k0[decltype(i_)::value]); }); });
    lds_barrier();
    int look_at = nit >= 4 ? 0 : nit;
#pragma unroll 1
    for (int it = 0; it + 1 < nit; ++it) {
        // (one offset of each and not all that they lead to kept over the loop)
        asm volatile("" : "+v"(src0), "+v"(k_off), "+v"(q_off), "+v"(v_off), "+v"(k_put), "+v"(v_put));
        products(yes, yes, rsrc_of(kgl, it + 2));
        if (it == look_at) {
            look_for_lost();
            look_at = it + 7 <= nit ? it + 3 : nit;
        }
        lds_barrier();                                              // the keys have been read, the values are there
        values(yes, NKG * it + kg, rsrc_of(vgl, it + 1));
        if (__any(m_new > m)) {
            const float alpha = pow2_diff(m - m_new, x2[1]);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
        }
        lds_barrier();                                              // the values have been read, the next keys are there
    }
    products(no, yes, rsrc_of(kgl, nit));
    look_for_lost();
    lds_barrier();
    values(no, 0, rsrc_of(kgl, nit));
    lds_barrier();

    // (what the end needs is worked out here, from a lane number that looks new, and not kept over the loop)
    int late = lane;
    asm volatile("" : "+v"(late));
    const int gr_e = late / QW, c_e = late % QW, row = q0 + QW * rg + c_e;
    const bool valid = row < Lq;
    const size_t row_off = (((size_t)b * Lq + (valid ? row : q0)) * H + h) * D;
    // from here on a wavefront finishes NR registers of its rows' O: from register r0 of block db0 on.  Register r of them is feature
    // QW ((r0 + r) / RPB) + FPT ((r0 + r) % RPB / 4) + 4 gr_e + r % 4 of those from QW db0 on.
    constexpr int NR = C::NR, OB = C::OB;
    const int db0 = kg * NR / C::RPB, r0 = kg * NR % C::RPB;
    auto feature = [&](int r) { return QW * db0 + QW * ((r0 + r) / C::RPB) + FPT * ((r0 + r) % C::RPB / 4) + 4 * gr_e + (r & 3); };
    const size_t gtok = (size_t)b * Lq + (valid ? row : q0);
    const size_t gi = a.g_per_token ? gtok : gtok * H + h;
    // ---- merge the four shares: everything relative to the largest maximum
    l = swap_sum<NG>(l);
    // A lane looks at 16 features of its row at a time.
    bool fits = l < INFINITY && lost == 0;
    constexpr int BPG = 16 / C::RPB;          // blocks with them
    const uint32_t zero = (uint32_t)zeros >> gr_e;
#pragma unroll
    for (int db = 0; db < DB; db += BPG) {
        float osq = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) osq = fmaf(o[db + i / C::RPB][i % C::RPB], o[db + i / C::RPB][i % C::RPB], osq);
        constexpr uint32_t quads = QW == 32 ? 0x55 : 0x1111;
        const float least = (~zero >> (QW / 4 * db) & quads) == 0 ? 0.f : 8.f * kPScale * kPScale;
        fits &= (osq >= l * least) & (osq < INFINITY);
    }
    const bool all_fit = __all(fits);
    ml = (float *)smem;                                             // [wavefront][maximum, sum, fits][row]
    if (gr_e == 0) {
        ml[wave * 96 + c_e] = m;
        ml[wave * 96 + 32 + c_e] = l;
    }
    if (late == 0) ml[wave * 96 + 64] = all_fit ? 0.f : 1.f;
    if (wave == 0 && late < C::CPR) {                               // by which each feature of O is too large, to its inverse
        const u32x4 s = __builtin_bit_cast(u32x4, v_scale);
        *(u32x4 *)(ml + 96 * C::NW + 4 * (late % C::CPR)) = u32x4{0x7f000000u - s[0], 0x7f000000u - s[1], 0x7f000000u - s[2], 0x7f000000u - s[3]};
    }
    __syncthreads();
    float misfits = 0.f;
#pragma unroll
    for (int w = 0; w < C::NW; ++w) misfits += ml[w * 96 + 64];
    float m_all = -FLT_MAX, l_all = 0.f;
#pragma unroll
    for (int w = 0; w < NKG; ++w) m_all = fmaxf(m_all, ml[(NKG * rg + w) * 96 + c_e]);
#pragma unroll
    for (int w = 0; w < NKG; ++w) l_all = fmaf(ml[(NKG * rg + w) * 96 + 32 + c_e], pow2_diff(ml[(NKG * rg + w) * 96 + c_e] - m_all, x2[1]), l_all);
    const float f = pow2_diff(m - m_all, x2[1]);
    f32x4 o_inv[NR / 4];
#pragma unroll
    for (int r = 0; r < NR; r += 4) o_inv[r / 4] = *(const f32x4 *)(ml + 96 * C::NW + feature(r));
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(__float_as_int(misfits)) != 0) return false;      // (the same in all wavefronts)
    float *mine = (float *)smem + wave * (DB * C::RPB * 64) + late;                                      // [wavefront][feature block][register][lane]
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < C::RPB; ++r) mine[(db * C::RPB + r) * 64] = o[db][r] * f;
    __syncthreads();
    const float *shares = (const float *)smem + (NKG * rg * DB * C::RPB + NR * kg) * 64 + late;
    float out[NR];
    l_all *= kPScale;
    const float inv_l = 1.0f / l_all;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NKG; ++w) sum += shares[(w * DB * C::RPB + r) * 64];
        // sum / l_all, the quotient corrected once
        const float q = sum * inv_l;
        out[r] = fmaf(fmaf(-q, l_all, sum), inv_l, q) * o_inv[r / 4][r & 3];
    }
    float sv[OB][KS][8], g_row = 1.0f;
    if (a.S != nullptr) {
#pragma unroll
        for (int ob = 0; ob < OB; ++ob) {
            const __amdgpu_buffer_rsrc_t Sg = make_rsrc(a.S + (size_t)bh * D * D, D * D * 4);
            const uint32_t off = 4 * (8 * gr_e * D + QW * (db0 + ob) + c_e);
#pragma unroll
            for (int t = 0; t < KS; ++t)
#pragma unroll
                for (int i = 0; i < 8; ++i) sv[ob][t][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(Sg, off + 4 * (8 * NG * t + i) * D, 0, 0));
        }
        if (a.g != nullptr && !a.g_per_element) g_row = a.g_is_bf16 ? (float)((const bf16_t *)a.g)[gi] : ((const float *)a.g)[gi];
        if (a.q_lin != nullptr) fetch_q((const float *)a.q_lin, late);    // the linear branch's own query (Eq. (3))
    }
    if (a.S != nullptr) {
        if (a.q_lin != nullptr) {
            __syncthreads();                                        // the shares have been read
            put_q((float *)smem, late);
            __syncthreads();
            q_inv = ((float *)smem)[2 * (QW * rg + c_e)];
            qss = ((float *)smem)[2 * (QW * rg + c_e) + 1];
        }
        const float rq = 1.0f / sqrtf(qss + a.l2_eps);
        float x[NR];
        static_for<0, OB>([&](auto ob_) {
            constexpr int ob = decltype(ob_)::value;
            float most = 0.f;
#pragma unroll
            for (int t = 0; t < KS; ++t)
#pragma unroll
                for (int i = 0; i < 8; ++i) most = fmaxf(most, fabsf(sv[ob][t][i]));
            most = swap_max<NG>(most);
            const f32x2 ss = scale_to(most, 12);     // every feature has a scale of its own
            const uint32_t zero = most == 0.f ? 0x7bff7bffu : 0u;     // (a feature of zeros lacks nothing)
            acc_t small = acc_t(0.f), main = acc_t(0.f), sizes = acc_t(0.f);
            static_for<0, KS>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                const Parts sp = split8([&](int i) { return sv[ob][t][i]; }, ss[0]);
                const Parts q = q_frag(t);
                small = mfma_f16(sp.hi, q.lo, small);
                small = mfma_f16(sp.lo, q.hi, small);
                main = mfma_f16(sp.hi, q.hi, main);
                if constexpr (t % (KS / 2) == 0) sizes = mfma_f16((sp.hi & 0x7fff7fffu) | zero, q.hi & 0x7fff7fffu, sizes);
            });
            main += small;
            constexpr int N = NR < C::RPB ? NR : C::RPB;            // registers of this block
            auto mine = [&](const acc_t &y, int i) {
                if constexpr (NR < C::RPB) return r0 == 0 ? y[i] : y[i + NR];
                else return y[i];
            };
            // What the lo parts lack, 2^-26 per feature beside factors of up to 2^13, is less than 2^-25 of products of size 2^16 and more
            // (which some of the features, at D = 128 a quarter, have to reach).
            float least = INFINITY, nan = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float inv = __shfl(ss[1], FPT * ((r0 + i) / 4) + 4 * gr_e + (i & 3), kWave);     // of the lane with that feature
                x[ob * C::RPB + i] = mine(main, i) * (inv * q_inv);
                least = fminf(least, mine(sizes, i));
                nan = fmaf(x[ob * C::RPB + i], 0.f, nan);          // of infinities too, which are no sums of halves either
            }
            if (__builtin_expect(__any(!(least >= 65536.f && nan == 0.f)), 0)) {
                const float *src = (const float *)(a.q_lin != nullptr ? a.q_lin : a.q) + row_off + 8 * gr_e;
                acc_t y = acc_t(0.f);
#pragma unroll
                for (int t = 0; t < KS; ++t)
#pragma unroll
                    for (int i = 0; i < 8; i += 4) {
                        const f32x4 q4 = *(const f32x4 *)(src + 8 * NG * t + i);
#pragma unroll
                        for (int j = 0; j < 4; ++j) y = mfma_f32(sv[ob][t][i + j], q4[j], y);
                    }
#pragma unroll
                for (int i = 0; i < N; ++i) x[ob * C::RPB + i] = mine(y, i);
            }
        });
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float g = g_row;                     // headwise or per-token gate, or one gate per output feature
            if (a.g != nullptr && a.g_per_element) {
                const size_t ge = gi * D + feature(r);
                g = a.g_is_bf16 ? (float)((const bf16_t *)a.g)[ge] : ((const float *)a.g)[ge];
            }
            out[r] = fmaf(g, x[r] * rq, out[r]);
        }
    }
    if (valid) {
        float *og = (float *)a.out + row_off;
#pragma unroll
        for (int r = 0; r < NR; r += 4) *(f32x4 *)(og + feature(r)) = f32x4{out[r], out[r + 1], out[r + 2], out[r + 3]};
    }
    return true;
}

// n_rb tiles of 64 rows per head, n_tiles in all; the first n_whole are served whole, the others as two tiles of 32 rows.
template <int D>
__global__ __launch_bounds__(512, 2) void fwd_f32_halves_kernel(FwdArgs a, int n_rb, int n_tiles, int n_whole, float scale_log2, float scale_err)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[F32HalfCfg<D, 32>::SMEM];
    int id = blockIdx.x, half = -1;
    if (id >= n_whole) {
        half = (id - n_whole) / (n_tiles - n_whole);
        id = n_whole + (id - n_whole) % (n_tiles - n_whole);
    }
    const int work = xcd_contiguous_id(id, n_tiles);                // the row blocks of a head share an XCD's L2
    const int bh = work / n_rb;
    int q0 = (work % n_rb) * 64, end = q0 + 64;
    const f32x2 x2 = {scale_log2, scale_err};
    bool done;
    if (half < 0) {
        done = fwd_f32_half_tile<D, 32>(a, x2, bh, q0, smem);
    } else {
        q0 += 32 * half;
        end = q0 + 32;
        if (q0 >= a.Lq) return;
        done = fwd_f32_half_tile<D, 16>(a, x2, bh, q0, smem);
    }
    // Four wavefronts for half of the rows each.  All tiles done again, 1560 tokens with a state, found before the key loop (infinite or
    // outsized first keys) and after it (everything else): 12 heads x 128 192 and 271 us (157 on fp32 products alone), 2 x 16 x 64 239 and 340
    // us (182).  (With 32-row tiles left to four of the eight wavefronts the first took 244 and 269 us.  A way out before the loop for values too
    // costs other launches 1-3 %.)
    if (!done) {
        const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
        constexpr int ML = F32Cfg<D, 32>::NW * 2 * 32 * 4, PART = F32Cfg<D, 32>::SMEM + ML;
        static_assert(2 * PART <= F32HalfCfg<D, 32>::SMEM && F32Cfg<D, 16>::SMEM <= F32Cfg<D, 32>::SMEM, "room for two tiles");
        int tid = threadIdx.x & 255;
        asm volatile("" : "+v"(tid));                               // (nothing of the other tile is kept for this one)
        unsigned char *mine = smem + part * PART;
        float (*ml)[2][32] = (float (*)[2][32])(mine + F32Cfg<D, 32>::SMEM);
        if (end > a.Lq) end = a.Lq;
        if (half < 0) fwd_f32_tile<D, 32, true>(a, x2, bh, q0 + 32 * part, end, tid, mine, ml);
        else fwd_f32_tile<D, 16, true>(a, x2, bh, q0 + 16 * part, end, tid, mine, ml);
    }
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

// Whether tiles of 64 rows on sums of halves are faster than `tiles` ones of 32 rows on fp32 products.  Their start and end are longer
// (scales, splitting, the search for lost bits) and the key loop is shorter; and while 32-row
// tiles find a CU for each of their halves these are 16-row ones.  In us, softmax alone, fp32 products and halves:
//   up to 128 tiles, D = 128: 4 heads, 1000 rows, 640 keys 19.0 and 19.0, 720 keys 21.9 and 21.4, 800 keys 24.4 and 23.9; D = 64: 2048 keys 29.3
//     and 29.8, 4096 keys 53.9 and 54.3 (2 heads, 1560 rows 58.1 and 54.3), 8192 keys 106 and 103;
//   beyond: D = 128, 200 tiles 64 keys 10.1 and 9.1; 600 tiles 32 keys 18.2 and 20.5, 48 keys 21.9 and 20.6, 128 keys 22.7 and 20.4;
//     D = 64, 200 tiles 64 keys 6.46 and 6.46, 256 keys 8.9 and 8.0, 400 tiles 64 keys 9.8 and 8.1; 608 tiles, where three workgroups of the
//     fp32 kernel share a CU: 384 keys 21.8 and 20.8, 512 keys 26.8 and 24.5;
//   up to 32 keys: as above, and a sum of so few rounds less often than operands lose bits (relative error at D = 128, 1 key 0 and 4.5e-8, 8
//     keys 1.1e-7 and 1.2e-7, 24 keys 1.5e-7 both);
//   rows that leave a row group empty: up to 32 of them 300 heads x 128, 500 keys 36 and 41; 65 to 96 a third more work: 150 heads, 90 rows, 512
//     keys 43.0 and 40.1.
bool halves_pay(const FwdArgs &a, long long tiles)
{
    const int n_rb = (a.Lq + 31) / 32;
    if (n_rb == 1 || a.Lkv <= 32) return false;
    if (n_rb == 3 && a.Lkv < 512) return false;
    if (a.D == 128) return tiles > kNumCu / 2 || a.Lkv >= 704;
    return tiles > 2 * kNumCu ? a.Lkv >= 384 : tiles > kNumCu / 2 || a.Lkv >= 4096;
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs &a, hipStream_t stream)
{
    const int n_rb = (a.Lq + 31) / 32;
    const long long n_tiles = (long long)n_rb * a.B * a.H;
    if (n_tiles <= 0 || n_tiles > 0x3fffffffLL) return hipErrorInvalidValue;
    const double c = (double)a.sm_scale * 1.4426950408889634;
    float scale_log2 = (float)c;
    if (fabs((double)scale_log2) > fabs(c)) scale_log2 = nextafterf(scale_log2, 0.f);
    const float scale_err = fmaxf((float)((c - (double)scale_log2) / (double)scale_log2), FLT_MIN);
    if (halves_pay(a, n_tiles)) {
        // as below, with twice the rows
        const int n_rb64 = (a.Lq + 63) / 64, n64 = (int)((long long)n_rb64 * a.B * a.H);
        const int rest = n64 % kNumCu, n_whole = rest > 0 && 2 * rest <= kNumCu ? n64 - rest : n64;
        const dim3 grid((unsigned)(2 * n64 - n_whole)), block(512);
        if (a.D == 64) return launch_kernel(fwd_f32_halves_kernel<64>, grid, block, stream, a, n_rb64, n64, n_whole, scale_log2, scale_err);
        if (a.D == 128) return launch_kernel(fwd_f32_halves_kernel<128>, grid, block, stream, a, n_rb64, n64, n_whole, scale_log2, scale_err);
        return hipErrorInvalidValue;
    }
    // Tiles beyond a multiple of one per CU are served by two workgroups of 16 rows each while those find a CU of their own:
    // they take half as long.  12 heads x 128, 1560 tokens (588 tiles, 76 beyond) 156 us, 4 heads, 500 tokens (64 tiles) 18 and
    // 30 us, 192 heads, 100 tokens (768 tiles, all whole) 37 us; with more than half of the CUs taken nothing would be shorter.
    const int rest = (int)(n_tiles % kNumCu);
    const bool halve = rest > 0 && 2 * rest <= kNumCu;
    const int n_whole = (int)n_tiles - (halve ? rest : 0);
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
