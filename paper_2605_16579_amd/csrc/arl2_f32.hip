// fp32-throughout variants of the two operations (for fp32 inputs), on the fp32 matrix instructions (gfx950):
//   out = softmax(q k^T * sm_scale) v + g * L2Norm(q) S             paper Eq. (2), (3), (5), (6)
//   S  <- gate * S + sum_i L2Norm(k_i)^T v_i                        paper Eq. (3), Eq. (4)
// v_mfma_f32_32x32x2_f32 multiplies and accumulates in fp32, so no step has reduced precision; exponentials and
// roots are the full-precision ones.
#include "arl2_device.h"

namespace arl2 {
namespace {

typedef __attribute__((address_space(3))) void lds_void;

// ---- readout ---------------------------------------------------------------------------------------
// Bound by the fp32 matrix rate (a 32 x 32 x 2 step takes 64 cycles for one dword per lane of each operand, so
// LDS and L2 have time to spare).  One workgroup owns 32 query rows of one (stream, head); its four wavefronts
// share the rows and take every fourth block of 32 keys, each with a running maximum, row sum and O of its own
// that are merged at the end.  Keys are split inside the workgroup because fp32 problems have few rows: 32-row
// wavefronts without the split leave most SIMDs of the chip empty.
//   S^T[key][q] = K Q^T    A = K rows from LDS, 16 bytes (four steps) per read;  B = q in registers
//   O^T[d][q]  += V^T P^T  A = V straight from global memory (a step reads two 128-byte row pieces);
//                          B = the accumulator registers of S^T as they are: register r of half-wave hh is key
//                          8 (r / 4) + 4 hh + r % 4, and that key's row of V is what the lane loads.
// A wavefront's K block travels straight from global memory to its own 32 rows of LDS (no registers, no barrier:
// nobody else reads it), requested while the second product of the block before it runs.  The rows are not padded
// (the direct load writes 16 bytes per lane in lane order); instead the lane at chunk j of row r loads chunk
// j ^ r, so that the rows a fragment read touches lie on different banks.
// The products of a row with a key or with the state are summed in several chains that are added at the end: one chain of
// D products is the larger error of the two that an output has (relative to 64 bits, two chains for the state: 2.14e-7 ->
// 1.57e-7 at D = 128; logits of +-20, chains of 16 products at D = 128 and two chains at D = 64: 1.11e-6 -> 4.4e-7 and
// 8.1e-7 -> 5.2e-7; a vector-ALU kernel with 16 lanes per row has 2.09e-7, 7.8e-7 and 7.9e-7).
// Measured, 12 heads x 128, 1560 tokens (15.7 GFLOP, 102 us at the 154 TFLOP/s that a large fp32 matrix product
// reaches): 194 us; the vector-ALU kernel, 16 lanes per query row and two passes over the keys, took 7160 us.
// 2 heads x 64, 64 tokens: 8.7 us against 38 us.
template <int D>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(FwdArgs a, int n_rb)
{
    constexpr int KT = D / 8;                 // 16-byte pieces of a row per half-wave
    constexpr int DB = D / 32;                // 32-feature blocks
    constexpr int CPR = D / 4;                // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;             // rows per direct load
    constexpr int NW = 4;                     // wavefronts = key groups
    constexpr int KBUF = 32 * D * 4;          // bytes of a K block, and of a wavefront's O
    __shared__ __attribute__((aligned(16))) unsigned char smem[NW * KBUF];
    __shared__ float ml[NW][2][32];           // maximum and row sum of each wavefront's share, per query row

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hh = lane >> 5, c = lane & 31;
    const int H = a.H, Lq = a.Lq, Lkv = a.Lkv;
    const int work = xcd_contiguous_id(blockIdx.x, gridDim.x);      // the row blocks of a head share an XCD's L2
    const int bh = work / n_rb, q0 = (work % n_rb) * 32;
    const int h = bh % H, b = bh / H;
    const int row = q0 + c;
    const bool valid = row < Lq;
    const uint32_t tok = (uint32_t)H * D * 4;                       // bytes of one token, all heads
    const size_t row_off = (((size_t)b * Lq + (valid ? row : q0)) * H + h) * D;
    const float *kg = (const float *)a.k + ((size_t)b * Lkv * H + h) * D;
    const float *vg = (const float *)a.v + ((size_t)b * Lkv * H + h) * D;

    // B operand of S^T: lane (row c, hh) holds features 8 t + 4 hh + 0..3 of its row
    f32x4 q[KT];
    auto load_q = [&](const float *src) {
        f32x4 ss = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            q[t] = *(const f32x4 *)(src + row_off + 8 * t + 4 * hh);
#pragma unroll
            for (int j = 0; j < 4; ++j) ss[j] = fmaf(q[t][j], q[t][j], ss[j]);
        }
        return xhalf_sum((ss[0] + ss[1]) + (ss[2] + ss[3]));
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
    float vr[2][4][DB];                       // V rows of four accumulator registers, current and next
    uint32_t v_off;                           // of this lane in the block's first row: 4 hh tokens and 4 c bytes
    auto fetch_v = [&](__amdgpu_buffer_rsrc_t r, auto quad_) {
        constexpr int quad = decltype(quad_)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                vr[quad & 1][j][db] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(r, v_off + (uint32_t)(8 * quad + j) * tok + 128 * db, 0, 0));
    };

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    // running maximum of the scaled logits (finite also while every logit was -inf); this lane's share of the row sum
    float m = -FLT_MAX, l = 0.f;

    if (wave < nblk) fetch_k(wave);
#pragma unroll 1
    for (int blk = wave; blk < nblk; blk += NW) {
        const __amdgpu_buffer_rsrc_t v_rsrc = rsrc_of(vg, blk);
        v_off = 4 * hh * tok + 4 * c;
        asm volatile("" : "+v"(v_off));       // (one offset and not sixteen kept over the loop)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // the K block has landed
        fetch_v(v_rsrc, std::integral_constant<int, 0>{});
        f32x16 s = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, s1 = s;
        if constexpr (D == 64) {                                    // even and odd steps
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const f32x4 ka = *(const f32x4 *)(kbuf + c * (D * 4) + 16 * ((2 * t + hh) ^ (c % CPR)));
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[j], q[t][j], s, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[j + 1], q[t][j + 1], s1, 0, 0, 0);
                }
            }
            s += s1;
        } else {                                                    // eight steps from zero, added up while the next eight run
            static_for<0, KT / 2 + 1>([&](auto g_) {
                constexpr int g = decltype(g_)::value;
                const f32x16 done = s1;
                if constexpr (g < KT / 2) {
                    f32x16 r = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                    static_for<2 * g, 2 * g + 2>([&](auto t_) {
                        constexpr int t = decltype(t_)::value;
                        const f32x4 ka = *(const f32x4 *)(kbuf + c * (D * 4) + 16 * ((2 * t + hh) ^ (c % CPR)));
                        static_for<0, 4>([&](auto j_) {
                            constexpr int j = decltype(j_)::value;
                            r = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[j], q[t][j], r, 0, 0, 0);
                        });
                    });
                    s1 = r;
                }
                if constexpr (g > 0) {
                    s = g == 1 ? done : s + done;
                    asm volatile("" : "+v"(s));                     // (otherwise all sums are kept and added at the end)
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the K block has been read: it may be overwritten
        if (blk + NW < nblk) fetch_k(blk + NW);

        if (32 * blk + 32 > Lkv) {                                  // keys past the end (last block only)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * blk + 8 * (r >> 2) + 4 * hh + (r & 3) >= Lkv) s[r] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        const float m_new = fmaxf(m, xhalf_max(mx) * a.sm_scale);
        if (__any(m_new > m)) {
            const float alpha = expf(m - m_new);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = expf(fmaf(s[r], a.sm_scale, -m));
            l += s[r];
        }
        static_for<0, 4>([&](auto quad_) {
            constexpr int quad = decltype(quad_)::value;
            if constexpr (quad < 3) fetch_v(v_rsrc, std::integral_constant<int, quad + 1>{});
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[quad & 1][j][db], s[4 * quad + j], o[db], 0, 0, 0);
        });
    }

    // ---- merge the four shares: everything relative to the largest maximum
    l = xhalf_sum(l);
    if (hh == 0) {
        ml[wave][0][c] = m;
        ml[wave][1][c] = l;
    }
    __syncthreads();                                                // also: no K block is read any more
    float m_all = ml[0][0][c];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, ml[w][0][c]);
    float l_all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l_all = fmaf(ml[w][1][c], expf(ml[w][0][c] - m_all), l_all);
    const float f = expf(m - m_all);
    float *ox = (float *)smem;                                      // [wavefront][feature block][register][lane]
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) ox[((wave * DB + db) * 16 + r) * 64 + lane] = o[db][r] * f;
    __syncthreads();
    // from here on a wavefront owns 32 output features
    if (wave >= DB) return;
    f32x16 out;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += ox[((w * DB + wave) * 16 + r) * 64 + lane];
        out[r] = s / l_all;
    }

    if (a.S != nullptr) {
        if (a.q_lin != nullptr) qss = load_q((const float *)a.q_lin);   // the linear branch's own query (Eq. (3))
        const float rq = 1.0f / sqrtf(qss + a.l2_eps);
        const float *Sg = a.S + (size_t)bh * D * D + 32 * wave + c;
        f32x16 inter = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, inter1 = inter;   // even and odd steps
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
                inter = __builtin_amdgcn_mfma_f32_32x32x2f32(Sg[(8 * t + 4 * hh + j) * D], q[t][j], inter, 0, 0, 0);
                inter1 = __builtin_amdgcn_mfma_f32_32x32x2f32(Sg[(8 * t + 4 * hh + j + 1) * D], q[t][j + 1], inter1, 0, 0, 0);
            }
        inter += inter1;
        const size_t gtok = (size_t)b * Lq + (valid ? row : q0);
        const size_t gi = a.g_per_token ? gtok : gtok * H + h;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float g = 1.0f;                  // headwise or per-token gate, or one gate per output feature
            if (a.g != nullptr) {
                const size_t ge = a.g_per_element ? gi * D + 32 * wave + 8 * (r >> 2) + 4 * hh + (r & 3) : gi;
                g = a.g_is_bf16 ? (float)((const bf16_t *)a.g)[ge] : ((const float *)a.g)[ge];
            }
            out[r] = fmaf(g, inter[r] * rq, out[r]);
        }
    }
    if (valid) {
        float *og = (float *)a.out + row_off + 32 * wave + 4 * hh;
#pragma unroll
        for (int p = 0; p < 4; ++p) *(f32x4 *)(og + 8 * p) = f32x4{out[4 * p], out[4 * p + 1], out[4 * p + 2], out[4 * p + 3]};
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

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs &a, hipStream_t stream)
{
    const int n_rb = (a.Lq + 31) / 32;
    const long long nwg = (long long)n_rb * a.B * a.H;
    if (nwg <= 0 || nwg > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg), block(256);
    if (a.D == 64) return launch_kernel(fwd_f32_kernel<64>, grid, block, stream, a, n_rb);
    if (a.D == 128) return launch_kernel(fwd_f32_kernel<128>, grid, block, stream, a, n_rb);
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
