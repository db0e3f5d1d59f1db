// Post-denoise state commit on bf16 MFMA (gfx950):
//   S <- gate * S + sum_i k'_i^T v_i,   k'_i = k_i / sqrt(|k_i|^2 + eps)     paper Eq. (3), Eq. (4)
//
// HBM-bound: every k and v element is read once.  The contraction runs over tokens, so both MFMA
// operands are needed token-major per feature; 64-token tiles of K and V are written to LDS row-major
// (as they arrive, 16-byte pieces) and read back through the transposing LDS read
// (ds_read_b64_tr_b16), which hands every lane four tokens of one feature.  To keep the fp32 state
// accurate the raw bf16 K (exact) is one operand and the row-scaled values r_i * v_i, split into
// bf16 hi + lo parts, are the other (two MFMAs per step, error ~2^-17; one bf16 rounding of the
// scaled values would cost ~1e-3 on the state).  The scale r_i = 1/sqrt(|k_i|^2 + eps) is computed
// from the K registers on their way to LDS (lane shuffles across the 16 lanes that share a row).
//
// Tokens are split over `nsplit` workgroups per (stream, head); each keeps the next tiles' loads in
// flight while it works on the current one and finally writes a D x D fp32 partial to the workspace.
// A second kernel adds the partials in split order and applies the gate to the old state, so the
// result is bit-identical from run to run (no floating-point atomics).
//
// Delta-rule variant (Eq. (4) literally, frame level):
//   S <- alpha S + beta K'^T (V - K' S)
// The partial kernel forms V - K' S tile by tile from the old state, which nothing writes before the reduce.
#include "arl2_device.h"

#include <type_traits>

namespace arl2 {
namespace {

constexpr int BT = 64;    // tokens per tile
constexpr int NT = 512;    // partial kernel: 8 wavefronts, two per SIMD
constexpr int NTR = 256;   // reduce kernels


constexpr int PFW = 3;     // tiles whose loads the plain commit's producer wavefronts keep in flight: HBM latency is several tile times
constexpr int PFD = 2;     // the same for the delta rule, which has fewer registers left (a third tile spills)

template <int D>
struct CommitCfg {
    static constexpr int CPR = D / 8;                   // 16-byte chunks per row
    static constexpr int ROW = 2 * D + 64;              // LDS bytes per tile row (conflict-free transposing reads)
    static constexpr int MAT = BT * ROW;                // one 64-token tile
    static constexpr int STAGE = 3 * MAT;               // K, V' hi, V' lo
    static constexpr int DH = D / 64;                   // 64-row halves of the output
    static constexpr int EB = D / 32;                   // 32-column blocks of the output
};

// Plain commit, producer / consumer form.  Staging a tile (row norms, scaling, hi/lo
// split: vector ALU) and contracting it (MFMA) take about the same time, and a wavefront does not overlap
// its own VALU work with its own MFMAs: wavefronts 0..3 (one per SIMD) only fetch and stage tile i + 1 into
// the other LDS stage while wavefronts 4..7 (one per SIMD) only run the MFMAs of tile i, each on a 64 x 64
// block of the partial; one workgroup barrier per tile hands the stages over.
template <int D>
__global__ __launch_bounds__(NT, 2) void commit_partial_ws_kernel(CommitArgs a)
{
    using C = CommitCfg<D>;
    constexpr int PT = NT / 2;                           // producer threads
    constexpr int KCHP = BT * C::CPR / PT;               // chunks per producer thread per tile (K and V each)
    constexpr int RPP = PT / C::CPR;                     // rows per pass of the producers
    constexpr int NE = D / 64;                           // 32-column blocks per consumer wavefront
    static_assert(KCHP >= 1 && NE >= 1, "unsupported head dimension");
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * C::STAGE];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hh = lane >> 5;
    const bool producer = wave < 4;
    const int split = blockIdx.x % a.nsplit;
    const int bh = blockIdx.x / a.nsplit;
    const int h = bh % a.H, b = bh / a.H;
    const int L = a.L, H = a.H;
    const uint32_t tok_bytes = (uint32_t)H * D * 2;
    const bf16_t *kg = (const bf16_t *)a.k + ((size_t)b * L * H + h) * D;
    const bf16_t *vg = (const bf16_t *)a.v + ((size_t)b * L * H + h) * D;
    const uint32_t range = (uint32_t)(L - 1) * tok_bytes + 2 * D;      // bytes of this head's slice
    const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(kg, range);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(vg, range);

    const int ntiles = (L + BT - 1) / BT;
    const int t_begin = (int)((long long)split * ntiles / a.nsplit);
    const int t_end = (int)((long long)(split + 1) * ntiles / a.nsplit);
    const int n = t_end - t_begin;

    // ---- producers: chunk i of a thread is row (tid / CPR) + RPP * i, 16-byte column tid % CPR
    const int lds_off = (tid / C::CPR) * C::ROW + 16 * (tid % C::CPR);
    u32x4 kr[PFW][KCHP], vr[PFW][KCHP];
    auto load_tile = [&](int tile, auto buf_) {     // a tile that is not this workgroup's is not requested
        constexpr int buf = decltype(buf_)::value;
        const uint32_t base = tile < t_end ? ((uint32_t)tile * BT + tid / C::CPR) * tok_bytes + 16 * (tid % C::CPR) : 0x80000000u;
#pragma unroll
        for (int i = 0; i < KCHP; ++i) {
            const uint32_t off = base + (uint32_t)i * RPP * tok_bytes;
            kr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off, 0, 0);
            vr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off, 0, 0);
        }
    };
    auto stage_tile = [&](int stage, auto buf_) {   // K as it is, and r * V split into bf16 hi + lo
        constexpr int buf = decltype(buf_)::value;
        unsigned char *sm = smem + stage * C::STAGE + lds_off;
#pragma unroll
        for (int i = 0; i < KCHP; ++i) {
            float ss = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float lo = __uint_as_float(kr[buf][i][w] << 16);
                const float hi = __uint_as_float(kr[buf][i][w] & 0xffff0000u);
                ss = fmaf(lo, lo, ss);
                ss = fmaf(hi, hi, ss);
            }
            ss = lane_group_sum<C::CPR>(ss);
            const float rn = fast_rsqrt(ss + a.l2_eps);
            // r * v as bf16 hi (truncated) + lo (rounded remainder): both members of a pair packed into one word
            u32x4 vh, vl;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t h0, h1;
                float l0, l1;
                split_bf16_trunc(__uint_as_float(vr[buf][i][w] << 16) * rn, h0, l0);
                split_bf16_trunc(__uint_as_float(vr[buf][i][w] & 0xffff0000u) * rn, h1, l1);
                vh[w] = (h0 >> 16) | h1;
                union { bf16x2 v; uint32_t u; } pk;
                pk.v[0] = to_bf16(l0);
                pk.v[1] = to_bf16(l1);
                vl[w] = pk.u;
            }
            unsigned char *p = sm + i * RPP * C::ROW;
            *(u32x4 *)(p) = kr[buf][i];
            *(u32x4 *)(p + C::MAT) = vh;
            *(u32x4 *)(p + 2 * C::MAT) = vl;
        }
    };

    // ---- consumers: wavefront 4 + cw owns rows 64 dh .. 64 dh + 63, column blocks e0 .. e0 + NE - 1
    const int cw = wave - 4;
    const bool consumer = !producer && cw * NE < C::DH * C::EB;
    const int dh = (cw * NE) / C::EB, e0 = (cw * NE) % C::EB;
    const int tr_off = (((lane & 15) >> 2) + 4 * hh) * C::ROW + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    f32x16 acc[2][NE];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][e][r] = 0.f;
    auto consume = [&](int stage) {
        const unsigned char *sm = smem + stage * C::STAGE + tr_off;
        // operand fragments of 16-token step t: tokens 16t + 4hh + 0..3 and 16t + 8 + 4hh + 0..3
        bf16x8 ka[2][2], bh_[2][NE], bl_[2][NE];
        auto load_step = [&](int t, int buf) {
            const unsigned char *row = sm + 16 * t * C::ROW;
#pragma unroll
            for (int i = 0; i < 2; ++i) ka[buf][i] = lds_read_tr_pair(row + 64 * (2 * dh + i), 8 * C::ROW);
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                bh_[buf][e] = lds_read_tr_pair(row + C::MAT + 64 * (e0 + e), 8 * C::ROW);
                bl_[buf][e] = lds_read_tr_pair(row + 2 * C::MAT + 64 * (e0 + e), 8 * C::ROW);
            }
        };
        load_step(0, 0);
#pragma unroll
        for (int t = 0; t < BT / 16; ++t) {
            if (t + 1 < BT / 16) load_step(t + 1, (t + 1) & 1);
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc[i][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[t & 1][i], bh_[t & 1][e], acc[i][e], 0, 0, 0);
                    acc[i][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[t & 1][i], bl_[t & 1][e], acc[i][e], 0, 0, 0);
                }
        }
    };

    // tile k of this workgroup (k = 0 .. n - 1) travels through register buffer k % PFW and LDS stage k % 2
    if (producer) {
        static_for<0, PFW>([&](auto i_) { load_tile(t_begin + decltype(i_)::value, i_); });
        if (n > 0) {
            stage_tile(0, std::integral_constant<int, 0>{});
            load_tile(t_begin + PFW, std::integral_constant<int, 0>{});
        }
    }
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += PFW) {
        static_for<0, PFW>([&](auto j_) {
            constexpr int j = decltype(j_)::value;
            const int i = i0 + j;
            if (i >= n) return;                          // uniform over the workgroup
            if (producer) {
                if (i + 1 < n) {
                    const std::integral_constant<int, (j + 1) % PFW> nb{};
                    stage_tile((i + 1) & 1, nb);
                    load_tile(t_begin + i + 1 + PFW, nb);
                }
            } else if (consumer) {
                consume(i & 1);
            }
            __syncthreads();
        });
    }

    // partial[bh][split][d][e]
    if (consumer) {
        float *part = (float *)a.workspace + ((size_t)bh * a.nsplit + split) * D * D;
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int d = 32 * (2 * dh + i) + 8 * (r >> 2) + 4 * hh + (r & 3);
                    const int col = 32 * (e0 + e) + (lane & 31);
                    part[(size_t)d * D + col] = acc[i][e][r];
                }
    }
}

// ---- delta rule: partial sums of K'^T (V - K' S) over this workgroup's tokens ------------------------------
// A wavefront owns 32 tokens of a tile and 32 columns of the state: it computes T = K S for them (A = token-major
// rows of K; B = the state's columns, held in registers for the whole walk as three bf16 parts: an error of the state is
// the same for every token and would add up), W = r (V - r T) in fp32 in the accumulator registers, and adds K^T W (A = K through the transposing read, B = W split into hi + lo, whose
// register order is the k-slot order of that read) to its D x 32 sums.  Nothing is exchanged between wavefronts
// before the end, where the token groups' sums are added in LDS.  The matrix work is little more than that of the expanded
// form K'^T V - (K'^T K') S (five products of K's size against four), but that form needs two D x D sums per split, a snapshot of the
// state and a third D x D x D product when the splits are added.
// Bound by latency: first loads, a few tiles of about 1.2 us each, the exchange at the end.  Measured with the reduce,
// 4 x 12 heads x 128, 1560 tokens (38 MB of keys and values): 23.6 us; the expanded form, five staged matrices per tile
// and a reduce of its own that multiplied by the state, took 40.3 us (24 + 18 of it in the kernels).  Largest error against
// 64 bits unchanged (rel 1.3e-6); with the state in two parts it was twice that at 6000 tokens.
template <int D>
struct DeltaCfg {
    static constexpr int CB = D / 32;                   // 32-column blocks
    static constexpr int TG = 8 / CB;                   // token groups: wavefronts that share a column block
    static constexpr int TT = 32 * TG;                  // tokens per tile
    static constexpr int CPR = D / 8;                   // 16-byte chunks per row
    static constexpr int ROW = 2 * D + 32;              // LDS bytes per row (conflict-free row and transposing reads)
    static constexpr int MAT = TT * ROW;
    static constexpr int STAGE = 2 * MAT + 4 * TT;      // K, V, r
    static constexpr int KCH = TT * CPR / NT;           // chunks per thread per tile (K and V each)
    static constexpr int RPP = NT / CPR;                // rows per pass
    static constexpr int OWN = 16 * CB / TG;            // accumulator registers that a token group adds up at the end
    static constexpr int XCH = TG * (TG - 1) * CB * OWN * 64 * 4;   // bytes exchanged there
    static constexpr int SMEM = 2 * STAGE > XCH ? 2 * STAGE : XCH;
};

template <int D>
__global__ __launch_bounds__(NT, 2) void commit_delta_partial_kernel(CommitArgs a)
{
    using C = DeltaCfg<D>;
    __shared__ __attribute__((aligned(16))) unsigned char smem[C::SMEM];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hh = lane >> 5, c = lane & 31;
    const int cb = wave % C::CB, tg = wave / C::CB;
    const int split = blockIdx.x % a.nsplit;
    const int bh = blockIdx.x / a.nsplit;
    const int h = bh % a.H, b = bh / a.H;
    const int L = a.L, H = a.H;
    const uint32_t tok_bytes = (uint32_t)H * D * 2;
    const bf16_t *kg = (const bf16_t *)a.k + ((size_t)b * L * H + h) * D;
    const bf16_t *vg = (const bf16_t *)a.v + ((size_t)b * L * H + h) * D;
    const uint32_t range = (uint32_t)(L - 1) * tok_bytes + 2 * D;      // bytes of this head's slice
    const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(kg, range);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(vg, range);

    const int ntiles = (L + C::TT - 1) / C::TT;
    const int t_begin = (int)((long long)split * ntiles / a.nsplit);
    const int t_end = (int)((long long)(split + 1) * ntiles / a.nsplit);

    // chunk i of this thread: row (tid / CPR) + RPP * i, 16-byte column tid % CPR; rows past the end read as zero, a
    // tile that is not this workgroup's is not requested
    u32x4 kr[PFD][C::KCH], vr[PFD][C::KCH];
    auto load_tile = [&](int tile, auto buf_) {
        constexpr int buf = decltype(buf_)::value;
        const uint32_t base = tile < t_end ? ((uint32_t)tile * C::TT + tid / C::CPR) * tok_bytes + 16 * (tid % C::CPR) : 0x80000000u;
#pragma unroll
        for (int i = 0; i < C::KCH; ++i) {
            const uint32_t off = base + (uint32_t)i * C::RPP * tok_bytes;
            kr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off, 0, 0);
            vr[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off, 0, 0);
        }
    };
    auto stage_tile = [&](unsigned char *st, auto buf_) {
        constexpr int buf = decltype(buf_)::value;
#pragma unroll
        for (int i = 0; i < C::KCH; ++i) {
            const int row = tid / C::CPR + C::RPP * i;
            float ss = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float lo = __uint_as_float(kr[buf][i][w] << 16);
                const float hi = __uint_as_float(kr[buf][i][w] & 0xffff0000u);
                ss = fmaf(lo, lo, ss);
                ss = fmaf(hi, hi, ss);
            }
            ss = lane_group_sum<C::CPR>(ss);
            unsigned char *p = st + row * C::ROW + 16 * (tid % C::CPR);
            *(u32x4 *)(p) = kr[buf][i];
            *(u32x4 *)(p + C::MAT) = vr[buf][i];
            if (tid % C::CPR == 0) *(float *)(st + 2 * C::MAT + 4 * row) = fast_rsqrt(ss + a.l2_eps);
        }
    };
    static_for<0, PFD>([&](auto i_) { load_tile(t_begin + decltype(i_)::value, i_); });

    // B operand of T: lane (column c, hh) holds rows 16 t + 8 hh + 0..7 of its column of the state
    bf16x8 sh[D / 16], sm[D / 16], sl[D / 16];
    {
        const float *Sg = a.S + (size_t)bh * D * D + 32 * cb + c;
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = Sg[(16 * t + 8 * hh + j) * D];
                sh[t][j] = to_bf16(x);
                const float x1 = x - (float)sh[t][j];
                sm[t][j] = to_bf16(x1);
                sl[t][j] = to_bf16(x1 - (float)sm[t][j]);
            }
    }
    f32x16 acc[C::CB];
#pragma unroll
    for (int d = 0; d < C::CB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[d][r] = 0.f;

    const int tr_off = (((lane & 15) >> 2) + 4 * hh) * C::ROW + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    for (int tile0 = t_begin; tile0 < t_end; tile0 += PFD) {
        static_for<0, PFD>([&](auto i_) {
            const int tile = tile0 + decltype(i_)::value;
            if (tile >= t_end) return;                  // uniform over the workgroup
            unsigned char *st = smem + ((tile - t_begin) & 1) * C::STAGE;
            stage_tile(st, i_);                         // waits for this tile's loads
            lds_barrier();                              // two stages: every wavefront is also done with the tile before last
            load_tile(tile + PFD, i_);
            const unsigned char *ks = st + 32 * tg * C::ROW;
            f32x16 tk = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < D / 16; ++t) {
                const bf16x8 ka = *(const bf16x8 *)(ks + c * C::ROW + 32 * t + 16 * hh);
                tk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, sh[t], tk, 0, 0, 0);
                tk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, sm[t], tk, 0, 0, 0);
                tk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, sl[t], tk, 0, 0, 0);
            }
            const float *rs = (const float *)(st + 2 * C::MAT) + 32 * tg + 4 * hh;
#pragma unroll
            for (int u = 0; u < 2; ++u) {               // 16 tokens: registers 8 u .. 8 u + 7 of T
                const unsigned char *kt = ks + tr_off + 16 * u * C::ROW;
                const bf16x8 v8 = lds_read_tr_pair(kt + C::MAT + 64 * cb, 8 * C::ROW);
                bf16x8 wh, wl;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 r4 = *(const f32x4 *)(rs + 16 * u + 8 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int j = 4 * q + e;
                        const float w = r4[e] * fmaf(-r4[e], tk[8 * u + j], (float)v8[j]);
                        wh[j] = to_bf16(w);
                        wl[j] = to_bf16(w - (float)wh[j]);
                    }
                }
#pragma unroll
                for (int d = 0; d < C::CB; ++d) {
                    const bf16x8 ka = lds_read_tr_pair(kt + 64 * d, 8 * C::ROW);
                    acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, wh, acc[d], 0, 0, 0);
                    acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, wl, acc[d], 0, 0, 0);
                }
            }
        });
    }

    // ---- the token groups' sums: group g adds and writes registers OWN g .. OWN g + OWN - 1, in group order
    __syncthreads();
    float *ex = (float *)smem;                          // [adding group][giving group][column block][register][lane]
    auto slot = [&](int to, int from) { return ex + (((to * (C::TG - 1) + from) * C::CB + cb) * C::OWN) * 64 + lane; };
    static_for<0, C::TG>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        if (tg == g) return;
        float *p = slot(g, tg - (tg > g ? 1 : 0));
#pragma unroll
        for (int r = 0; r < C::OWN; ++r) p[64 * r] = acc[(C::OWN * g + r) / 16][(C::OWN * g + r) % 16];
    });
    __syncthreads();
    float *part = (float *)a.workspace + ((size_t)bh * a.nsplit + split) * D * D + 32 * cb + c;
    static_for<0, C::TG>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        if (tg != g) return;
#pragma unroll
        for (int r = 0; r < C::OWN; ++r) {
            float sum = 0.f;
#pragma unroll
            for (int f = 0; f < C::TG; ++f)
                sum += f == g ? acc[(C::OWN * g + r) / 16][(C::OWN * g + r) % 16] : slot(g, f - (f > g ? 1 : 0))[64 * r];
            const int d = 32 * ((C::OWN * g + r) / 16) + 8 * ((C::OWN * g + r) % 16 >> 2) + 4 * hh + (r & 3);
            part[(size_t)d * D] = sum;
        }
    });
}

// S[bh] = gate[bh] * S[bh] + beta[bh] * sum_{split ascending} partial[bh][split]   (no beta: 1)
template <int NS>
__global__ __launch_bounds__(NTR) void commit_reduce_kernel(CommitArgs a, int vec_per_head)
{
    const int bh = blockIdx.x / (vec_per_head / NTR);
    const int vi = (blockIdx.x % (vec_per_head / NTR)) * NTR + threadIdx.x;
    const size_t head_elems = (size_t)vec_per_head * 4;
    const f32x4 *part = (const f32x4 *)((const float *)a.workspace + (size_t)bh * a.nsplit * head_elems) + vi;
    f32x4 *Sg = (f32x4 *)(a.S + (size_t)bh * head_elems);
    const float gate = a.gate[bh], beta = a.beta != nullptr ? a.beta[bh] : 1.f;
    const f32x4 old = Sg[vi];
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    // all loads of a batch are issued before the adds; the adds run in split order
    for (int s0 = 0; s0 < a.nsplit; s0 += NS) {
        f32x4 x[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            x[j] = (s0 + j < a.nsplit) ? part[(size_t)(s0 + j) * vec_per_head] : zero;
        }
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] += x[j][c];
    }
    f32x4 res;
#pragma unroll
    for (int c = 0; c < 4; ++c) res[c] = fmaf(gate, old[c], beta * sum[c]);
    Sg[vi] = res;
}

}  // namespace

int commit_nsplit(int B, int H, int L)
{
    const int ntiles = (L + BT - 1) / BT;
    const long long bh = (long long)B * H;
    long long want = (192 + bh - 1) / bh;      // enough workgroups in flight to saturate HBM
    if (want < 1) want = 1;
    if (want > ntiles) want = ntiles;
    if (want > 32) want = 32;
    return (int)want;
}

hipError_t launch_commit_reduce_bf16(const CommitArgs &a, hipStream_t stream)
{
    const int vec_per_head = a.D * a.D / 4;        // multiple of 256 for D in {64, 128}
    const long long rwg = (long long)a.B * a.H * (vec_per_head / NTR);
    if (rwg <= 0 || rwg > 0x7fffffffLL) return hipErrorInvalidValue;
    return launch_kernel(commit_reduce_kernel<8>, dim3((unsigned)rwg), dim3(NTR), stream, a, vec_per_head);
}

// The interface's workspace holds twice the plain commit's partial sums and one more per head; the delta rule, whose workgroups
// fill a CU each (254 registers), may use all of it.
int commit_delta_max_nsplit(int B, int H, int L) { return 2 * commit_nsplit(B, H, L) + 1; }

// Splits of the delta rule: one workgroup per CU where the workspace allows it, then as few as keep the longest split as short.
template <int D>
hipError_t launch_delta(CommitArgs a, hipStream_t stream)
{
    const int ntiles = (a.L + DeltaCfg<D>::TT - 1) / DeltaCfg<D>::TT;
    const long long bh = (long long)a.B * a.H;
    long long want = kNumCu / bh;
    if (want > a.nsplit) want = a.nsplit;
    if (want > ntiles) want = ntiles;
    if (want < 1) want = 1;
    const int per = (int)((ntiles + want - 1) / want);
    a.nsplit = (ntiles + per - 1) / per;
    const hipError_t e = launch_kernel(commit_delta_partial_kernel<D>, dim3((unsigned)(bh * a.nsplit)), dim3(NT), stream, a);
    return e != hipSuccess ? e : launch_commit_reduce_bf16(a, stream);
}

hipError_t launch_commit_bf16(const CommitArgs &a, hipStream_t stream)
{
    const long long nwg = (long long)a.B * a.H * a.nsplit;
    if (nwg <= 0 || nwg > 0x7fffffffLL || (a.D != 64 && a.D != 128)) return hipErrorInvalidValue;
    // the kernels address one stream's K (or V) with 32-bit byte offsets
    if ((long long)(a.L + 4 * BT) * a.H * a.D * 2 > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.beta != nullptr) return a.D == 128 ? launch_delta<128>(a, stream) : launch_delta<64>(a, stream);
    const hipError_t e = a.D == 128 ? launch_kernel(commit_partial_ws_kernel<128>, dim3((unsigned)nwg), dim3(NT), stream, a)
                                    : launch_kernel(commit_partial_ws_kernel<64>, dim3((unsigned)nwg), dim3(NT), stream, a);
    return e != hipSuccess ? e : launch_commit_reduce_bf16(a, stream);
}

}  // namespace arl2
