// Branch-mix gate on bf16 MFMA (gfx950):
//   G[b][l][n] = sigmoid( sum_j x[b][l][j] Wg[n][j] )                        paper Eq. (6)
// x is the layer's hidden state [B][L][dm], dm = H D; Wg holds one row of dm weights per gate output:
// one per head (the paper's headwise gate) or a single one (the scalar gate of its gate ablation, Tab. 4).
// HBM-bound: x is read once (2 H flop per byte).  Computed transposed, G^T[h][l] = Wg x^T, so that both
// operands are read as rows; the H <= 32 heads occupy the rows of one 32 x 32 MFMA tile (rows >= H are
// zero).  One workgroup owns 32 tokens and walks the hidden dimension in chunks of 512 columns: the chunk
// of x travels HBM -> registers -> LDS as whole 1 KB row pieces (fragment loads straight from global
// memory touch 32 cache lines per instruction and made the kernel request-bound), two LDS buffers, the
// next chunk in flight while the four wavefronts each contract a quarter of the current one; their
// partial sums are added in LDS.
//
// More than 32 gate outputs per token (the element-wise gate of the same ablation, one per feature: Wg is
// dm x dm) make the projection a dense matrix product and MFMA-bound: gate_dense_kernel below.
#include "arl2_device.h"

#include <type_traits>

namespace arl2 {
namespace {

constexpr int NT = 256;
constexpr int CW = 512;                  // columns of x per chunk
constexpr int XROW = 2 * CW + 16;        // LDS bytes per token row of a chunk (conflict-free 16-byte reads)
constexpr int XCH = 32 * (2 * CW / 16) / NT;   // 16-byte pieces of a chunk per thread

__global__ __launch_bounds__(NT) void gate_proj_kernel(GateArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char xs[2][32 * XROW];
    static_assert(sizeof(float) * 4 * 16 * 64 <= 32 * XROW, "the partial sums reuse the first chunk buffer");
    float (*part)[16][64] = reinterpret_cast<float (*)[16][64]>(&xs[0][0]);   // [wavefront][register][lane], after the last chunk
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, hh = lane >> 5, c = lane & 31;
    const int dm = a.dm, H = a.n_out;                    // rows of Wg = gate outputs per token
    const long long tok0 = (long long)blockIdx.x * 32;   // first token (over streams and chunk positions)
    const long long ntok = (long long)a.B * a.L;

    const uint32_t x_bytes = (uint32_t)(ntok * dm * 2), w_bytes = (uint32_t)H * dm * 2;
    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(a.x, x_bytes);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(a.Wg, w_bytes);
    // lanes whose head does not exist read zeros
    const uint32_t w_row = c < H ? (uint32_t)c * dm * 2 : w_bytes;

    // piece i of this thread in a chunk: token row (tid + NT i) / 64, 16-byte column (tid + NT i) % 64
    const int nchunk = (dm + CW - 1) / CW;
    // Three chunks are requested at once (one memory latency for 1536 columns, the hidden size of the
    // paper's model), then staged and contracted one after the other.
    constexpr int GRP = 3;
    u32x4 xr[GRP][XCH];
    auto fetch = [&](int ch, auto j_) {                  // chunk ch of the 32 token rows into register set j
        constexpr int j = decltype(j_)::value;
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            const int id = tid + NT * i, row = id / (2 * CW / 16), col = id % (2 * CW / 16);
            const int colb = 2 * CW * ch + 16 * col;                       // byte column in the row of x
            const bool ok = tok0 + row < ntok && colb < 2 * dm;
            xr[j][i] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, ok ? (uint32_t)((tok0 + row) * dm * 2 + colb) : x_bytes, 0, 0);
        }
    };
    f32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int KS = CW / 16 / 4;                      // k-steps of a chunk per wavefront
    auto contract = [&](int ch, auto j_) {               // stage register set j as chunk ch, then this wavefront's quarter of it
        constexpr int j = decltype(j_)::value;
        unsigned char *buf = xs[ch & 1];
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            const int id = tid + NT * i, row = id / (2 * CW / 16), col = id % (2 * CW / 16);
            *(u32x4 *)(buf + row * XROW + 16 * col) = xr[j][i];
        }
        // A = Wg rows from global memory (few rows, L2-resident)
        union { u32x4 u; bf16x8 v; } wa[KS];
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const uint32_t colb = 2 * CW * ch + 32 * (KS * wave + i) + 16 * hh;
            wa[i].u = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, (w_row < w_bytes && colb < (uint32_t)(2 * dm)) ? w_row + colb : w_bytes, 0, 0);
        }
        __syncthreads();                                 // the chunk is in LDS (the other buffer was last read a barrier ago)
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const bf16x8 xb = *(const bf16x8 *)(buf + c * XROW + 32 * (KS * wave + i) + 16 * hh);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[i].v, xb, acc, 0, 0, 0);
        }
    };
    const std::integral_constant<int, 0> J0{};
    const std::integral_constant<int, 1> J1{};
    const std::integral_constant<int, 2> J2{};
    for (int ch = 0; ch < nchunk; ch += GRP) {           // chunks past the last one read zeros and are skipped
        fetch(ch, J0);
        if (ch + 1 < nchunk) fetch(ch + 1, J1);
        if (ch + 2 < nchunk) fetch(ch + 2, J2);
        contract(ch, J0);
        if (ch + 1 < nchunk) contract(ch + 1, J1);
        if (ch + 2 < nchunk) contract(ch + 2, J2);
    }
    __syncthreads();                                     // every wavefront has read its last chunk
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][r][lane] = acc[r];
    __syncthreads();
    // thread (register r, lane) of the first 1024 elements: head n = 8 (r / 4) + 4 hh + r % 4, token tok0 + c
    for (int i = tid; i < 16 * 64; i += NT) {
        const int r = i >> 6, ln = i & 63;
        const int n = 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3);
        const long long tok = tok0 + (ln & 31);
        if (n < H && tok < ntok) {
            const float s = (part[0][r][ln] + part[1][r][ln]) + (part[2][r][ln] + part[3][r][ln]);
            const float g = 1.0f / (1.0f + __expf(-s));
            if (a.g_is_bf16) ((bf16_t *)a.g)[tok * H + n] = to_bf16(g);
            else ((float *)a.g)[tok * H + n] = g;
        }
    }
}

// ---- dense projection: G[tok][n] = sigmoid( sum_j x[tok][j] Wg[n][j] ) for any number of outputs n ----
// One workgroup owns TM tokens x TN outputs, each wavefront 64 tokens x TN / WN outputs (2 x NB MFMA
// blocks).  The hidden dimension is walked in steps of 64 columns: the 128-byte row pieces of x and Wg
// travel straight from memory into one of ST LDS stages, up to ST - 1 steps ahead, one barrier per step.  (The
// 16-byte chunks of a row are stored at chunk ^ (row / 2 % 8): a fragment read touches one chunk of 32 rows, which would
// share banks otherwise, and a direct load leaves no room for padding.)  Three shapes:
//   128 x 128, four wavefronts, four stages    while every workgroup has a CU to itself: nothing else hides its loads
//   128 x 128, four wavefronts, two stages     two workgroups per CU, one multiplies while the other waits
//   256 x 256, eight wavefronts of 64 x 128    large problems: half the LDS and L2 traffic per flop
// Bound by the matrix cores inside a round (about two thirds busy with two workgroups per CU), outside it by the launch,
// the first loads and the last stores, about 10 us.  Measured against loads through registers into padded LDS rows, fp32
// gate, dm outputs of dm columns: 4680 tokens, dm 1536 39.9 -> 31.5 us; 1560 tokens 25.0 -> 19.7 us; 18720 tokens
// 129 -> 106 us; 37440 tokens 235 -> 209 us; 999 tokens, dm 320 10.8 -> 9.2 us.  A 256 x 128 shape was nowhere better than
// the best of these by more than 4 %.
constexpr int GK = 64;                        // hidden columns per step
constexpr int GROW = 2 * GK;                  // LDS bytes per staged row piece

template <int TM, int TN, int NTH, int ST>
__global__ __launch_bounds__(NTH, NTH / 256) void gate_dense_kernel(GateArgs a, int n_ntile)
{
    constexpr int NW = NTH / 64;
    constexpr int WM = TM / 64, WN = NW / WM;            // wavefronts along tokens, along outputs
    constexpr int NB = TN / WN / 32;                     // 32-output blocks per wavefront
    constexpr int XP = TM / 8 / NW, WP = TN / 8 / NW;    // loads of 8 rows per wavefront and step: x, Wg
    constexpr int STG = (TM + TN) * GROW;
    constexpr int OROW = 64 + 4, OBYTES = 32 * OROW * 4; // 32 tokens x 64 outputs of a wavefront on their way out
    static_assert(WM * WN == NW && NB * 32 * WN == TN && XP * 8 * NW == TM && WP * 8 * NW == TN && NB % 2 == 0, "tile shape");
    static_assert(ST >= 2 && ST * STG <= 160 * 1024, "stages");
    static_assert(NW * OBYTES <= ST * STG, "the wavefronts' output tiles reuse the stages");
    __shared__ __attribute__((aligned(1024))) unsigned char sm[ST * STG];   // [stage][x rows, Wg rows]
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hh = lane >> 5, c = lane & 31;
    const int wm = wave % WM, wn = wave / WM;
    const int dm = a.dm, N = a.n_out;
    const long long ntok = (long long)a.B * a.L;
    // consecutive workgroups of an XCD share a token tile and walk over the outputs: x is fetched once
    const int work = xcd_contiguous_id(blockIdx.x, gridDim.x);
    const long long tok0 = (long long)(work / n_ntile) * TM;
    const int n0 = (work % n_ntile) * TN;

    const uint32_t x_bytes = (uint32_t)(ntok * dm * 2), w_bytes = (uint32_t)((long long)N * dm * 2);
    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(a.x, x_bytes);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(a.Wg, w_bytes);
    const int nk = dm / GK;                              // dm is a multiple of 64

    // Load i of this wavefront fills the rows 8 (NW i + wave) + 0..7, lane = (row lane / 8, chunk lane % 8).  Byte
    // offsets at step 0; rows past the end point beyond the buffer at every step (and read as zero)
    const uint32_t colb = 16 * ((lane & 7) ^ (4 * (wave & 1) + (lane >> 4)));
    uint32_t xoff[XP], woff[WP];
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const long long row = tok0 + 8 * (NW * i + wave) + (lane >> 3);
        xoff[i] = row < ntok ? (uint32_t)(row * dm * 2) + colb : 0x80000000u;
    }
#pragma unroll
    for (int i = 0; i < WP; ++i) {
        const long long row = n0 + 8 * (NW * i + wave) + (lane >> 3);
        woff[i] = row < N ? (uint32_t)(row * dm * 2) + colb : 0x80000000u;
    }
    const uint32_t lds0 = lds_address(sm) + 1024 * wave;
    auto fetch = [&](int kc, int st) __attribute__((always_inline)) {   // step kc into stage st; XP + WP loads also past the last step
        const uint32_t kb = kc < nk ? 2 * GK * kc : 0x80000000u;
#pragma unroll
        for (int i = 0; i < XP; ++i) load_to_lds(x_rsrc, kc < nk ? xoff[i] + kb : kb, lds0 + st * STG + 1024 * NW * i);
#pragma unroll
        for (int i = 0; i < WP; ++i) load_to_lds(w_rsrc, kc < nk ? woff[i] + kb : kb, lds0 + st * STG + TM * GROW + 1024 * NW * i);
    };
    f32x16 acc[2][NB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // fragments of one 16-column k-step of a stage, in two sets: the next k-step is read while the current one is multiplied
    bf16x8 xa[2][2], wb[2][NB];
    const unsigned char *xs = sm + (64 * wm + c) * GROW, *ws = sm + (TM + 32 * NB * wn + c) * GROW;
    const int swz = (c >> 1) & 7;                        // the same for all rows c + 32 i
    auto read = [&](int st, auto t_) __attribute__((always_inline)) {
        constexpr int t = decltype(t_)::value;
        const int ch = st * STG + 16 * ((2 * t + hh) ^ swz);
#pragma unroll
        for (int i = 0; i < 2; ++i) xa[t & 1][i] = *(const bf16x8 *)(xs + 32 * i * GROW + ch);
#pragma unroll
        for (int j = 0; j < NB; ++j) wb[t & 1][j] = *(const bf16x8 *)(ws + 32 * j * GROW + ch);
    };
    auto multiply = [&](auto t_) __attribute__((always_inline)) {
        constexpr int t = decltype(t_)::value;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[t & 1][i], wb[t & 1][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int T = GK / 16;

    // Step kc lives in stage kc % ST.  A step's barrier stands before its last k-step, whose fragments are in registers by
    // then: past it every wavefront has read the stage, which takes the loads of step kc + ST, and the first fragments of
    // step kc + 1 arrive under the last products.  The loads of the ST - 2 steps after that may still be in flight.
    static_for<0, ST>([&](auto s_) { fetch(decltype(s_)::value, decltype(s_)::value); });
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((ST - 1) * (XP + WP)) : "memory");
    read(0, std::integral_constant<int, 0>{});
    for (int k0 = 0; k0 < nk; k0 += ST) {
        static_for<0, ST>([&](auto s_) __attribute__((always_inline)) {
            constexpr int st = decltype(s_)::value;
            if (k0 + st >= nk) return;                   // uniform over the workgroup
            static_for<0, T - 1>([&](auto t_) __attribute__((always_inline)) {
                read(st, std::integral_constant<int, decltype(t_)::value + 1>{});
                multiply(t_);
            });
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((ST - 2) * (XP + WP)) : "memory");
            fetch(k0 + st + ST, st);
            read((st + 1) % ST, std::integral_constant<int, 0>{});
            multiply(std::integral_constant<int, T - 1>{});
        });
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // nothing in flight, every stage read

    // Epilogue through LDS, a wavefront for itself, 32 tokens x 64 outputs at a time: accumulator register r of block (i, j)
    // is token 64 wm + 32 i + 8 (r / 4) + 4 hh + r % 4, output 32 (NB wn + j) + c; the rows are read back 16 bytes of
    // fp32 per lane, so that a store instruction writes four row pieces of 256 bytes.
    float *ot = reinterpret_cast<float *>(sm + wave * OBYTES);
    const bool vec = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(a.g) & 15) == 0;   // every row of g starts 16-byte (bf16: 8-byte) aligned
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jp = 0; jp < NB; jp += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) ot[(8 * (r >> 2) + 4 * hh + (r & 3)) * OROW + 32 * j + c] = acc[i][jp + j][r];
#pragma unroll
            for (int it = 0; it < 8; ++it) {             // (a wavefront's LDS operations complete in order)
                const int row = 4 * it + (lane >> 4), n = n0 + 32 * (NB * wn + jp) + 4 * (lane & 15);
                const long long tok = tok0 + 64 * wm + 32 * i + row;
                f32x4 s = *(const f32x4 *)(ot + row * OROW + 4 * (lane & 15));
                if (tok >= ntok || n >= N) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = 1.0f / (1.0f + __expf(-s[e]));
                if (vec) {
                    if (a.g_is_bf16) {
                        bf16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = to_bf16(s[e]);
                        *(bf16x4 *)((bf16_t *)a.g + tok * N + n) = o;
                    } else {
                        *(f32x4 *)((float *)a.g + tok * N + n) = s;
                    }
                } else {
                    for (int e = 0; e < 4 && n + e < N; ++e) {
                        if (a.g_is_bf16) ((bf16_t *)a.g)[tok * N + n + e] = to_bf16(s[e]);
                        else ((float *)a.g)[tok * N + n + e] = s[e];
                    }
                }
            }
        }
}

template <int TM, int TN, int NTH, int ST>
hipError_t launch_gate_dense(const GateArgs &a, long long ntok, hipStream_t stream)
{
    const long long n_ntile = (a.n_out + TN - 1) / TN, n_mtile = (ntok + TM - 1) / TM;
    if (n_mtile * n_ntile > 0x7fffffffLL) return hipErrorInvalidValue;
    return launch_kernel(gate_dense_kernel<TM, TN, NTH, ST>, dim3((unsigned)(n_mtile * n_ntile)), dim3(NTH), stream, a, (int)n_ntile);
}

}  // namespace

hipError_t launch_gate_proj_bf16(const GateArgs &a, hipStream_t stream)
{
    const long long ntok = (long long)a.B * a.L;
    const long long nwg = (ntok + 31) / 32;
    if (nwg <= 0 || nwg > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.n_out < 1 || a.dm % 16 != 0) return hipErrorInvalidValue;
    // x and Wg are addressed with 32-bit byte offsets
    if (ntok * a.dm * 2 > 0x7fffffffLL || (long long)a.n_out * a.dm * 2 > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.n_out > 32) {
        if (a.dm % GK != 0) return hipErrorInvalidValue;
        // One workgroup per CU: 128 x 128 with deep stages (256 tiles of dm 2048: 25.1 us, with two stages 28.8).  Beyond,
        // the shape with the shorter sum of rounds, one of large tiles taking as long as about 1.5 of small ones
        // (measured 1.47 to 1.6): 564 small or 144 large tiles of dm 1536 47.9 and 46.5 us, 1764 or 444 128 and 106 us,
        // 444 or 114 31.5 and 47.7 us; 1512 or 384 of dm 3072, where the rule is indifferent, 171 and 169 us.
        const long long small = ((ntok + 127) / 128) * ((a.n_out + 127) / 128), big = ((ntok + 255) / 256) * ((a.n_out + 255) / 256);
        if (small <= kNumCu) return launch_gate_dense<128, 128, 256, 4>(a, ntok, stream);
        const long long small_rounds = (small + 2 * kNumCu - 1) / (2 * kNumCu), big_rounds = (big + kNumCu - 1) / kNumCu;
        return 3 * big_rounds <= 2 * small_rounds ? launch_gate_dense<256, 256, 512, 2>(a, ntok, stream)
                                                  : launch_gate_dense<128, 128, 256, 2>(a, ntok, stream);
    }
    return launch_kernel(gate_proj_kernel, dim3((unsigned)nwg), dim3(NT), stream, a);
}

}  // namespace arl2
