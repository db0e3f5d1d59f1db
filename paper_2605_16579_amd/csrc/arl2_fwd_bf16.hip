// Read-only denoising pass on bf16 MFMA (gfx950):
//   out = softmax(q k^T * sm_scale) v + g * L2Norm(q) S            paper Eq. (2), (3), (5), (6)
//
// One workgroup owns 256 query rows of one (stream, head): eight wavefronts with 32 of them each, or at D = 64 four with 64
// (`Whole`); or half a tile, 128 rows: eight wavefronts, two on the same rows with half of every key tile each (two key
// groups), or in launches of more tiles than CUs at D = 64 four with 32 rows each and one key group.  A SIMD has two
// wavefronts, of one workgroup or two, with 256 registers each.  Everything is computed transposed so that no operand is
// re-laid out between the two GEMMs:
//
//   S^T[kv][q]  = K[kv][:] . Q[q][:]      A = K tile rows from LDS,  B = Q fragments in registers
//   O^T[d][q]  += V^T[d][kv] . P^T[kv][q] A = V^T fragments from LDS, B = exp'd S^T accumulators
//
// With v_mfma_f32_32x32x16_bf16 a lane holds one query column (lane % 32) of the S^T
// accumulator, so the softmax row statistics are in-lane reductions plus one exchange
// between the two half-waves.  The accumulator registers of S^T are exactly a B operand of
// the second GEMM (k-slot j of half-wave hh is key 16t + 8(j/4) + 4hh + j%4); the matching
// V^T fragments come from the row-major V tile in LDS through the transposing LDS read
// (ds_read_b64_tr_b16), four keys per read.
//
// The unit of the schedule is a slot, the softmax of one 32-key block beside the first GEMM of the next block and the
// second GEMM of the previous one (see `slot`).  K/V tiles travel (buffer loads, zero beyond the last key) into an LDS
// ring with one workgroup barrier per tile: straight, requested two barriers ahead, or through registers (two key groups, and
// eight wavefronts at D = 64, where that is the faster by up to 3 %).  12 heads x 128, 14400 keys: 1.51 us per 64-key tile
// straight, 1.61 us through registers (on zeros, where power does not bound it, 1.09 and 1.15 us).  At 65 to 400 rows and
// 64 KB or more from token to token (256 heads x 128) straight copies are the slower by up to 7 %; 192 heads, 257 to 700 rows
// are 2 to 4 % the faster.  The softmax is optimistic: the running maximum
// starts as the first block's, probabilities are taken relative to it as it stands, and only when a lane's share of
// the row sum shows that a logit exceeded it by more than ~2^7 is the block maximum computed, the running maximum
// raised, the accumulators rescaled and the block redone.  This removes the per-block maximum reduction and the
// accumulator rescale from the steady state without changing the normalised result.  (Row sums use plain fp32 adds:
// the bf16 dot product measured far slower next to MFMAs, and so did 4 x 4 x 4 MFMAs against a matrix of ones.)
//
// Epilogue (fused linear readout): O_inter^T[e][q] = S^T[e][d] . Q^T[d][q] with the fp32
// state split into bf16 hi + lo parts, staged row-major through LDS and read
// transposed like V, the raw bf16 q fragments as B operand, and the L2 norm of q applied as an
// fp32 per-column scale.  The linear branch may read a query of its own (Eq. (3): RoPE(phi_q(Q))):
// either given as an array, or computed here from the pre-map rows and the head's D x D matrix, in
// which case the rotated, rounded accumulators of that small GEMM are used as the B fragments
// directly.  The gate is one value per (token, head) (Eq. (6)), per token, or per output feature.
//
// What bounds it: the matrix cores and, on real data, the power they draw (a launch that fills the chip holds the
// clock at 1.73 to 1.83 GHz, by card).  Measured for one pass with state and gate, 12 heads x 128:
//   4680 tokens (228 tiles of 256 rows)   123 us; 3 x 24 heads x 64, 999 tokens (288 tiles) 28 us; 1560 tokens (156 half tiles) 26.5 us, 38 us with 84 whole tiles;
//   2 x 3 heads, 328 tokens (18 half tiles) 11.9 us, 15.6 us with 12 whole ones (17 us with query rows loaded fragment by
//   fragment, the tiles of the prologue one after the other and the first block's exponentials computed twice).
#include "arl2_device.h"

#include <type_traits>

namespace arl2 {
namespace {

constexpr int BN = 64;    // keys per tile
constexpr int NSTAGE = 4; // LDS ring depth (a power of two)
constexpr int kStoreStep0 = 4;   // the tile copy's LDS writes begin in this step of an interval's second slot

template <int D, int KG, int RB, int NW>
struct FwdCfg {
    static constexpr int NT = 64 * NW;           // threads per workgroup
    static constexpr int RG = NW / KG;           // wavefronts that share their rows' keys with KG - 1 others each
    static constexpr int WR = 32 * RB;           // query rows per wavefront
    static constexpr int BM = WR * RG;           // query rows per workgroup
    static constexpr int KS = D / 16;            // k-steps of the QK^T contraction
    static constexpr int DB = D / 32;            // 32-row blocks of O^T
    static constexpr int CPR = D / 8;            // 16-byte chunks per row
    static constexpr int KROW = 2 * D + 16;      // LDS bytes per K row (padded: conflict-free b128 reads)
    static constexpr int VROW = 2 * D + 64;      // LDS bytes per V row (padded: conflict-free transposing reads)
    // Direct copy: tiles go from memory into LDS without passing through registers, 1 KB per instruction.
    static constexpr bool DIRECT = KG == 1 && (D == 128 || NW == 4);
    static constexpr int GROUP_ROWS = 512 / D;   // rows of such a kilobyte
    static constexpr int GROUP = D == 128 ? 1024 + 16 : 1024;    // LDS bytes from one to the next
    static constexpr int K_BYTES = DIRECT ? BN / GROUP_ROWS * GROUP : BN * KROW;
    static constexpr int V_BYTES = DIRECT ? BN / GROUP_ROWS * GROUP : BN * VROW;
    static constexpr int STAGE = K_BYTES + V_BYTES;   // one K/V tile
    static constexpr int KV_BYTES = (KG == 1 ? NSTAGE : 2) * STAGE;
    static constexpr int DBW = DB / KG;          // 32-feature blocks of the output that a wavefront finishes
    static constexpr int SS_BYTES = D * VROW;    // one bf16 part of the state staged [d][e]
    static constexpr int ST_BYTES = 2 * SS_BYTES;
    static constexpr int SCH = (D * CPR + NT - 1) / NT;   // 8-float state pieces per thread
    static constexpr int OUT_BYTES = BM * KROW;  // output staging [q][e]
    // fused feature map: half of Wq[h] (D/2 rows) plus, per wavefront, the rotation tables of its tokens
    static constexpr int WH_BYTES = (D / 2) * KROW;
    static constexpr int TST = D / 2 + 2;        // floats per staged table row (conflict-free 8-byte reads)
    static constexpr int TAB_BYTES = 2 * WR * TST * 4;
    static constexpr int FM_BYTES = WH_BYTES + RG * TAB_BYTES;
    static constexpr int WCH = ((D / 2) * CPR + NT - 1) / NT;     // 16-byte chunks of the Wq half per thread
    static constexpr int TCH = WR * (D / 8) / 64;                 // 16-byte chunks of one table tile per lane
    // one key group: the query rows pass through ring stages 2 and on, and what they need beyond them
    static constexpr int Q_GROUPS = WR / GROUP_ROWS;     // of a wavefront's query rows
    static constexpr int Q_BYTES = DIRECT ? Q_GROUPS * GROUP : WR * KROW;
    static constexpr int Q_END = KG == 1 ? 2 * STAGE + NW * Q_BYTES : 0;
    static constexpr int RING_END = Q_END > KV_BYTES ? Q_END : KV_BYTES;
    static constexpr int SMEM0 = (RING_END > ST_BYTES ? (RING_END > OUT_BYTES ? RING_END : OUT_BYTES)
                                                      : (ST_BYTES > OUT_BYTES ? ST_BYTES : OUT_BYTES));
    static constexpr int SMEM1 = SMEM0 > FM_BYTES ? SMEM0 : FM_BYTES;
    // with two key groups the ring is half as large and the state has room of its own behind it
    static constexpr int S_OFF = KG == 1 ? 0 : KV_BYTES;
    static constexpr int ML_OFF = KG == 1 ? SMEM1 : (KV_BYTES + ST_BYTES > SMEM1 ? KV_BYTES + ST_BYTES : SMEM1);
    static constexpr int SMEM = ML_OFF + (KG == 1 ? 0 : NW * 2 * 32 * 4);
    static_assert(SMEM <= 160 * 1024, "more LDS than a CU has");
    static_assert(KG == 1 || NW * RB * DBW * 16 * 64 * 4 <= KV_BYTES, "the partial outputs pass through the ring");
    static constexpr int KCH = BN * CPR / NT;    // 16-byte chunks per thread per tile (K and V each)
    static constexpr int ROWS_PER_PASS = NT / CPR;
    static constexpr int S_LEN = KS;             // K fragments of one 32-key block, each for RB MFMAs
    static constexpr int PV_LEN = 2 * DB;        // V^T fragments of one 32-key block, each for RB MFMAs
    static constexpr int RING = 4;               // fragment registers in flight from LDS
    static constexpr int PF = RING - 1;          // operand fragments are read from LDS this many steps ahead
    // LDS reads a full slot issues after step `first` (its own fragments, then the next slot's; S fragments,
    // at even positions, are one read, V^T fragments two)
    static constexpr int lds_reads_from(int first)
    {
        int c = 0;
        for (int n = first; n < S_LEN + PV_LEN; ++n) c += ((n + PF) & 1) == 0 ? 1 : 2;
        return c;
    }
    // the copy's writes go into every other step if they all fit, else into every step
    static constexpr int STORE_STRIDE = kStoreStep0 + 4 * KCH - 2 < S_LEN + PV_LEN ? 2 : 1;
    static constexpr int LAST_STORE = kStoreStep0 + STORE_STRIDE * (2 * KCH - 1);
    static constexpr int LDS_AFTER_COPY = lds_reads_from(LAST_STORE + 1);
    static_assert(LAST_STORE < S_LEN + PV_LEN && 2 * KCH - 1 < S_LEN + PV_LEN, "the copy must fit into one slot");
    static_assert(KCH >= 1, "tile too small for the workgroup");
    static_assert(S_LEN % RING == 0 && PV_LEN % RING == 0, "chain lengths must be multiples of the fragment ring");
};

// The running maximum is raised only when a lane's share of a tile's row sum (32 probabilities taken
// relative to the running maximum) reaches this value, i.e. some logit exceeded it by more than ~2^7.
constexpr float kRowSumLimit = 4096.0f;


// Two kilobytes straight into LDS (16 bytes per lane, lane l to lds + 16 l; the second OFF2 bytes further).  The
// instruction's offset moves the source address as well, so `off2` is less by as much.  M0 carries the LDS address and is
// the statement's output, so that the compiler knows it overwritten (it does not honour M0 in a list of clobbers; with the
// address as an input in M0 whole tiles of D = 128 take 0.2 % longer).  The loads have no output register: the caller waits on
// vmcnt before the bytes are read.
template <int OFF2>
__device__ __forceinline__ void load_pair_to_lds(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, uint32_t off2, uint32_t lds)
{
    uint32_t m0;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %4, 0 offen lds\n\tbuffer_load_dwordx4 %3, %4, 0 offen offset:%5 lds"
                 : "={m0}"(m0) : "s"(lds), "v"(off), "v"(off2), "s"(rsrc), "n"(OFF2) : "memory");
}
// Workgroup barrier after all but the last N of this wavefront's loads have arrived, and all of its LDS reads.
template <int N>
__device__ __forceinline__ void direct_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Query tile qt (of FwdCfg's BM rows) of (stream, head) bh, by one workgroup.
template <int D, int KG, int RB, int NW, bool FUSED_MAP>
__device__ __forceinline__ void fwd_tile(const FwdArgs &a, float scale_log2, int bh, int qt, unsigned char *smem)
{
    using C = FwdCfg<D, KG, RB, NW>;
    constexpr int BM = C::BM, NT = C::NT, WR = C::WR;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c = lane & 31, hh = lane >> 5;
    const int rg = wave % C::RG, kg = wave / C::RG;       // row group and key group of this wavefront

    const int h = bh % a.H, b = bh / a.H;
    const int H = a.H, Lq = a.Lq, Lkv = a.Lkv;

    const bf16_t *kgl = (const bf16_t *)a.k + ((size_t)b * Lkv * H + h) * D;
    const bf16_t *vgl = (const bf16_t *)a.v + ((size_t)b * Lkv * H + h) * D;
    const uint32_t tok_bytes = (uint32_t)H * D * 2;                       // one token, all heads
    const uint32_t kv_range = (uint32_t)(Lkv - 1) * tok_bytes + 2 * D;    // bytes of this head's K (or V) slice
    const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(kgl, kv_range);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(vgl, kv_range);

    // ---- Q fragments (B operand of S^T = K Q^T): lane (c, hh) holds Q[row][16 t + 8 hh + 0..7]
    const int q0 = qt * BM + rg * WR;
    bf16x8 qf[RB][C::KS];
    float qss[RB];                    // |row|^2 over the full head dimension
    // The rows travel whole (16-byte chunks, D / 8 lanes per row) through LDS rows of KROW bytes to the fragments:
    // fragment loads straight from memory touch 32 cache lines per instruction.  The key groups of a row group move
    // a share of its rows each.  Rows past the last query read as zero.
    constexpr int QCH = WR * C::CPR / 64 / KG;             // chunks per lane
    const int q_rows = Lq - qt * BM < BM ? Lq - qt * BM : BM;
    const __amdgpu_buffer_rsrc_t q_rsrc = make_rsrc((const bf16_t *)a.q + ((size_t)(b * (size_t)Lq + qt * BM) * H + h) * D,
                                                    (uint32_t)(q_rows - 1) * tok_bytes + 2 * D);
    auto fetch_rows = [&](u32x4 *x) {
#pragma unroll
        for (int i = 0; i < QCH; ++i) {
            const int id = lane + 64 * (kg * QCH + i);
            x[i] = __builtin_amdgcn_raw_buffer_load_b128(q_rsrc, (uint32_t)(WR * rg + id / C::CPR) * tok_bytes + 16 * (id % C::CPR), 0, 0);
        }
    };
    auto put_rows = [&](unsigned char *dst, const u32x4 *x) {
#pragma unroll
        for (int i = 0; i < QCH; ++i) {
            const int id = lane + 64 * (kg * QCH + i);
            *(u32x4 *)(dst + (id / C::CPR) * C::KROW + 16 * (id % C::CPR)) = x[i];
        }
    };
    // Direct copy: fragment offsets, 64-byte (D = 64: 32-byte) column x of K row c and 64-byte column x of V row vr + 4 hh
    int kdx[4] = {}, vdx[4] = {};
    auto get_rows = [&](const unsigned char *src) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int t = 0; t < C::KS; ++t) {
                if constexpr (C::DIRECT) qf[rb][t] = *(const bf16x8 *)(src + rb * (C::K_BYTES / 2) + (D == 128 ? kdx[t / 2] + 32 * (t & 1) : kdx[t]));
                else qf[rb][t] = *(const bf16x8 *)(src + (32 * rb + c) * C::KROW + 32 * t + 16 * hh);
            }
    };
    // the same fragments straight from memory (the other query arrays of the epilogue)
    auto row_token = [&](int rb) -> size_t {              // rows past the last query read row 0, unused
        const int qrow = q0 + 32 * rb + c;
        return b * (size_t)Lq + (qrow < Lq ? qrow : 0);
    };
    auto load_rows = [&](const bf16_t *src, bf16x8 (*x)[C::KS]) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const bf16_t *row = src + (row_token(rb) * H + h) * D + 8 * hh;
#pragma unroll
            for (int t = 0; t < C::KS; ++t) x[rb][t] = *(const bf16x8 *)(row + 16 * t);
        }
    };
    auto square_rows = [&]() {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            float ss = 0.f;
#pragma unroll
            for (int t = 0; t < C::KS; ++t)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float f = (float)qf[rb][t][j];
                    ss = fmaf(f, f, ss);
                }
            qss[rb] = xhalf_sum(ss);
        }
    };

    // ---- global -> registers -> LDS copies: 16-byte chunks, chunk id = tid + NT*i -> (row, col)
    u32x4 kst[C::KCH], vst[C::KCH];
    const uint32_t g_off0 = (uint32_t)(tid / C::CPR) * tok_bytes + 16 * (tid % C::CPR);   // chunk 0 of tile 0
    const int lds_k_off = (tid / C::CPR) * C::KROW + 16 * (tid % C::CPR);
    const int lds_v_off = (tid / C::CPR) * C::VROW + 16 * (tid % C::CPR);
    uint32_t g_off = g_off0;          // chunk 0 of the next tile to load

    auto load_k = [&](int tile, u32x4 *x) {
#pragma unroll
        for (int i = 0; i < C::KCH; ++i)
            x[i] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, g_off0 + (uint32_t)(tile * BN + i * C::ROWS_PER_PASS) * tok_bytes, 0, 0);
    };
    auto load_v = [&](int tile, u32x4 *x) {
#pragma unroll
        for (int i = 0; i < C::KCH; ++i)
            x[i] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, g_off0 + (uint32_t)(tile * BN + i * C::ROWS_PER_PASS) * tok_bytes, 0, 0);
    };
    auto store_k = [&](int stage, const u32x4 *x) {
#pragma unroll
        for (int i = 0; i < C::KCH; ++i) *(u32x4 *)(smem + stage * C::STAGE + lds_k_off + i * C::ROWS_PER_PASS * C::KROW) = x[i];
    };
    auto store_v = [&](int stage, const u32x4 *x) {
#pragma unroll
        for (int i = 0; i < C::KCH; ++i)
            *(u32x4 *)(smem + stage * C::STAGE + C::K_BYTES + lds_v_off + i * C::ROWS_PER_PASS * C::VROW) = x[i];
    };
    // the same copy in pieces.  One key group: the loads of a tile (chunk h of K and of V), its stores (piece p).
    auto load_tile_part = [&](auto h_) {
        constexpr int h = decltype(h_)::value;
        const uint32_t off = g_off + (uint32_t)h * C::ROWS_PER_PASS * tok_bytes;
        kst[h] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off, 0, 0);
        vst[h] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off, 0, 0);
        if constexpr (h == C::KCH - 1) g_off += BN * tok_bytes;
    };
    auto store_tile_part = [&](int stage, auto p_) {
        constexpr int p = decltype(p_)::value;
        unsigned char *smK = smem + stage * C::STAGE;
        if constexpr ((p & 1) == 0) *(u32x4 *)(smK + lds_k_off + (p >> 1) * C::ROWS_PER_PASS * C::KROW) = kst[p >> 1];
        else *(u32x4 *)(smK + C::K_BYTES + lds_v_off + (p >> 1) * C::ROWS_PER_PASS * C::VROW) = vst[p >> 1];
    };
    // Several key groups, interval j: piece p of K(j + 2) or V(j) from its register into LDS, then the same piece
    // of K(j + 3) or V(j + 1) is requested (g_off: V(j + 1)).
    auto copy_part = [&](int stage, auto p_) {
        constexpr int p = decltype(p_)::value, h = p >> 1;
        store_tile_part(stage, p_);
        const uint32_t off = g_off + (uint32_t)h * C::ROWS_PER_PASS * tok_bytes;
        if constexpr ((p & 1) == 0) kst[h] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off + 2 * BN * tok_bytes, 0, 0);
        else vst[h] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off, 0, 0);
        if constexpr (p == 2 * C::KCH - 1) g_off += BN * tok_bytes;
    };

    // Direct copy.  A copy of whole kilobytes cannot pad rows to keep the fragment reads free of bank conflicts; the 16-byte
    // chunks x of a row r are exchanged instead:
    //   D = 128: at (r / 4) GROUP + 256 (r % 4) + 16 (x ^ 4 (r % 4)), the groups of four rows 16 bytes apart;
    //   D = 64:  at 128 r + 16 (x ^ r / 2 % 8) in K tiles (32 rows are read at one chunk), and 128 r + 16 (x ^ 4 (r / 2 % 2)) in
    //            V tiles (four rows at four chunks).
    // A wavefront moves two kilobytes of K and of V; a tile is requested two barrier intervals before it is read.
    const uint32_t lds0 = lds_address(smem);
    uint32_t dsrc[2][2] = {};         // source offsets of the lane's two chunks of K and V, from BELOW bytes below the tile
    constexpr int BELOW = D == 128 ? 64 : 0;
    if constexpr (C::DIRECT) {
        static_assert(!C::DIRECT || BN / C::GROUP_ROWS == 2 * NW, "two kilobytes of K and of V per wavefront");
        const int vr = (lane >> 2) & 3;
        if constexpr (D == 128) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                kdx[x] = (c >> 2) * C::GROUP + 256 * (c & 3) + 64 * (x ^ (c & 3)) + 16 * hh;
                vdx[x] = hh * C::GROUP + 256 * vr + 64 * (x ^ vr) + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
            }
            dsrc[0][0] = (uint32_t)(8 * wave + (lane >> 4)) * tok_bytes + 16 * ((lane & 15) ^ (4 * (lane >> 4))) + BELOW;
            dsrc[0][1] = dsrc[0][0] + 4 * tok_bytes - C::GROUP;        // (4 tok_bytes >= 1024, hence the 64 bytes)
            dsrc[1][0] = dsrc[0][0];
            dsrc[1][1] = dsrc[0][1];
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) kdx[x] = 128 * c + 32 * (x ^ ((c >> 2) & 3)) + 16 * (hh ^ ((c >> 1) & 1));
#pragma unroll
            for (int x = 0; x < 2; ++x) vdx[x] = 128 * (vr + 4 * hh) + 64 * (x ^ (vr >> 1)) + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
            const uint32_t row = (uint32_t)(16 * wave + (lane >> 3)) * tok_bytes;
#pragma unroll
            for (int i = 0; i < 2; ++i) {                              // (8 tok_bytes >= 1024)
                dsrc[0][i] = row + i * (8 * tok_bytes - C::GROUP) + 16 * ((lane & 7) ^ (4 * i + (lane >> 4)));
                dsrc[1][i] = row + i * (8 * tok_bytes - C::GROUP) + 16 * ((lane & 7) ^ (4 * ((lane >> 4) & 1)));
            }
        }
    }
    // K (PART 0) or V (PART 1) of a tile; past the last key nothing is read and zeros are stored.
    auto direct_part = [&](int tile, auto part_) {
        constexpr int PART = decltype(part_)::value;
        const int left = (int)kv_range - tile * (int)(BN * tok_bytes);
        const bf16_t *base = (PART ? vgl : kgl) + (ptrdiff_t)tile * BN * H * D - BELOW / 2;
        load_pair_to_lds<C::GROUP>(make_rsrc(base, left > 0 ? (uint32_t)left + BELOW : 0), dsrc[PART][0], dsrc[PART][1],
                                   lds0 + (tile & (NSTAGE - 1)) * C::STAGE + PART * C::K_BYTES + 2 * wave * C::GROUP);
    };
    // This wavefront's query rows, laid out like those of a K tile, to `lds`.
    auto direct_rows = [&](uint32_t lds) {
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc((const bf16_t *)a.q + ((size_t)(b * (size_t)Lq + qt * BM) * H + h) * D - BELOW / 2,
                                                      (uint32_t)(q_rows - 1) * tok_bytes + 2 * D + BELOW);
#pragma unroll
        for (int g = 0; g < C::Q_GROUPS; g += 2) {
            const uint32_t off = (uint32_t)(WR * rg + C::GROUP_ROWS * (g - 2 * wave)) * tok_bytes;
            load_pair_to_lds<C::GROUP>(rsrc, dsrc[0][0] + off, dsrc[0][1] + off, lds + g * C::GROUP);
        }
    };
    auto direct_tile = [&](int tile) { static_for<0, 2>([&](auto part_) { direct_part(tile, part_); }); };

    // lane roles inside a 32-key block
    const int k_frag_off = c * C::KROW + 16 * hh;                                   // + 32*t
    const int v_frag_off = (((lane & 15) >> 2) + 4 * hh) * C::VROW + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);

    // ---- running softmax state and accumulators
    f32x16 o_acc[C::DB][RB];     // O^T blocks
    f32x16 s_acc[2][RB];         // S^T of the key block whose softmax runs, and of the next one
    bf16x8 pf[2][RB][2];         // P^T fragments (B operands of the second GEMM): two per key block
    bf16x8 fr[C::RING];          // A-operand fragments in flight from LDS
    float m_run[RB];             // running max of scaled logits (log2 domain)
    float l_run[RB] = {};        // this lane's share of the running sum
    auto clear_output = [&]() {
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int r = 0; r < 16; ++r) o_acc[db][rb][r] = 0.f;
    };

    // Byte offsets in the ring of the K rows / V rows of this wavefront's 32-key block `blk`: half blk % 2 of tile
    // blk / 2, or with two key groups half kg of tile blk.
    auto k_block = [&](int blk) -> int {
        if constexpr (C::DIRECT) return ((blk >> 1) & (NSTAGE - 1)) * C::STAGE + (blk & 1) * (C::K_BYTES / 2);
        else if constexpr (KG == 1) return ((blk >> 1) & (NSTAGE - 1)) * C::STAGE + (blk & 1) * 32 * C::KROW;
        else return (blk & 1) * C::STAGE + kg * 32 * C::KROW;
    };
    auto v_block = [&](int blk) -> int {
        if constexpr (C::DIRECT) return ((blk >> 1) & (NSTAGE - 1)) * C::STAGE + C::K_BYTES + (blk & 1) * (C::K_BYTES / 2);
        else if constexpr (KG == 1) return ((blk >> 1) & (NSTAGE - 1)) * C::STAGE + C::K_BYTES + (blk & 1) * 32 * C::VROW;
        else return (blk & 1) * C::STAGE + C::K_BYTES + kg * 32 * C::VROW;
    };
    auto first_key = [&](int blk) -> int { return KG == 1 ? 32 * blk : BN * blk + 32 * kg; };
    // A-operand fragments: k-step n of S^T = K Q^T (a K row piece), and MFMA n of O^T += V^T P^T
    // (16-key step n / DB, row block n % DB: a transposed V piece).
    auto k_frag = [&](const unsigned char *kp, auto n_) -> bf16x8 {
        constexpr int n = decltype(n_)::value;
        if constexpr (C::DIRECT && D == 128) return *(const bf16x8 *)(kp + kdx[n / 2] + 32 * (n & 1));
        else if constexpr (C::DIRECT) return *(const bf16x8 *)(kp + kdx[n]);
        else return *(const bf16x8 *)(kp + k_frag_off + 32 * n);
    };
    auto v_frag = [&](const unsigned char *vp, auto n_) -> bf16x8 {
        constexpr int n = decltype(n_)::value;
        // keys 16u + 4hh + 0..3 and 16u + 8 + 4hh + 0..3
        if constexpr (C::DIRECT) return lds_read_tr_pair(vp + vdx[n % C::DB] + (n / C::DB) * (C::V_BYTES / 4), C::V_BYTES / 8);
        else return lds_read_tr_pair(vp + v_frag_off + 16 * (n / C::DB) * C::VROW + 64 * (n % C::DB), 8 * C::VROW);
    };
    // Products of a step: K fragment n (or V^T fragment n) with the query rows (the probabilities) of every row block.
    auto s_mfma = [&](auto buf_, auto n_, bf16x8 x) {
        constexpr int buf = decltype(buf_)::value, t = decltype(n_)::value;
        const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        static_for<0, RB>([&](auto r_) {
            constexpr int rb = decltype(r_)::value;
            if constexpr (t == 0) s_acc[buf][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[rb][t], zero, 0, 0, 0);
            else s_acc[buf][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qf[rb][t], s_acc[buf][rb], 0, 0, 0);
        });
    };
    auto pv_mfma = [&](auto buf_, auto n_, bf16x8 x) {
        constexpr int buf = decltype(buf_)::value, u = decltype(n_)::value / C::DB, db = decltype(n_)::value % C::DB;
        static_for<0, RB>([&](auto r_) {
            constexpr int rb = decltype(r_)::value;
            o_acc[db][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, pf[buf][rb][u], o_acc[db][rb], 0, 0, 0);
        });
    };
    // exp2 of the 16 logits per lane of one key block relative to the running maximum -> its two P^T
    // fragments; returns this lane's share of the row sum.  (Only on the rare path that raises the maximum.)
    auto exp_block = [&](auto par_, auto r_) -> float {
        constexpr int PAR = decltype(par_)::value, rb = decltype(r_)::value;
        const float mneg = -m_run[rb];
        float psum = 0.f;
        static_for<0, 8>([&](auto i_) {
            constexpr int r = 2 * decltype(i_)::value;
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s_acc[PAR][rb][r], scale_log2, mneg));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s_acc[PAR][rb][r + 1], scale_log2, mneg));
            psum += p0 + p1;
            pf[PAR][rb][r >> 3][r & 7] = to_bf16(p0);
            pf[PAR][rb][r >> 3][(r & 7) + 1] = to_bf16(p1);
        });
        return psum;
    };

    // One slot of the software pipeline, on key block j (logits in s_acc[j % 2], produced one slot earlier):
    //   matrix pipe:  S(j+1) = K_{j+1} Q^T  -> s_acc[(j+1) % 2]     (KS MFMAs, if the block exists)
    //                 O^T += V_{j-1}^T P_{j-1}^T                      (2 DB MFMAs, if j > 0)
    //   vector ALU:   softmax of block j -> its P^T fragments and row-sum share
    // Neither MFMA chain depends on this slot's vector work, so every step issues one MFMA, the LDS read of
    // the operand fragment needed PF MFMAs later (at the end of the slot: of the next slot's first chain)
    // and a slice of the softmax; the slices are themselves staggered (scale of logit v+2, exponential of
    // logit v+1, sum and conversion of logit v) so that no instruction waits for the one before it.
    // copy_: 0 nothing; 1 this slot also requests the next K/V tile from global memory (early steps);
    // 2 it also writes that tile, by now in registers, into ring stage `cstage`, one 16-byte piece per thread
    // every other step, so that the copy runs under the MFMAs instead of in a burst before the barrier; 3 (several key
    // groups) the whole copy of an interval and its barrier, as soon as the slot has requested its last fragment: the
    // fragments requested after that are the next slot's, from the tiles that the barrier publishes; 4 the same for the last
    // tile, whose V is all that is left to store (into stage `cstage`).  Direct copy: 5 the barrier, as soon as the slot has
    // requested its last fragment (those requested after it are the next slot's); 6 the loads of tile `cstage`.
    auto slot = [&](auto par_, auto has_s_, auto has_pv_, auto next_s_, auto masked_, int j, auto copy_, int cstage) {
        constexpr int PAR = decltype(par_)::value;
        constexpr int COPY = decltype(copy_)::value;
        constexpr bool HAS_S = decltype(has_s_)::value, HAS_PV = decltype(has_pv_)::value;
        constexpr bool NEXT_S = decltype(next_s_)::value, MASKED = decltype(masked_)::value;
        constexpr int SL = HAS_S ? C::S_LEN : 0, NS = SL + (HAS_PV ? C::PV_LEN : 0);
        constexpr int NL = 16 * RB, LPS = NL / NS;   // logits per lane, and per step
        static_assert(NS % C::RING == 0 && NL % NS == 0, "slot length");
        const unsigned char *kp = smem + k_block(j + 1);
        const unsigned char *vp = smem + v_block(j - 1);
        const unsigned char *np = smem + k_block(j + 2);      // next slot: S(j+2) (if any) and PV(j)
        const unsigned char *nvp = smem + v_block(j);
        float x[NL], ps0[RB] = {}, ps1[RB] = {};
        int key0 = first_key(j) + 4 * hh;            // key of the lane's first logit
        if constexpr (MASKED && RB > 1) asm volatile("" : "+v"(key0));    // (sixteen keys would otherwise be kept from the first block to the last)
        auto op_scale = [&](auto v_) {               // logit v: scaled, relative to the running maximum
            constexpr int v = decltype(v_)::value;
            if constexpr (v < NL) {
                constexpr int rb = v >> 4, r = v & 15;
                if constexpr (MASKED) {              // keys past the end of the sequence (last tile only)
                    if (key0 >= Lkv - (8 * (r >> 2) + (r & 3))) s_acc[PAR][rb][r] = -INFINITY;
                }
                x[v] = fmaf(s_acc[PAR][rb][r], scale_log2, -m_run[rb]);
            }
        };
        auto op_exp = [&](auto v_) {
            constexpr int v = decltype(v_)::value;
            if constexpr (v < NL) x[v] = __builtin_amdgcn_exp2f(x[v]);
        };
        auto op_sum = [&](auto v_) {                 // row-sum share, and the P^T pair (v-1, v) for odd v
            constexpr int v = decltype(v_)::value;
            constexpr int rb = v >> 4, u = (v >> 3) & 1;
            if constexpr (v & 1) {
                ps1[rb] += x[v];
                bf16x2 pk = {to_bf16(x[v - 1]), to_bf16(x[v])};
                asm volatile("" : "+v"(pk));         // the conversion stays in this step
                pf[PAR][rb][u][(v & 7) - 1] = pk[0];
                pf[PAR][rb][u][v & 7] = pk[1];
            } else {
                ps0[rb] += x[v];
            }
        };
        // MFMA n of the slot: with both chains present they alternate (S at even n), so that MFMAs which
        // accumulate into the same registers are never issued back to back
        auto is_s = [](int n) constexpr { return HAS_S && (!HAS_PV || (n & 1) == 0); };
        auto idx = [](int n) constexpr { return HAS_S && HAS_PV ? n >> 1 : n; };
        auto fetch = [&](auto m_) {                  // requests the A fragment of MFMA m (m >= NS: of the next slot)
            constexpr int m = decltype(m_)::value;
            if constexpr (m < NS) {
                if constexpr (is_s(m)) fr[m % C::RING] = k_frag(kp, std::integral_constant<int, idx(m)>{});
                else fr[m % C::RING] = v_frag(vp, std::integral_constant<int, idx(m)>{});
            } else {
                // the next slot has a second GEMM (this slot's block) in every case; its S chain alternates with it
                constexpr int mm = m - NS;
                if constexpr (NEXT_S && (mm & 1) == 0) fr[m % C::RING] = k_frag(np, std::integral_constant<int, (mm >> 1)>{});
                else fr[m % C::RING] = v_frag(nvp, std::integral_constant<int, (NEXT_S ? mm >> 1 : mm)>{});
            }
        };
        static_for<0, NS>([&](auto n_) {
            constexpr int n = decltype(n_)::value;
            fetch(std::integral_constant<int, n + C::PF>{});
            if constexpr (is_s(n)) s_mfma(std::integral_constant<int, PAR ^ 1>{}, std::integral_constant<int, idx(n)>{}, fr[n % C::RING]);
            else pv_mfma(std::integral_constant<int, PAR ^ 1>{}, std::integral_constant<int, idx(n)>{}, fr[n % C::RING]);
            if constexpr (COPY == 1 && (n & 1) == 1 && n / 2 < C::KCH) load_tile_part(std::integral_constant<int, n / 2>{});
            if constexpr (COPY == 2 && n >= kStoreStep0 && n <= C::LAST_STORE && (n - kStoreStep0) % C::STORE_STRIDE == 0)
                store_tile_part(cstage, std::integral_constant<int, (n - kStoreStep0) / C::STORE_STRIDE>{});
            if constexpr (COPY == 5 && n == NS - C::PF - 1) direct_barrier<4>();
            if constexpr (COPY == 6 && (n == 1 || n == 5)) direct_part(cstage, std::integral_constant<int, n / 4>{});
            if constexpr (COPY == 3 || COPY == 4) {
                static_for<0, 2 * C::KCH>([&](auto p_) {
                    constexpr int p = decltype(p_)::value;
                    if constexpr (p * (NS - C::PF) / (2 * C::KCH) == n) {
                        if constexpr (COPY == 3) copy_part(PAR, p_);
                        else if constexpr (p & 1) store_tile_part(cstage, p_);
                    }
                });
                if constexpr (n == NS - C::PF - 1) lds_barrier();
            }
            if constexpr (n == 0) {
                op_scale(std::integral_constant<int, 0>{});
                op_scale(std::integral_constant<int, 1>{});
                op_exp(std::integral_constant<int, 0>{});
            }
            static_for<0, LPS>([&](auto i_) {
                constexpr int v = n * LPS + decltype(i_)::value;
                op_scale(std::integral_constant<int, v + 2>{});
                op_exp(std::integral_constant<int, v + 1>{});
                op_sum(std::integral_constant<int, v>{});
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        // Rarely a logit exceeded the running maximum (which starts as the first block's) by more than the
        // threshold: take the true block maximum, raise the running maximum, rescale, redo the block.
        bool over = false;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            ps0[rb] += ps1[rb];
            over |= !(ps0[rb] < kRowSumLimit);
        }
        if (__builtin_expect(__any(over), 0)) {      // wave-uniform; also true for inf and NaN
            // (compile-time loops: the compiler unrolls nothing on a path it is told to be rare)
            static_for<0, RB>([&](auto b_) {
                constexpr int rb = decltype(b_)::value;
                float mx = s_acc[PAR][rb][0];
                static_for<1, 16>([&](auto r_) { mx = fmaxf(mx, s_acc[PAR][rb][decltype(r_)::value]); });
                mx = xhalf_max(mx) * scale_log2;
                const float m_new = fmaxf(m_run[rb], mx);
                const float alpha = m_new == m_run[rb] ? 1.0f : __builtin_amdgcn_exp2f(m_run[rb] - m_new);
                m_run[rb] = m_new;
                l_run[rb] *= alpha;
                if constexpr (HAS_PV)
                    static_for<0, C::DB>([&](auto db_) {
                        static_for<0, 16>([&](auto r_) { o_acc[decltype(db_)::value][rb][decltype(r_)::value] *= alpha; });
                    });
                ps0[rb] = exp_block(par_, b_);
            });
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) l_run[rb] += ps0[rb];
    };

    const std::false_type no{};
    const std::true_type yes{};
    const std::integral_constant<int, 0> par0{};
    const std::integral_constant<int, 1> par1{};
    const std::integral_constant<int, 0> copy0{};
    const std::integral_constant<int, 1> copy1{};
    const std::integral_constant<int, 2> copy2{};
    const std::integral_constant<int, 3> copy3{};
    const std::integral_constant<int, 4> copy4{};
    const std::integral_constant<int, 5> copy5{};
    const std::integral_constant<int, 6> copy6{};

    // S(0), plain: nothing to overlap it with
    auto first_product = [&]() {
        const unsigned char *kp = smem + k_block(0);
        const unsigned char *np = smem + k_block(1);
        static_for<0, C::PF>([&](auto m_) { fr[decltype(m_)::value] = k_frag(kp, m_); });
        static_for<0, C::S_LEN>([&](auto n_) {
            constexpr int n = decltype(n_)::value;
            constexpr int m = n + C::PF;
            if constexpr (m < C::S_LEN) fr[m % C::RING] = k_frag(kp, std::integral_constant<int, m>{});
            else fr[m % C::RING] = k_frag(np, std::integral_constant<int, m - C::S_LEN>{});
            s_mfma(par0, n_, fr[n % C::RING]);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // The running maximum starts as the true maximum of the first block (which always holds a key: with two key groups
    // Lkv > 32), so that its slot need not find out by computing every exponential twice.
    auto first_maximum = [&]() {
        int key0 = first_key(0) + 4 * hh;
        if constexpr (RB > 1) asm volatile("" : "+v"(key0));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                mx = fmaxf(mx, key0 < Lkv - (8 * (r >> 2) + (r & 3)) ? s_acc[0][rb][r] : -INFINITY);
            }
            m_run[rb] = fmaxf(xhalf_max(mx) * scale_log2, -FLT_MAX);     // finite also where every logit of the block is -inf
        }
    };
    // second GEMM of the last key block `blk` of parity P (its first fragments are in flight)
    auto last_product = [&](auto p_, int blk) {
        const unsigned char *vp = smem + v_block(blk);
        static_for<0, C::PV_LEN>([&](auto n_) {
            constexpr int n = decltype(n_)::value;
            constexpr int m = n + C::PF;
            if constexpr (m < C::PV_LEN) fr[m % C::RING] = v_frag(vp, std::integral_constant<int, m>{});
            pv_mfma(p_, n_, fr[n % C::RING]);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    const float *Sg = a.S != nullptr ? a.S + ((size_t)b * H + h) * D * D : nullptr;
    unsigned char *smHi = smem + C::S_OFF, *smLo = smHi + C::SS_BYTES;
    f32x4 sr[C::SCH][2];
    auto load_state = [&]() {         // 8-float pieces: row id / CPR, column piece id % CPR
#pragma unroll
        for (int i = 0; i < C::SCH; ++i) {
            const int id = tid + NT * i;
            if (id < D * C::CPR) {
                const float *sp = Sg + (size_t)(id / C::CPR) * D + 8 * (id % C::CPR);
                sr[i][0] = *(const f32x4 *)(sp);
                sr[i][1] = *(const f32x4 *)(sp + 4);
            }
        }
    };
    auto store_state = [&]() {        // split into bf16 hi + lo, row-major [d][e]
#pragma unroll
        for (int i = 0; i < C::SCH; ++i) {
            const int id = tid + NT * i;
            if (id < D * C::CPR) {
                union { u32x4 u; bf16x8 v; } hi, lo;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float x = sr[i][j >> 2][j & 3];
                    const bf16_t hb = to_bf16(x);
                    hi.v[j] = hb;
                    lo.v[j] = to_bf16(x - (float)hb);
                }
                const int off = (id / C::CPR) * C::VROW + 16 * (id % C::CPR);
                *(u32x4 *)(smHi + off) = hi.u;
                *(u32x4 *)(smLo + off) = lo.u;
            }
        }
    };
    constexpr bool EARLY_STATE = KG > 1 && !FUSED_MAP;   // the state goes to LDS before the key loop
    // D = 128 with the query rows kept to the end: 29 registers spilled with two endings (120 bytes of scratch per lane), none
    // with one: 64 heads, 328 tokens 15.3 us with, 12.9 us without the spill.  The other forms have registers left, and with
    // one ending they are 2 to 5 % slower (12 heads x 64, 200 tokens: 6.9 us against 7.2 us).
    constexpr bool ONE_ENDING = D == 128 && !FUSED_MAP;

    if constexpr (KG == 1) {
        // Two row blocks: a single tile gets an empty second one, whose keys are all masked, and the first tile's keys are
        // masked in any case (with a path of its own for a single tile registers would spill).
        const int nt0 = (Lkv + BN - 1) / BN, ntiles = RB > 1 && nt0 == 1 ? 2 : nt0;
        // ---- prologue: tiles 0 and 1 into the ring, all their loads and those of the query rows in flight together
        {
            u32x4 k1[C::KCH], v1[C::KCH], x[QCH];
            if constexpr (C::DIRECT) {
                if (q0 < Lq) direct_rows(lds0 + 2 * C::STAGE + wave * C::Q_BYTES);
                direct_tile(0);
                direct_tile(1);
            } else {
                load_k(0, kst);
                if (q0 < Lq) fetch_rows(x);
                load_v(0, vst);
                load_k(1, k1);
                load_v(1, v1);
                store_k(0, kst);
            }
            unsigned char *mine = smem + 2 * C::STAGE + wave * C::Q_BYTES;       // in stages that tile 2 and on will use
            if constexpr (C::DIRECT) {
                asm volatile("s_waitcnt vmcnt(8)" ::: "memory");                 // the query rows are there, the two tiles may not
            } else {
                if (q0 < Lq) put_rows(mine, x);
                store_v(0, vst);
                store_k(1, k1);
                store_v(1, v1);
            }
            if (q0 < Lq) {              // (wavefronts without rows keep off the LDS: 128 rows over 300 keys 8.7 -> 8.2 us)
                get_rows(mine);
                square_rows();
            }
        }
        if constexpr (C::DIRECT) direct_barrier<0>();
        else __syncthreads();

        // Interval i covers the slots of key blocks 2i and 2i+1: they read K of tiles i and i+1 and V of tiles i-1 and i.
        // Direct copy: the barrier of interval i stands near the end of its first slot.  Behind it tile i-1 is no longer read
        // and tile i+3 is requested into its stage; tile i+1, requested two barriers earlier, has arrived when all loads but
        // the last tile's have.
        // Else the barrier closes the interval: tile i+2 is fetched into registers at its start and written at its end to the ring
        // stage of tile i-2 (four stages); the barrier that closes the interval publishes it.
        auto close_interval = [&](int i) {
            store_k((i + 2) & (NSTAGE - 1), kst);
            store_v((i + 2) & (NSTAGE - 1), vst);
            __syncthreads();
        };
        auto load_tile = [&](int tile) {
            load_k(tile, kst);
            load_v(tile, vst);
        };
        g_off += 3 * BN * tok_bytes;
        if constexpr (C::DIRECT) direct_tile(2);
        if (q0 < Lq) {
            first_product();
            if constexpr (C::DIRECT) direct_tile(3);
            else load_tile(2);
            first_maximum();
            if constexpr (RB > 1) {
                slot(par0, yes, no, yes, yes, 0, copy0, 0);
                clear_output();
                slot(par1, yes, yes, yes, yes, 1, copy0, 0);
            } else if (ntiles == 1) {
                slot(par0, yes, no, no, yes, 0, copy0, 0);
                clear_output();
                slot(par1, no, yes, no, yes, 1, copy0, 0);
            } else {
                slot(par0, yes, no, yes, no, 0, copy0, 0);
                clear_output();
                slot(par1, yes, yes, yes, no, 1, copy0, 0);
            }
            if constexpr (!C::DIRECT) close_interval(0);
#pragma unroll 1
            for (int i = 1; i < ntiles - 1; ++i) {
                if constexpr (C::DIRECT) {
                    slot(par0, yes, yes, yes, no, 2 * i, copy5, 0);
                    slot(par1, yes, yes, yes, no, 2 * i + 1, copy6, i + 3);
                    continue;
                }
                slot(par0, yes, yes, yes, no, 2 * i, copy1, 0);
                slot(par1, yes, yes, yes, no, 2 * i + 1, copy2, (i + 2) & (NSTAGE - 1));
                // the writes are complete once at most the LDS reads issued after the last of them are still
                // outstanding (LDS operations complete in order); those reads stay in flight across the barrier
                lds_barrier_keep<C::LDS_AFTER_COPY>();
            }
            if (ntiles > 1) {
                const int i = ntiles - 1;
                slot(par0, yes, yes, no, yes, 2 * i, copy0, 0);
                slot(par1, no, yes, no, yes, 2 * i + 1, copy0, 0);
            }
            last_product(par1, 2 * ntiles - 1);
        } else {
            // A wavefront whose rows all lie past the last query (the ragged last workgroup of a head) only
            // helps to move the tiles: the same loads, stores and barriers, no arithmetic.  Its rows are never
            // stored.
            clear_output();
            if constexpr (C::DIRECT) {
                direct_tile(3);
#pragma unroll 1
                for (int i = 1; i < ntiles - 1; ++i) {
                    direct_barrier<4>();
                    direct_tile(i + 3);
                }
            } else {
                load_tile(2);
                close_interval(0);
#pragma unroll 1
                for (int i = 1; i < ntiles - 1; ++i) {
                    load_tile(i + 2);
                    close_interval(i);
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) l_run[rb] = 1.0f;
        }
        // the loads of the tiles past the last one write zeros into the ring: they end before it is used for anything else
        if constexpr (C::DIRECT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        // ---- several key groups: a wavefront works on one 32-key block of every tile, one slot per tile.  Slot j reads
        // K(j + 1) and V(j - 1); K(j + 2) and V(j) are written during it, so two ring stages are enough.
        const int nt0 = (Lkv + BN - 1) / BN, nt = nt0 > 1 ? nt0 : 2;     // a second, empty tile where there is only one
        {
            u32x4 k0[C::KCH], k1[C::KCH], x[QCH];
            load_k(0, k0);
            fetch_rows(x);
            load_k(1, k1);
            load_k(2, kst);
            load_v(0, vst);
            g_off += BN * tok_bytes;
            store_k(0, k0);
            put_rows(smem + C::S_OFF + rg * WR * C::KROW, x);
            static_assert(KG == 1 || C::RG * WR * C::KROW <= C::ST_BYTES, "the query rows pass through the state's room");
            store_k(1, k1);
        }
        lds_barrier();
        if (EARLY_STATE && Sg != nullptr) load_state();      // arrives under the first products
        if (q0 < Lq) {
            get_rows(smem + C::S_OFF + rg * WR * C::KROW);
            square_rows();
            first_product();
            lds_barrier();            // every wavefront has read K(0), whose stage slot 0 overwrites, and its query rows
            first_maximum();
            slot(par0, yes, no, yes, yes, 0, copy3, 0);
            if (EARLY_STATE && Sg != nullptr) store_state();
            clear_output();
            int j = 1;
#pragma unroll 1
            for (; j + 1 < nt - 1; j += 2) {
                slot(par1, yes, yes, yes, no, j, copy3, 0);
                slot(par0, yes, yes, yes, no, j + 1, copy3, 0);
            }
            if (j < nt - 1) {
                slot(par1, yes, yes, yes, no, j, copy3, 0);
                ++j;
            }
            // the last slot has no first product: its fragments start with V(nt - 2)
            const unsigned char *vp = smem + v_block(j - 1);
            static_for<0, C::PF>([&](auto m_) { fr[decltype(m_)::value] = v_frag(vp, m_); });
            // An ending for each parity, or one, to whose registers the even parity's logits and probabilities are moved: with
            // two the largest form of this function does not fit the registers.
            if constexpr (ONE_ENDING) {
                if ((j & 1) == 0) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        s_acc[1][rb] = s_acc[0][rb];
                        pf[0][rb][0] = pf[1][rb][0];
                        pf[0][rb][1] = pf[1][rb][1];
                    }
                }
                slot(par1, no, yes, no, yes, j, copy4, j & 1);
                last_product(par1, j);
            } else if (j & 1) {
                slot(par1, no, yes, no, yes, j, copy4, 1);
                last_product(par1, j);
            } else {
                slot(par0, no, yes, no, yes, j, copy4, 0);
                last_product(par0, j);
            }
        } else {                      // rows past the last query: moves the tiles and the state only
            lds_barrier();
            if (EARLY_STATE && Sg != nullptr) store_state();
            clear_output();
#pragma unroll 1
            for (int j = 0; j < nt; ++j) {
                static_for<0, 2 * C::KCH>([&](auto p_) { copy_part(j & 1, p_); });
                lds_barrier();
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                l_run[rb] = 1.0f;
                m_run[rb] = 0.f;
            }
        }
    }

    // ---- epilogue ------------------------------------------------------------------------
    // The output blocks that this wavefront finishes: all of its rows' features, or with several key groups a share of
    // them, after the groups' partial results (each relative to its own maximum) have been exchanged through LDS.
    f32x16 out[C::DBW][RB];
    const int db0 = KG == 1 ? 0 : C::DBW * kg;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) l_run[rb] = xhalf_sum(l_run[rb]);
    if constexpr (KG == 1) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float inv_l = 1.0f / l_run[rb];
#pragma unroll
            for (int db = 0; db < C::DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) out[db][rb][r] = o_acc[db][rb][r] * inv_l;
        }
    } else {
        static_assert(KG <= 2 && (KG == 1 || RB == 1), "the exchange is written for two key groups of 32 rows");
        float *ml = (float *)(smem + C::ML_OFF);                       // [wavefront][maximum, sum][row]
        f32x4 *ox = (f32x4 *)smem;                                     // [wavefront][block][register quad][lane]
        const int peer = wave ^ C::RG;
        ml[(wave * 2 + hh) * 32 + c] = hh ? l_run[0] : m_run[0];
        __syncthreads();                                               // the ring is no longer read
#pragma unroll
        for (int i = 0; i < C::DBW; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {                              // the peer's blocks go to the peer
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = kg ? o_acc[i][0][4 * q + e] : o_acc[C::DBW + i][0][4 * q + e];
                ox[((wave * C::DBW + i) * 4 + q) * 64 + lane] = x;
            }
        const float m_peer = ml[peer * 2 * 32 + c], l_peer = ml[(peer * 2 + 1) * 32 + c];
        const float mm = fmaxf(m_run[0], m_peer);
        const float f0 = __builtin_amdgcn_exp2f(m_run[0] - mm), f1 = __builtin_amdgcn_exp2f(m_peer - mm);
        const float inv_l = 1.0f / fmaf(l_run[0], f0, l_peer * f1);
        const float f = f0 * inv_l, f_peer = f1 * inv_l;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C::DBW; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 x = ox[((peer * C::DBW + i) * 4 + q) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    out[i][0][4 * q + e] = fmaf(kg ? o_acc[C::DBW + i][0][4 * q + e] : o_acc[i][0][4 * q + e], f, x[e] * f_peer);
            }
    }

    if (Sg != nullptr) {
        size_t gi[RB];
        float g_row[RB];                                      // requested here, used after the products
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            gi[rb] = a.g_per_token ? row_token(rb) : row_token(rb) * H + h;
            g_row[rb] = 1.0f;
            if (a.g != nullptr && !a.g_per_element)
                g_row[rb] = a.g_is_bf16 ? (float)((const bf16_t *)a.g)[gi[rb]] : ((const float *)a.g)[gi[rb]];
        }
        // O_inter^T[e][q] = sum_d S[d][e] * q[q][d]: the fp32 state is split into bf16 hi + lo parts
        // (fp32 accumulate), both staged row-major [d][e] in LDS and read as S^T fragments through the
        // transposing LDS read, exactly like V.
        if (a.q_lin != nullptr) {
            // the linear branch has a query of its own (Eq. (3): its feature map differs from the
            // softmax branch's): take its fragments and its squared norm instead
            load_rows((const bf16_t *)a.q_lin, qf);
            square_rows();
        }
        // Fused feature map of the linear branch (Eq. (3)): q_lin^T[e][row] = sum_d Wq[e][d] xq[row][d], rotated
        // pair by pair, is never stored: the accumulator registers, rounded to bf16, are the B fragments of
        // the readout (k-slot j of half-wave hh is feature 16t + 8(j/4) + 4hh + j%4, as for P^T above).
        // Wq[h] passes through LDS in two halves of D/2 output rows (whole rows in, fragments out) and every
        // wavefront stages the rotation table rows of its 32 tokens in a region of its own: read straight
        // from global memory, fragment by fragment, these operands cost ~13 us of cache-line requests.
        if constexpr (FUSED_MAP) {
            bf16x8 xf[RB][C::KS];
            load_rows((const bf16_t *)a.xq, xf);
            unsigned char *smW = smem;                                           // D/2 rows of Wq[h], KROW bytes each
            float *cosT = (float *)(smem + C::WH_BYTES + rg * C::TAB_BYTES);   // [WR][TST] tables of this wavefront's rows
            float *sinT = cosT + WR * C::TST;
            const bool rope = a.cs != nullptr;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) qss[rb] = 0.f;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                __syncthreads();                      // the K/V ring (or the previous half of Wq) is no longer read
#pragma unroll
                for (int i = 0; i < C::WCH; ++i) {    // chunk id: row id / CPR of this half, 16-byte column id % CPR
                    const int id = tid + NT * i;
                    const int wr = id / C::CPR, wc = id % C::CPR;
                    if (wr < D / 2)
                        *(u32x4 *)(smW + wr * C::KROW + 16 * wc) =
                            *(const u32x4 *)((const bf16_t *)a.Wq + ((size_t)h * D + half * (D / 2) + wr) * D + 8 * wc);
                }
                if (half == 0 && rope && kg == 0) {
#pragma unroll
                    for (int i = 0; i < C::TCH; ++i) {
                        const int id = lane + 64 * i;
                        const int tk = id / (D / 8), col = id % (D / 8);
                        const int trow = q0 + tk < Lq ? q0 + tk : Lq - 1;
                        const u32x4 cv = *(const u32x4 *)(a.cs + (size_t)trow * (D / 2) + 4 * col);
                        const u32x4 sv = *(const u32x4 *)(a.sn + (size_t)trow * (D / 2) + 4 * col);
                        u32x2 *cd = (u32x2 *)(cosT + tk * C::TST + 4 * col), *sd = (u32x2 *)(sinT + tk * C::TST + 4 * col);
                        cd[0] = u32x2{cv[0], cv[1]};
                        cd[1] = u32x2{cv[2], cv[3]};
                        sd[0] = u32x2{sv[0], sv[1]};
                        sd[1] = u32x2{sv[2], sv[3]};
                    }
                }
                __syncthreads();
#pragma unroll
                for (int e2 = 0; e2 < C::DB / 2; ++e2) {
                    const int eb = half * (C::DB / 2) + e2;
                    f32x16 acc[RB];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[rb][r] = 0.f;
#pragma unroll
                    for (int t = 0; t < C::KS; ++t) {
                        const bf16x8 wf = *(const bf16x8 *)(smW + (32 * e2 + c) * C::KROW + 32 * t + 16 * hh);
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf[rb][t], acc[rb], 0, 0, 0);
                    }
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        if (rope) {
#pragma unroll
                            for (int j4 = 0; j4 < 4; ++j4) {      // registers 4 j4 .. +3: features 32 eb + 8 j4 + 4 hh + 0..3
                                const f32x2 c2 = *(const f32x2 *)(cosT + (32 * rb + c) * C::TST + 16 * eb + 4 * j4 + 2 * hh);
                                const f32x2 s2 = *(const f32x2 *)(sinT + (32 * rb + c) * C::TST + 16 * eb + 4 * j4 + 2 * hh);
#pragma unroll
                                for (int p = 0; p < 2; ++p) {
                                    const float y0 = acc[rb][4 * j4 + 2 * p], y1 = acc[rb][4 * j4 + 2 * p + 1];
                                    acc[rb][4 * j4 + 2 * p] = y0 * c2[p] - y1 * s2[p];
                                    acc[rb][4 * j4 + 2 * p + 1] = fmaf(y0, s2[p], y1 * c2[p]);
                                }
                            }
                        }
#pragma unroll
                        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const bf16_t y = to_bf16(acc[rb][8 * tt + j]);
                                qf[rb][2 * eb + tt][j] = y;
                                qss[rb] = fmaf((float)y, (float)y, qss[rb]);
                            }
                    }
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) qss[rb] = xhalf_sum(qss[rb]);
        }
        if constexpr (!EARLY_STATE) {
            __syncthreads();                              // every wave is done with the K/V ring
            load_state();
            store_state();
            __syncthreads();
        }
        f32x16 inter[C::DBW][RB];
#pragma unroll
        for (int db = 0; db < C::DBW; ++db)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int r = 0; r < 16; ++r) inter[db][rb][r] = 0.f;
        // k-slot j of half-wave hh must be d = 16t + 8hh + j to match q fragments loaded from memory, and
        // d = 16t + 8(j/4) + 4hh + j%4 to match fragments that were accumulator registers (fused feature map)
        const int s_row = FUSED_MAP ? ((lane & 15) >> 2) + 4 * hh : 8 * hh + ((lane & 15) >> 2);
        const int s_second = (FUSED_MAP ? 8 : 4) * C::VROW;
        const int s_frag_off = s_row * C::VROW + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
#pragma unroll
        for (int t = 0; t < C::KS; ++t)
#pragma unroll
            for (int db = 0; db < C::DBW; ++db) {
                const unsigned char *p = smHi + s_frag_off + 16 * t * C::VROW + 64 * (db0 + db);
                const bf16x8 sh = lds_read_tr_pair(p, s_second), sl = lds_read_tr_pair(p + C::SS_BYTES, s_second);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) inter[db][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sh, qf[rb][t], inter[db][rb], 0, 0, 0);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) inter[db][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sl, qf[rb][t], inter[db][rb], 0, 0, 0);
            }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float gq = (1.0f / sqrtf(qss[rb] + a.l2_eps)) * g_row[rb];       // gate * L2 norm scale for this lane's query row
            if (a.g != nullptr && a.g_per_element) {
                // one gate per output feature: registers 4 j .. 4 j + 3 of block db are features 32 db + 8 j + 4 hh + 0..3
#pragma unroll
                for (int db = 0; db < C::DBW; ++db)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const size_t ge = gi[rb] * D + 32 * (db0 + db) + 8 * j + 4 * hh;
                        float g4[4];
                        if (a.g_is_bf16) {
                            const bf16x4 x = *(const bf16x4 *)((const bf16_t *)a.g + ge);
#pragma unroll
                            for (int i = 0; i < 4; ++i) g4[i] = (float)x[i];
                        } else {
                            const f32x4 x = *(const f32x4 *)((const float *)a.g + ge);
#pragma unroll
                            for (int i = 0; i < 4; ++i) g4[i] = x[i];
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            out[db][rb][4 * j + i] = fmaf(gq * g4[i], inter[db][rb][4 * j + i], out[db][rb][4 * j + i]);
                    }
            } else {
#pragma unroll
                for (int db = 0; db < C::DBW; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) out[db][rb][r] = fmaf(gq, inter[db][rb][r], out[db][rb][r]);
            }
        }
    }

    // Transpose through LDS so that rows are written as contiguous 16-byte pieces, each wavefront its own block of
    // WR rows x 32 DBW features.  With two key groups the block lies where the wavefront has just read its peer's
    // partial result (nobody else touches that part); with one it may lie where others still read the state.
    constexpr int OROW = 64 * C::DBW + 16, OCPR = 4 * C::DBW;          // LDS bytes and 16-byte chunks per row
    static_assert(WR * OROW <= RB * C::DBW * 16 * 64 * 4, "the block fits the peer's partial result");
    unsigned char *region = smem + (KG == 1 ? wave * WR * OROW : (wave ^ C::RG) * (C::DBW * 16 * 64 * 4));
    if (KG == 1 || FUSED_MAP) __syncthreads();
#pragma unroll
    for (int db = 0; db < C::DBW; ++db)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                bf16x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = to_bf16(out[db][rb][4 * j4 + i]);
                *(bf16x4 *)(region + (32 * rb + c) * OROW + 2 * (32 * db + 8 * j4 + 4 * hh)) = w;
            }
    bf16_t *og = (bf16_t *)a.out;
#pragma unroll
    for (int i = 0; i < WR * OCPR / 64; ++i) {
        const int idx = lane + 64 * i;
        const int row = idx / OCPR, col = idx % OCPR;
        const int orow = q0 + row;
        if (orow < Lq) {
            const u32x4 x = *(const u32x4 *)(region + row * OROW + 16 * col);
            *(u32x4 *)(og + ((size_t)(b * (size_t)Lq + orow) * H + h) * D + 32 * db0 + 8 * col) = x;
        }
    }
}

// How the workgroups of a launch divide the query tiles: whole 256-row tiles, half tiles of 128 rows with two key groups, or
// whole tiles first (D = 64: or none) and half ones behind them, which at D = 64 have one key group.
enum FwdSplit { kWhole, kHalves, kHalvesLast };

struct FwdGrid {
    int n_qtiles;        // 256-row tiles per head (kHalves: 128-row tiles)
    int n_tiles;         // all tiles
    int n_whole;         // kHalvesLast: tiles that are served whole
    int ragged_last;
    int one_per_cu;      // kWhole, D = 64: workgroups of eight wavefronts with 32 rows each, not of four with 64
};

// Whole tiles.  D = 128: eight wavefronts of 32 rows, whose accumulators fill the registers.  D = 64: four wavefronts of 64
// rows, for which every operand fragment read from LDS serves two products, and two workgroups per CU.  While there is at most
// one tile per CU, where four wavefronts would each be alone on a SIMD, eight of 32 rows here too.  With a state, tails
// halved, eight wavefronts and four: 12 heads x 64, 4680 tokens (228 tiles) 77 and 82 us; 3 x 24 heads, 999 tokens (288 tiles)
// 33.3 and 27.6 us; 8 x 12 heads, 4680 tokens 579 and 529 us.
// The half tiles behind whole ones have the whole tiles' number of wavefronts, at D = 64 four, and with that one key group.
template <int D>
struct Whole {
    static constexpr int RB = D == 64 ? 2 : 1, NW = 8 / RB;
    static constexpr int SMEM = FwdCfg<D, 1, RB, NW>::SMEM, SMEM8 = FwdCfg<D, 1, 1, 8>::SMEM;
    static_assert(D == 128 || SMEM <= 80 * 1024, "two workgroups per CU");
};

template <int D, FwdSplit SPLIT, bool FUSED_MAP>
__global__ __launch_bounds__(SPLIT == kWhole || SPLIT == kHalves ? 512 : 64 * Whole<D>::NW, 2)
void fwd_bf16_kernel(FwdArgs a, FwdGrid g, float scale_log2)
{
    constexpr int RB = Whole<D>::RB, NW = SPLIT == kHalves ? 8 : Whole<D>::NW, KH = NW / 4;     // KH: key groups of a half tile
    constexpr bool TWO_FORMS = SPLIT == kWhole && RB > 1;       // the launch says how much LDS
    constexpr int SMEM1 = Whole<D>::SMEM, SMEM2 = FwdCfg<D, KH, 1, NW>::SMEM;
    __shared__ __attribute__((aligned(16))) unsigned char fixed_smem[TWO_FORMS ? 16 : SPLIT == kWhole ? SMEM1 : SPLIT == kHalves ? SMEM2 : SMEM1 > SMEM2 ? SMEM1 : SMEM2];
    extern __shared__ __attribute__((aligned(16))) unsigned char launch_smem[];
    unsigned char *smem = TWO_FORMS ? launch_smem : fixed_smem;
    int id = blockIdx.x, half = -1;
    if (SPLIT == kHalvesLast && id >= g.n_whole) {
        const int n_rest = g.n_tiles - g.n_whole;
        half = (id - g.n_whole) / n_rest;
        id = g.n_whole + (id - g.n_whole) % n_rest;
    }
    int qt, bh;
    if (g.ragged_last) {
        // Several rounds of workgroups, and the last query tile of every head is ragged (its workgroup has
        // idle wavefronts and finishes early): every XCD takes B H / 8 heads, their full tiles first, head
        // by head, and their ragged tiles at the end of its dispatch order, where a short job shortens the
        // last, partly filled round (workgroup ids go round the 8 XCDs in dispatch order).
        const int x = id % kNumXcd, loc = id / kNumXcd;
        const int heads_x = a.B * a.H / kNumXcd, n_full = g.n_qtiles - 1;
        if (loc < heads_x * n_full) {
            bh = x * heads_x + loc / n_full;
            qt = loc % n_full;
        } else {
            bh = x * heads_x + (loc - heads_x * n_full);
            qt = n_full;
        }
    } else {
        const int work = xcd_contiguous_id(id, g.n_tiles);
        qt = work % g.n_qtiles;
        bh = work / g.n_qtiles;
    }
    if constexpr (SPLIT == kWhole) {
        if constexpr (TWO_FORMS) {
            if (g.one_per_cu) {
                fwd_tile<D, 1, 1, 8, FUSED_MAP>(a, scale_log2, bh, qt, smem);
                return;
            }
        }
        fwd_tile<D, 1, RB, NW, FUSED_MAP>(a, scale_log2, bh, qt, smem);
    } else if constexpr (SPLIT == kHalves) {
        fwd_tile<D, KH, 1, NW, FUSED_MAP>(a, scale_log2, bh, qt, smem);
    } else if (half < 0) {
        fwd_tile<D, 1, RB, NW, FUSED_MAP>(a, scale_log2, bh, qt, smem);
    } else if ((2 * qt + half) * 128 < a.Lq) {
        fwd_tile<D, KH, 1, NW, FUSED_MAP>(a, scale_log2, bh, 2 * qt + half, smem);
    }
}

template <int D, FwdSplit SPLIT>
hipError_t launch_fwd(const FwdArgs &a, FwdGrid g, float scale_log2, hipStream_t stream)
{
    // (a tile of up to 128 rows has no second half)
    const int n_wg = SPLIT == kHalvesLast && a.Lq > 128 ? 2 * g.n_tiles - g.n_whole : g.n_tiles;
    const bool eight = SPLIT == kHalves || Whole<D>::NW == 8 || (SPLIT == kWhole && g.one_per_cu);
    const dim3 grid((unsigned)n_wg), block(eight ? 512 : 256);
    const unsigned lds = SPLIT != kWhole || Whole<D>::NW == 8 ? 0 : g.one_per_cu ? Whole<D>::SMEM8 : Whole<D>::SMEM;
    if (a.xq != nullptr) return launch_kernel_lds(fwd_bf16_kernel<D, SPLIT, true>, grid, block, lds, stream, a, g, scale_log2);
    return launch_kernel_lds(fwd_bf16_kernel<D, SPLIT, false>, grid, block, lds, stream, a, g, scale_log2);
}

// Whether `tiles` query tiles of up to `rows` rows are faster in half tiles of two key groups, as far as rows and keys decide
// it.  Such a half tile has a longer start and end (the key groups' exchange); what it shortens is the key loop.  Half against
// whole tiles of eight wavefronts, in us, softmax alone (with a state, gate or fused map the lines are the same):
//   more than 128 rows, so that halving makes more workgroups: from two key tiles on (128 heads x 128, 200 rows: 64 keys
//     7.7 and 7.4, 65 keys 7.6 and 8.5; x 64: 5.7 and 5.3, 5.7 and 6.1);
//   up to 128 rows, where two wavefronts share a loop and nothing else is gained: 24 heads x 128, 128 rows: 384 keys 9.6
//     and 8.9, 640 keys 12.3 and 11.9, 1024 keys 16.5 and 16.5; 64 rows: 640 keys 11.7 and 11.8; 24 heads x 64, 64 rows: 384
//     keys 7.0 and 6.7, 512 keys 7.8 and 7.8, 640 keys 8.7 and 8.9;
//   the same on more than three quarters of the CUs at D = 128, where reading keys and values is the bound and whole tiles
//     have more of them in flight: 256 heads, 128 rows: 1536 keys 37 and 35, 2048 keys 49 and 57.
template <int D>
bool halves_pay(int rows, int keys, long long tiles)
{
    if (rows > 128) return keys > BN;                    // (two key groups need a key each in the first tile)
    if (D == 128 && 4 * tiles > 3 * kNumCu) return keys >= 32 * BN;
    return keys >= (D == 128 ? 10 : 8) * BN;
}

// D = 64, more 256-row tiles than CUs: whether tiles of 128 rows, four wavefronts with 32 each, serve the whole launch.  Where
// the 64-row wavefronts of a whole tile find no rows, or only one key tile, they are slower than the eight of 32 rows that
// they replaced; the small tiles are slower than neither.  In us, softmax alone, eight wavefronts / 64-row ones / small tiles:
//   up to 128 rows, which leave two of the four 64-row wavefronts without any: 288 heads, 65 rows, 64 keys 7.1 / 8.3 / 5.1; 128
//     rows, 384 keys 14.0 / 15.9 / 11.1; 512 heads, 128 rows, 640 keys 21.2 / 25.6 / 21.9; 2048 heads, 128 rows, 1024 keys
//     149 / 136 / 122; up to 64 rows, one wavefront's, it is the other way from eight key tiles on while two rounds of tiles
//     are not full: 320 heads, 64 rows, 640 keys 18.5 / 15.5 / 16.5; 426 heads, 2048 keys 44.8 / 37.1 / 38.8; 464 heads, 1024
//     keys 27.8 / 27.7 / 26.4;
//   one key tile, to which the 64-row wavefronts add an empty one: 200 heads, 384 rows 9.0 / 9.7 / 8.3, 600 rows 12.7 / 13.7 /
//     10.1; 256 heads, 1000 rows 22.1 / 19.8 / 18.5; beyond four rounds they have made up for it: 768 heads, 1000 rows
//     57.8 / 46.8 / 48.4.
bool small_tiles_pay(int rows, int keys, int tiles)
{
    if (rows > 128) return keys <= BN && tiles <= 4 * kNumCu;
    return rows > 64 || keys < 8 * BN || 4 * tiles > 7 * kNumCu;
}

template <int D>
hipError_t launch_fwd(const FwdArgs &a, hipStream_t stream)
{
    const float scale_log2 = a.sm_scale * 1.4426950408889634f;
    const long long heads = (long long)a.B * a.H;
    const long long q256 = (a.Lq + 255) / 256, q128 = (a.Lq + 127) / 128;
    if (heads * q128 > 0x3fffffffLL) return hipErrorInvalidValue;
    FwdGrid g = {};
    g.n_qtiles = (int)q256;
    g.n_tiles = g.n_whole = (int)(heads * q256);
    // more workgroups than CUs, a ragged last query tile per head, and whole heads per XCD
    g.ragged_last = g.n_tiles > kNumCu && a.Lq % 256 != 0 && q256 > 1 && heads % kNumXcd == 0;
    // Half tiles while they run as one round: 1024 tokens x 16 heads x 128 19.6 us against 27.1 us for whole tiles, x 32
    // heads (256 half tiles) 23.4 against 28.7 us; with the fused map, whose matrix half as many rows share, 24.6 against 31.8
    // and 28.4 against 33.7 us; just beyond, x 48 heads, 43.9 against 34.9 us.
    if (heads * q128 <= kNumCu && halves_pay<D>(a.Lq, a.Lkv, heads)) {
        g.n_qtiles = (int)q128;
        g.n_tiles = (int)(heads * q128);
        g.ragged_last = 0;
        return launch_fwd<D, kHalves>(a, g, scale_log2, stream);
    }
    if constexpr (D == 64)
        if (g.n_tiles > kNumCu && small_tiles_pay(a.Lq, a.Lkv, g.n_tiles)) {
            g.n_whole = 0;
            return launch_fwd<D, kHalvesLast>(a, g, scale_log2, stream);
        }
    // The tail of a launch of several rounds: when at most half of the CUs would have a tile in it, these tiles are halved.
    // D = 128: a half tile takes 0.57 of the time of a whole one, so that 2048 tokens x 66 heads (2.06 rounds) take 156 instead
    // of 172 us, 1000 tokens x 272 heads (4.25 rounds) 174 instead of 180 us, and with the fused map 172 and 200 us instead of
    // 186 and 206 us.  D = 64, where a round is 256 tiles too, as the two workgroups of a CU share its time: 2048 tokens x 66
    // heads 82.5 instead of 93.9 us, 1000 tokens x 272 heads 79.6 instead of 85.2 us, with the fused map 92 and 95 instead of
    // 106 and 103 us.  Nothing changes where more than half of the CUs have work in the last round: 1024 tokens x 100 heads x 64
    // (1.56 rounds) 35.9 us, 40.1 us halved.
    // With up to 128 rows in the tail's tiles the whole ones of D = 64 leave wavefronts idle: 136 heads, 257 rows and keys
    // 13.0 us, 10.6 us halved (10.7 us with eight wavefronts of 32 rows); 192 heads, 384 rows and keys 16.8 and 13.8 us; so
    // these are halved in a second round for any number of keys.  Beyond it the line is halves_pay's, of which D = 64 could do
    // without: 272 heads, 300 rows, 70 keys (2.13 rounds) 12.5 us, 11.1 us halved (13.7 us with eight wavefronts).
    const int rest = g.n_tiles % kNumCu;
    const int tail_rows = g.ragged_last || q256 == 1 ? (a.Lq - 1) % 256 + 1 : 256;
    const bool pays = (D == 64 && tail_rows <= 128 && g.n_tiles <= 2 * kNumCu) || halves_pay<D>(tail_rows, a.Lkv, rest);
    if (g.n_tiles > kNumCu && rest > 0 && 2 * rest <= kNumCu && pays) {
        g.n_whole = g.n_tiles - rest;
        return launch_fwd<D, kHalvesLast>(a, g, scale_log2, stream);
    }
    g.one_per_cu = g.n_tiles <= kNumCu;
    return launch_fwd<D, kWhole>(a, g, scale_log2, stream);
}

}  // namespace

hipError_t launch_fwd_bf16(const FwdArgs &a, hipStream_t stream)
{
    // the kernel addresses one stream's K (or V) with 32-bit byte offsets
    if ((long long)(a.Lkv + 4 * BN) * a.H * a.D * 2 > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.D == 128) return launch_fwd<128>(a, stream);
    if (a.D == 64) return launch_fwd<64>(a, stream);
    return hipErrorInvalidValue;
}

}  // namespace arl2
