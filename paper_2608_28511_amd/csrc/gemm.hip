// Grouped bf16 GEMM on gfx950 MFMA for the routed experts (grouped GEMM over
// expert segments, Section 5.2), their backward, and the dense latent
// projections.
//
// One kernel template covers every product of the layer:
//
//   ROWS mode   C[r, n] = sum_k A[r, k] * B_e[k, n] for the rows r of expert
//               e's segment [offsets[e], offsets[e+1]) (forward up/down and
//               the two dgrads), or for all M rows when offsets is NULL
//               (dense latent projections).
//   KGRP mode   C_e[m, n] = sum_{r in segment e} A[r, m] * B[r, n]  (wgrad:
//               the contraction runs over the expert's ragged rows).
//
// Four block tiles on 512 threads, 8 wavefronts, in a 2 x 4 grid but for one
// (v_mfma_f32_16x16x32_bf16):
//   phased 256 x 256 (phased.h), 64 k per k tile: the dense weight gradients, and
//     ROWS launches and the experts' weight gradients where its coarser tile
//     count does not cost a round (take_phased, launch_grouped_wgrad2).  Its two
//     groups of waves alternate between reading fragments and multiplying, so
//     the matrix pipes are busy 80-90% of the k loop (the 128-row tile: 67%);
//     under it the chip is power bound: 1.6-1.75 GHz at 1.2-1.36 PFLOP/s.
//   128 x 256, 64 k per stage, 3-stage ring of 48 KB stages: the other ROWS
//     launches and the shortest weight gradients;
//   128 x 128, 4-stage ring of 32 KB stages, waves of 32 x 64 in a 4 x 2 grid:
//     the smallest ROWS launches (rows_kind);
//   256 x 256, 32 k per stage, 4-stage ring of 32 KB stages: the products over
//     an MX-FP8 A that are long enough, and the weight gradients of many experts
//     with few rows each.
// For all but the first neither the MFMAs nor copy bandwidth bound the kernel: all
// eight waves read after each barrier and then all multiply, and the waits
// are on LDS and copy latency.
// One workgroup fills a CU's LDS, so each SIMD runs two wavefronts: one wave's
// address arithmetic, barrier and LDS latency overlap the other's MFMAs.
//
// Operands never pass through registers on their way to LDS: every 16-byte
// chunk is copied by a buffer load with an LDS destination into the LDS
// ring, all but one stage in flight while one is consumed.  Each operand
// keeps the layout it has in HBM:
//   K-contiguous source  -> LDS rows of 64 or 32 k (XOR-swizzled by row),
//                           MFMA fragments read with ds_read_b128;
//   M/N-contiguous source (weights stored [D, F] / [F, D], both wgrad
//                           operands) -> LDS k-rows of BM or BN elements
//                           (chunk pairs XOR-swizzled by k), fragments read
//                           with two ds_read_b64_tr_b16, the gfx950 LDS
//                           transpose read, so no VALU transposition at all.
// A DMA lane's LDS destination is fixed by its lane id, so the swizzles are
// applied by permuting which global chunk each lane fetches.  Lanes whose
// chunk lies outside the operand (ragged expert rows, k / n tails) fetch a
// zero chunk instead, so partial tiles need no special path.
//
// The MFMA takes the weight-side fragment as its first operand, so each
// lane's four accumulators hold four consecutive output columns of one row.
//
// ROWS mode runs persistently: one workgroup per CU walks its share of the
// output tiles, and the DMA ring runs over the flattened sequence of (tile,
// k step) pairs, so the first two k steps of a workgroup's next tile are
// already loading while it finishes the current one.  Output tiles are
// written through a 16 KB LDS slice (16 x 64 bf16 per wave) so that every
// store is 16 contiguous bytes and one store instruction covers 8 whole
// 128-byte rows; stores go through a range-checked buffer descriptor, so
// rows past the tile's end and columns past N are dropped by the hardware.
// Squared-ReLU (up projection) is fused there, and so is the dgrad's
// product with the activation derivative, whose saved pre-activation each
// lane loads at its accumulators' positions.
//
// The up projection can also read its A operand as the MX-FP8 dispatch
// payload (gemm_rows_mx_kernel): codes and block scales travel through the
// same ring and each lane decodes its fragment right before the MFMA, with a
// result identical to decoding first (see MxDma and mx_frag).
//
// KGRP mode (weight gradients) takes (expert, m-tile, n-tile) items, one per
// workgroup or, on the phased tile, claimed by persistent workgroups.  The items of
// an expert take two m-tiles at a time across all n-tiles, so that those an XCD
// runs together keep their operand rows in its L2.  The fp32 tile leaves through LDS
// as whole row pieces, non-temporally but for the cases of GradStore.
//
// Expert segments are located through device-side tile tables (expert,
// first row, end row of every 128-row and every 256-row tile, built from the
// routing offsets on the device): no host reads the routing counts.  Work item w of the
// grid-wide order is tile (m, n) of an ordering that takes 8 m-tiles at a
// time across all n-tiles, and the items a round of workgroups processes
// together on one XCD are consecutive, so they share A rows and expert
// weights in that XCD's L2.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "phased.h"
#include "schedule.h"
#include "tile_dma.h"

namespace moe {

constexpr int BN = 256;
constexpr int kGemmThreads = kWaves * 64;
constexpr int kEpiWaveBytes = 16 * 64 * 2;      // 16 x 64 bf16 staging block per wave
constexpr int kEpiBytes = kWaves * kEpiWaveBytes;  // 16 KB
constexpr int kGroupM = 8;

// Block tile BM x BN with KD contraction elements per ring stage and a ring
// of STAGES stages.  AMX: A is MX-FP8 (codes, one byte per element, and the
// stage's block scales; see MxDma) instead of bf16.
template <int BM_, int KD_, int STAGES_, bool AMX_ = false, int BN_ = 256>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, KD = KD_, kStages = STAGES_;
    static constexpr bool kAmx = AMX_;
    static constexpr int kWaveN = BN / 64;      // waves side by side, 64 columns each
    static constexpr int kWaveRows = BM / (kWaves / kWaveN);
    static constexpr int MI = kWaveRows / 16;   // A fragments (16 rows) per wave
    static constexpr int kKK = KD / 32;         // MFMA k steps per stage
    static constexpr int kCodeBytes = BM * KD;  // AMX: the stage's codes, then its scale words
    static constexpr int kSclBytes = AMX_ ? kWaves * 64 * 4 : 0;
    static constexpr int kABytes = AMX_ ? kCodeBytes + kSclBytes : BM * KD * 2;
    static constexpr int kBBytes = BN * KD * 2;
    static constexpr int kStageBytes = kABytes + kBBytes;
    static constexpr int kRingBytes = kStages * kStageBytes;
    static constexpr int kFrag = 16 * KD * 2;   // bytes between 16-row fragments of the row layout
    static constexpr int kFragA = AMX_ ? 16 * KD : kFrag;
};
using TileS = Tile<128, 64, 3>;   // 144 KB ring (+16 KB epilogue staging)
using TileL = Tile<256, 32, 4>;   // 128 KB ring
using TileN = Tile<128, 64, 4, false, 128>;   // 128 KB ring; waves of 32 rows
using TileSX = Tile<128, 64, 3, true>;   // MX-FP8 A: 126 KB ring
using TileLX = Tile<256, 32, 4, true>;   // 104 KB ring
static_assert(TileN::kRingBytes + kEpiBytes <= 160 * 1024 &&
                  TileS::kRingBytes + kEpiBytes <= 160 * 1024 && TileL::kRingBytes + kEpiBytes <= 160 * 1024 &&
                  TileSX::kRingBytes + kEpiBytes <= 160 * 1024 && TileLX::kRingBytes + kEpiBytes <= 160 * 1024,
              "LDS budget");

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// MX-FP8 A operand (codes [R, Kd] uint8, E8M0 scales [R, Kd / 32] uint8):
// per stage each wave copies one 16-byte chunk of codes (rows of KD bytes,
// fp8 row layout) and one scale word.  A row's scale bytes are not 4-byte
// aligned, so every row gets a window of kLPR words starting at the aligned
// word at or below its first block of the stage; the fragment read takes its
// byte at offset (row * nb + kb) & 3 of the window.  The scale descriptor
// spans the whole array rounded up to 4 bytes: rows past R read zero, and
// rows past a tile's end (zero codes) read other rows' finite scales.
template <class T>
struct MxDma {
    static constexpr int kLPR = kWaves * 64 / T::BM;   // scale words per row
    static_assert(kLPR * T::BM == kWaves * 64 && 3 + T::kKK <= 4 * kLPR, "scale window");
    static constexpr int kSlots = 2;                     // copies per wave and stage
    DmaTile<true, T::BM, T::KD / 2, kWaves, 1> codes;    // code pairs as 16-bit elements
    static_assert(decltype(codes)::kSlots == 1, "one code chunk per wave and stage");
    i32x4 srs;       // wave-uniform
    uint32_t srow;   // (row0 + this lane's window row) * nb
    uint32_t sword;  // byte of this lane's word in the window
    uint32_t kb;     // first block of the next stage

    __device__ __forceinline__ void init(const uint8_t* q, const uint8_t* scale, uint32_t scale_bytes,
                                         int64_t row0, int64_t row_hi, int Kd, int wave, int lane) {
        codes.init((const uint16_t*)q, Kd / 2, row0, row_hi, 0, Kd / 2, wave, lane);
        srs = buf_rsrc(scale, scale_bytes);
        const int p = wave * 64 + lane;
        srow = (uint32_t)((row0 + p / kLPR) * (Kd / 32));
        sword = (uint32_t)(4 * (p % kLPR));
        kb = 0;
    }
    template <bool KTAIL, int I0, int I1>
    __device__ __forceinline__ void issue(uint32_t tile_lds, int64_t k_rem, int wave) {
        codes.template issue<KTAIL, 0, 1>(tile_lds, k_rem / 2, wave);
        dma4(srs, ((srow + kb) & ~3u) + sword, tile_lds + T::kCodeBytes + (uint32_t)wave * 256u);
        kb += T::kKK;
    }
};

// bf16 MFMA fragment of 8 MX-FP8 codes sharing one E8M0 scale byte s8:
// code * 2^(s8 - 127).  v_cvt_scalef32_pk_bf16_fp8 takes the scale from the
// exponent field of an fp32 operand; for every finite code at every scale
// byte up to 246 (the largest the encoder emits) its result equals the exact
// decode, bf16 subnormals included (checked exhaustively on gfx950).
__device__ __forceinline__ bf16x8 mx_frag(u32x2 c, uint32_t s8) {
    const float sc = __uint_as_float(s8 << 23);
    const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[0], sc, false);
    const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[0], sc, true);
    const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[1], sc, false);
    const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[1], sc, true);
    const u32x4 w = {__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1),
                     __builtin_bit_cast(uint32_t, p2), __builtin_bit_cast(uint32_t, p3)};
    return __builtin_bit_cast(bf16x8, w);
}

struct GemmArgs {
    const uint16_t* A;
    const uint16_t* B;
    void* C;
    const uint16_t* aux_in;   // EPI_DRELU2: pre-activation u, same layout as C
    uint16_t* aux_out;        // EPI_RELU2: pre-activation u (may be null)
    const int32_t* offsets;   // [E+1] expert row segments (KGRP mode)
    const int32_t* order;     // KGRP pair launch: experts by descending row count (the item order)
    const int4* tiles;        // ROWS mode: per 128-row tile {expert, row0, row_end, 0}; null = dense
    const int32_t* mtile_total;  // ROWS mode with tiles: device count of valid 128-row m-tiles
    const int4* tiles_l;      // the same for 256-row tiles
    const int32_t* mtile_total_l;
    const int32_t* a_perm;    // ROWS mode, bf16 A gathered: row r of the product is A row a_perm[r] / a_div
    int a_div;
    uint32_t a_mul;           // v / a_div = v * a_mul >> a_shift for 0 <= v < 2^31
    int a_shift;
    int64_t a_src_rows;       // rows of the gathered A
    const uint8_t* A_scale;   // MX-FP8 A: E8M0 scales [R, Kd / 32]
    uint32_t scale_bytes;     // R * Kd / 32 rounded up to a multiple of 4
    int64_t lda, ldb, ldc;
    int64_t b_stride;         // elements between experts' B (ROWS mode)
    int64_t c_stride;         // elements between experts' C (KGRP mode)
    int64_t M;                // dense rows (ROWS, no offsets) or output rows (KGRP)
    int64_t R;                // rows of the activation buffers: segments are clamped to [0, R)
    int N, Kd, E;
    int m_tiles, n_tiles;
    int m_tiles_l;            // ROWS mode: m-tiles of 256 rows (dense) or their static bound
    int accumulate;           // EPI_F32: C += product instead of C = product
    int store;                // phased KGRP: GradStore of C
};

// Wait until stage `cur` of `total` has landed when stages cur + 1 ..
// cur + T::kStages - 2 (those that exist) may still be in flight: copies
// complete in order, so at most that many stages' worth may be outstanding.
template <class T, int kPerStage>
__device__ __forceinline__ void wait_stage(int cur, int total) {
    const int ahead = total - 1 - cur;
    if constexpr (T::kStages >= 4) {
        if (ahead >= 2) { wait_vmcnt<2 * kPerStage>(); return; }
    }
    if constexpr (T::kStages >= 3) {
        if (ahead >= 1) { wait_vmcnt<kPerStage>(); return; }
    }
    wait_vmcnt<0>();
}

// One KD-wide stage of the main loop for stage slot S of the ring: read the
// fragments of each 32-wide k step, send the copies of the stage kStages - 1
// ahead (half of B after the second k step's reads when a stage has two),
// and accumulate.  `next` says whether there is a stage to copy; nrem is the
// contraction length left from its start.
// AMX: sb is the lane's scale byte of the stage's first block in slot 0.
template <class T, bool A_K, bool B_K, bool KTAIL, int S, class DA, class DB, int NA, int NB>
__device__ __forceinline__ void mma_stage(f32x4 (&acc)[T::MI][4], const uint32_t (&abase)[NA],
                                          const uint32_t (&bbase)[2][NB], DA& da, DB& db, bool next,
                                          int64_t nrem, uint32_t ldsA, uint32_t ldsB, int wave,
                                          uint32_t sb = 0) {
    constexpr int NS = (S + T::kStages - 1) % T::kStages;
    constexpr int kSA = DA::kSlots, kSB = DB::kSlots;
#pragma unroll
    for (int kk = 0; kk < T::kKK; ++kk) {
        bf16x8 af[T::MI], bfg[4];
#pragma unroll
        for (int i = 0; i < T::MI; ++i) {
            if constexpr (T::kAmx) {
                // volatile: the compiler would pair these reads (512 bytes
                // apart) into ds_read2st64_b64, whose two addresses per lane
                // share banks (measured: 2.6x the LDS cycles)
                const u32x2 c =
                    *(const volatile lds_u32x2*)(uintptr_t)(abase[kk] + S * T::kABytes + i * T::kFragA);
                const uint32_t s8 =
                    *(const lds_u8*)(uintptr_t)(sb + S * T::kABytes + i * 16 * 4 * MxDma<T>::kLPR + kk);
                af[i] = mx_frag(c, s8);
            } else if constexpr (A_K) {
                af[i] = lds_b128(abase[kk] + S * T::kABytes + i * T::kFrag);
            } else {
                af[i] = lds_tr_pair(abase[i] + S * T::kABytes + kk * 64 * T::BM, 8 * T::BM);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            constexpr uint32_t so = (S & 1) * T::kBBytes;
            if constexpr (B_K) bfg[j] = lds_b128(bbase[S >> 1][kk] + so + j * T::kFrag);
            else bfg[j] = lds_tr_pair(bbase[S >> 1][j] + so + kk * 64 * T::BN, 8 * T::BN);
        }
        if (next) {
            if (T::kKK == 1) {
                da.template issue<KTAIL, 0, kSA>(ldsA + NS * T::kABytes, nrem, wave);
                db.template issue<KTAIL, 0, kSB>(ldsB + NS * T::kBBytes, nrem, wave);
            } else if (kk == 0) {
                da.template issue<KTAIL, 0, kSA>(ldsA + NS * T::kABytes, nrem, wave);
                db.template issue<KTAIL, 0, kSB / 2>(ldsB + NS * T::kBBytes, nrem, wave);
            } else {
                db.template issue<KTAIL, kSB / 2, kSB>(ldsB + NS * T::kBBytes, nrem, wave);
            }
        }
#pragma unroll
        for (int i = 0; i < T::MI; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfg[j], af[i], acc[i][j], 0, 0, 0);
    }
}

// Per-lane fragment bases of the A (BM-wide) and B (BN-wide) operands.
template <class T, bool A_K, bool B_K, int NA, int NB>
__device__ __forceinline__ void frag_bases(uint32_t (&abase)[NA], uint32_t (&bbase)[2][NB], uint32_t ldsA,
                                           uint32_t ldsB, int wm, int wn, int lane) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
        abase[i] = ldsA + (T::kAmx ? mx_row_base<T::KD>(wm * T::kWaveRows, i, lane)
                           : A_K  ? row_base<T::KD>(wm * T::kWaveRows, i, lane)
                                  : col_base<T::BM>(wm * T::kWaveRows + i * 16, lane));
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const uint32_t o = B_K ? row_base<T::KD>(wn * 64, j, lane) : col_base<T::BN>(wn * 64 + j * 16, lane);
        bbase[0][j] = ldsB + o;                    // stages 0 and 1
        bbase[1][j] = ldsB + 2 * T::kBBytes + o;   // stages 2 and 3 (immediate offsets reach 64 KB)
    }
}

template <int MI>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[MI][4]) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Calls step(integral_constant<S>, g) for g = g0 .. g0 + kStages - 1 (those
// below total), S the ring slot of step g.
template <int kStages, class F>
__device__ __forceinline__ void ring_round(F&& step, int g0, int total) {
    step(std::integral_constant<int, 0>{}, g0);
    if (g0 + 1 < total) step(std::integral_constant<int, 1 % kStages>{}, g0 + 1);
    if constexpr (kStages >= 3)
        if (g0 + 2 < total) step(std::integral_constant<int, 2 % kStages>{}, g0 + 2);
    if constexpr (kStages >= 4)
        if (g0 + 3 < total) step(std::integral_constant<int, 3 % kStages>{}, g0 + 3);
}

// ---------------------------------------------------------------------------
// KGRP mode (wgrad): C_e[m, n] = sum over expert e's rows r of A[r, m] B[r, n],
// fp32 output.  One workgroup per (expert, m-tile, n-tile).
template <class T>
__device__ __forceinline__ void kgrp_item(const GemmArgs& p, int e, int in, char* smem);

// The pair launch's items are those of the expert order (slot r = the
// expert with the r-th most rows), each slot holding problem 0's items, then
// problem 1's.  Workgroups go to XCDs round-robin, so workgroup b is the
// (b / 8)-th of XCD b % 8, and every XCD runs its items in the order below:
//   heavy slots (the leading ones, at most 8, whose expert holds more than
//   R / 16 rows: its two gradients are then over half an XCD's fair share)
//   are cut into chunks of kKgChunk consecutive items, chunk c going to XCD
//   c % 8, so every XCD holds an equal share of the longest contractions
//   (whole units left the XCD with the busiest experts of a Zipf routing
//   at ~1.2x its share);
//   the other slots' units (one expert, one problem) follow whole, dealt
//   in rounds of 8 that alternate direction (unit 8k + i to XCD i, or 7 - i
//   when k is odd, counted from the XCD after the last heavy chunk), so
//   the units' decreasing sizes even out across XCDs, and the items an XCD
//   runs together keep one expert's operand rows in its L2 (cutting them
//   too cost 2.6% on a balanced routing).
// Each XCD's share is padded to the same length; the padding comes last.
constexpr int kKgChunk = 8;

struct KgItem {
    int r, q, in;   // slot, problem, item; r < 0: padding
};

// The expert order's buffer: E ranks, then one claim counter per XCD, each in
// a 128-byte line of its own.
constexpr int kClaimStride = 32;
__host__ __device__ __forceinline__ int order_claims(int E) { return (E + kClaimStride - 1) / kClaimStride * kClaimStride; }
size_t expert_order_bytes(int E) { return (size_t)(order_claims(E) + kXcds * kClaimStride) * 4; }

// Slots whose expert holds more than R / 16 rows: a prefix of the order.
__device__ __forceinline__ int heavy_slots(const GemmArgs& p) {
    typedef const __attribute__((address_space(4))) int32_t* cptr;
    const cptr ord = (cptr)p.order, off = (cptr)p.offsets;
    const int n = p.E < kXcds ? p.E : kXcds;
    const int R = (int)p.R;
    int h = 0;
    for (; h < n; ++h) {
        int e = ord[h];
        e = (e >= 0 && e < p.E) ? e : h;
        int lo = off[e], hi = off[e + 1];
        lo = lo < 0 ? 0 : (lo > R ? R : lo);
        hi = hi < lo ? lo : (hi > R ? R : hi);
        if ((int64_t)(hi - lo) * 16 <= p.R) break;
    }
    return h;
}

// heavy0, heavy1: the two problems' items in a heavy slot (per0 and per1, unless
// those are cut smaller).
__device__ __forceinline__ KgItem kg_item(unsigned b, int E, int per0, int per1, int H, int heavy0, int heavy1) {
    const int per = heavy0 + heavy1, perm = per0 > per1 ? per0 : per1;
    const int64_t heavy = (int64_t)H * per;
    const int n_hc = (int)((heavy + kKgChunk - 1) / kKgChunk);
    const int x = (int)(b % kXcds), j = (int)(b / kXcds);
    const int nhx = n_hc > x ? (n_hc - x + kXcds - 1) / kXcds : 0;   // heavy chunks on XCD x
    KgItem it{-1, 0, 0};
    if (perm == 0) return it;
    if (j < nhx * kKgChunk) {
        const int64_t g = (int64_t)(x + kXcds * (j / kKgChunk)) * kKgChunk + j % kKgChunk;
        if (g >= heavy) return it;
        it.r = (int)(g / per);
        const int rem = (int)(g - (int64_t)it.r * per);
        it.q = rem >= heavy0 ? 1 : 0;
        it.in = rem - it.q * heavy0;
        return it;
    }
    const int jj = j - nhx * kKgChunk, k = jj / perm;
    const int xp = ((x - n_hc) % kXcds + kXcds) % kXcds;
    const int u = kXcds * k + ((k & 1) ? kXcds - 1 - xp : xp);
    const int r = H + u / 2, q = u & 1, in = jj - k * perm;
    if (r >= E || in >= (q ? per1 : per0)) return it;
    return KgItem{r, q, in};
}

// Items of XCD x in kg_item's order, its padding after the last one left out.
__device__ __forceinline__ int kg_count(int x, int E, int per0, int per1, int H, int heavy0, int heavy1) {
    const int perm = per0 > per1 ? per0 : per1;
    const int n_hc = (int)(((int64_t)H * (heavy0 + heavy1) + kKgChunk - 1) / kKgChunk);
    const int nhx = n_hc > x ? (n_hc - x + kXcds - 1) / kXcds : 0;
    const int xp = ((x - n_hc) % kXcds + kXcds) % kXcds;
    const int units = 2 * (E - H), full = units / kXcds;
    const int pos = (full & 1) ? kXcds - 1 - xp : xp;
    return nhx * kKgChunk + (full + (pos < units % kXcds ? 1 : 0)) * perm;
}

// Does the busiest expert's contraction, on the phased tile 1.35 us a k tile and
// 10.5 an item, outlast a workgroup's share of the work, items_per_wg of every expert?
// Halving the heavy items' rows costs about as much as it gains at 1.2 shares:
// 6 and 14% lost at 1.05 and 1.2 (16 experts x 2,433 rows, 1,584 x 1,104; 7 x 2,321, 664 x
// 3,328, all of them heavy), 7-20% won beyond.
__device__ __forceinline__ bool outlasts(const GemmArgs& p, float items_per_wg) {
    typedef const __attribute__((address_space(4))) int32_t* cptr;
    int e = ((cptr)p.order)[0];
    e = (e >= 0 && e < p.E) ? e : 0;
    const float rows = (float)(((cptr)p.offsets)[e + 1] - ((cptr)p.offsets)[e]);
    constexpr float kRow = 1.35f / 64, kItem = 10.5f;
    return rows * kRow + kItem > 1.25f * ((float)p.R * kRow + (float)p.E * kItem) * items_per_wg;
}

// The pair launch's grid: every XCD's longest possible share (8 heavy slots).
inline int64_t kg_grid(int E, int64_t per0, int64_t per1) {
    const int64_t per = per0 + per1, perm = per0 > per1 ? per0 : per1;
    const int64_t n_hc = ((E < kXcds ? E : kXcds) * per + kKgChunk - 1) / kKgChunk;
    return kXcds * ((n_hc + kXcds - 1) / kXcds * kKgChunk + (2 * (int64_t)E + kXcds - 1) / kXcds * perm);
}

// Two weight gradients over the same expert segments in one launch, items
// placed as above, so each gradient's long contractions overlap the other's
// instead of each launch ending on its own tail.
template <class T>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_kgrp2_kernel(GemmArgs p0, GemmArgs p1) {
    __shared__ __attribute__((aligned(1024))) char smem[T::kRingBytes];
    const int per0 = p0.m_tiles * p0.n_tiles, per1 = p1.m_tiles * p1.n_tiles;
    const KgItem it = kg_item(blockIdx.x, p0.E, per0, per1, heavy_slots(p0), per0, per1);
    if (it.r < 0) return;
    const GemmArgs& p = it.q ? p1 : p0;
    const int eo = ((const __attribute__((address_space(4))) int32_t*)p0.order)[it.r];
    const int e = (eo >= 0 && eo < p0.E) ? eo : it.r;
    kgrp_item<T>(p, e, it.in, smem);
}

// Two m-tiles at a time across all n-tiles: the ~32 items an XCD runs
// together then share two m-tiles of A rows and a run of n-tiles of B
// rows, which fit its L2 (all m-tiles at a time did not: the 31.5B
// shape's wgrad 3286 -> ~3100 us; groups of 4 and 8 fell in between).
constexpr int kKgM = 2;

// fp32 store of a wave's MI x 16 rows x 64 columns from row rbase and column
// cbase of C_e, through the wave's 4 KB LDS slice: per 16-row block 16 x 64 fp32
// go there (16-byte chunk c of row r at c ^ r) and come back as whole
// 256-byte row pieces, 4 rows per store instruction, written
// non-temporally: the gradient is not read here, and full lines keep the
// bypassing writes efficient while the operand rows stay in L2.  (Also where
// rows start beside a line and a piece fills one of three: cached stores would
// move the cost to the launches that follow, see GradStore.)
template <int MI>
__device__ __forceinline__ void kgrp_store(const f32x4 (&acc)[MI][4], const GemmArgs& p, int e, uint32_t ep, int rbase,
                                           int cbase, int lane) {
    const int r = lane & 15;
    const int rq = lane >> 4, c = lane & 15;
    const int ncol = cbase + c * 4;
    float* const C = (float*)p.C + (int64_t)e * p.c_stride + ncol;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ch = (j * 4 + (lane >> 4)) ^ r;
            *(__attribute__((address_space(3))) f32x4*)(uintptr_t)(ep + (uint32_t)(r * 256 + ch * 16)) = acc[i][j];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rr = q * 4 + rq;
            const f32x4 v =
                *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)(ep + (uint32_t)(rr * 256 + ((c ^ rr) * 16)));
            const int64_t m = rbase + i * 16 + rr;
            if (m < p.M && ncol < p.N) __builtin_nontemporal_store(v, (f32x4*)(C + m * p.ldc));
        }
    }
}

// Item `in` (an m-tile, n-tile pair) of expert e.
template <class T>
__device__ __forceinline__ void kgrp_item(const GemmArgs& p, int e, int in, char* smem) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar LDS offsets
    const int wm = wave >> 2, wn = wave & 3;
    const int width = kKgM * p.n_tiles;
    const int grp = in / width, first_m = grp * kKgM;
    const int gsz = (p.m_tiles - first_m) < kKgM ? (p.m_tiles - first_m) : kKgM;
    const int in2 = in - grp * width;
    const int mt = first_m + in2 % gsz, nt = in2 / gsz;
    const int64_t row0 = (int64_t)mt * T::BM;
    const int64_t row_hi = (row0 + T::BM) < p.M ? (row0 + T::BM) : p.M;
    int64_t k_begin = p.offsets[e], k_end = p.offsets[e + 1];
    k_begin = k_begin < 0 ? 0 : (k_begin > p.R ? p.R : k_begin);
    k_end = k_end < k_begin ? k_begin : (k_end > p.R ? p.R : k_end);
    const int64_t n0 = (int64_t)nt * BN;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const uint32_t ldsB = lds0, ldsA = lds0 + T::kStages * T::kBBytes;

    DmaTile<false, T::BM, T::KD> da;
    DmaTile<false, BN, T::KD> db;
    da.init(p.A, p.lda, row0, row_hi, k_begin, k_end, wave, lane);
    db.init(p.B, p.ldb, n0, (int64_t)p.N, k_begin, k_end, wave, lane);
    constexpr int kSA = DmaTile<false, T::BM, T::KD>::kSlots, kSB = DmaTile<false, BN, T::KD>::kSlots;
    constexpr int kPerStage = kSA + kSB;

    uint32_t abase[T::MI], bbase[2][4];
    frag_bases<T, false, false>(abase, bbase, ldsA, ldsB, wm, wn, lane);

    f32x4 acc[T::MI][4];
    zero_acc(acc);

    const int64_t klen = k_end - k_begin;
    const int nk = (int)((klen + T::KD - 1) / T::KD);

    auto step = [&](auto stage_c, int kt) {
        constexpr int S = decltype(stage_c)::value;
        wait_stage<T, kPerStage>(kt, nk);
        stage_barrier();
        mma_stage<T, false, false, true, S>(acc, abase, bbase, da, db, kt + T::kStages - 1 < nk,
                                            klen - (int64_t)(kt + T::kStages - 1) * T::KD, ldsA, ldsB, wave);
    };

    if (nk > 0) {
        for (int q = 0; q < T::kStages - 1 && q < nk; ++q) {
            da.template issue<true, 0, kSA>(ldsA + q * T::kABytes, klen - (int64_t)q * T::KD, wave);
            db.template issue<true, 0, kSB>(ldsB + q * T::kBBytes, klen - (int64_t)q * T::KD, wave);
        }
        for (int kt = 0; kt < nk; kt += T::kStages) ring_round<T::kStages>(step, kt, nk);
    }

    __syncthreads();   // the ring is free
    kgrp_store<T::MI>(acc, p, e, lds0 + (uint32_t)wave * 4096u, (int)row0 + wm * (T::BM / 2), (int)n0 + wn * 64, lane);
}

// ---------------------------------------------------------------------------
// ROWS mode, persistent.

struct RowsTile {
    int e, row0, row_hi, n0;  // rows and columns are below 2^31
};

static_assert(kSchedGroupM == kGroupM, "schedule runs and dense groups take the same m-tiles");

template <int BM, int BN>
__device__ __forceinline__ RowsTile rows_tile(const GemmArgs& p, const int4* tiles, int m_count, int n_tiles, int w,
                                              int m_base) {
    typedef const __attribute__((address_space(4))) int32_t* cptr;
    // item w of the m-tiles [m_base, m_base + m_count) x all n-tiles, taken a
    // group of m-tiles at a time across all n-tiles: with a tile table the
    // groups are its runs of one expert's m-tiles (cut at the share's ends),
    // dense rows take kGroupM m-tiles at a time
    int mt, nt;
    if (tiles != nullptr) {
        // item w lies in the run that holds m-tile m_base + w / n_tiles (a
        // run of s m-tiles covers s * n_tiles consecutive items); the table
        // is written by an earlier launch and read-only here: scalar loads
        // through the constant address space
        const int q = m_base + w / n_tiles;
        const int packed = ((cptr)(tiles + q))[3];
        int a = packed >> 4, b = a + (packed & 15);
        a = a > m_base ? a : m_base;
        b = b < m_base + m_count ? b : m_base + m_count;
        if (a > q || b <= q) { a = q; b = q + 1; }   // an entry that does not hold q: take q alone
        const int s = b - a;
        const int in = w - (a - m_base) * n_tiles;
        mt = a + in % s;
        nt = in / s;
        nt = nt < n_tiles ? nt : n_tiles - 1;
    } else {
        const int width = kGroupM * n_tiles;
        const int group = w / width;
        const int first_m = group * kGroupM;
        const int gsz = (m_count - first_m) < kGroupM ? (m_count - first_m) : kGroupM;
        const int in = w - group * width;
        mt = m_base + first_m + in % gsz;
        nt = in / gsz;
    }
    mt = __builtin_amdgcn_readfirstlane(mt);
    RowsTile t;
    if (tiles != nullptr) {
        const __attribute__((address_space(4))) int32_t* ti =
            (const __attribute__((address_space(4))) int32_t*)(tiles + mt);
        t.e = ti[0];
        t.row0 = ti[1];
        t.row_hi = ti[2];
    } else {
        t.e = 0;
        t.row0 = mt * BM;
        t.row_hi = (t.row0 + BM) < p.M ? (t.row0 + BM) : (int)p.M;
    }
    t.n0 = nt * BN;
    return t;
}

// Buffer descriptor over rows [row0, row0 + nrows) of a row-major bf16 matrix:
// accesses at byte offsets >= nrows * ldc * 2 are dropped (stores) or read as
// zero (loads) by the hardware.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* base, int64_t row0, int64_t nrows,
                                                            int64_t ldc) {
    const uint16_t* b = (const uint16_t*)base + row0 * ldc;
    const int32_t bytes = nrows > 0 ? (int32_t)(nrows * ldc * 2) : 0;
    return __builtin_amdgcn_make_buffer_rsrc((void*)b, 0, bytes, 0x00020000);
}

constexpr uint32_t kDropOffset = 0x80000000u;  // beyond any descriptor's range
constexpr int kNonTemporal = 2;                // cache policy of a buffer store

// Staged epilogue of one 64 x 64 wave tile (EPI_BF16 / EPI_RELU2 /
// EPI_DRELU2): per 16-row block, the accumulators go to the wave's LDS slice
// as bf16 (chunk c of row r at c ^ (r & 7)), come back as 16-byte row pieces
// and leave as two buffer_store_dwordx4 of 8 rows x 128 bytes each.  OUT:
// 0 = the product (squared-ReLU applied for EPI_RELU2; times 2 max(u, 0),
// u from uu at the accumulators' positions, for EPI_DRELU2), 1 = the raw
// product (pre-activation).
template <int EPI, int OUT, int MI>
__device__ __forceinline__ void staged_store(const f32x4 (&acc)[MI][4], void* C, int64_t ldc, int N,
                                             int64_t rbase, int64_t nrows, int64_t cbase,
                                             uint32_t ep, int lane, const u32x2 (*uu)[4] = nullptr) {
    const __amdgpu_buffer_rsrc_t rs = rows_rsrc(C, rbase, nrows, ldc);
    const int r = lane & 15;
    const uint32_t wr = ep + (uint32_t)(r * 128 + (lane >> 4 & 1) * 8);
    const int rr0 = lane >> 3, c = lane & 7;
    const bool col_ok = cbase + c * 8 < N;
    const uint32_t ld = (uint32_t)ldc;   // a tile's offsets stay below 2^31 (at most 256 rows of 65536)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 a = acc[i][j];
            float v0 = a[0], v1 = a[1], v2 = a[2], v3 = a[3];
            if constexpr (EPI == EPI_RELU2 && OUT == 0) {
                v0 = relu_f32(v0); v1 = relu_f32(v1); v2 = relu_f32(v2); v3 = relu_f32(v3);
                v0 *= v0; v1 *= v1; v2 *= v2; v3 *= v3;
            }
            if constexpr (EPI == EPI_DRELU2) {
                const u32x2 u = uu[i][j];
                v0 = v0 * 2.f * relu_f32(bf16_lo(u[0]));
                v1 = v1 * 2.f * relu_f32(bf16_hi(u[0]));
                v2 = v2 * 2.f * relu_f32(bf16_lo(u[1]));
                v3 = v3 * 2.f * relu_f32(bf16_hi(u[1]));
            }
            const int ch = 2 * j + (lane >> 5);
            const u32x2 w = {pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
            *(lds_u32x2*)(uintptr_t)(wr + (uint32_t)((ch ^ (r & 7)) * 16)) = w;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int rr = q * 8 + rr0;
            const u32x4 v = *(const lds_u32x4*)(uintptr_t)(ep + (uint32_t)(rr * 128 + ((c ^ (rr & 7)) * 16)));
            const int row = i * 16 + rr;
            const uint32_t off = (row < nrows && col_ok) ? ((uint32_t)row * ld + (uint32_t)cbase + c * 8) * 2 : kDropOffset;
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, off, 0, 0);
        }
    }
}

// dgrad epilogue: C = bf16(acc * 2 max(u, 0)) with u read from aux_in at the
// accumulators' own positions (8 bytes per lane and fragment), written by
// staged_store.  The sixteen u loads are issued by drelu2_load at the tile's
// first k step (right after its barrier, before that step's operand
// copies), so they have long completed when the epilogue uses them: its
// waits never reach the copies in flight at the tile's end.
template <int MI>
__device__ __forceinline__ void drelu2_load(u32x2 (&uu)[MI][4], const uint16_t* aux_in, int64_t ldc, int N,
                                            int64_t rbase, int64_t nrows, int64_t cbase, int lane) {
    const __amdgpu_buffer_rsrc_t ru = rows_rsrc(aux_in, rbase, nrows, ldc);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = i * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = (int)cbase + j * 16 + 4 * (lane >> 4);
            const uint32_t off =
                (row < nrows && col < N) ? ((uint32_t)row * (uint32_t)ldc + (uint32_t)col) * 2 : kDropOffset;
            uu[i][j] = __builtin_amdgcn_raw_buffer_load_b64(ru, off, 0, 0);
        }
    }
}

// fp32 epilogue: each lane's four accumulators of a fragment are four
// consecutive columns of one row, stored as one 16-byte buffer store (with
// `accumulate`, added to what C holds there).  The descriptor spans only this
// wave's rows, so rows past the tile and columns past N are dropped.
template <int MI>
__device__ __forceinline__ void f32_store(const f32x4 (&acc)[MI][4], float* C, int64_t ldc, int N,
                                          int64_t rbase, int64_t nrows, int64_t cbase, bool accumulate,
                                          int lane) {
    const int64_t rows = nrows < MI * 16 ? nrows : MI * 16;
    const int32_t bytes = rows > 0 ? (int32_t)(rows * ldc * 4) : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(C + rbase * ldc), 0, bytes,
                                                                        0x00020000);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = i * 16 + (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = (int)cbase + j * 16 + 4 * (lane >> 4);
            const uint32_t off =
                (row < rows && col < N) ? ((uint32_t)row * (uint32_t)ldc + (uint32_t)col) * 4 : kDropOffset;
            f32x4 v = acc[i][j];
            if (accumulate) {
                const u32x4 o = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
                v[0] += __uint_as_float(o[0]);
                v[1] += __uint_as_float(o[1]);
                v[2] += __uint_as_float(o[2]);
                v[3] += __uint_as_float(o[3]);
            }
            const u32x4 w = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                             __float_as_uint(v[3])};
            __builtin_amdgcn_raw_buffer_store_b128(w, rs, off, 0, 0);
        }
    }
}

// C[r, n] = sum_k A[r, k] B_e[k, n] over the grid-wide list of output tiles
// (expert segments from the tile table `tiles` with m_total valid m-tiles,
// or all M rows when it is null), in tiles of T::BM rows.  A is K-contiguous
// (ROW layout); B is N-contiguous (B_K false: weights stored [Kd, N]) or
// K-contiguous (B_K true: transposed weights of the dgrads).  KTAIL: Kd is
// not a multiple of 64.
template <class T, bool B_K, int EPI, bool KTAIL>
__device__ __forceinline__ void rows_body(const GemmArgs& p, char* smem, const int4* tiles, int m_total) {
    constexpr int BM = T::BM, BN = T::BN, MI = T::MI, KD = T::KD, kStages = T::kStages;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::kWaveN, wn = wave % T::kWaveN;

    // Each XCD's G / 8 workgroups (workgroups go to XCDs round-robin) take a
    // contiguous eighth of the m-tiles, all n-tiles, in group-M order; this
    // workgroup takes items w = lx + j * (G / 8) of its XCD's share.  The
    // tile list is expert-major, so an expert's weights stream through one
    // XCD's L2 (two where a share boundary splits the expert) instead of
    // every XCD whose m-tile groups touch it.
    const int G = gridDim.x;   // a multiple of kXcds
    const int Gx = G / kXcds;
    const int xcd = (int)(blockIdx.x % kXcds), lx = (int)(blockIdx.x / kXcds);
    const int m_base = (int)((int64_t)m_total * xcd / kXcds);
    const int m_count = (int)((int64_t)m_total * (xcd + 1) / kXcds) - m_base;
    const int n_tiles = BN == 256 ? p.n_tiles : (p.N + BN - 1) / BN;
    const int n_work = m_count * n_tiles;
    const int n_mine = lx < n_work ? (n_work - lx + Gx - 1) / Gx : 0;
    const int nk = (p.Kd + KD - 1) / KD;
    const int g_total = n_mine * nk;  // (tile, k step) pairs
    if (g_total == 0) return;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const uint32_t ldsB = lds0, ldsA = lds0 + kStages * T::kBBytes;
    const uint32_t ep = lds0 + T::kRingBytes + (uint32_t)wave * kEpiWaveBytes;

    using DA = std::conditional_t<T::kAmx, MxDma<T>, DmaTile<true, BM, KD>>;
    DA da;
    DmaTile<B_K, BN, KD> db;
    constexpr int kSA = DA::kSlots, kSB = DmaTile<B_K, BN, KD>::kSlots;
    constexpr int kPerStage = kSA + kSB;
    auto dma_tile = [&](int j) {
        const RowsTile t = rows_tile<BM, BN>(p, tiles, m_count, n_tiles, lx + j * Gx, m_base);
        if constexpr (T::kAmx)
            da.init((const uint8_t*)p.A, p.A_scale, p.scale_bytes, t.row0, t.row_hi, p.Kd, wave, lane);
        else if (p.a_perm != nullptr)
            da.init_gather(p.A, p.lda, p.a_perm, p.a_div, p.a_src_rows, t.row0, t.row_hi, wave, lane);
        else
            da.init(p.A, p.lda, t.row0, t.row_hi, 0, p.Kd, wave, lane);
        db.init(p.B + (int64_t)t.e * p.b_stride, p.ldb, t.n0, (int64_t)p.N, 0, p.Kd, wave, lane);
    };

    constexpr int kNB = B_K ? T::kKK : 4;
    uint32_t abase[T::kKK], bbase[2][kNB];
    frag_bases<T, true, B_K>(abase, bbase, ldsA, ldsB, wm, wn, lane);

    f32x4 acc[MI][4];
    zero_acc(acc);

    // AMX: the lane's rows are r0 + 16 i; their scale windows sit 4 * kLPR
    // bytes apart, and all share the in-window byte offset (row * nb + kb) & 3.
    const int nb = p.Kd / 32;
    const int r0_lane = wm * T::kWaveRows + (lane & 15);
    uint32_t sbase = 0, rnb = 0;
    if constexpr (T::kAmx) {
        sbase = ldsA + T::kCodeBytes + (uint32_t)r0_lane * 4u * MxDma<T>::kLPR;
        rnb = (uint32_t)(r0_lane * nb);
    }

    // DMA of the first kStages - 1 steps; kd / jd track the next step to send.
    int kd = 0, jd = 0;
    for (int q = 0; q < kStages - 1 && q < g_total; ++q) {
        if (kd == 0) dma_tile(jd);
        const int rem = p.Kd - kd * KD;
        da.template issue<KTAIL, 0, kSA>(ldsA + q * T::kABytes, rem, wave);
        db.template issue<KTAIL, 0, kSB>(ldsB + q * T::kBBytes, rem, wave);
        if (++kd == nk) { kd = 0; ++jd; }
    }

    int kc = 0;   // k step of the tile being computed
    int jc = 0;   // its index in this workgroup's list
    RowsTile cur = rows_tile<BM, BN>(p, tiles, m_count, n_tiles, lx, m_base);
    u32x2 uu[MI][4];   // dgrad: the tile's pre-activations

    auto step = [&](auto stage_c, int g) {
        constexpr int S = decltype(stage_c)::value;
        // Stages g .. g + kStages - 2 are in flight and stage g must have
        // landed.  Stores of an epilogue may still be in flight; they are
        // not counted, so the wait covers this stage's copies whichever way
        // they complete (loads complete in order among themselves).
        wait_stage<T, kPerStage>(g, g_total);
        stage_barrier();
        if constexpr (EPI == EPI_DRELU2)
            if (kc == 0)
                drelu2_load(uu, p.aux_in, p.ldc, p.N, cur.row0 + wm * T::kWaveRows,
                            cur.row_hi - (cur.row0 + wm * T::kWaveRows), cur.n0 + wn * 64, lane);
        const bool next = g + kStages - 1 < g_total;
        if (next && kd == 0) dma_tile(jd);
        uint32_t sb = 0;
        if constexpr (T::kAmx) sb = sbase + (((uint32_t)(cur.row0 * nb + kc * T::kKK) + rnb) & 3u);
        mma_stage<T, true, B_K, KTAIL, S>(acc, abase, bbase, da, db, next, p.Kd - kd * KD, ldsA, ldsB, wave,
                                          sb);
        if (++kd == nk) { kd = 0; ++jd; }
        if (kc == nk - 1) {
            const int rbase = cur.row0 + wm * T::kWaveRows;
            const int nrows = cur.row_hi - rbase;
            const int cbase = cur.n0 + wn * 64;
            if constexpr (EPI == EPI_DRELU2) {
                staged_store<EPI, 0, MI>(acc, p.C, p.ldc, p.N, rbase, nrows, cbase, ep, lane, uu);
            } else if constexpr (EPI == EPI_F32) {
                f32_store(acc, (float*)p.C, p.ldc, p.N, rbase, nrows, cbase, p.accumulate != 0, lane);
            } else {
                staged_store<EPI, 0, MI>(acc, p.C, p.ldc, p.N, rbase, nrows, cbase, ep, lane);
                if constexpr (EPI == EPI_RELU2)
                    if (p.aux_out != nullptr)
                        staged_store<EPI, 1, MI>(acc, p.aux_out, p.ldc, p.N, rbase, nrows, cbase, ep, lane);
            }
            zero_acc(acc);
            kc = 0;
            ++jc;
            if (jc < n_mine) cur = rows_tile<BM, BN>(p, tiles, m_count, n_tiles, lx + jc * Gx, m_base);
        } else {
            ++kc;
        }
    };

    for (int g = 0; g < g_total; g += kStages) ring_round<kStages>(step, g, g_total);
}

// rows_body on the phased 256 x 256 tile: the same work list over 256-row
// tiles.  Around each output tile's k loop the two groups of waves fall into
// step, and what both need to do then is done once, at the same time: writing
// the tile (128 KB a CU, at 64 bytes a clock 2,048 of its ~3,900 clocks) and
// preparing the tile after the next.  A tile switch inside the k loop costs no
// memory latency: the workgroup's tiles are listed in LDS at the start, the
// perm entries of a tile's gathered rows are copied to LDS two tiles ahead,
// and its descriptors and row offsets are ready when its copies begin.  All
// copies in flight have landed before the stores are issued, so the next k
// tile waits for neither.  (Writing the tile in pieces during the memory parts
// of the phases instead, where the other group multiplies, was slower: 1.77 ->
// 1.87 ms on 24 experts x 4,779 rows, 2,688 -> 3,520, because the groups' pieces
// then follow each other.)
// Measured, phased / 128- and 256-row tiles of one barrier per stage, up and
// down projection: 64 experts x 768 rows (2,048 -> 1,024) 237 / 285 and 214 /
// 249 us; 256 uneven experts x 256 rows (2,048 -> 2,688) 855 / 986 and 790 /
// 880; 512 x 704 (672 -> 1,856) 1,034 / 1,158 and 832 / 1,013; 192 x 597 (2,688 ->
// 3,520) 1,983 / 2,290 and 1,881 / 2,231; 24 x 4,779 of the same 1,674 / 1,966 and
// 1,600 / 1,935 (1.30 and 1.36 PFLOP/s).
constexpr int kPermBytes = kWaves * 256;                                        // 64 entries per wave
constexpr int kPermOff = TileP::kRingBytes + kEpiBytes;
constexpr int kListOff = kPermOff + kPermBytes;
constexpr int kListTiles = (160 * 1024 - kListOff) / (int)sizeof(RowsTile);     // 896

// v, opaque to the optimiser: what is derived from it is computed where it is
// used instead of being held in registers over the k loop.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Work item w as in rows_tile, in per-lane code.
template <int BM>
__device__ __forceinline__ RowsTile rows_tile_lane(const GemmArgs& p, const int4* tiles, int m_count, int w,
                                                   int m_base) {
    RowsTile t;
    int mt, nt;
    if (tiles != nullptr) {
        const int q = m_base + w / p.n_tiles;
        const int packed = tiles[q].w;
        int a = packed >> 4, b = a + (packed & 15);
        a = a > m_base ? a : m_base;
        b = b < m_base + m_count ? b : m_base + m_count;
        if (a > q || b <= q) { a = q; b = q + 1; }
        const int s = b - a;
        const int in = w - (a - m_base) * p.n_tiles;
        mt = a + in % s;
        nt = in / s;
        nt = nt < p.n_tiles ? nt : p.n_tiles - 1;
        const int4 e = tiles[mt];
        t.e = e.x;
        t.row0 = e.y;
        t.row_hi = e.z;
    } else {
        const int width = kGroupM * p.n_tiles;
        const int group = w / width;
        const int first_m = group * kGroupM;
        const int gsz = (m_count - first_m) < kGroupM ? (m_count - first_m) : kGroupM;
        const int in = w - group * width;
        mt = m_base + first_m + in % gsz;
        nt = in / gsz;
        t.e = 0;
        t.row0 = mt * BM;
        t.row_hi = (t.row0 + BM) < p.M ? (t.row0 + BM) : (int)p.M;
    }
    t.n0 = nt * BN;
    return t;
}

// At least two k tiles (Kd > 64): tile jc + 1 is prepared before tile jc's
// second-last k tile starts sending it.
// Items lx + j * Gx of the XCD's m-tiles [m_base, m_base + m_count), 0 <= j < n_mine <= kListTiles.
template <bool B_K, int EPI, bool KTAIL>
__device__ __forceinline__ void rows_list_phased(const GemmArgs& p, char* smem, const int4* tiles, int m_base,
                                                 int m_count, int lx, int Gx, int n_mine) {
    constexpr int BM = TileP::BM;
    const int tid = threadIdx.x, lane_ = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int nk = (p.Kd + TileP::KD - 1) / TileP::KD;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const uint32_t ep = lds0 + TileP::kRingBytes + (uint32_t)wave * kEpiWaveBytes;
    const uint32_t perm_lds = lds0 + kPermOff + (uint32_t)wave * 256u;
    RowsTile* list = (RowsTile*)(smem + kListOff);
    for (int j = tid; j < n_mine; j += kGemmThreads)
        list[j] = rows_tile_lane<BM>(p, tiles, m_count, lx + j * Gx, m_base);
    __syncthreads();
    auto tile_at = [&](int j) {
        const RowsTile t = list[j];
        RowsTile u;
        u.e = __builtin_amdgcn_readfirstlane(t.e);
        u.row0 = __builtin_amdgcn_readfirstlane(t.row0);
        u.row_hi = __builtin_amdgcn_readfirstlane(t.row_hi);
        u.n0 = __builtin_amdgcn_readfirstlane(t.n0);
        return u;
    };

    Phased<true, B_K, KTAIL> ph;
    ph.wave = wave;
    ph.bases(lds0, wm, wn, lane_);
    ph.nkd = nk;
    ph.k_len = p.Kd;

    // Gathered A: lane l < 32 of a wave brings the perm entry of tile row
    // 128 (l / 16) + 16 wave + l % 16, the rows whose chunks the wave copies.
    const bool gather = !B_K && p.a_perm != nullptr;
    auto fetch_perm = [&](const RowsTile& t) {
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the last entries are read
        const int lane = fresh(lane_);
        const uint32_t row = (uint32_t)((lane >> 4) * 128 + wave * 16 + (lane & 15));
        const int n = t.row_hi - t.row0;
        dma4(buf_rsrc(p.a_perm + t.row0, (uint32_t)(n > 0 ? n * 4 : 0)), lane < 32 ? row * 4u : kDmaDrop, perm_lds);
    };
    // nxt: the tile after the one being sent; its operands' descriptors and, with
    // gathered rows, its chunks are prepared where both groups are in step.
    // ahead: the tile after that one, whose perm entries are on their way.
    using PH = Phased<true, B_K, KTAIL>;
    struct Next {
        i32x4 a, b;
        int cols;
        uint32_t off[2][2];
    } nxt;
    RowsTile cur = tile_at(0);
    RowsTile ahead = cur;
    auto prepare = [&]() {   // tile `ahead`, whose perm entries have landed
        const RowsTile& t = ahead;
        if (gather) {
            const int lane = fresh(lane_);
            nxt.a = buf_rsrc(p.A, (uint32_t)(p.a_src_rows * p.lda * 2));
            PH::DA::gathered_chunks(nxt.off, p.lda, p.a_src_rows, lane, [&](int h, int i) {
                const int r = h * 16 + i * 8 + (lane >> 3);
                const int v = *(const __attribute__((address_space(3))) int*)(uintptr_t)(perm_lds + r * 4);
                const bool in = t.row0 + h * 128 + (wave * 2 + i) * 8 + (lane >> 3) < t.row_hi;
                const uint32_t tok = (uint32_t)(((uint64_t)(uint32_t)v * p.a_mul) >> p.a_shift);
                return in && v >= 0 ? (int)tok : -1;
            });
        } else {
            nxt.a = PH::DA::span(p.A, p.lda, t.row0, t.row_hi, 0, p.Kd);
        }
        nxt.b = PH::DB::span(p.B + (int64_t)t.e * p.b_stride, p.ldb, t.n0, p.N, 0, p.Kd);
        nxt.cols = p.N - t.n0;
    };
    auto look_ahead = [&](int j) {
        ahead = tile_at(j);
        if (gather) fetch_perm(ahead);
    };
    auto take = [&]() {
        const int lane = fresh(lane_);
        ph.da.rs = nxt.a;
        ph.db.rs = nxt.b;
        ph.da.first_chunks(p.lda, 0, wave, lane);
        if (gather) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i) ph.da.off[h][i] = nxt.off[h][i];
        }
        ph.db.first_chunks(p.ldb, nxt.cols, wave, lane);
    };
    int jd = 0;
    auto next_tile = [&]() {
        if (++jd < n_mine) {
            take();
        } else {
            ph.da.stop();
            ph.db.stop();
        }
    };
    look_ahead(0);
    if (gather) wait_vmcnt<0>();
    prepare();
    take();
    if (n_mine > 1) {
        look_ahead(1);
        if (gather) wait_vmcnt<0>();
        prepare();
        if (n_mine > 2) look_ahead(2);   // its perm entries land with the first k tiles' copies
    }
    ph.start(next_tile);

    f32x4 acc0[4][4], acc1[4][4];
    for (int jc = 0; jc < n_mine; ++jc) {
        const int r0 = cur.row0 + wm * 64, cbase = cur.n0 + wn * 64;
        // a wave whose 64 rows of a half, or whose columns, are all padding has no products there
        const bool on0 = cbase < p.N && r0 < cur.row_hi, on1 = cbase < p.N && r0 + 128 < cur.row_hi;
        zero_acc(acc0);
        zero_acc(acc1);
        if (wm == 1) asm volatile("s_barrier" ::: "memory");   // group 1 one barrier behind
        if (on0 && on1) {
            ph.template k_tile<true, true>(acc0, acc1, true, true, next_tile);
            for (int kc = 1; kc < nk; ++kc) ph.template k_tile<true, false>(acc0, acc1, true, true, next_tile);
        } else {
            ph.template k_tile<false, true>(acc0, acc1, on0, on1, next_tile);
            for (int kc = 1; kc < nk; ++kc) ph.template k_tile<false, false>(acc0, acc1, on0, on1, next_tile);
        }
        if (wm == 0) asm volatile("s_barrier" ::: "memory");   // in step again: both groups write at once
        const int lane = fresh(lane_);
        // tile jc + 2 (jc + 1 is being sent); its perm entries landed during this tile's second k tile
        if (jc + 2 < n_mine) prepare();
        wait_vmcnt<0>();   // the next k tile is a FRESH one
        if (jc + 3 < n_mine) look_ahead(jc + 3);
        auto leave = [&](const f32x4 (&acc)[4][4], int rbase) {
            const int nrows = cur.row_hi - rbase;
            if constexpr (EPI == EPI_DRELU2) {
                u32x2 uu[4][4];
                drelu2_load(uu, p.aux_in, p.ldc, p.N, rbase, nrows, cbase, lane);
                staged_store<EPI, 0, 4>(acc, p.C, p.ldc, p.N, rbase, nrows, cbase, ep, lane, uu);
            } else if constexpr (EPI == EPI_F32) {
                f32_store(acc, (float*)p.C, p.ldc, p.N, rbase, nrows, cbase, p.accumulate != 0, lane);
            } else {
                staged_store<EPI, 0, 4>(acc, p.C, p.ldc, p.N, rbase, nrows, cbase, ep, lane);
                if constexpr (EPI == EPI_RELU2)
                    if (p.aux_out != nullptr)
                        staged_store<EPI, 1, 4>(acc, p.aux_out, p.ldc, p.N, rbase, nrows, cbase, ep, lane);
            }
        };
        if (on0) leave(acc0, r0);
        if (on1) leave(acc1, r0 + 128);
        if (jc + 1 < n_mine) cur = tile_at(jc + 1);
    }
    wait_vmcnt<0>();   // no copy into LDS outlives the workgroup
}

template <bool B_K, int EPI, bool KTAIL>
__device__ __forceinline__ void rows_body_phased(const GemmArgs& p, char* smem, const int4* tiles, int m_total) {
    const int Gx = gridDim.x / kXcds;   // the grid is a multiple of kXcds
    const int xcd = (int)(blockIdx.x % kXcds), lx = (int)(blockIdx.x / kXcds);
    const int m_base = (int)((int64_t)m_total * xcd / kXcds);
    const int m_count = (int)((int64_t)m_total * (xcd + 1) / kXcds) - m_base;
    const int n_work = m_count * p.n_tiles;
    const int n_mine = lx < n_work ? (n_work - lx + Gx - 1) / Gx : 0;
    for (int j0 = 0; j0 < n_mine; j0 += kListTiles) {
        __syncthreads();   // the last list is no longer read
        rows_list_phased<B_K, EPI, KTAIL>(p, smem, tiles, m_base, m_count, lx + j0 * Gx, Gx,
                                          n_mine - j0 < kListTiles ? n_mine - j0 : kListTiles);
    }
}

// fp32 store of a wave's 64 rows x 64 columns to C (its first row, ldc apart),
// columns from cbase, through 2 KB of LDS: 16 rows x 32 columns at a time
// (16-byte chunk c of row r at c ^ (r & 7)), read back as whole 128-byte row
// pieces, 8 rows per store instruction.  Rows from `rows` and columns from N on are
// dropped.
template <int POLICY>
__device__ __forceinline__ void kgrp_store_half(const f32x4 (&acc)[4][4], float* C, int64_t ldc, int rows, int N,
                                                uint32_t ep, int cbase, int lane) {
    rows = rows < 64 ? rows : 64;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)C, 0, rows > 0 ? (int32_t)(rows * ldc * 4) : 0, 0x00020000);
    const int r = lane & 15, rr0 = lane >> 3, c = lane & 7;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; jj += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int ch = (j * 4 + (lane >> 4)) ^ (r & 7);
                *(__attribute__((address_space(3))) f32x4*)(uintptr_t)(ep + (uint32_t)(r * 128 + ch * 16)) =
                    acc[i][jj + j];
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int rr = q * 8 + rr0;
                const u32x4 v = *(const lds_u32x4*)(uintptr_t)(ep + (uint32_t)(rr * 128 + ((c ^ (rr & 7)) * 16)));
                const int row = i * 16 + rr, col = cbase + jj * 16 + c * 4;
                const uint32_t off =
                    (row < rows && col < N) ? ((uint32_t)row * (uint32_t)ldc + (uint32_t)col) * 4 : kDropOffset;
                __builtin_amdgcn_raw_buffer_store_b128(v, rs, off, 0, POLICY);
            }
        }
}

// The same for the four waves side by side, 256 columns from n0: 8 rows x 256 columns
// at a time through 8 KB of LDS that they share (gb; chunk c of row r at
// c ^ 4 (r & 7)), a whole row of the tile per store instruction, non-temporal.
// Every wave of the workgroup calls it.
__device__ __forceinline__ void kgrp_store_rows(const f32x4 (&acc)[4][4], float* C, int64_t ldc, int rows, int N,
                                                uint32_t gb, int n0, int wn, int lane) {
    rows = rows < 64 ? rows : 64;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)C, 0, rows > 0 ? (int32_t)(rows * ldc * 4) : 0, 0x00020000);
    const int r = lane & 15, col = n0 + lane * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if ((r >> 3) == s) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int ch = (wn * 16 + j * 4 + (lane >> 4)) ^ ((r & 7) * 4);
                    *(__attribute__((address_space(3))) f32x4*)(uintptr_t)(gb + (uint32_t)((r & 7) * 1024 + ch * 16)) =
                        acc[i][j];
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // written, by all four
            u32x4 v[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int rr = wn * 2 + q;
                v[q] = *(const lds_u32x4*)(uintptr_t)(gb + (uint32_t)(rr * 1024 + ((lane ^ (rr * 4)) * 16)));
            }
            stage_barrier();   // read, by all four
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int row = i * 16 + s * 8 + wn * 2 + q;
                const uint32_t off =
                    (row < rows && col < N) ? ((uint32_t)row * (uint32_t)ldc + (uint32_t)col) * 4 : kDropOffset;
                __builtin_amdgcn_raw_buffer_store_b128(v[q], rs, off, 0, kNonTemporal);
            }
        }
}

// How a weight gradient (C, ldc; `bytes`: all that the launch writes) leaves:
//   kLinePieces    rows start on cache lines: 128-byte pieces, whole lines,
//                  non-temporal (see kgrp_store);
//   kCachedPieces  they do not, and the last-level cache holds all of it: cached
//                  128-byte pieces, whose partial lines merge in L2;
//   kTileRows      they do not, and it is larger: whole rows of the tile, seven lines of
//                  nine whole, non-temporal.
// Non-temporal 128-byte pieces off the lines only ever fill parts of two, which costs
// up to 2.4 times.  Cached, a gradient beyond the last-level cache is still dirty there
// when the launch ends, and the launches after it pay for its way to memory:
// 36 experts x 275 rows, 2,224 x 2,000, gradients 384 us and the up projection after
// them 184, as tile rows 395 and 144; 163 x 77, 1,552 x 1,552, 700 and 267, 756 and 212.
// Over 300 random shapes whole passes take 0.989 of what cached stores of all took.
enum GradStore { kLinePieces, kCachedPieces, kTileRows };
constexpr int64_t kHeldBytes = (int64_t)220 << 20;   // of the 256 MB last-level cache

static GradStore grad_store(const void* C, int64_t ldc, int64_t bytes) {
    if ((((uintptr_t)C | (uintptr_t)(ldc * 4)) & 127) == 0) return kLinePieces;
    return bytes <= kHeldBytes ? kCachedPieces : kTileRows;
}

// The items of dense weight gradients: `whole` tiles over all rows, then the
// other tiles in `chunks` pieces of chunk_rows rows each (chunk-major, so that
// what runs together shares operand rows), whose partial tiles tile_sum_kernel
// adds in order.  items: all of them, pieces counted.
// A partial tile has the rows and columns of the largest tile, not 256 of each.
struct DensePlan {
    int whole, chunks, chunk_rows, items;
    int piece_rows, piece_ld;
};

constexpr int kKgTabOff = TileP::kRingBytes + kWaves * 2048;
constexpr int kKgSlotOff = kKgTabOff + 3 * kMaxExperts * 4;
static_assert(kKgSlotOff + 4 * 32 <= 160 * 1024, "LDS budget");

// The pair launch on the phased tile, one workgroup per CU that runs items of
// its XCD's order until none is left: its first two by position, then each
// claimed from the XCD's counter while an earlier item is written.  The copies
// of the next item start during the last two k tiles of the current one, so
// neither a workgroup launch nor a cold pipeline stands between items, and an
// item's stores drain under the next one's first k tile.  The matrix pipes are
// busy 71% of the launch at 24 experts x 4,779 rows (2,688 x 3,520), against
// 74-78% of the row products: both operands take two LDS transpose reads a
// fragment.  Heavy slots (see kg_item) whose longest contraction would outlast
// the device's even share of the work are taken in items of 128 rows, whose
// second halves have no products (114 Zipf-loaded experts x 1,677 rows, 568 x 448,
// 43,949 of them one expert's: 836 -> 684 us; 26 x 572, 800 x 1,008: 136 -> 113; whole
// passes over 150 Zipf loads of two rounds and more take 0.985).
// Measured, this / one 256-row item a workgroup and one barrier
// a stage: 3,530 / 3,820 us; 128 Zipf-loaded experts x 1,024 rows (2,048 x
// 1,024) 1,130-1,180 / 1,230.
//
// DENSE: the weight gradients of dense projections, all rows one segment.  The
// items of a DensePlan follow each other over the grid, a round of every XCD's
// workgroups taking consecutive ones.
template <bool DENSE>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_kgrp2_phased_kernel(GemmArgs p0, GemmArgs p1,
                                                                            int32_t* __restrict__ claims,
                                                                            DensePlan plan, float* __restrict__ part) {
    __shared__ __attribute__((aligned(1024))) char smem[160 * 1024];
    const int tid = threadIdx.x, lane_ = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const uint32_t ep = lds0 + TileP::kRingBytes + (uint32_t)wave * 2048u;
    int32_t* const tab_e = (int32_t*)(smem + kKgTabOff);      // per slot of the expert order: expert,
    int32_t* const tab_k = tab_e + kMaxExperts;                   // first row,
    int32_t* const tab_n = tab_k + kMaxExperts;                   // row count
    struct Slot {
        int q, e, k_begin, k_len, row0, n0, bm;   // q < 0: no item; e < 0: padding of the order; bm: rows
    };
    Slot* const slots = (Slot*)(smem + kKgSlotOff);

    const int Gx = (int)gridDim.x / kXcds, x = (int)(blockIdx.x % kXcds), lx = (int)(blockIdx.x / kXcds);
    const int E = p0.E, R = (int)p0.R;
    const int per0 = p0.m_tiles * p0.n_tiles, per1 = p1.m_tiles * p1.n_tiles;
    int H = 0, n_x = 0, heavy0 = per0, heavy1 = per1, bm_heavy = TileP::BM;
    if constexpr (!DENSE) {
        for (int r = tid; r < E; r += kGemmThreads) {
            int e = p0.order[r];
            e = (e >= 0 && e < E) ? e : r;
            int lo = p0.offsets[e], hi = p0.offsets[e + 1];
            lo = lo < 0 ? 0 : (lo > R ? R : lo);
            hi = hi < lo ? lo : (hi > R ? R : hi);
            tab_e[r] = e;
            tab_k[r] = lo;
            tab_n[r] = hi - lo;
        }
        H = heavy_slots(p0);
        if (H > 0 && outlasts(p0, (float)(per0 + per1) / (float)gridDim.x)) {
            bm_heavy = 128;
            heavy0 = (int)(p0.M + 127) / 128 * p0.n_tiles;
            heavy1 = (int)(p1.M + 127) / 128 * p1.n_tiles;
        }
        n_x = kg_count(x, E, per0, per1, H, heavy0, heavy1);
    }
    // item `in` of problem q, bm rows high: 512 rows at a time across all n-tiles
    auto place = [&](Slot& s, int q, int in, int bm) {
        const int n_tiles = q ? p1.n_tiles : p0.n_tiles, m_tiles = ((int)(q ? p1.M : p0.M) + bm - 1) / bm;
        const int group = kKgM * TileP::BM / bm, width = group * n_tiles;
        const int grp = in / width, first_m = grp * group;
        const int gsz = (m_tiles - first_m) < group ? (m_tiles - first_m) : group;
        const int in2 = in - grp * width;
        s.q = q;
        s.bm = bm;
        s.row0 = (first_m + in2 % gsz) * bm;
        s.n0 = in2 / gsz * TileP::BN;
    };
    auto describe = [&](int j, int slot) {
        Slot s{-1, -1, 0, 0, 0, 0, TileP::BM};
        if constexpr (DENSE) {
            const int g = j * (int)gridDim.x + x * Gx + lx;
            int in = g;
            s.e = 0;   // 0: straight to C, else piece e - 1 of the partial tiles
            s.k_len = R;
            if (g >= plan.whole && plan.chunks > 1) {
                const int tail = per0 + per1 - plan.whole, t = g - plan.whole, c = t / tail;
                in = plan.whole + (t - c * tail);
                s.e = 1 + (t - c * tail) * plan.chunks + c;
                s.k_begin = c * plan.chunk_rows < R ? c * plan.chunk_rows : R;
                s.k_len = R - s.k_begin < plan.chunk_rows ? R - s.k_begin : plan.chunk_rows;
            }
            if (g < plan.items) place(s, in >= per0 ? 1 : 0, in >= per0 ? in - per0 : in, TileP::BM);
        } else if (j < n_x) {
            const KgItem it = kg_item((unsigned)(j * kXcds + x), E, per0, per1, H, heavy0, heavy1);
            s.q = 0;
            if (it.r >= 0) {
                s.e = tab_e[it.r];
                s.k_begin = tab_k[it.r];
                s.k_len = tab_n[it.r];
                place(s, it.q, it.in, it.r < H ? bm_heavy : TileP::BM);
            }
        }
        slots[slot] = s;
    };
    __syncthreads();
    // the second by position in reverse: the items come largest first
    if (tid < 2) describe(DENSE ? tid : (tid ? 2 * Gx - 1 - lx : lx), tid);
    __syncthreads();
    auto item = [&](int j) {
        const Slot s = slots[j & 3];
        Slot u;
        u.q = __builtin_amdgcn_readfirstlane(s.q);
        u.e = __builtin_amdgcn_readfirstlane(s.e);
        u.k_begin = __builtin_amdgcn_readfirstlane(s.k_begin);
        u.k_len = __builtin_amdgcn_readfirstlane(s.k_len);
        u.row0 = __builtin_amdgcn_readfirstlane(s.row0);
        u.n0 = __builtin_amdgcn_readfirstlane(s.n0);
        u.bm = __builtin_amdgcn_readfirstlane(s.bm);
        return u;
    };
    // at least two k tiles, so that the copies run at most one item ahead
    auto k_tiles = [](int len) { return len > TileP::KD ? (len + TileP::KD - 1) / TileP::KD : 2; };

    using PH = Phased<false, false, false>;
    PH ph;
    ph.wave = wave;
    ph.bases(lds0, wm, wn, lane_);
    ph.k_len = 0;   // column-contiguous operands: the descriptors end the contraction
    int jd = 0;
    auto take = [&](const Slot& s) {
        const int lane = fresh(lane_);
        const GemmArgs& p = s.q > 0 ? p1 : p0;
        const int M = s.e < 0 ? 0 : (int)p.M;
        ph.da.rs = PH::DA::span(p.A, p.lda, s.row0, M, s.k_begin, s.k_begin + s.k_len);
        ph.db.rs = PH::DB::span(p.B, p.ldb, s.n0, p.N, s.k_begin, s.k_begin + s.k_len);
        ph.da.first_chunks(p.lda, min(M - s.row0, s.bm), wave, lane);
        ph.db.first_chunks(p.ldb, p.N - s.n0, wave, lane);
        ph.nkd = k_tiles(s.k_len);
    };
    auto next_tile = [&]() {
        const Slot s = item(++jd);
        if (s.q >= 0) {
            take(s);
        } else {
            ph.da.stop();
            ph.db.stop();
        }
    };
    Slot cur = item(0);
    if (cur.q < 0) return;
    take(cur);
    ph.start(next_tile);

    f32x4 acc0[4][4], acc1[4][4];
    for (int jc = 0;; ++jc) {
        const GemmArgs& p = cur.q > 0 ? p1 : p0;
        const int M = cur.e < 0 ? 0 : (int)p.M;
        const int r0 = cur.row0 + wm * 64, cbase = cur.n0 + wn * 64;
        const bool on0 = cbase < p.N && r0 < M;
        const bool on1 = cur.bm > 128 && cbase < p.N && r0 + 128 < M;
        const int nk = k_tiles(cur.k_len);
        zero_acc(acc0);
        zero_acc(acc1);
        if (wm == 1) asm volatile("s_barrier" ::: "memory");   // group 1 one barrier behind
        if (on0 && on1) {
            ph.k_tile<true, true>(acc0, acc1, true, true, next_tile);
            for (int kc = 1; kc < nk; ++kc) ph.k_tile<true, false>(acc0, acc1, true, true, next_tile);
        } else {
            ph.k_tile<false, true>(acc0, acc1, on0, on1, next_tile);
            for (int kc = 1; kc < nk; ++kc) ph.k_tile<false, false>(acc0, acc1, on0, on1, next_tile);
        }
        if (wm == 0) asm volatile("s_barrier" ::: "memory");   // in step again: both groups write at once
        wait_vmcnt<0>();   // the next k tile is a FRESH one
        const Slot nxt = item(jc + 1);
        int next = jc + 2;
        if constexpr (!DENSE)
            if (nxt.q >= 0 && tid == 0) next = 2 * Gx + atomicAdd(claims + kClaimStride * x, 1);
        const int lane = fresh(lane_);
        // C at row r0 and column c0 of the columns below
        float* C = (float*)p.C + (int64_t)cur.e * p.c_stride + (int64_t)r0 * p.ldc;
        int64_t ldc = p.ldc;
        int c0 = 0, store = p.store;
        if constexpr (DENSE)
            if (cur.e > 0) {
                C = part + ((int64_t)(cur.e - 1) * plan.piece_rows + wm * 64) * plan.piece_ld;
                ldc = plan.piece_ld;
                c0 = cur.n0;
                store = kLinePieces;
            }
        if (store == kTileRows) {
            const uint32_t gb = lds0 + TileP::kRingBytes + (uint32_t)wm * 8192u;
            kgrp_store_rows(acc0, C, ldc, M - r0, p.N, gb, cur.n0, wn, lane);
            if (cur.bm > 128 && cur.row0 + 128 < M)
                kgrp_store_rows(acc1, C + 128 * ldc, ldc, M - r0 - 128, p.N, gb, cur.n0, wn, lane);
        } else if (store == kLinePieces) {
            if (on0) kgrp_store_half<kNonTemporal>(acc0, C, ldc, M - r0, p.N - c0, ep, cbase - c0, lane);
            if (on1) kgrp_store_half<kNonTemporal>(acc1, C + 128 * ldc, ldc, M - r0 - 128, p.N - c0, ep, cbase - c0, lane);
        } else {
            if (on0) kgrp_store_half<0>(acc0, C, ldc, M - r0, p.N - c0, ep, cbase - c0, lane);
            if (on1) kgrp_store_half<0>(acc1, C + 128 * ldc, ldc, M - r0 - 128, p.N - c0, ep, cbase - c0, lane);
        }
        if (nxt.q < 0) break;
        if (tid == 0) describe(next, (jc + 2) & 3);
        cur = nxt;
    }
    wait_vmcnt<0>();   // no copy into LDS outlives the workgroup
}

// Rounds of the busiest XCD: ceil(m / 8) m-tiles times n_tiles items over its
// G / 8 workgroups.
__host__ __device__ __forceinline__ int tile_rounds(int m_tiles, int n_tiles, int G) {
    const int Gx = G / kXcds;
    return ((m_tiles + kXcds - 1) / kXcds * n_tiles + Gx - 1) / Gx;
}

// The tile of a bf16 ROWS launch, from the m-tile counts of both heights
// (every workgroup reads the same counts, so the whole grid takes the same
// body): the phased 256-row tile when its rounds cost less than those of the
// 128-row tile.  Measured against each other (480 random loads of 6 to 300 experts,
// 1,400 launches: geometric mean and range of phased / 128-row time, by the ratio of their
// rounds): up to 2 rounds of 128-row tiles 1 : 2 0.83 (0.63-1.13), 1 : 1 1.18; 3 to 6
// rounds 0.5 0.82, 0.6 0.87, 0.65 0.95 (0.78-1.12), 0.75 0.97 (0.81-1.18), 0.8 1.01, 1.0
// 1.08; 7 and more 0.5 0.79, 0.6 0.86, 0.65 0.93, 0.7 0.92, 0.75 0.97, 1.0 1.02.  Dense
// rows (660 products of 512 to 16,384): 1 : 2 0.79, 2 : 4 0.78, 3 : 5 0.85, 2 : 3 0.95
// (0.79-1.07), 3 : 4 1.06, which the line leaves out.  The
// down projection of 256 uneven experts x 256 rows (2,688 -> 2,048), 14 : 21 rounds: 809-820
// against 940 us.
constexpr int kPhasedRoundPct = 135;
__host__ __device__ __forceinline__ bool take_phased(int m_small, int m_tall, int n_tiles, int G) {
    return tile_rounds(m_tall, n_tiles, G) * kPhasedRoundPct < tile_rounds(m_small, n_tiles, G) * 100;
}

// MX-FP8 A: relative time of one 256-row tile against two 128-row tiles (a
// third fewer operand bytes per product; measured 0.91 over the five layer
// shapes' real routing counts).
constexpr int kTallTileCostPct = 91;
__device__ __forceinline__ bool take_tall_tiles(int m_small, int m_tall, int n_tiles, int G) {
    return 2 * tile_rounds(m_tall, n_tiles, G) * kTallTileCostPct < 100 * tile_rounds(m_small, n_tiles, G);
}

constexpr int kRowsSmemBytes = 160 * 1024;
static_assert(TileS::kRingBytes + kEpiBytes <= kRowsSmemBytes && kListOff < kRowsSmemBytes, "LDS budget");

// The ROWS launch.  kMaybePhased: the launch may take the phased tile, which
// the kernel decides from the tile schedule's counts (known only after
// routing); otherwise the kernel holds one 128-row body alone, 256 or (kNarrow)
// 128 columns wide (see rows_kind).
enum RowsKind { kWide, kNarrow, kMaybePhased };
template <bool B_K, int EPI, bool KTAIL, RowsKind KIND>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_rows_kernel(GemmArgs p) {
    __shared__ __attribute__((aligned(1024))) char smem[kRowsSmemBytes];
    typedef const __attribute__((address_space(4))) int32_t* cnt_ptr;
    // the table's count, never beyond the table (the builder caps it too)
    const int m_small = p.mtile_total != nullptr ? min(*(cnt_ptr)p.mtile_total, p.m_tiles) : p.m_tiles;
    if constexpr (KIND == kMaybePhased) {
        const int m_tall = p.mtile_total_l != nullptr ? min(*(cnt_ptr)p.mtile_total_l, p.m_tiles_l) : p.m_tiles_l;
        if (take_phased(m_small, m_tall, p.n_tiles, (int)gridDim.x)) {
            rows_body_phased<B_K, EPI, KTAIL>(p, smem, p.tiles_l, m_tall);
            return;
        }
    }
    rows_body<std::conditional_t<KIND == kNarrow, TileN, TileS>, B_K, EPI, KTAIL>(p, smem, p.tiles, m_small);
}

constexpr int kRowsMxSmemBytes =
    (TileSX::kRingBytes > TileLX::kRingBytes ? TileSX::kRingBytes : TileLX::kRingBytes) + kEpiBytes;

// The ROWS launch over an MX-FP8 A (the up projection reading the dispatch
// payload as sent): the same bodies with the codes and scales in the ring
// and the decode in the fragment read; the tile height is chosen as above.
template <int EPI, bool KTAIL>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_rows_mx_kernel(GemmArgs p) {
    __shared__ __attribute__((aligned(1024))) char smem[kRowsMxSmemBytes];
    typedef const __attribute__((address_space(4))) int32_t* cnt_ptr;
    // the table's count, never beyond the table (the builder caps it too)
    const int m_small = p.mtile_total != nullptr ? min(*(cnt_ptr)p.mtile_total, p.m_tiles) : p.m_tiles;
    const int m_tall = p.mtile_total_l != nullptr ? min(*(cnt_ptr)p.mtile_total_l, p.m_tiles_l) : p.m_tiles_l;
    if (take_tall_tiles(m_small, m_tall, p.n_tiles, (int)gridDim.x)) {
        rows_body<TileLX, false, EPI, KTAIL>(p, smem, p.tiles_l, m_tall);
        return;
    }
    rows_body<TileSX, false, EPI, KTAIL>(p, smem, p.tiles, m_small);
}

static_assert(kSchedBM[0] == TileS::BM && kSchedBM[1] == TileL::BM, "schedule tile heights");

__global__ __launch_bounds__(1024) void tile_schedule_kernel(const int32_t* __restrict__ offsets, int E, int R,
                                                              SchedPart small, SchedPart large) {
    build_tile_schedule(offsets, E, R, small, large);
}

int gemm_tile_m() { return TileS::BM; }

size_t gemm_schedule_bytes(int E, int64_t R) {
    return sched_part_bytes(E, R, TileS::BM) + sched_part_bytes(E, R, TileL::BM);
}

// Compute units of the current device, read once per device.
int cu_count() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    static std::once_flag once[64];
    static int cus[64];
    std::call_once(once[dev], [dev] {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus[dev] = n;
    });
    return cus[dev];
}

// The persistent grid: one workgroup per CU (a multiple of the XCD count).
static int64_t persistent_grid() {
    int64_t G = (cu_count() / kXcds) * kXcds;
    return G < kXcds ? kXcds : G;
}

// Workgroups of a ROWS launch: never more than the static bound on the
// number of output tiles (0: nothing to do).
static int64_t rows_grid(const GemmArgs& a) {
    const int64_t bound = (int64_t)a.m_tiles * a.n_tiles;
    if (bound <= 0) return 0;
    const int64_t G = persistent_grid();
    const int64_t need = (bound + kXcds - 1) / kXcds * kXcds;
    return need < G ? need : G;
}

// Workgroups that take the 128-column tiles of every XCD's m-tiles in one
// round.  Expert segments: m-tiles sum to ceil(c / 128) <= 1 + (c - 1) / 128 over
// the experts with rows, at most min(R, E) of them.
static int64_t narrow_grid(const GemmArgs& a) {
    const int64_t used = std::min<int64_t>(a.R, a.E);
    const int64_t m = a.tiles != nullptr ? std::min<int64_t>(a.m_tiles, used + (a.R - used) / TileN::BM) : a.m_tiles;
    return (m + kXcds - 1) / kXcds * ((a.N + TileN::BN - 1) / TileN::BN) * kXcds;
}

// The body of a ROWS launch, G workgroups of the full width.
// Narrow: the tiles of half the width take a single round.  Such a launch is one
// chain of k tiles a workgroup, bound by the latency of each; half the tile
// takes 0.65-0.75 of the wide one's time (us, wide / narrow: 8 experts x 128 rows,
// 256 -> 512 8.3 / 6.8 and back 11.9 / 8.4; 8 x 32, 2,048 -> 1,024 29.2 / 20.5; 8 x 8,
// 2,688 -> 3,520 37.9 / 27.7; dense 1,024 x 2,688 x 2,688 37.6 / 27.5; dense 32 x 2,688 x
// 672, whose few wide tiles share one XCD, 98 / 24).  At narrow rounds 2 against
// wide rounds 1 it takes 0.98-1.25, at 3 : 2 0.97, at 4 : 2 1.04-1.21; 2 : 2 takes 0.65, but
// the counts behind it are a bound and routing may leave the wide tile one round.
// Phased, dense rows: the rule itself.
// Expert segments, whose counts the host does not know: not with a single
// round of 128-row tiles, and not below 80 rows per expert, where routing
// without strong skew leaves no expert over 128 rows and both heights the same
// tiles (of 1,400 launches of random loads ten below it, with 26 to 75 rows an
// expert, would have gained 2-15%).  Such launches are short, and the kernel with
// both bodies costs them up to 1 us (18.0 against 17.6 us at 1,024 rows of 8
// experts, 43.8 against 43.0 us at 1,024 rows of 64).  The phased body needs two k tiles.
static RowsKind rows_kind(const GemmArgs& a, int64_t G) {
    if (narrow_grid(a) <= persistent_grid()) return kNarrow;
    if (a.Kd <= TileP::KD) return kWide;
    const bool phased = a.tiles == nullptr
                            ? take_phased(a.m_tiles, a.m_tiles_l, a.n_tiles, (int)G)
                            : tile_rounds(a.m_tiles, a.n_tiles, (int)G) > 1 && a.R >= 80 * (int64_t)a.E;
    return phased ? kMaybePhased : kWide;
}

template <bool B_K, int EPI, bool KTAIL>
static void launch_rows_kernel(const GemmArgs& a, hipStream_t st) {
    const int64_t wide = rows_grid(a);
    const RowsKind kind = rows_kind(a, wide);
    const dim3 G((unsigned)(kind == kNarrow ? narrow_grid(a) : wide)), B(kGemmThreads);
    if (kind == kNarrow)
        hipLaunchKernelGGL((gemm_rows_kernel<B_K, EPI, KTAIL, kNarrow>), G, B, 0, st, a);
    else if (kind == kWide)
        hipLaunchKernelGGL((gemm_rows_kernel<B_K, EPI, KTAIL, kWide>), G, B, 0, st, a);
    else
        hipLaunchKernelGGL((gemm_rows_kernel<B_K, EPI, KTAIL, kMaybePhased>), G, B, 0, st, a);
}

template <bool B_K, int EPI>
static hipError_t launch_rows(const GemmArgs& a, hipStream_t st) {
    if (rows_grid(a) == 0) return hipSuccess;
    if (a.Kd % TileS::KD != 0)
        launch_rows_kernel<B_K, EPI, true>(a, st);
    else
        launch_rows_kernel<B_K, EPI, false>(a, st);
    return launch_check(st);
}

template <int EPI>
static hipError_t launch_rows_mx(const GemmArgs& a, hipStream_t st) {
    const int64_t G = rows_grid(a);
    if (G == 0) return hipSuccess;
    if (a.Kd % TileS::KD != 0)
        hipLaunchKernelGGL((gemm_rows_mx_kernel<EPI, true>), dim3((unsigned)G), dim3(kGemmThreads), 0, st, a);
    else
        hipLaunchKernelGGL((gemm_rows_mx_kernel<EPI, false>), dim3((unsigned)G), dim3(kGemmThreads), 0, st, a);
    return launch_check(st);
}

static hipError_t launch_rows_epi(const GemmArgs& a, bool b_kmajor, int epi, hipStream_t st) {
    if (!b_kmajor) {
        if (epi == EPI_BF16) return launch_rows<false, EPI_BF16>(a, st);
        if (epi == EPI_RELU2) return launch_rows<false, EPI_RELU2>(a, st);
        if (epi == EPI_F32) return launch_rows<false, EPI_F32>(a, st);
    } else {
        if (epi == EPI_BF16) return launch_rows<true, EPI_BF16>(a, st);
        if (epi == EPI_DRELU2) return launch_rows<true, EPI_DRELU2>(a, st);
        if (epi == EPI_F32) return launch_rows<true, EPI_F32>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tile_schedule(const int32_t* offsets, int E, int64_t R, void* sched, hipStream_t st) {
    hipLaunchKernelGGL(tile_schedule_kernel, dim3(1), dim3(1024), 0, st, offsets, E, (int)R,
                       sched_part(sched, E, R, false), sched_part(sched, E, R, true));
    return launch_check(st);
}

// The operand-independent part of a ROWS launch: B, C, sizes and both tile
// heights' schedule tables (the kernel picks one from their counts).
static void rows_args(GemmArgs& a, const moe_bf16* B, int64_t ldb, int64_t b_stride, void* C, int64_t ldc,
                      moe_bf16* aux_out, const void* sched, int E, int64_t R, int N, int Kd) {
    a.B = B; a.C = C; a.aux_out = aux_out;
    a.ldb = ldb; a.ldc = ldc; a.b_stride = b_stride;
    a.M = R; a.R = R; a.N = N; a.Kd = Kd; a.E = E;
    a.n_tiles = (N + BN - 1) / BN;
    if (sched != nullptr) {
        const SchedPart ss = sched_part((void*)sched, E, R, false), sl = sched_part((void*)sched, E, R, true);
        a.tiles = ss.tiles;
        a.mtile_total = ss.mtile_start + E;  // mtile_start[E]
        a.m_tiles = ss.max_tiles;
        a.tiles_l = sl.tiles;
        a.mtile_total_l = sl.mtile_start + E;
        a.m_tiles_l = sl.max_tiles;
    } else {
        a.m_tiles = (int)((R + TileS::BM - 1) / TileS::BM);
        a.m_tiles_l = (int)((R + TileL::BM - 1) / TileL::BM);
    }
}

hipError_t launch_grouped_rows(const moe_bf16* A, int64_t lda, const moe_bf16* B, int64_t ldb,
                               int64_t b_stride, bool b_kmajor, void* C, int64_t ldc, int epi,
                               const moe_bf16* aux_in, moe_bf16* aux_out, const void* sched,
                               int E, int64_t R, int N, int Kd, hipStream_t st, bool accumulate) {
    if (R == 0) return hipSuccess;
    // the DMA descriptor of an N-contiguous B spans its whole contraction
    if (!b_kmajor && (int64_t)Kd * ldb * 2 >= kMaxDmaBytes) return hipErrorInvalidValue;
    GemmArgs a{};
    a.A = A; a.aux_in = aux_in;
    a.accumulate = accumulate ? 1 : 0;
    a.lda = lda;
    rows_args(a, B, ldb, b_stride, C, ldc, aux_out, sched, E, R, N, Kd);
    return launch_rows_epi(a, b_kmajor, epi, st);
}

hipError_t launch_grouped_rows_gather(const moe_bf16* X, int64_t ldx, int64_t x_rows, const int32_t* perm, int div,
                                      const moe_bf16* B, int64_t ldb, int64_t b_stride, void* C, int64_t ldc, int epi,
                                      moe_bf16* aux_out, const void* sched, int E, int64_t R, int N, int Kd,
                                      hipStream_t st) {
    if (R == 0) return hipSuccess;
    if ((int64_t)Kd * ldb * 2 >= kMaxDmaBytes || x_rows * ldx * 2 >= kMaxDmaBytes || div < 1)
        return hipErrorInvalidValue;
    GemmArgs a{};
    a.A = X;
    a.lda = ldx;
    a.a_perm = perm;
    a.a_div = div;
    // s = 31 + ceil(log2 div), m = ceil(2^s / div): m * div - 2^s < div <= 2^(s - 31), so v * m >> s is exact
    int sh = 31;
    while (((int64_t)1 << (sh - 31)) < div) ++sh;
    a.a_shift = sh;
    a.a_mul = (uint32_t)((((uint64_t)1 << sh) + div - 1) / div);
    a.a_src_rows = x_rows;
    rows_args(a, B, ldb, b_stride, C, ldc, aux_out, sched, E, R, N, Kd);
    return launch_rows_epi(a, false, epi, st);
}

hipError_t launch_grouped_rows_mx(const uint8_t* Aq, const uint8_t* A_scale, const moe_bf16* B, int64_t ldb,
                                  int64_t b_stride, void* C, int64_t ldc, int epi, moe_bf16* aux_out,
                                  const void* sched, int E, int64_t R, int N, int Kd, hipStream_t st) {
    if (R == 0) return hipSuccess;
    if (Kd <= 0 || Kd % 32 != 0 || ((uintptr_t)Aq & 15u) != 0) return hipErrorInvalidValue;
    if ((int64_t)Kd * ldb * 2 >= kMaxDmaBytes) return hipErrorInvalidValue;
    const int64_t scale_bytes = (R * (Kd / 32) + 3) / 4 * 4;
    if (scale_bytes >= kMaxDmaBytes) return hipErrorInvalidValue;
    GemmArgs a{};
    a.A = (const uint16_t*)Aq;
    a.A_scale = A_scale;
    a.scale_bytes = (uint32_t)scale_bytes;
    a.lda = Kd;
    rows_args(a, B, ldb, b_stride, C, ldc, aux_out, sched, E, R, N, Kd);
    if (epi == EPI_BF16) return launch_rows_mx<EPI_BF16>(a, st);
    if (epi == EPI_RELU2) return launch_rows_mx<EPI_RELU2>(a, st);
    return hipErrorInvalidValue;
}


constexpr int kPhasedGradPct = 152;   // cost of a round of phased items, of one of 128-row items

// Both weight gradients of the expert FFN in one launch (gemm_kgrp2_kernel),
// items of the experts with the most rows first.
hipError_t launch_grouped_wgrad2(const moe_bf16* A0, int64_t lda0, const moe_bf16* B0, int64_t ldb0, float* C0,
                                 int64_t ldc0, int64_t c_stride0, int M0, int N0, const moe_bf16* A1, int64_t lda1,
                                 const moe_bf16* B1, int64_t ldb1, float* C1, int64_t ldc1, int64_t c_stride1, int M1,
                                 int N1, const int32_t* offsets, const int32_t* order, int E, int64_t R,
                                 hipStream_t st) {
    if (R * (lda0 > ldb0 ? lda0 : ldb0) * 2 >= kMaxDmaBytes || R * (lda1 > ldb1 ? lda1 : ldb1) * 2 >= kMaxDmaBytes)
        return hipErrorInvalidValue;
    if (order == nullptr || E < 1 || E > kMaxExperts) return hipErrorInvalidValue;
    GemmArgs a[2] = {};
    const moe_bf16* As[2] = {A0, A1};
    const moe_bf16* Bs[2] = {B0, B1};
    float* Cs[2] = {C0, C1};
    const int64_t lda[2] = {lda0, lda1}, ldb[2] = {ldb0, ldb1}, ldc[2] = {ldc0, ldc1}, cs[2] = {c_stride0, c_stride1};
    const int Ms[2] = {M0, M1}, Ns[2] = {N0, N1};
    int64_t items[2] = {0, 0};   // of 128-row and of 256-row tiles
    for (int q = 0; q < 2; ++q) {
        a[q].A = As[q]; a[q].B = Bs[q]; a[q].C = Cs[q]; a[q].offsets = offsets; a[q].order = order;
        a[q].lda = lda[q]; a[q].ldb = ldb[q]; a[q].ldc = ldc[q]; a[q].c_stride = cs[q];
        a[q].M = Ms[q]; a[q].R = R; a[q].N = Ns[q]; a[q].E = E;
        for (int h = 0; h < 2; ++h)
            items[h] += (int64_t)E * ((Ms[q] + kSchedBM[h] - 1) / kSchedBM[h]) * ((Ns[q] + BN - 1) / BN);
    }
    // The phased tile when its rounds of items over the device cost less, as in
    // take_phased, but not for fewer than two rounds or a k tile of rows an expert.
    // Measured, phased / 128-row: rounds 1 : 2 0.82 on even loads, but 1.04 and 1.29
    // where the loads vary as exp(0.7 z) or by Zipf's law, because the busiest
    // expert's items, twice as long, are then the whole time; 2 : 4 0.86-0.90, 0.83
    // and 1.0; 4 : 8 and more 0.80, 0.79 and 0.88.
    // With fewer rows the stores take most of the time.  Where rows start on 64-byte
    // pieces, one 256-row item a workgroup costs least (whole passes of forward
    // and backward, 36 shapes: 0.96 of the 128-row tile's, phased 0.98; 184 experts x
    // 24 rows, 1,120 x 3,168: the gradients 945 us, phased 993; below a round the
    // 128-row tile: 7 experts x 22 rows, 416 x 416, 6.9 and 9.2).  Where they do not, and
    // every 256-byte store covers parts of three cache lines, the more workgroups
    // store at once the better: 128-row items (0.96 of phased, 256-row items 1.01), but
    // for gradients that the last-level cache holds, whose cached stores the
    // phased tile makes (0.98 of the 128-row tile's).
    const int64_t G = persistent_grid();
    const bool few = R < TileP::KD * (int64_t)E;
    const int64_t bytes = (int64_t)E * (c_stride0 + c_stride1) * 4;
    for (int q = 0; q < 2; ++q) a[q].store = grad_store(Cs[q], ldc[q], bytes);
    const bool on64 = ((ldc0 | ldc1) & 15) == 0 && (((uintptr_t)C0 | (uintptr_t)C1) & 63) == 0;
    const bool phased = few ? !on64 && bytes <= kHeldBytes && items[1] > G
                            : items[1] >= 2 * G &&
                                  (items[1] + G - 1) / G * kPhasedGradPct < (items[0] + G - 1) / G * 100;
    const bool tall = phased || (few ? on64 && items[1] >= G : items[1] >= 4 * G);
    for (int q = 0; q < 2; ++q) {
        a[q].m_tiles = (Ms[q] + kSchedBM[tall] - 1) / kSchedBM[tall];
        a[q].n_tiles = (Ns[q] + BN - 1) / BN;
    }
    const int64_t n_wg =
        kg_grid(E, (int64_t)a[0].m_tiles * a[0].n_tiles, (int64_t)a[1].m_tiles * a[1].n_tiles);
    if (n_wg > 0x7fffffff) return hipErrorInvalidConfiguration;
    if (phased)
        hipLaunchKernelGGL(gemm_kgrp2_phased_kernel<false>, dim3((unsigned)G), dim3(kGemmThreads), 0, st, a[0], a[1],
                           const_cast<int32_t*>(order) + order_claims(E), DensePlan{}, (float*)nullptr);
    else if (tall)
        hipLaunchKernelGGL(gemm_kgrp2_kernel<TileL>, dim3((unsigned)n_wg), dim3(kGemmThreads), 0, st, a[0], a[1]);
    else
        hipLaunchKernelGGL(gemm_kgrp2_kernel<TileS>, dim3((unsigned)n_wg), dim3(kGemmThreads), 0, st, a[0], a[1]);
    return launch_check(st);
}

// The plan of the dense weight gradients M0 x N0 and M1 x N1 over R rows on the 256
// workgroups of a device (a device of another size runs the same plan, so the
// sums' order is the same): whole rounds of tiles over all rows, then the rest
// cut into the number of pieces whose rounds take least.  In units of one k
// tile (1.5 us): a piece costs its k tiles and 4 more (start, stores, the
// workgroups' spread), the sum of the pieces 0.035 per 256 KB of partial tiles read or
// written (5 TB/s) and 2 for its launch.  A chunk has at least two k tiles; there are
// at most 64 chunks (of a single tile 64 leave a few us to win) and 128 MB of
// partial tiles.
static DensePlan dense_plan(int64_t R, int M0, int N0, int M1, int N1) {
    constexpr int64_t G = 256;
    auto tiles = [](int M, int N) {
        return (int64_t)((M + TileP::BM - 1) / TileP::BM) * ((N + TileP::BN - 1) / TileP::BN);
    };
    const int64_t n = tiles(M0, N0) + tiles(M1, N1);
    const int64_t nk = (R + TileP::KD - 1) / TileP::KD, tail = n % G;
    const int rows = std::min(std::max(M0, M1), TileP::BM), cols = std::min(std::max(N0, N1), TileP::BN);
    DensePlan best{(int)(n - tail), 1, (int)R, (int)n, rows, (cols + 31) / 32 * 32};   // rows of whole cache lines
    const double piece = 0.035 * best.piece_rows * best.piece_ld / (TileP::BM * TileP::BN);
    double cost = 0;
    for (int64_t c = 1; tail > 0 && (c == 1 || (c <= 64 && tail * c <= 2 * G && 2 * c <= nk)); ++c) {
        const int64_t per = (nk + c - 1) / c;
        const double t = (double)((tail * c + G - 1) / G) * (double)(per + 4) +
                         (c > 1 ? piece * (double)(tail * (2 * c + 1)) + 2 : 0);
        if (c == 1 || t < cost) {
            cost = t;
            best.chunks = (int)c;
            best.chunk_rows = c > 1 ? (int)(per * TileP::KD) : (int)R;
            best.items = (int)(n - tail + tail * c);
        }
    }
    return best;
}

size_t dense_wgrad_ws_bytes(int64_t R, int M0, int N0, int M1, int N1) {
    const DensePlan pl = dense_plan(R, M0, N0, M1, N1);
    return pl.chunks > 1 ? (size_t)(pl.items - pl.whole) * pl.piece_rows * pl.piece_ld * 4 : 0;
}

// C tiles from `whole` on = the sum of their partial tiles, chunks ascending.
// Bandwidth-bound: one thread adds four columns, one block four rows.
__global__ __launch_bounds__(256) void tile_sum_kernel(GemmArgs p0, GemmArgs p1, DensePlan plan,
                                                       const float* __restrict__ part) {
    int in = plan.whole + (int)blockIdx.y;
    const int64_t piece = (int64_t)plan.piece_rows * plan.piece_ld;
    const float* src = part + (int64_t)blockIdx.y * plan.chunks * piece;
    const int per0 = p0.m_tiles * p0.n_tiles;
    const GemmArgs& p = in >= per0 ? p1 : p0;
    if (in >= per0) in -= per0;
    const int width = kKgM * p.n_tiles;
    const int grp = in / width, first_m = grp * kKgM;
    const int gsz = (p.m_tiles - first_m) < kKgM ? (p.m_tiles - first_m) : kKgM;
    const int in2 = in - grp * width;
    const int row = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6), col = ((int)threadIdx.x & 63) * 4;
    const int m = (first_m + in2 % gsz) * TileP::BM + row, n = in2 / gsz * TileP::BN + col;
    if (m >= p.M || n >= p.N) return;
    src += row * plan.piece_ld + col;
    f32x4 s = *(const f32x4*)src;
#pragma unroll 4
    for (int c = 1; c < plan.chunks; ++c) {
        const f32x4 v = *(const f32x4*)(src + c * piece);
        s[0] += v[0]; s[1] += v[1]; s[2] += v[2]; s[3] += v[3];
    }
    float* dst = (float*)p.C + (int64_t)m * p.ldc + n;   // 4-byte aligned
    dst[0] = s[0]; dst[1] = s[1]; dst[2] = s[2]; dst[3] = s[3];
}

// C_q [M_q, N_q] = A_q^T B_q over R rows, q = 0 and (M1 > 0) 1, in one launch and
// the sum of the pieces.  One problem at a time left each with its own partly
// empty last round, and equal chunks of all tiles wrote every tile twice or
// more: both gradients of 16,384 rows (2,688 x 3,520) took 2 x (360 + 40) us in
// 128-row tiles of two chunks, and take 546 + 12 (1.14 PFLOP/s) here; the router's
// (2,688 x 576) took 83 + 21 in nine chunks, and take 60 + 12 + 5 with the planes' sum.
hipError_t launch_dense_wgrad2(const moe_bf16* A0, const moe_bf16* B0, float* C0, int M0, int N0, const moe_bf16* A1,
                               const moe_bf16* B1, float* C1, int M1, int N1, int64_t R, void* ws, hipStream_t st) {
    const int widest = std::max(std::max(M0, N0), std::max(M1, N1));
    if (R * widest * 2 >= kMaxDmaBytes) return hipErrorInvalidValue;
    GemmArgs a[2] = {};
    const moe_bf16* As[2] = {A0, A1};
    const moe_bf16* Bs[2] = {B0, B1};
    float* Cs[2] = {C0, C1};
    const int Ms[2] = {M0, M1}, Ns[2] = {N0, N1};
    for (int q = 0; q < 2; ++q) {
        a[q].A = As[q]; a[q].B = Bs[q]; a[q].C = Cs[q];
        a[q].lda = Ms[q]; a[q].ldb = Ns[q]; a[q].ldc = Ns[q];
        a[q].M = Ms[q]; a[q].R = R; a[q].N = Ns[q];
        a[q].m_tiles = (Ms[q] + TileP::BM - 1) / TileP::BM;
        a[q].n_tiles = (Ns[q] + BN - 1) / BN;
        a[q].store = grad_store(Cs[q], Ns[q], ((int64_t)M0 * N0 + (int64_t)M1 * N1) * 4);
    }
    const DensePlan pl = dense_plan(R, M0, N0, M1, N1);
    if (pl.items == 0) return hipSuccess;
    const int64_t G = std::min<int64_t>(persistent_grid(), (pl.items + kXcds - 1) / kXcds * kXcds);
    hipLaunchKernelGGL(gemm_kgrp2_phased_kernel<true>, dim3((unsigned)G), dim3(kGemmThreads), 0, st, a[0], a[1],
                       (int32_t*)nullptr, pl, (float*)ws);
    hipError_t err = launch_check(st);
    if (err != hipSuccess || pl.chunks == 1) return err;
    hipLaunchKernelGGL(tile_sum_kernel, dim3((unsigned)((pl.piece_rows + 3) / 4), (unsigned)((pl.items - pl.whole) / pl.chunks)), dim3(256), 0, st, a[0], a[1], pl,
                       (const float*)ws);
    return launch_check(st);
}

// Experts ranked by row count, most first (ties to the lower index):
// order[rank] = e, and the pair launch's claim counters behind it, zeroed.
// One workgroup; each thread counts, for its experts, the
// experts that come before them.
__global__ __launch_bounds__(1024) void expert_order_kernel(const int32_t* __restrict__ offsets, int E, int R,
                                                            int32_t* __restrict__ order) {
    __shared__ int32_t cnt[1024];
    for (int i = threadIdx.x; i < kXcds * kClaimStride; i += 1024) order[order_claims(E) + i] = 0;
    for (int e = threadIdx.x; e < E; e += 1024) {
        int lo = offsets[e], hi = offsets[e + 1];
        lo = lo < 0 ? 0 : (lo > R ? R : lo);
        hi = hi < lo ? lo : (hi > R ? R : hi);
        cnt[e] = hi - lo;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 1024) {
        const int c = cnt[e];
        int rank = 0;
        for (int f = 0; f < E; ++f) rank += (cnt[f] > c || (cnt[f] == c && f < e)) ? 1 : 0;
        order[rank] = e;
    }
}

hipError_t launch_expert_order(const int32_t* offsets, int E, int64_t R, int32_t* order, hipStream_t st) {
    hipLaunchKernelGGL(expert_order_kernel, dim3(1), dim3(1024), 0, st, offsets, E, (int)R, order);
    return launch_check(st);
}


}  // namespace moe
