// The phased 256 x 256 tile of the grouped GEMM: two groups of four waves that
// take turns at the matrix pipes.
//
// A k tile (64 deep) is four phases per wave, each a memory part M (LDS
// fragment reads, two operand copies) and a compute part C (16 MFMAs), with a
// workgroup barrier after each part.  Group 1 (waves 4..7) runs one barrier
// behind group 0, and waves w and w + 4 share a SIMD, so while one wave of a
// SIMD computes, the other reads the fragments of its next 16 MFMAs: neither
// barrier nor LDS latency leaves the pipe idle, which is what bounds a
// schedule in which all eight waves read and then all compute.
//
//   wave (wm, wn) of 2 x 4: rows {64 wm .. +63} of both 128-row halves of the
//   tile, columns 64 wn .. +63; accumulators acc0 hold half 0, acc1 half 1.
//   Phases of k tile t (k0, k1: its 32-deep k steps):
//     0: read A half 0 k0                      acc0 += A0 k0 * B k0
//     1: read A half 0 k1, B k1                acc0 += A0 k1 * B k1
//     2: read A half 1 k0                      acc1 += A1 k0 * B k0
//     3: read A half 1 k1, B k0 of t + 1       acc1 += A1 k1 * B k1
//   Every accumulator takes its k steps in ascending order, so the results are
//   those of the 128-row tile, bit for bit.
//
// LDS holds two k tiles, each as four 16 KB pieces, and every phase sends one
// piece (two 1 KB copies per wave) into the slot whose last reader was an
// earlier phase.  A piece is waited for in the phase before the one that
// reads it, by every wave, and that phase's barriers order it before the
// readers; five pieces (80 KB) stay in flight.
//   N-contiguous B (pieces by k step, full 512-byte rows of 256 columns):
//     sent in phase 0: A1(t+1), 1: Bk0(t+2), 2: A0(t+2), 3: Bk1(t+2); each is
//     read six phases later, so every phase waits until 10 copies are left.
//   K-contiguous B (pieces by 128 columns, full 128-byte rows of 64 k, so
//     that no copy reads half a cache line):
//     sent in phase 0: A0(t+1), 1: A1(t+1), 2: B0(t+2), 3: B1(t+2); both B
//     pieces are read in phases 3 and 1.
#pragma once

#include "tile_dma.h"

namespace moe {

struct TileP {
    static constexpr int BM = 256, BN = 256, KD = 64;
    static constexpr int kPiece = 16 * 1024;
    static constexpr int kBuf = 2 * kPiece;        // one operand of one k tile
    static constexpr int kABytes = 2 * kBuf;       // two k tiles of A, then two of B
    static constexpr int kRingBytes = 2 * kABytes;
};

// Copy state of one operand: two pieces per k tile, two 1 KB slots per wave
// and piece.  ROWL: K-contiguous source, piece h = rows [128 h, 128 h + 128)
// of the tile as LDS rows of 64 k.  Otherwise an M/N-contiguous source, whose
// pieces are columns [128 h, +128) x 64 k (KSPLIT false) or k rows [32 h, +32)
// x 256 columns (KSPLIT true).  Chunks outside the operand read as zero.
template <bool ROWL, bool KSPLIT>
struct PieceDma {
    static_assert(!(ROWL && KSPLIT), "a K-contiguous operand is cut by rows");
    static constexpr int kOff = KSPLIT ? 1 : 2;
    i32x4 rs;              // wave-uniform
    uint32_t kstep;        // bytes from a lane's chunk to its next one, wave-uniform
    uint32_t off[kOff][2];
    int kpos;              // ROWL: k offset of the lane's chunks in the k tile

    // The tile's descriptor: rows (or columns) from x0, contraction from k_begin.
    __device__ __forceinline__ static i32x4 span(const uint16_t* __restrict__ src, int64_t ld, int64_t x0,
                                                 int64_t x_hi, int64_t k_begin, int64_t k_end) {
        if constexpr (ROWL) {
            const int64_t x_end = x0 + 256 < x_hi ? x0 + 256 : x_hi;
            const int64_t rows = x_end > x0 ? x_end - x0 : 0;
            return buf_rsrc(src + x0 * ld + k_begin, (uint32_t)(rows * ld * 2));
        } else {
            const int64_t krows = k_end > k_begin ? k_end - k_begin : 0;
            return buf_rsrc(src + k_begin * ld + x0, (uint32_t)(krows > 0 ? krows * ld * 2 - x0 * 2 : 0));
        }
    }
    // The lane's first chunks in it; cols = columns of the operand from x0 on
    // (ROWL: unused).
    __device__ __forceinline__ void first_chunks(int64_t ld, int cols, int wave, int lane) {
        if constexpr (ROWL) {
            kstep = TileP::KD * 2;
            const int c = (lane & 7) ^ (lane >> 3);   // rswz of row 8 * slot + lane / 8
            kpos = c * 8;
            const uint32_t o = (uint32_t)(((wave * 16 + (lane >> 3)) * (uint32_t)ld + c * 8) * 2);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i) off[h][i] = o + (uint32_t)((h * 128 + i * 8) * 2) * (uint32_t)ld;
        } else if constexpr (KSPLIT) {
            kstep = (uint32_t)(32 * ld * 2);
            kpos = 0;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = (wave * 2 + i) * 2 + (lane >> 5);
                const int c = (lane & 31) ^ cswz(k);
                off[0][i] = c * 8 < cols ? (uint32_t)((k * (uint32_t)ld + c * 8) * 2) : kDmaDrop;
            }
        } else {
            kstep = (uint32_t)(TileP::KD * ld * 2);
            kpos = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int k = (wave * 2 + i) * 4 + (lane >> 4);
                    const int c = h * 16 + ((lane & 15) ^ cswz(k));
                    off[h][i] = c * 8 < cols ? (uint32_t)((k * (uint32_t)ld + c * 8) * 2) : kDmaDrop;
                }
        }
    }

    // Gathered rows: the descriptor spans the whole source, and the lane's row
    // of each slot is source row idx(h, i), dropped outside [0, src_rows).
    template <class Idx>
    __device__ __forceinline__ static void gathered_chunks(uint32_t (&o)[2][2], int64_t ld, int64_t src_rows,
                                                           int lane, Idx&& idx) {
        static_assert(ROWL, "gathered rows need the row layout");
        const int c = (lane & 7) ^ (lane >> 3);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int tok = idx(h, i);
                o[h][i] = (uint32_t)tok < (uint64_t)src_rows ? ((uint32_t)tok * (uint32_t)ld + c * 8) * 2 : kDmaDrop;
            }
    }

    // Every later copy reads zeros without touching memory (past the last k tile).
    __device__ __forceinline__ void stop() { rs[2] = 0; }

    // Send piece H of the operand's next k tile to LDS byte dst.  KTAIL (ROWL):
    // chunks at or past k_rem, the contraction left from the k tile's start,
    // read as zero.
    template <int H, bool KTAIL>
    __device__ __forceinline__ void send(uint32_t dst, int k_rem, int wave) {
        constexpr int h = KSPLIT ? 0 : H;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t o = off[h][i];
            if constexpr (KTAIL && ROWL) o = kpos < k_rem ? o : kDmaDrop;
            dma16(rs, o, dst + (uint32_t)(wave * 2 + i) * 1024u);
            off[h][i] += kstep;
        }
    }
};

// The k-tile stream of one workgroup.  next_tile(da, db) starts the copies of
// the output tile that follows (or stops them past the last one).
template <bool A_ROW, bool B_ROW, bool KTAIL>
struct Phased {
    using DA = PieceDma<A_ROW, false>;
    using DB = PieceDma<B_ROW, !B_ROW>;
    DA da;
    DB db;
    uint32_t ldsA, ldsB;          // first byte of A's and B's pieces
    uint32_t abase[A_ROW ? 2 : 4], bbase[B_ROW ? 2 : 4];
    bf16x8 a[4], b0[4], b1[4];
    int kd, nkd;                  // the k tile being sent, of nkd in its output tile
    int k_len;                    // its contraction length
    uint32_t par;                 // kBuf * (parity of the k tile being computed)
    int wave;

    __device__ __forceinline__ void bases(uint32_t lds0, int wm, int wn, int lane) {
        ldsA = lds0;
        ldsB = lds0 + TileP::kABytes;
        if constexpr (A_ROW) {
            abase[0] = ldsA + row_base<64>(wm * 64, 0, lane);
            abase[1] = ldsA + row_base<64>(wm * 64, 1, lane);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) abase[i] = ldsA + col_base<128>(wm * 64 + i * 16, lane);
        }
        if constexpr (B_ROW) {
            bbase[0] = ldsB + row_base<64>(wn * 64, 0, lane);
            bbase[1] = ldsB + row_base<64>(wn * 64, 1, lane);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) bbase[j] = ldsB + col_base<256>(wn * 64 + j * 16, lane);
        }
    }

    // on: the wave's 64 rows of the half hold a row of the tile.
    template <int H, int KK>
    __device__ __forceinline__ void read_a(bool on) {
        if (!on) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (A_ROW) a[i] = lds_b128(abase[KK] + H * TileP::kPiece + i * 2048);
            else a[i] = lds_tr_pair(abase[i] + H * TileP::kPiece + KK * 32 * 256, 4 * 256);
        }
    }
    template <int KK>
    __device__ __forceinline__ void read_b(bf16x8 (&b)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (B_ROW) b[j] = lds_b128(bbase[KK] + j * 2048);
            else b[j] = lds_tr_pair(bbase[j] + KK * TileP::kPiece, 4 * 512);
        }
    }
    template <int N>
    __device__ __forceinline__ void flip(uint32_t (&base)[N], uint32_t nxt) {   // to the other k tile's pieces
#pragma unroll
        for (int i = 0; i < N; ++i) base[i] += nxt - par;
    }
    __device__ __forceinline__ void settle() {   // this wave's LDS reads done, then the barrier
        stage_barrier();
        __builtin_amdgcn_sched_barrier(0);
    }
    // Padding rows cost no matrix work where all 64 of a wave's rows are padding.
    __device__ __forceinline__ void mma(f32x4 (&acc)[4][4], const bf16x8 (&b)[4], bool on) {
        if (on) {
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }

    // The copies that precede the first k tile, and its B k0 fragments.  The
    // caller has initialised da and db for the first output tile.
    template <class Next>
    __device__ __forceinline__ void start(Next&& next_tile) {
        par = 0;
        kd = 0;
        if constexpr (!B_ROW) {
            send_b<0>(0);
            send_a<0>(0);
            send_b<1>(0);
            send_a<1>(0);
            advance(next_tile);
            send_b<0>(TileP::kBuf);
            send_a<0>(TileP::kBuf);
            send_b<1>(TileP::kBuf);
        } else {
            send_b<0>(0);
            send_b<1>(0);
            send_a<0>(0);
            send_a<1>(0);
            advance(next_tile);
            send_b<0>(TileP::kBuf);
            send_b<1>(TileP::kBuf);
        }
        wait_vmcnt<0>();   // the first k tile is a FRESH one
        stage_barrier();
        read_b<0>(b0);
    }
    template <int H>
    __device__ __forceinline__ void send_a(uint32_t buf) {
        da.template send<H, KTAIL>(ldsA + buf + H * TileP::kPiece, k_len - kd * TileP::KD, wave);
    }
    template <int H>
    __device__ __forceinline__ void send_b(uint32_t buf) {
        db.template send<H, KTAIL>(ldsB + buf + H * TileP::kPiece, k_len - kd * TileP::KD, wave);
    }
    template <class Next>
    __device__ __forceinline__ void advance(Next&& next_tile) {
        if (++kd == nkd) {
            kd = 0;
            next_tile();
        }
    }

    // One k tile; on0 and on1: the wave's rows of the two halves are not all padding.
    // FULL: both hold one, known at compile time (a branch around the reads and
    // products of each phase costs ~4% of the loop).  FRESH: every copy sent
    // before this k tile has landed, so only copies sent during it are waited
    // for: an output tile's stores, still on their way, hold nothing up.
    template <bool FULL, bool FRESH, class Next>
    __device__ __forceinline__ void k_tile(f32x4 (&acc0)[4][4], f32x4 (&acc1)[4][4], bool on0, bool on1,
                                           Next&& next_tile) {
        const uint32_t nxt = par ^ TileP::kBuf;
        if constexpr (FULL) on0 = on1 = true;
        // phase 0
        read_a<0, 0>(on0);
        if constexpr (!B_ROW) {
            send_a<1>(nxt);
            if constexpr (!FRESH) wait_vmcnt<10>();
        } else {
            send_a<0>(nxt);
        }
        settle();
        mma(acc0, b0, on0);
        // phase 1
        read_a<0, 1>(on0);
        read_b<1>(b1);
        flip(bbase, nxt);
        if constexpr (!B_ROW) {
            advance(next_tile);
            send_b<0>(par);
            if constexpr (!FRESH) wait_vmcnt<10>();
        } else {
            send_a<1>(nxt);
            if constexpr (!FRESH) wait_vmcnt<8>();
        }
        settle();
        mma(acc0, b1, on0);
        // phase 2
        read_a<1, 0>(on1);
        if constexpr (!B_ROW) {
            send_a<0>(par);
            if constexpr (!FRESH) wait_vmcnt<10>();
        } else {
            advance(next_tile);
            send_b<0>(par);
            if constexpr (!FRESH) wait_vmcnt<6>();
        }
        settle();
        mma(acc1, b0, on1);
        // phase 3
        read_a<1, 1>(on1);
        read_b<0>(b0);
        flip(abase, nxt);
        send_b<1>(par);
        if constexpr (B_ROW) wait_vmcnt<6>();   // A0(t+1), sent in phase 0, is read in the next phase
        else if constexpr (!FRESH) wait_vmcnt<10>();
        settle();
        mma(acc1, b1, on1);
        par = nxt;
    }
};

}  // namespace moe
