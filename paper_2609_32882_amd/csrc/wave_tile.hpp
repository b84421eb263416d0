// Building blocks of the one-wave attention kernel (attn_fwd_wave.hip): 64-row
// bf16 tiles in unpadded, XOR-swizzled LDS rows, their asynchronous copies and
// their fragment reads.
//
// A tile is two half-tiles of 32 rows.  Tile row y lies at LDS row y; the
// 16-byte chunk c of a row lies at chunk c ^ wt_swizzle(y).  64 banks of 4
// bytes are 16 chunks, so with 256-byte rows (D = 128) the bank of a piece is
// its physical chunk.
//  - A row read (wave_frags::row, ds_read_b128) serves 16 lanes per clock, which
//    read one chunk c of the 16 rows of a 16-row block: the swizzle gives
//    those rows 16 different bank groups.
//  - A transposing read (wave_frags::col, ds_read_b64_tr_b16) serves a half-wave
//    per clock: 4 consecutive chunks (an aligned group) of 4 consecutive rows.
//    The high two bits of the swizzle differ among those rows, so the groups
//    fall on disjoint banks.
// No padding and no row permutation: a half-tile is a whole number of 1 KB
// copies, every fourth of which has the same per-lane source offset (the
// swizzle repeats after 16 rows), so four offset registers serve all tiles.
#pragma once

#include "common.hpp"

namespace vsa2 {

template <int RB>
__host__ __device__ constexpr int wt_swizzle(int y) {
    static_assert(RB == 256, "row bytes");
    return ((y & 3) << 2) | ((y >> 2) & 3);
}

// Asynchronous copies of half-tiles of 32 rows of RB bytes by one wave.
template <int RB>
struct wave_copy {
    static constexpr int HALF = 32 * RB;          // bytes of a half-tile
    static constexpr int ND = HALF / 1024;        // copies per half-tile
    int off[4];                                   // copy j: source offset off[j % 4] + 1024 j

    __device__ __forceinline__ explicit wave_copy(int lane) {
        constexpr int LPR = RB / 16;              // lanes (16-byte chunks) per row
        constexpr int RPC = 64 / LPR;             // rows per copy
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = lane / LPR;
            off[i] = r * RB + ((lane % LPR) ^ wt_swizzle<RB>(i * RPC + r)) * 16;
        }
    }
    // Copy j of the half-tile at g (wave-uniform) to LDS address lds.  A copy
    // that is not live fetches the half-tile's first 16 bytes in every lane:
    // the number of copies in flight stays what the waits count on.
    template <int J>
    __device__ __forceinline__ void issue(uint32_t lds, uint64_t g, bool live) const {
        const uint64_t b = g + (J / 4) * 4096;
        const uint32_t l = lds + (J / 4) * 4096;
        const int o = live ? off[J % 4] : 0;
        uint64_t at;                              // the waits of dma16
        asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 offset:%4"
                     : "=&s"(at)
                     : "s"(l), "v"(o), "s"(b), "n"((J % 4) * 1024)
                     : "memory", "m0");
    }
};

__device__ __forceinline__ uint32_t lds_addr(const char* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)p));
}

// Per-lane LDS addresses of the fragments of a tile.
template <int RB>
struct wave_frags {
    static constexpr int KS = RB / 32;   // 16-column groups of a row (k-steps over the head dim)
    static constexpr int MT = RB / 64;   // 32-column groups
    int row_at[KS];                      // row fragment of k-step ks: row_at[ks] + half-tile offset
    int col_at[MT][2];                   // column fragment: col_at[mt][r] + 16-row step offset

    __device__ __forceinline__ explicit wave_frags(int lane) {
        const int half = lane >> 5;
        // row fragments take rows in the slot-swapped view (lane s reads tile
        // row swap_bits_2_3(s)), which makes a lane's 16 accumulator rows two
        // runs of 8 consecutive tile rows
        const int y = swap_bits_2_3(lane & 31);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) row_at[ks] = y * RB + ((2 * ks + half) ^ wt_swizzle<RB>(y)) * 16;
        const int i = lane & 15, G = lane >> 4;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int yy = 8 * (G >> 1) + 4 * r + (i >> 2);
                const int c = 4 * mt + 2 * (G & 1) + ((i & 3) >> 1);
                col_at[mt][r] = yy * RB + (c ^ wt_swizzle<RB>(yy)) * 16 + 8 * (i & 1);
            }
    }
    // A operand, rows of half-tile t (32 rows), columns 16 ks .. 16 ks + 15
    __device__ __forceinline__ void row(frag_bf16& f, const char* tile, int t, int ks) const {
        load_frag(f, tile + row_at[ks] + t * 32 * RB);
    }
    // A operand of the transposed use: columns 32 mt .. + 31 as output rows,
    // tile rows 32 t + 16 kk .. + 15 as the contraction
    __device__ __forceinline__ void col(frag_bf16& f, const char* tile, int t, int kk, int mt) const {
        typedef short v4i16 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
        v4i16 r2[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
            r2[r] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(tile + col_at[mt][r] + (32 * t + 16 * kk) * RB));
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8_t;
        const s16x8_t w = {r2[0][0], r2[0][1], r2[0][2], r2[0][3], r2[1][0], r2[1][1], r2[1][2], r2[1][3]};
        f.v = __builtin_bit_cast(bf16x8_t, w);
    }
};

// acc += a b with the accumulators in AGPRs (the vector registers hold the
// scores): the instruction is written out because the compiler is asked for
// the VGPR form everywhere else.  The compiler does not know that it is an
// MFMA, so the waits that MFMAs need are the caller's: a and b are fragments
// that LDS reads delivered or packing finished well before (at least two
// instructions), and mma_drain comes before anything but another mma_acc
// touches the accumulators.
__device__ __forceinline__ void mma_acc(f32x16_t& acc, const frag_bf16& a, const frag_bf16& b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a.v), "v"(b.v));
}
// The mma_acc issued so far have written their results (32 wait states; an
// 8-pass MFMA needs at most 19 before a vector instruction reads them), and
// no instruction moves across.
__device__ __forceinline__ void mma_drain() {
    lds_order();
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    lds_order();
}

// The same for code inside a kernel's loop that changes the accumulators: the
// values it reads are defined here, so no copy of them is made earlier.
template <int M, int N>
__device__ __forceinline__ void acc_settle(f32x16_t (&acc)[M][N]) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[i][j]));
}

// ---------------------------------------------------------------------------
// Pacing: the waves of one XCD that walk lists of about the same length keep
// near the same list position, so that the tiles they gather are shared
// through the XCD's L2.
//
// Per XCD the call's workspace holds PACE_SLOTS words; the wave of the XCD's
// j-th row keeps its position in word j mod PACE_SLOTS (1 + steps since the
// launch began; the sign bit once the row is done).  A row starts at the
// multiple of its length nearest to the highest position (the rows resident
// together start and end together; one that starts late catches up).  Before a
// step a wave waits while a quarter of the rows at work are more than
// PACE_SLACK steps behind it.  This only ever delays a wave: no result depends
// on it, and a wave gives up waiting after PACE_POLLS polls per row (another
// launch among the resident waves, rows that share a word).
// (One word each and plain stores: a shared counter takes 0.1 us per atomic.)
// ---------------------------------------------------------------------------
constexpr int PACE_SLOTS = 256;                // 1 KB: one 16-byte copy per lane
static_assert(PACE_BYTES == 8 * 4 * PACE_SLOTS, "one block of words per XCD");
constexpr int PACE_SLACK = 2;
constexpr int PACE_POLLS = 256;

__device__ __forceinline__ int xcc_id() {
    uint32_t x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    return static_cast<int>(x & 7u);
}

struct pace_clock {
    uint64_t words;       // this XCD's words
    const uint32_t* copy; // 1 KB of LDS that receives them
    int at;               // byte offset of this wave's own word
    int base;             // position at which this wave's row starts
    int polls;            // left

    // The words, on their way to LDS (one vector-memory operation).
    __device__ __forceinline__ void request() const {
        const uint32_t l = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)copy));
        uint64_t from;
        asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 sc1"
                     : "=&s"(from)
                     : "s"(l), "v"(static_cast<int>(threadIdx.x * 16)), "s"(words)
                     : "memory", "m0");
    }
    __device__ __forceinline__ void store(uint32_t x) const {
        uint64_t active;                          // put back as it was
        asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, 1\n\tglobal_store_dword %1, %2, %3\n\ts_mov_b64 exec, %0"
                     : "=&s"(active)
                     : "v"(at), "v"(x), "s"(words)
                     : "memory");
    }
    __device__ __forceinline__ void seen(int (&w)[4]) const {
        const int4 x = *reinterpret_cast<const int4*>(reinterpret_cast<const char*>(copy) + threadIdx.x * 16);
        w[0] = x.x; w[1] = x.y; w[2] = x.z; w[3] = x.w;
    }
    // Joins (the words requested before) for a row of about `len` steps.
    __device__ __forceinline__ void join(float len) {
        int w[4];
        seen(w);
        int hi = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) hi = max(hi, w[i] & 0x7fffffff);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) hi = max(hi, __shfl_xor(hi, off, 64));
        base = __builtin_amdgcn_readfirstlane(static_cast<int>(rintf(static_cast<float>(hi - 1) / len) * len));
        step(0);
    }
    __device__ __forceinline__ void step(int done) const { store(static_cast<uint32_t>(base + done + 1)); }
    __device__ __forceinline__ void leave(int done) const { store(static_cast<uint32_t>(base + done + 1) | 0x80000000u); }
    __device__ __forceinline__ bool ahead(int step) const {
        int w[4];
        seen(w);
        const int own = base + step + 1 - PACE_SLACK;
        int work = 0, behind = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            work += __popcll(__ballot(w[i] > 0));
            behind += __popcll(__ballot(w[i] > 0 && w[i] < own));
        }
        return 4 * behind > work;
    }
    __device__ __forceinline__ void wait(int step) {
        while (ahead(step) && polls > 0) {
            --polls;
            __builtin_amdgcn_s_sleep(4);
            request();
            vm_wait<0>();
        }
    }
};

}  // namespace vsa2
