// Block-sparse attention forward for bf16 and D = 128, one wave per query block
// (VSA2 Sec. 2.1 with a block mask, Sec. 2.2 Eq. block_sparse).  attn_fwd.hip
// states the computation and which launches and heads come here.
//
// What bounds the two-wave kernel at 720p (40 heads, top-120, 5.76M pairs, 189
// GB of K/V gathers): its waves stall on each other's barriers and on LDS
// reads, and 85 GB of the gathers miss the L2s, which pull at most about 7
// TB/s.  Here:
//  - One wave owns all 64 queries: every K and V^T fragment read from LDS feeds
//    two MFMAs instead of one (half the LDS reads), and there are no barriers.
//    Its 128 accumulators and 64 Q registers live in AGPRs (one wave per SIMD).
//  - The wave is its own pipeline over half-tiles of 32 keys: while the softmax
//    of half-tile i runs on the vector unit, the MFMAs compute S of half-tile
//    i + 1 and P V of half-tile i - 1, one MFMA to one element (one exponential
//    and about 3.5 other vector instructions) per slot.  Without memory (tiles
//    left in LDS) this takes 7.6 ms at 720p, 1.6 PFLOP/s.
//  - No row max per tile: p = 2^(s c - m) against a reference m that is raised
//    (and the tile redone) only when the lane's sum of a tile passes 2^8.
//  - Each half-tile's buffer is refilled as soon as its last fragment is read;
//    three of the four are in flight.
//  - Paced walks (wave_tile.hpp): the waves of an XCD stay within a few list
//    entries of each other.  Unpaced, this kernel outruns the L2s: 139 GB of
//    misses, 19.9 ms; paced 54 GB, 13.2 to 13.8 ms a call by the box (14.5 to
//    15.1 ms for the two-wave kernel); with every gather an L2 hit 11.5 ms.
#include <type_traits>

#include "wave_tile.hpp"
#include "internal.hpp"

namespace vsa2 {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;

template <int I> using ic = std::integral_constant<int, I>;
template <int N, typename Fn>
__device__ __forceinline__ void for_each_ic(Fn&& fn) {
    if constexpr (N > 0) {
        for_each_ic<N - 1>(fn);
        fn(ic<N - 1>{});
    }
}

// The V tile of an entry outside [0, N): its scores are masked, and its
// probabilities, all 0, need a V whose products are 0 (a real tile may hold
// infinities), so that the entry can go through the pipeline like any other.
__device__ const uint4 zero_tile[2 * wave_copy<256>::HALF / 16] = {};

template <bool COMP, bool PAD>
__global__ __launch_bounds__(64, 1) void attn_fwd_wave_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t col_cap,
    bf16_t* __restrict__ o, float* __restrict__ lse, bf16_t* __restrict__ o_lo, int Hq, int Hkv, int N, float c_log2,
    int period, const int32_t* __restrict__ order, uint32_t* __restrict__ pace, const float* __restrict__ even,
    cube_grid grid, block_flag_layout fl) {
    using F = frag_bf16;
    constexpr int D = 128;
    constexpr int RB = 2 * D;
    constexpr int KS = D / 16, MT = D / 32;
    constexpr int ND = wave_copy<RB>::ND, HALF = wave_copy<RB>::HALF;
    constexpr int64_t TILE = 2 * HALF;
    constexpr int AHEAD = 3;                        // fragments requested ahead of their products
    __shared__ __align__(1024) char lds[4 * HALF];   // K low, K high, V low, V high
    __shared__ __align__(1024) uint32_t pace_lds[PACE_SLOTS];
    const char* k_lds = lds;
    const char* v_lds = lds + 2 * HALF;

    const int lane = threadIdx.x, half = lane >> 5;
    const int64_t item = xcd_item(blockIdx.x, gridDim.x);
    // the order permutes rows within a head; a grid's size fits in 32 bits
    const int64_t bh = static_cast<uint32_t>(item) / static_cast<uint32_t>(N);
    const float avg = even[bh];              // this head's average list length
    if (!(avg > 0.f)) return;                // uneven lists: a head of the two-wave kernel
    const int64_t row = work_row(order, item, gridDim.x);
    const int n = static_cast<int>(row - bh * N);
    const int b = static_cast<int>(static_cast<uint32_t>(bh) / static_cast<uint32_t>(Hq));
    const int h = static_cast<int>(bh) - b * Hq;
    const int64_t kvh = static_cast<int64_t>(b) * Hkv + h / (Hq / Hkv);
    const int64_t L = static_cast<int64_t>(N) * 64;
    const uint64_t kb = reinterpret_cast<uint64_t>(k + kvh * L * D), vb = reinterpret_cast<uint64_t>(v + kvh * L * D);
    const int64_t qtok = bh * L + static_cast<int64_t>(n) * 64 + (lane & 31);   // + 32 qt
    const uint64_t qmask = PAD ? cube_real_mask(grid, n, lane) : ~0ull;

    int64_t e0 = row_ptr[row], e1 = row_ptr[row + 1];
    e0 = e0 < 0 ? 0 : (e0 > col_cap ? col_cap : e0);
    e1 = e1 < e0 ? e0 : (e1 > col_cap ? col_cap : e1);
    const int cnt = __builtin_amdgcn_readfirstlane(static_cast<int>(e1 - e0));

    F qf[2][KS];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) load_frag(qf[qt][ks], q + (qtok + 32 * qt) * D + ks * 16 + half * 8);
    if constexpr (PAD) {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
            if (!((qmask >> (32 * qt + (lane & 31))) & 1)) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) qf[qt][ks] = F{};
            }
    }
    bool big = false;
    if constexpr (COMP) {
        big = byte_of(scalar_load_i32(byte_word(fl.q, row)), row);
        if (!big && scalar_load_i32(fl.any_kv + kvh) != 0) {
            bool hit = false;
            for (int64_t e = e0 + lane; e < e1; e += 64) {
                const int c = col_idx[e];
                if (c >= 0 && c < N && fl.kv[kvh * N + c]) hit = true;
            }
            big = __any(hit);
        }
    }
    // rows about as long as the head's average are paced, from their list's
    // first entry; the others start at the phase of their place in the launch
    const bool paced = __builtin_amdgcn_readfirstlane(fabsf(cnt - avg) <= avg * (1.f / 16) ? 1 : 0) != 0;
    pace_clock clk;
    clk.words = reinterpret_cast<uint64_t>(pace + xcc_id() * PACE_SLOTS);
    clk.copy = pace_lds;
    clk.at = 4 * static_cast<int>((blockIdx.x >> 3) % PACE_SLOTS);
    clk.polls = PACE_POLLS;
    clk.base = 0;
    const int s0 = paced ? 0 : __builtin_amdgcn_readfirstlane(
        static_cast<int>(sweep_start(col_idx, e0, cnt, blockIdx.x >> 3, period, N)));
    if (paced) {
        clk.request();
    }
    const wave_copy<RB> cp(lane);
    const wave_frags<RB> fr(lane);
    const uint32_t l0 = lds_addr(lds);

#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            settle(qf[qt][ks]);
            pin_agpr(qf[qt][ks]);
        }
    f32x16_t oacc[2][MT];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[qt][mt][i] = 0.f;
        }
    float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f}, lr[2] = {0.f, 0.f};

    // the list, 64 entries at a time in a register (lane i: entry 64 w + i of
    // the walk); entries outside [0, N) read as -1
    int ents = -1;
    bool any = false;                 // an entry inside [0, N) was met
    auto load_ents = [&](int w) {
        const int j = 64 * w + lane;
        int c = -1;
        if (j < cnt) {
            const int t = s0 + j;
            c = col_idx[e0 + (t >= cnt ? t - cnt : t)];
        }
        ents = (c >= 0 && c < N) ? c : -1;
        any = any || __ballot(ents >= 0) != 0;
    };
    auto walk = [&](auto two_term) {
        constexpr bool TWO = decltype(two_term)::value;
        constexpr int PT = TWO ? 2 : 1;
        f32x16_t s[2][2];            // scores of the two half-tiles: s[t][qt]
        u32x4_t pw[2][2][2][PT];      // P fragments: [t][kk][qt][hi, lo], 4 words each
        F ring[4];

        // block of walk position j (wave-uniform); -1 for positions past the
        // list (not live) and entries outside [0, N), which copy block 0's K
        // (masked) and a V of zeros
        auto ent_at = [&](int j) -> int { return __builtin_amdgcn_readlane(ents, j & 63); };

        struct src { uint64_t k, v; bool live; };
        const uint64_t zb = reinterpret_cast<uint64_t>(zero_tile);
        auto src_of = [&](int c, bool live) {
            const int64_t at = static_cast<int64_t>(c < 0 ? 0 : c) * TILE;
            return src{kb + at, c < 0 ? zb : vb + at, live};
        };
        auto fetch_row = [&](auto f, int t, int ks) { fr.row(ring[decltype(f)::value & 3], k_lds, t, ks); };
        auto fetch_col = [&](auto f, int t, int u) { fr.col(ring[decltype(f)::value & 3], v_lds, t, u / MT, u % MT); };

        auto p_frag = [](const u32x4_t& w) {
            F f;
            f.v = __builtin_bit_cast(bf16x8_t, w);
            return f;
        };

        // One step of the pipeline (one half-tile): softmax of s[T], with
        // S of the next half-tile (s[1 - T]) and P V of the previous one
        // (half 1 - T) in its shadow.
        auto step = [&](auto t_, auto do_s_, auto do_pv_, auto next_, uint64_t dma_a, uint64_t dma_b, bool live_a,
                        bool live_b, uint64_t kmask) {
            constexpr int T = decltype(t_)::value, U = 1 - T;
            constexpr bool DO_S = decltype(do_s_)::value, DO_PV = decltype(do_pv_)::value;
            constexpr bool NEXT = decltype(next_)::value;     // the next step starts with an S product
            constexpr int NFS = DO_S ? KS : 0, NFV = DO_PV ? 2 * MT : 0, NF = NFS + NFV;
            constexpr int SLOTS = 2 * NFS + 2 * PT * NFV;
            constexpr int PER = (32 + SLOTS - 1) / SLOTS;
            constexpr int DPS = (ND + 2 * (KS - AHEAD) - 1) / (2 * (KS - AHEAD));   // copies per slot
            if constexpr (PAD) {
                if (kmask != ~0ull) {
                    asm volatile("");      // stays a branch (not 32 selects on every tile)
                    const uint32_t lm = static_cast<uint32_t>(kmask >> (T * 32 + half * 8));
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            s[T][qt][i] = ((lm >> ((i >> 3) * 16 + (i & 7))) & 1u) ? s[T][qt][i] : -INFINITY;
                }
            } else {
                if (kmask == 0) {
                    asm volatile("");
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int i = 0; i < 16; ++i) s[T][qt][i] = -INFINITY;
                }
            }
            float x[32];
            float ps[2] = {0.f, 0.f}, pr[2] = {0.f, 0.f};
            auto el_fma = [&](int e) {
                const int qt = (e >> 3) & 1;
                x[e] = fmaf(s[T][qt][8 * (e >> 4) + (e & 7)], c_log2, -m[qt]);
            };
            auto el_exp = [&](int e) { x[e] = fast_exp2(x[e]); };
            auto el_sum = [&](int e) {
                const int qt = (e >> 3) & 1, kk = e >> 4, w = (e & 7) >> 1;
                ps[qt] += x[e];
                if (e & 1) {
                    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
                    const bf16x2_t one = __builtin_bit_cast(bf16x2_t, 0x3f803f80u);
                    const uint32_t hi = pack2_bf16(x[e - 1], x[e]);
                    pw[T][kk][qt][0][w] = hi;
                    if constexpr (TWO) {
                        const uint32_t lo = pack2_bf16(x[e - 1] - __uint_as_float(hi << 16),
                                                       x[e] - __uint_as_float(hi & 0xffff0000u));
                        pw[T][kk][qt][PT - 1][w] = lo;
                        pr[qt] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, lo), one, pr[qt], false);
                    }
                    pr[qt] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, hi), one, pr[qt], false);
                }
            };
            auto elements = [&](int slot) {     // the vector work of one slot
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int e = slot * PER + i;
                    if (e >= 2 * PER && e - 2 * PER < 32) el_sum(e - 2 * PER);
                    if (e >= PER && e - PER < 32) el_exp(e - PER);
                    if (e < 32) el_fma(e);
                }
            };
            if constexpr (!DO_S) {      // no products before: request the first column fragments here
                vm_wait<2 * ND>();
                for_each_ic<AHEAD>([&](auto f) { fetch_col(f, U, decltype(f)::value); });
            }
            // slots: one MFMA each, with its share of the vector work, of the
            // fragment requests and of the copies
            for_each_ic<SLOTS>([&](auto slot_) {
                constexpr int SL = decltype(slot_)::value;
                constexpr bool IN_S = SL < 2 * NFS;
                constexpr int F_ = IN_S ? SL / 2 : NFS + (SL - 2 * NFS) / (2 * PT);      // fragment in use
                constexpr int SUB = IN_S ? SL % 2 : (SL - 2 * NFS) % (2 * PT);
                constexpr int PSL = IN_S ? SL : SL - 2 * NFS;                              // slot of the phase
                if constexpr (SUB == 0) {
                    constexpr int R = F_ + AHEAD;                                          // fragment to request
                    if constexpr (R < NFS) fetch_row(ic<R>{}, U, R);
                    else if constexpr (R < NF) {
                        if constexpr (R == NFS) vm_wait<2 * ND>();
                        fetch_col(ic<R>{}, U, R - NFS);
                    } else if constexpr (NEXT) {
                        if constexpr (R == NF) vm_wait<2 * ND>();
                        fetch_row(ic<R>{}, T, R - NF);
                    }
                }
                for_each_ic<DPS>([&](auto d_) {
                    constexpr int J = PSL * DPS + decltype(d_)::value;
                    if constexpr (J < ND && DO_S && DO_PV) {
                        if constexpr (IN_S) cp.template issue<J>(l0 + 2 * HALF + (1 - U) * HALF, dma_a, live_a);
                        else cp.template issue<J>(l0 + U * HALF, dma_b, live_b);
                    }
                });
                if constexpr (IN_S) {
                    constexpr int ks = F_, qt = SUB;
                    if constexpr (ks == 0) {
                        const f32x16_t z = {};
                        s[U][qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[F_ & 3].v, qf[qt][ks].v, z, 0, 0, 0);
                    } else {
                        mma(s[U][qt], ring[F_ & 3], qf[qt][ks]);
                    }
                } else {
                    constexpr int u = F_ - NFS, kk = u / MT, mt = u % MT, qt = SUB & 1, lo = SUB >> 1;
                    mma_acc(oacc[qt][mt], ring[F_ & 3], p_frag(pw[U][kk][qt][lo]));
                }
                elements(SL);
                lds_order();
            });
#pragma unroll
            for (int sl = SLOTS; sl < SLOTS + 2; ++sl) elements(sl);
            // the running reference m: p = 2^(s c - m) stays below 2^8 (its
            // sum over the lane's 16 keys is checked in place of a row max
            // per tile); otherwise m rises to the row max and the tile is redone
            if (__any(!(ps[0] <= 256.f) || !(ps[1] <= 256.f))) {
                acc_settle(oacc);
#pragma unroll
                for (int qt = 0; qt < 2; ++qt) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[T][qt][i]);
                    mx = fmaxf(mx, swap_half(mx)) * c_log2;
                    const float mn = fmaxf(m[qt], mx);
                    if (mn != -INFINITY) {
                        const float alpha = fast_exp2(m[qt] - mn);
                        l[qt] *= alpha;
                        lr[qt] *= alpha;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int i = 0; i < 16; ++i) oacc[qt][mt][i] *= alpha;
                        m[qt] = mn;
                    }
                    ps[qt] = pr[qt] = 0.f;
                }
#pragma unroll
                for (int e = 0; e < 32; ++e) {
                    const int qt = (e >> 3) & 1;
                    const float sv = s[T][qt][8 * (e >> 4) + (e & 7)];
                    x[e] = sv == -INFINITY ? 0.f : fast_exp2(fmaf(sv, c_log2, -m[qt]));   // NaN stays
                    el_sum(e);
                }
            }
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                l[qt] += ps[qt];
                lr[qt] += pr[qt];
            }
            // the fragments are whole here, long before the products that take them
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int p = 0; p < PT; ++p) asm volatile("" : "+v"(pw[T][kk][qt][p]));
        };
        auto kmask_of = [&](int c) -> uint64_t {
            if (c < 0) return 0;
            if constexpr (PAD) return cube_real_mask(grid, c, lane);
            return ~0ull;
        };

        load_ents(0);
        int c_cur = ent_at(0);
        int c_nxt = cnt > 1 ? ent_at(1) : -1;
        src cur = src_of(c_cur, true), nxt = src_of(c_nxt, cnt > 1);
        // Copies go out in the order the steps use them, and every wait finds
        // the two half-tiles issued after the one it needs still in flight:
        // K low, K high | K low', V low | K high' | then in the loop V high,
        // K low'', V low', K high'', ... (' next block).
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0, cur.k, true); });
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0 + HALF, cur.k + HALF, true); });
        vm_wait<ND>();
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[0][qt][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            F f;
            fr.row(f, k_lds, 0, ks);
            mma(s[0][0], f, qf[0][ks]);
            mma(s[0][1], f, qf[1][ks]);
        }
        lds_order();
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0, nxt.k, nxt.live); });
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0 + 2 * HALF, cur.v, true); });
        vm_wait<2 * ND>();
        for_each_ic<AHEAD>([&](auto f) { fetch_row(f, 1, decltype(f)::value); });
        constexpr auto yes = std::true_type{};
        constexpr auto no = std::false_type{};
        step(ic<0>{}, yes, no, no, 0, 0, false, false, kmask_of(c_cur));
        if (paced) {
            clk.join(avg);
            clk.request();
        }
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0 + HALF, nxt.k + HALF, nxt.live); });
        vm_wait<2 * ND>();
        for_each_ic<AHEAD>([&](auto f) { fetch_row(f, 0, decltype(f)::value); });
        for (int j = 0; j + 1 < cnt; ++j) {
            const bool more = j + 2 < cnt;
            if (more && ((j + 2) & 63) == 0) load_ents((j + 2) >> 6);
            const int c_far = more ? ent_at(j + 2) : -1;
            const src far = src_of(c_far, more);
            if (paced) {
                clk.wait(j);
                clk.step(j + 1);
                clk.request();
            }
            step(ic<1>{}, yes, yes, yes, cur.v + HALF, far.k, true, more, kmask_of(c_cur));
            step(ic<0>{}, yes, yes, yes, nxt.v, far.k + HALF, true, more, kmask_of(c_nxt));
            c_cur = c_nxt;
            c_nxt = c_far;
            cur = nxt;
            nxt = far;
        }
        for_each_ic<ND>([&](auto j) { cp.template issue<decltype(j)::value>(l0 + 3 * HALF, cur.v + HALF, true); });
        step(ic<1>{}, no, yes, no, 0, 0, false, false, kmask_of(c_cur));
        vm_wait<0>();
        asm volatile("s_nop 3");
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                F f;
                fr.col(f, v_lds, 1, kk, mt);
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int p = 0; p < PT; ++p) mma_acc(oacc[qt][mt], f, p_frag(pw[1][kk][qt][p]));
            }
        mma_drain();
    };
    if (cnt > 0) {
        if (COMP && big) walk(std::true_type{});
        else walk(std::false_type{});
        if (paced) clk.leave(cnt - 1);
    }
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const bool q_real = !PAD || ((qmask >> (32 * qt + (lane & 31))) & 1);
        const float lt = q_real ? l[qt] + swap_half(l[qt]) : 0.f;     // a padding query has no output
        const float lrt = q_real ? lr[qt] + swap_half(lr[qt]) : 0.f;
        // keys but no score above -inf: no weights to divide by
        const float none = any && m[qt] == -INFINITY ? __builtin_nanf("") : 0.f;
        const float inv = lrt > 0.f ? 1.0f / lrt : none;
        const int64_t tok = qtok + 32 * qt;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int d0 = mt * 32 + g4 * 8 + half * 4;
                float ov[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) ov[j] = q_real ? oacc[qt][mt][g4 * 4 + j] * inv : 0.f;
                const uint32_t w0 = pack2_bf16(ov[0], ov[1]), w1 = pack2_bf16(ov[2], ov[3]);
                *reinterpret_cast<uint2*>(o + tok * D + d0) = make_uint2(w0, w1);
                if constexpr (COMP) {
                    const uint32_t r0 = pack2_bf16(ov[0] - __uint_as_float(w0 << 16),
                                                   ov[1] - __uint_as_float(w0 & 0xffff0000u));
                    const uint32_t r1 = pack2_bf16(ov[2] - __uint_as_float(w1 << 16),
                                                   ov[3] - __uint_as_float(w1 & 0xffff0000u));
                    *reinterpret_cast<uint2*>(o_lo + tok * D + d0) = make_uint2(r0, r1);
                }
            }
        if (half == 0) lse[tok] = lt > 0.f ? (m[qt] + log2f(lt)) * 0.6931471805599453f : -INFINITY;
    }
}

hipError_t launch_attn_fwd_wave(const void* q, const void* k, const void* v, const int32_t* row_ptr,
                                const int32_t* col_idx, int64_t col_cap, void* o, float* lse, void* o_lo,
                                const int32_t* order, uint32_t* pace, const float* even, int64_t rows, int Hq,
                                int Hkv, int N, const cube_grid& cg, const block_flag_layout& fl, hipStream_t s) {
    const float c = 1.4426950408889634f / sqrtf(128.f);
    auto go = [&](auto comp, auto pad) {
        constexpr bool COMP = decltype(comp)::value, PAD = decltype(pad)::value;
        hipLaunchKernelGGL((attn_fwd_wave_kernel<COMP, PAD>), dim3(static_cast<unsigned>(rows)), dim3(64), 0, s,
                           static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                           static_cast<const bf16_t*>(v), row_ptr, col_idx, col_cap, static_cast<bf16_t*>(o), lse,
                           static_cast<bf16_t*>(o_lo), Hq, Hkv, N, c,
                           resident_per_xcd<attn_fwd_wave_kernel<COMP, PAD>>(64), order, pace, even, cg, fl);
    };
    if (o_lo) {
        if (cg.padded) go(std::true_type{}, std::true_type{}); else go(std::true_type{}, std::false_type{});
    } else {
        if (cg.padded) go(std::false_type{}, std::true_type{}); else go(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace vsa2
