// Modular products of the CRT halves with the reduction on the matrix cores.
//
// A product t = a b of two NL-limb numbers (LB-bit limbs, F = LB NL) is reduced
// by folding its high half: t = t_lo + sum_i d_i 2^(F + pos_i) with byte digits
// d_i of t_hi, and 2^(F + pos_i) = W_i mod m is a table of the modulus alone.
// Every chunk of a tile shares its modulus, so sum_i d_i W_i over a tile is a
// matrix product: W's digits (rows: digits of the result, columns: digits of
// t_hi) times the tile's digits, int8 MFMA with exact 32-bit sums.  The result
// r = t_lo + sum_i d_i W_i = a b mod m is below 2^F + 2^(F-4), again an operand:
// a chain of products needs no other reduction and no Montgomery form.  The
// VALU only forms a b (a square: half of it), where a Montgomery product also
// spends NL^2 multiply-adds on its reduction.
//
// Digits.  A limb x < 2^31 gives four: the bytes of (x + 0x00808080) ^ 0x00808080,
// the low three signed, the top one not, sum = x.  Digit 4 k + j stands at bit
// LB k + 8 j, of t_hi (4 NLP columns of W) and of W_i itself (4 NLP rows), NLP =
// NL rounded up to 4.
//
// Sums.  A column sum is below NL (3*128 + 2^(LB-24) + 1) 128 in size; the
// accumulators start at a bias at or above that (a power of two; 0 for rows
// that W cannot reach), so the sums that leave the matrix cores are never
// negative.  All biases together are made a multiple of m by adding the digits
// of -sum mod m (fold_setup_kernel writes both, as the start values).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pmk_internal.hpp"

namespace pmk {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr uint32_t kDigitBias = 0x00808080u;

// Table of one prime (bytes): the start values of the 4 NLP rows (32-bit), then
// W for the 32 x 32 MFMA.  W's tile (m, s): rows 32 m .. (32, in the last tile
// 16 when NLP is 4 modulo 8) by columns 32 s .. (32, the last step likewise
// 16), stored in operand order: lane half h of row i holds 16 (8) successive
// columns, 16 h (8 h) on.
template <int NL, int LB>
struct FoldShape {
    static constexpr int NLP = (NL + 3) / 4 * 4;
    static constexpr int FULL = NLP / 8;              // K steps of 32 digits
    static constexpr bool HALF = NLP % 8 != 0;        // and one of 16
    static constexpr int STEPS = FULL + (HALF ? 1 : 0);
    static constexpr int TILES = STEPS;               // row tiles (W is square)
    static constexpr int DIGITS = 4 * NLP;
    static constexpr int INIT_BYTES = 4 * DIGITS;
    static constexpr int BYTES = INIT_BYTES + DIGITS * DIGITS;
    PMK_HD static constexpr int rows(int m) { return m < FULL ? 32 : 16; }
    PMK_HD static constexpr int tile_off(int m, int s) { return INIT_BYTES + m * 32 * DIGITS + s * rows(m) * 32; }
    // byte of W's element (row, column)
    PMK_HD static constexpr int element(int row, int col) {
        const int m = row / 32, s = col / 32, n = s < FULL ? 16 : 8;  // columns per lane half
        return tile_off(m, s) + (col % 32 / n * rows(m) + row % 32) * n + col % n;
    }
};

// One wave's view of the table in LDS.
struct FoldLds {
    const uint8_t *w;  // FoldShape::BYTES bytes
};

// The next instruction at an 8-byte boundary (kernels_impl.hpp, code alignment).
__device__ __forceinline__ void fold_align() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile(".p2align 3");
    __builtin_amdgcn_sched_barrier(0);
}

// v_permlane32_swap: x = [x.lo | y.lo], y = [x.hi | y.hi] (halves of 32 lanes)
__device__ __forceinline__ void swap32(uint32_t &x, uint32_t &y) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}

// Order in which the MFMAs of one product are issued, between which of its
// multiply-adds.  Issued back to back they stall their wave (each keeps the
// matrix core for 32 cycles); one per kPace VALU instructions they run beside
// the column products.  Column c of the product is k = NL - 2 + c in the high
// part (c <= NL), then k = c - NL - 1.  MFMA n belongs to row tile tile(n), K step
// step(n), half n & 1 of the chunks: the steps of tiles 0 and 1 as their digits
// are ready, then tiles 2, 3, ... in turn, two tiles' sums in registers at a
// time.
template <int NL, int LB, bool SQR>
struct FoldOrder {
    using S = FoldShape<NL, LB>;
    static constexpr int kPace = 10;
    static constexpr int COLS = 2 * NL + 1;
    static constexpr int TOTAL = 2 * S::TILES * S::STEPS;
    int first[COLS + 1] = {};  // MFMAs [first[c], first[c + 1]) are issued in column c,
    int at[TOTAL] = {};        // each after this many of its multiply-adds

    static constexpr int tile(int n) { return n < 4 * S::STEPS ? (n / 2) & 1 : 2 + (n - 4 * S::STEPS) / (2 * S::STEPS); }
    static constexpr int step(int n) { return n < 4 * S::STEPS ? n / 4 : (n - 4 * S::STEPS) / 2 % S::STEPS; }
    static constexpr int k_of(int c) { return c <= NL ? NL - 2 + c : c - NL - 1; }
    static constexpr int lo(int k) { return k - NL + 1 > 0 ? k - NL + 1 : 0; }
    // first operand indices [lo, end) of column k (the square term apart)
    static constexpr int end(int k) { return SQR ? (k + 1) / 2 : (k < NL ? k + 1 : NL); }
    static constexpr int mads(int c) { return c > NL && k_of(c) >= NL - 2 ? 0 : end(k_of(c)) - lo(k_of(c)); }
    constexpr FoldOrder() {
        int next = 0, work = 0, ready = 0, limbs = 0;
        for (int c = 0; c < COLS; ++c) {
            first[c] = next;
            const bool high = c <= NL;
            const int k = k_of(c);
            // last tile whose accumulators are free
            const int can = high ? 1 : k / 8 + (k % 8 == 7 ? 2 : 1);
            for (int o = 0; o <= mads(c); ++o) {
                if (work >= kPace && next < TOTAL && step(next) < ready && tile(next) <= can) {
                    at[next++] = o;
                    work = 0;
                }
                ++work;
            }
            // a tile's last MFMAs come no later than its first use
            if (!high && k % 8 == 0)
                while (next < TOTAL && (next < 4 * S::STEPS || tile(next) <= k / 8)) at[next++] = mads(c);
            work += high ? 4 : 8;
            if (high && k >= NL) {
                ++limbs;
                if (c == NL) ++limbs;  // the top limb follows the last column
                ready = limbs == NL ? S::STEPS : limbs / 8;
            }
        }
        first[COLS] = next;
    }
};

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// The fold of one product.  high<i>(x) takes limb i of t_hi in order; mfma<n>()
// issues MFMA n; low<k>(u, v) gives u, v with u + 2^16 v = limb k of sum d_i W_i.
template <int NL, int LB, typename Order>
struct Folder {
    using S = FoldShape<NL, LB>;
    FoldLds f;
    int lane;
    uint32_t dig[S::NLP];  // digits; after the swaps operand B of the two halves of the tile
    v16i c0[2], c1[2];     // sums of row tiles m, m + 1: chunks 0-31, chunks 32-63
    v4i w[3];              // operand A, read ahead (a half step uses two registers)
    uint32_t u1, v1;       // the odd limb of the current pair

    __device__ __forceinline__ Folder(FoldLds f_, int lane_) : f(f_), lane(lane_) {
#pragma unroll
        for (int i = NL; i < S::NLP; ++i) dig[i] = 0;
        load_w<0>();
        load_w<1>();
    }
    template <int M>
    __device__ __forceinline__ void start() {
        const int *p = (const int *)f.w + 32 * M + 4 * (lane >> 5);
        v16i a{};
#pragma unroll
        for (int g = 0; g < (M < S::FULL ? 4 : 2); ++g) {
            const v4i x = *(const v4i *)(p + 8 * g);
            a[4 * g] = x[0], a[4 * g + 1] = x[1], a[4 * g + 2] = x[2], a[4 * g + 3] = x[3];
        }
        c0[M & 1] = a;
        c1[M & 1] = a;
    }
    template <int J>
    __device__ __forceinline__ void load_w() {  // operand A of MFMAs 2 J, 2 J + 1
        if constexpr (2 * J < Order::TOTAL) {
            constexpr int m = Order::tile(2 * J), s = Order::step(2 * J);
            const int row = S::rows(m) == 32 ? (lane & 31) : (lane & 15);
            const int at = (lane >> 5) * S::rows(m) + row;
            if constexpr (s < S::FULL) {
                w[J % 3] = *(const v4i *)(f.w + S::tile_off(m, s) + 16 * at);
            } else {
                const v2i x = *(const v2i *)(f.w + S::tile_off(m, s) + 8 * at);
                w[J % 3][0] = x[0];
                w[J % 3][1] = x[1];
            }
        }
    }
    template <int N>
    __device__ __forceinline__ void mfma() {
        constexpr int m = Order::tile(N), s = Order::step(N), h = N & 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (h == 0) {
            load_w<N / 2 + 2>();
            if constexpr (s == 0) start<m>();
        }
        const v4i a = w[N / 2 % 3];
        v16i &c = h ? c1[m & 1] : c0[m & 1];
        if constexpr (s < S::FULL) {
            constexpr int i = 8 * s + 4 * h;
            const v4i x = {(int)dig[i], (int)dig[i + 1], (int)dig[i + 2], (int)dig[i + 3]};
            c = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, x, c, 0, 0, 0);
        } else {
            constexpr int i = 8 * s + 2 * h;
            const long wl = (long)(((uint64_t)(uint32_t)a[1] << 32) | (uint32_t)a[0]);
            const long x = (long)(((uint64_t)dig[i + 1] << 32) | dig[i]);
            c = __builtin_amdgcn_mfma_i32_32x32x16_i8(wl, x, c, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // limb I of t_hi (below 2^31)
    template <int I>
    __device__ __forceinline__ void high(uint32_t x) {
        dig[I] = (x + kDigitBias) ^ kDigitBias;
        if constexpr (I % 8 == 7 || (I == NL - 1 && !S::HALF)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) swap32(dig[I / 8 * 8 + j], dig[I / 8 * 8 + 4 + j]);
        } else if constexpr (I == NL - 1) {
#pragma unroll
            for (int j = 0; j < 2; ++j) swap32(dig[8 * S::FULL + j], dig[8 * S::FULL + 2 + j]);
        }
    }
    template <int K>
    __device__ __forceinline__ void low(uint32_t &u, uint32_t &v) {
        constexpr int m = K / 8, g = (K % 8) / 2;
        if constexpr (K % 2 == 0) {
            const v16i &a = c0[m & 1], &b = c1[m & 1];
            u = (uint32_t)a[4 * g] + ((uint32_t)a[4 * g + 1] << 8);
            v = (uint32_t)a[4 * g + 2] + ((uint32_t)a[4 * g + 3] << 8);
            u1 = (uint32_t)b[4 * g] + ((uint32_t)b[4 * g + 1] << 8);
            v1 = (uint32_t)b[4 * g + 2] + ((uint32_t)b[4 * g + 3] << 8);
            swap32(u, u1);
            swap32(v, v1);
        } else {
            u = u1;
            v = v1;
        }
    }
};

// r = a b mod m (SQR: a^2, b = 2 a limb by limb) for limbs below 2^LB, the top
// one below 2^LB + 2^(LB-4); r likewise.  Columns NL-2 .. 2 NL - 2 come first:
// they give t_hi, short of the carry out of column NL - 3, which goes into
// limb NL-2 later and stays below 2^-20 of 2^F (t_lo then is that much above
// 2^F).  one = 1, k16 = 2^16, held in registers so that adding a 32-bit value to a
// 64-bit sum is one multiply-add.
template <int NL, int LB, bool SQR>
__device__ __forceinline__ void fold_mul(uint32_t (&r)[NL], const uint32_t (&a)[NL], const uint32_t (&b)[NL],
                                         FoldLds f, int lane, uint32_t one, uint32_t k16) {
    static_assert((NL * 1.15 + 0.01) * (double)(1ull << LB) * (double)(1ull << LB) < 18446744073709551615.0,
                  "column sums may overflow 64 bits");
    constexpr uint32_t MASK = (1u << LB) - 1u;
    using Order = FoldOrder<NL, LB, SQR>;
    static constexpr Order ord{};
    Folder<NL, LB, Order> fo(f, lane);
    uint32_t top[2];  // limbs NL-2, NL-1 of t_lo
    uint64_t acc = 0;
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, Order::COLS>([&](auto cc) {
        constexpr int c = cc(), k = Order::k_of(c);
        constexpr bool high = c <= NL;
        constexpr int lo = Order::lo(k), n = Order::mads(c);
        if constexpr (c == NL + 1) acc = 0;
        auto products = [&](int from, int to) {
            // at 56 limbs a stretch can start with a reload from scratch: waited for before
            // the alignment
            if constexpr (NL == 56) {
                __builtin_amdgcn_sched_barrier(0);
                if (from < to) asm volatile("" ::"v"(a[lo + from]), "v"(b[k - lo - from]));
            }
            fold_align();
#pragma unroll
            for (int i = lo + from; i < lo + to; ++i) acc += (uint64_t)a[i] * b[k - i];
        };
        static_for<ord.first[c], ord.first[c + 1]>([&](auto nn) {
            constexpr int m = nn();
            products(m == ord.first[c] ? 0 : ord.at[m - 1 > 0 ? m - 1 : 0], ord.at[m]);
            fo.template mfma<m>();
        });
        products(ord.first[c] == ord.first[c + 1] ? 0 : ord.at[ord.first[c + 1] > 0 ? ord.first[c + 1] - 1 : 0], n);
        if constexpr (SQR && k % 2 == 0 && (high || k < NL - 2)) acc += (uint64_t)a[k / 2] * a[k / 2];
        if constexpr (high) {
            const uint32_t x = (uint32_t)acc & MASK;
            if constexpr (k < NL) top[k - (NL - 2)] = x;
            else fo.template high<k - NL>(x);
            acc >>= LB;
            if constexpr (c == NL) fo.template high<NL - 1>((uint32_t)acc);
        } else {
            if constexpr (k >= NL - 2) acc += top[k - (NL - 2)];
            uint32_t u, v;
            fo.template low<k>(u, v);
            fold_align();
            acc += (uint64_t)v * k16;
            acc += (uint64_t)u * one;
            r[k] = k < NL - 1 ? (uint32_t)acc & MASK : (uint32_t)acc;
            acc >>= LB;
        }
        asm volatile("" : "+v"(acc));
        __builtin_amdgcn_sched_barrier(0);
    });
}

}  // namespace pmk
