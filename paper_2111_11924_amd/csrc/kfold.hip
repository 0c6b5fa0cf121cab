// Tables of the fold forms (fold.hpp), written once per key table.
//
// W_i = 2^(F + pos_i) mod m, one lane per i, by one Montgomery reduction each
// from the key record's constants: with R = 2^(lbh nlh) and e = F + pos_i -
// lbh nlh, MM(R^2, 2^e) = 2^(F + pos_i) (MM(R^3, 2^(e - lbh nlh)) where 2^e does not
// lie below R).  A block takes one (key, prime) at a time, a lane per column of a form.
// The lanes' sums lie in a buffer of the caller's, not in private memory, which the
// runtime would set aside for every wave that fits the chip (up to 3 GB, and abort the
// queue where that is not free).
//
// Bound by the latency of those sums: each pass over them takes eight
// rows of the product.  16 8192-bit keys: 29.1 ms with a row per pass and the columns in
// five rounds, 2.9 here; 128 4096-bit keys 10.3 and 2.1.
#include <algorithm>

#include "fold.hpp"
#include "mont.hpp"

namespace pmk {

namespace {

constexpr int kRows = 8;  // rows of a product per pass over its sums

struct SetupArgs {
    const uint32_t *keys;  // key records
    uint8_t *out;          // two tables of `size` bytes per key
    uint32_t size;
    uint32_t items;        // (key, prime) pairs
    uint64_t *sums;        // per block: SetupShape::WORDS
};

constexpr int setup_threads(FoldForm f) { return (4 * f.nl + 4 + 63) / 64 * 64; }

// a lane's column of numbers in a block's part of the buffer
template <typename T, int THREADS>
struct Column {
    T *p;
    __device__ T &operator[](int j) const { return p[j * THREADS]; }
};

// t[from ..] += sum_r x[r] 2^(LB r) times the NL limbs of n, without the columns below `skip`
template <int NL, typename T64>
__device__ void add_rows(T64 t, int from, const uint32_t (&x)[kRows], const uint32_t *n, int skip) {
    uint32_t w[kRows] = {};  // n's limbs j, j - 1, ...
    for (int j = 0; j < NL + kRows - 1; ++j) {
#pragma unroll
        for (int r = kRows - 1; r > 0; --r) w[r] = w[r - 1];
        w[0] = j < NL ? n[j] : 0u;
        if (j < skip) continue;
        uint64_t s = t[from + j];
#pragma unroll
        for (int r = 0; r < kRows; ++r) s += (uint64_t)x[r] * w[r];
        t[from + j] = s;
    }
}

// r = t R^-1 mod n, canonical (R = 2^(LB NL), t below R n, 2 NL + kRows limbs, overwritten)
template <int NL, int LB, typename T64, typename T32>
__device__ void redc(T32 r, T64 t, const uint32_t *n, uint32_t n0) {
    constexpr uint32_t MASK = (1u << LB) - 1u;
    uint64_t c = 0;
    for (int i = 0; i < NL; i += kRows) {
        const int rows = NL - i < kRows ? NL - i : kRows;
        uint32_t m[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            m[k] = 0;
            if (k >= rows) continue;
            uint64_t s = t[i + k] + c;
#pragma unroll
            for (int l = 0; l < k; ++l) s += (uint64_t)m[l] * n[k - l];
            m[k] = ((uint32_t)s * n0) & MASK;
            c = (s + (uint64_t)m[k] * n[0]) >> LB;
        }
        add_rows<NL>(t, i, m, n, rows);
    }
    for (int j = 0; j < NL; ++j) {
        c += t[NL + j];
        r[j] = (uint32_t)c & MASK;
        c >>= LB;
    }
    // below 2 n: subtract n unless that borrows
    int32_t bw = 0;
    for (int j = 0; j < NL; ++j) bw = ((int32_t)r[j] - (int32_t)n[j] + bw) >> 31;
    if (bw) return;
    for (int j = 0; j < NL; ++j) {
        const int32_t v = (int32_t)r[j] - (int32_t)n[j] + bw;
        r[j] = (uint32_t)v & MASK;
        bw = v >> 31;
    }
}

// bits [at, at + len) of nl limbs of lb bits, len <= 29
template <typename T32>
__device__ uint32_t bits_of(T32 x, int nl, int lb, int at, int len) {
    const int k = at / lb, sh = at % lb;
    const uint64_t lo = k < nl ? x[k] : 0u, hi = k + 1 < nl ? x[k + 1] : 0u;
    return (uint32_t)((lo | hi << lb) >> sh) & ((1u << len) - 1u);
}

// A column of W per lane of a block; two lanes more sum the rows' biases mod m.  The
// rows' start values are their biases plus the digits of minus that sum mod m.
template <int CB, bool LANE>
struct SetupShape {
    static constexpr Geom G = make_geom(CB);
    static constexpr FoldForm f = LANE ? fold_lane(CB) : fold_group(CB);
    static constexpr int THREADS = setup_threads(f), COLS = 4 * f.nl;
    static constexpr int SUMS = 2 * G.nlh + kRows;                             // 64-bit words of a lane
    static constexpr int WORDS = THREADS * SUMS + (THREADS * G.nlh + 1) / 2;  // of a block, with a residue per lane
    static_assert(THREADS >= COLS + 4 && COLS % 64 < 60, "lanes and columns for the sum of the biases");
};

template <int CB, bool LANE>
__device__ void fold_setup_item(const SetupArgs &a, uint32_t item, uint64_t *buf, uint32_t (&sums)[2][make_geom(CB).nlh]) {
    using S = SetupShape<CB, LANE>;
    constexpr Geom G = S::G;
    constexpr int NLH = G.nlh, LBH = G.lbh, RB = NLH * LBH, THREADS = S::THREADS;
    constexpr uint32_t MASK = (1u << LBH) - 1u;
    constexpr FoldForm f = S::f;
    constexpr int P = CB / 2, F = f.lb * f.nl, COLS = S::COLS;
    static_assert(F >= P + 17 && F >= RB && F + f.lb * f.nl < 3 * RB, "fold position");
    const uint32_t *hr = a.keys + (size_t)(item >> 1) * G.stride + G.off_half[0] + (item & 1) * G.h_size;
    const uint32_t *n = hr + G.h_m;
    const uint32_t n0 = hr[G.h_m0];
    uint8_t *tab = a.out + (size_t)item * a.size + (LANE ? fold_table(CB).lane : fold_table(CB).group);
    auto element = [](int row, int col) {
        if constexpr (LANE) return FoldShape<f.nl, f.lb>::element(row, col);
        // row tile row / 16, K step col / 64: 16 bytes of lane 16 (col / 16 % 4) + row % 16
        else
            return 16 * f.nl +
                   ((row / 16 * fold_group_steps(CB) + col / 64) * 64 + col / 16 % 4 * 16 + row % 16) * 16 + col % 16;
    };
    const int i = threadIdx.x;
    const Column<uint64_t, THREADS> t{buf + i};
    const Column<uint32_t, THREADS> x{(uint32_t *)(buf + THREADS * S::SUMS) + i};
    if (i < COLS + 2)
        for (int j = 0; j < S::SUMS; ++j) t[j] = 0;
    if (i < COLS) {
        int e = F + f.lb * (i / 4) + 8 * (i % 4) - RB;
        const uint32_t *c = hr + (e < RB ? G.h_rr : G.h_rrr);
        if (e >= RB) e -= RB;
        const int q = e / LBH, sh = e % LBH;
        uint32_t below = 0;  // c 2^e
        for (int j = 0; j < NLH; ++j) {
            const uint32_t v = c[j];
            t[q + j] = ((uint64_t)v << sh | below) & MASK;
            below = (uint32_t)((uint64_t)v << sh >> LBH);
        }
        t[q + NLH] = below;
        redc<NLH, LBH>(x, t, n, n0);
        for (int k = 0; k < f.nl; ++k) {
            const uint32_t d = (bits_of(x, NLH, LBH, f.lb * k, f.lb) + kDigitBias) ^ kDigitBias;
            for (int j = 0; j < 4; ++j) tab[element(4 * k + j, i)] = (uint8_t)(d >> (8 * j));
        }
    } else if (i < COLS + 2) {
        // sum of the biases lo + R hi: MM(lo, R) or MM(hi, R^2); its limbs in the column of
        // the lane two further, which has none
        const Column<uint64_t, THREADS> z{buf + i + 2};
        for (int j = 0; j < 2 * NLH; ++j) z[j] = 0;
        for (int k = 0; k < f.nl; ++k)
            for (int j = 0; j < 4; ++j) {
                const int at = f.lb * k + 8 * j;
                z[at / LBH] += (uint64_t)fold_bias(f, P, k, j, !LANE) << (at % LBH);
            }
        uint64_t c = 0;
        for (int j = 0; j < 2 * NLH; ++j) {
            c += z[j];
            z[j] = c & MASK;
            c >>= LBH;
        }
        const int hi = i - COLS;
        for (int j = 0; j < NLH; j += kRows) {
            uint32_t rows[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) rows[r] = j + r < NLH ? (uint32_t)z[hi * NLH + j + r] : 0u;
            add_rows<NLH>(t, j, rows, hr + (hi ? G.h_rr : G.h_one), 0);
        }
        redc<NLH, LBH>(x, t, n, n0);
        for (int j = 0; j < NLH; ++j) sums[hi][j] = x[j];
    }
    __syncthreads();
    if (i == 0) {
        // minus the sum: m - lo - hi, plus m where that is negative
        int32_t bw = 0;
        for (int j = 0; j < NLH; ++j) {
            const int32_t v = (int32_t)n[j] - (int32_t)sums[0][j] - (int32_t)sums[1][j] + bw;
            x[j] = (uint32_t)v & MASK;
            bw = v >> LBH;
        }
        if (bw < 0) {
            uint32_t cy = 0;
            for (int j = 0; j < NLH; ++j) {
                const uint32_t v = x[j] + n[j] + cy;
                x[j] = v & MASK;
                cy = v >> LBH;
            }
        }
        uint32_t *init = (uint32_t *)tab;
        for (int k = 0; k < f.nl; ++k) {
            const uint32_t d = bits_of(x, NLH, LBH, f.lb * k, f.lb);
            for (int j = 0; j < 4; ++j)
                init[4 * k + j] = fold_bias(f, P, k, j, !LANE) + (j < 3 ? (d >> (8 * j)) & 255u : d >> 24);
        }
    }
    __syncthreads();
}

template <int CB, bool LANE>
__global__ __launch_bounds__(setup_threads(LANE ? fold_lane(CB) : fold_group(CB))) void fold_setup_kernel(SetupArgs a) {
    __shared__ uint32_t sums[2][make_geom(CB).nlh];
    uint64_t *buf = a.sums + (size_t)blockIdx.x * SetupShape<CB, LANE>::WORDS;
    for (uint32_t item = blockIdx.x; item < a.items; item += gridDim.x) fold_setup_item<CB, LANE>(a, item, buf, sums);
}

template <int CB>
constexpr uint64_t block_words() {
    if constexpr (fold_lane(CB).nl != 0)
        return std::max(SetupShape<CB, true>::WORDS, SetupShape<CB, false>::WORDS);
    else
        return SetupShape<CB, false>::WORDS;
}

// blocks: as many as `words` words hold
template <int CB>
int setup(const SetupArgs &a, uint64_t words, hipStream_t s) {
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(a.items, words / block_words<CB>());
    if constexpr (fold_lane(CB).nl != 0) {
        hipLaunchKernelGGL((fold_setup_kernel<CB, true>), dim3(blocks), dim3(SetupShape<CB, true>::THREADS), 0, s, a);
        const int e = (int)hipGetLastError();
        if (e) return e;
    }
    hipLaunchKernelGGL((fold_setup_kernel<CB, false>), dim3(blocks), dim3(SetupShape<CB, false>::THREADS), 0, s, a);
    return (int)hipGetLastError();
}

template <int CB>
uint64_t setup_words(uint32_t count) {
    // up to 128 MiB: 64 blocks at 8192 bits
    return block_words<CB>() * std::max<uint64_t>(1, std::min<uint64_t>(2ull * count, (128ull << 20) / 8 / block_words<CB>()));
}

}  // namespace

uint64_t fold_setup_words(int cls, uint32_t count) {
    switch (kClassBits[cls]) {
        case 1024: return setup_words<1024>(count);
        case 2048: return setup_words<2048>(count);
        case 3072: return setup_words<3072>(count);
        case 4096: return setup_words<4096>(count);
        case 6144: return setup_words<6144>(count);
        case 8192: return setup_words<8192>(count);
        default: return 0;
    }
}

int launch_fold_setup(int cls, const uint32_t *keys, uint32_t count, uint8_t *fold, uint64_t *sums, uint64_t words,
                      void *stream) {
    const SetupArgs a{keys, fold, fold_table(kClassBits[cls]).size, 2 * count, sums};
    hipStream_t s = (hipStream_t)stream;
    switch (kClassBits[cls]) {
        case 1024: return setup<1024>(a, words, s);
        case 2048: return setup<2048>(a, words, s);
        case 3072: return setup<3072>(a, words, s);
        case 4096: return setup<4096>(a, words, s);
        case 6144: return setup<6144>(a, words, s);
        case 8192: return setup<8192>(a, words, s);
        default: return 0;
    }
}

}  // namespace pmk
