// Tables of the fold forms (fold.hpp), written once per key table.
//
// W_i = 2^(F + pos_i) mod m, one lane per i, by one Montgomery product each
// from the key record's constants: with R = 2^(lbh nlh) and e = F + pos_i -
// lbh nlh, MM(R^2, 2^e) = 2^(F + pos_i) (MM(R^3, 2^(e - lbh nlh)) where 2^e does not
// lie below R).  Rolled loops: the setup of a whole key table takes less time
// than its upload.
#include "fold.hpp"
#include "mont.hpp"

namespace pmk {

namespace {

constexpr int kMaxHalf = 152;   // limbs of the largest CRT half
constexpr int kSetupBlock = 128;

struct SetupArgs {
    const uint32_t *keys;  // key records
    uint8_t *out;          // two tables of `size` bytes per key
    uint32_t size;
};

// r = a b R^-1 mod n, canonical; nl limbs of lb bits, a b < R n
__device__ void mm(uint32_t *r, const uint32_t *a, const uint32_t *b, const uint32_t *n, uint32_t n0, int nl, int lb) {
    const uint32_t mask = (1u << lb) - 1u;
    uint64_t t[kMaxHalf];
    for (int j = 0; j < nl; ++j) t[j] = 0;
    for (int i = 0; i < nl; ++i) {
        const uint32_t bi = b[i];
        uint64_t c = t[0] + (uint64_t)a[0] * bi;
        const uint32_t m = ((uint32_t)c * n0) & mask;
        c = (c + (uint64_t)m * n[0]) >> lb;
        for (int j = 1; j < nl; ++j) t[j - 1] = t[j] + (uint64_t)a[j] * bi + (uint64_t)m * n[j];
        t[nl - 1] = 0;
        t[0] += c;
    }
    uint64_t c = 0;
    for (int j = 0; j < nl; ++j) {
        c += t[j];
        r[j] = (uint32_t)c & mask;
        c >>= lb;
    }
    // below 2 n: subtract n unless that borrows
    int32_t bw = 0;
    for (int j = 0; j < nl; ++j) bw = ((int32_t)r[j] - (int32_t)n[j] + bw) >> 31;
    if (bw) return;
    for (int j = 0; j < nl; ++j) {
        const int32_t v = (int32_t)r[j] - (int32_t)n[j] + bw;
        r[j] = (uint32_t)v & mask;
        bw = v >> 31;
    }
}

// bits [at, at + len) of nl limbs of lb bits, len <= 29
__device__ uint32_t bits_of(const uint32_t *x, int nl, int lb, int at, int len) {
    const int k = at / lb, sh = at % lb;
    const uint64_t lo = k < nl ? x[k] : 0u, hi = k + 1 < nl ? x[k + 1] : 0u;
    return (uint32_t)((lo | hi << lb) >> sh) & ((1u << len) - 1u);
}

// One block per (key, prime): the columns of W over the lanes, and the start
// values of the rows: their biases plus the digits of -(sum of the biases) mod m.
template <int CB>
__global__ __launch_bounds__(kSetupBlock) void fold_setup_kernel(SetupArgs a) {
    constexpr Geom G = make_geom(CB);
    constexpr int NLH = G.nlh, LBH = G.lbh, RB = NLH * LBH;
    constexpr FoldTable T = fold_table(CB);
    const uint32_t *hr = a.keys + (size_t)(blockIdx.x >> 1) * G.stride + G.off_half[0] + (blockIdx.x & 1) * G.h_size;
    const uint32_t *n = hr + G.h_m;
    const uint32_t n0 = hr[G.h_m0];
    uint8_t *out = a.out + (size_t)blockIdx.x * a.size;
    constexpr int P = CB / 2;
    auto form = [&](auto f_, bool loose, uint8_t *tab, auto element) {
        constexpr FoldForm f = decltype(f_)::value();
        constexpr int F = f.lb * f.nl;
        static_assert(F >= P + 17 && F >= RB && F + f.lb * f.nl < 3 * RB, "fold position");
        uint32_t x[NLH], b[NLH];
        for (int i = threadIdx.x; i < 4 * f.nl; i += kSetupBlock) {
            int e = F + f.lb * (i / 4) + 8 * (i % 4) - RB;
            const uint32_t *c = hr + (e < RB ? G.h_rr : G.h_rrr);
            if (e >= RB) e -= RB;
            for (int j = 0; j < NLH; ++j) b[j] = j == e / LBH ? 1u << (e % LBH) : 0u;
            mm(x, c, b, n, n0, NLH, LBH);
            for (int k = 0; k < f.nl; ++k) {
                const uint32_t d = (bits_of(x, NLH, LBH, f.lb * k, f.lb) + kDigitBias) ^ kDigitBias;
                for (int j = 0; j < 4; ++j) tab[element(4 * k + j, i)] = (uint8_t)(d >> (8 * j));
            }
        }
        if (threadIdx.x) return;
        // sum of the biases, lo + R hi
        uint64_t z[2 * NLH];
        for (int j = 0; j < 2 * NLH; ++j) z[j] = 0;
        for (int k = 0; k < f.nl; ++k)
            for (int j = 0; j < 4; ++j) {
                const int at = f.lb * k + 8 * j;
                z[at / LBH] += (uint64_t)fold_bias(f, P, k, j, loose) << (at % LBH);
            }
        uint64_t c = 0;
        for (int j = 0; j < 2 * NLH; ++j) {
            c += z[j];
            z[j] = c & ((1u << LBH) - 1u);
            c >>= LBH;
        }
        uint32_t y[NLH];
        for (int j = 0; j < NLH; ++j) b[j] = (uint32_t)z[j];
        mm(x, hr + G.h_rr, b, n, n0, NLH, LBH);
        for (int j = 0; j < NLH; ++j) b[j] = (uint32_t)z[NLH + j];
        mm(y, hr + G.h_rrr, b, n, n0, NLH, LBH);
        c = 0;
        for (int j = 0; j < NLH; ++j) {
            c += (uint64_t)x[j] + y[j];
            x[j] = (uint32_t)c & ((1u << LBH) - 1u);
            c >>= LBH;
            b[j] = j == 0;
        }
        mm(y, x, b, n, n0, NLH, LBH);  // the sum mod m
        int32_t bw = 0;
        for (int j = 0; j < NLH; ++j) {  // m - that
            const int32_t v = (int32_t)n[j] - (int32_t)y[j] + bw;
            x[j] = (uint32_t)v & ((1u << LBH) - 1u);
            bw = v >> 31;
        }
        uint32_t *init = (uint32_t *)tab;
        for (int k = 0; k < f.nl; ++k) {
            const uint32_t d = bits_of(x, NLH, LBH, f.lb * k, f.lb);
            for (int j = 0; j < 4; ++j)
                init[4 * k + j] = fold_bias(f, P, k, j, loose) + (j < 3 ? (d >> (8 * j)) & 255u : d >> 24);
        }
    };
    if constexpr (fold_lane(CB).nl) {
        struct Lane {
            static constexpr FoldForm value() { return fold_lane(CB); }
        };
        using S = FoldShape<fold_lane(CB).nl, fold_lane(CB).lb>;
        form(Lane{}, false, out + T.lane, [](int row, int col) { return S::element(row, col); });
    }
    if constexpr (fold_group(CB).nl) {
        struct Group {
            static constexpr FoldForm value() { return fold_group(CB); }
        };
        // row tile row / 16, K step col / 64: 16 bytes of lane 16 (col / 16 % 4) + row % 16
        form(Group{}, true, out + T.group, [](int row, int col) {
            return 16 * fold_group(CB).nl +
                   ((row / 16 * fold_group_steps(CB) + col / 64) * 64 + col / 16 % 4 * 16 + row % 16) * 16 + col % 16;
        });
    }
}

template <int CB>
int setup(const SetupArgs &a, uint32_t count, hipStream_t s) {
    hipLaunchKernelGGL(fold_setup_kernel<CB>, dim3(2 * count), dim3(kSetupBlock), 0, s, a);
    return (int)hipGetLastError();
}

}  // namespace

int launch_fold_setup(int cls, const uint32_t *keys, uint32_t count, uint8_t *fold, void *stream) {
    const SetupArgs a{keys, fold, fold_table(kClassBits[cls]).size};
    hipStream_t s = (hipStream_t)stream;
    switch (kClassBits[cls]) {
        case 1024: return setup<1024>(a, count, s);
        case 2048: return setup<2048>(a, count, s);
        case 3072: return setup<3072>(a, count, s);
        case 4096: return setup<4096>(a, count, s);
        case 6144: return setup<6144>(a, count, s);
        case 8192: return setup<8192>(a, count, s);
        default: return 0;
    }
}

}  // namespace pmk
