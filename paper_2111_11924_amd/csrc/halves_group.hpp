// CRT halves in the fold form with a number spread over a block (fold.hpp):
// launches too small to fill the chip, and the classes whose numbers do not fit
// one lane.
//
// A block of WV waves works on 16 chunks of one tile, modulo one prime.  Lane
// (q, n) of a wave (q = lane / 16, n = lane % 16) computes, for chunk n, the
// columns k = 4 m + q and k + NL of a product for the wave's share of the m in
// [0, NL / 4): every m costs the same, NL + 4 multiply-adds (a square about
// half).  Its limbs of the reduced result are the same k: row tile m of the
// 16 x 16 MFMA gives lane (q, n) the four digits of limb 4 m + q, so a wave
// needs W's row tiles of its own m only and keeps them in registers for the
// whole exponentiation (RES of the K steps; the rest is read from L2 each time).
// Four exchanges per product go through LDS: the carries of the columns, the
// digits of t_hi, the carries of the folded limbs, and the result as the next
// operand.
//
// Operands lie in LDS in four copies per chunk, copy c shifted by c limbs, so
// that lane (q, n) reads b_(4 D + q - 3 .. 4 D + q) as one aligned 16-byte
// load; zeros stand below limb 0 and above limb NL - 1.
//
// Limbs are loose: a column's sum splits into limb, carry and second carry
// (LB bits each), added once without rippling on.  t_lo is then below 2^(F+1), and
// so is an operand, up to the folded sum; t_hi's top limb is below 2^(LB+2).
//
// Bound by the chain of one number: per product the columns, the MFMA steps and the
// four exchanges follow one another.  1 MiB under 64 2048-bit keys 4.38 ms with
// four lanes per number, 2.95 here; 100 KiB under 16 keys 17.1 / 6.3 ms at 4096
// bits, 43.6 / 15.8 at 6144 and 94.3 / 34.5 at 8192 with eight.
#pragma once

namespace pmk {

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <int CB, int WV>
struct GroupShape {
    static constexpr int NL = fold_group(CB).nl, LB = fold_group(CB).lb;
    static constexpr int NM = NL / 4;                  // limb groups, row tiles
    static constexpr int CM = (NM + WV - 1) / WV;      // of them per wave,
    static constexpr int LAST = NM - (WV - 1) * CM;    // the last wave maybe fewer
    static_assert(LAST > 0, "every wave has work");
    static constexpr int KS = fold_group_steps(CB);    // K steps of 64 digits
    static constexpr int RES = fold_group_resident(CB) < KS ? fold_group_resident(CB) : KS;
    static constexpr int CHUNK = 3;
    static constexpr int CP = NL + 4;                  // words of one copy
    static constexpr int SN = 4 * CP + 4;              // words of a chunk's copies
    static constexpr int DS = 16 * KS + 4;             // words of a chunk's digits
    static constexpr int X = 0, Y = 16 * SN, P = 32 * SN, D = P + 2 * 16 * (2 * NL + 2), C = D + 16 * DS;
    static constexpr int WORDS = C + 16 * (NL + 1);
    static constexpr uint32_t MASK = (1u << LB) - 1u;
};

// Global memory through pointers of its own address space: made from a generic
// pointer that went through an opaque copy (fresh), an access is a flat one,
// which counts as an LDS access too and so holds up the next barrier.
typedef __attribute__((address_space(1))) uint32_t global_u32;
typedef const __attribute__((address_space(1))) uint8_t global_u8;
typedef const __attribute__((address_space(1))) v4i global_v4i;

// barrier over the block's LDS accesses only: global loads stay in flight
PMK_DEV void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// acc += products of limbs 4 I .. 4 I + 3 of a with v = b_(4 D + q - 3 .. 4 D + q)
PMK_DEV void block4(uint64_t &acc, u4 a, u4 v) {
    acc += (uint64_t)a[0] * v[3];
    acc += (uint64_t)a[1] * v[2];
    acc += (uint64_t)a[2] * v[1];
    acc += (uint64_t)a[3] * v[0];
}

// Keeps the products issued so far ahead of the loads that follow: the compiler
// otherwise gathers the loads of the whole column loop at its start and spills.
template <int CM>
PMK_DEV void hold(uint64_t (&lo)[CM], uint64_t (&hi)[CM]) {
#pragma unroll
    for (int j = 0; j < CM; ++j) asm volatile("" : "+v"(lo[j]), "+v"(hi[j]));
    __builtin_amdgcn_sched_barrier(0);
}

constexpr int kAhead = 2;  // steps between a load from LDS and its use

// Columns 4 m + q (lo) and those + NL (hi) for the m of wave W.  a: the lane's
// chunk, unshifted copy; v: the copy shifted by q, in 16-byte groups.
template <int CB, int WV, int W, int CM>
PMK_DEV void group_columns(uint64_t (&lo)[CM], uint64_t (&hi)[CM], const u4 *a, const u4 *v) {
    using G = GroupShape<CB, WV>;
    constexpr int M0 = W * G::CM, M1 = M0 + G::CM < G::NM ? M0 + G::CM : G::NM, NM = G::NM;
    // v groups: [j] for lo, [CM + j] for hi, group m - i (+ NM) of m = M0 + j;
    // a's group and the two groups entering the windows are loaded kAhead steps early
    u4 win[2 * G::CM] = {}, aq[kAhead] = {}, lq[kAhead] = {}, hq[kAhead] = {};
    auto fetch = [&](int i) {  // what step i needs new
        if (i >= NM) return;
        aq[i % kAhead] = a[i];
        if (i > 0 && M0 - i >= 0) lq[i % kAhead] = v[M0 - i];
        if (i >= M0) hq[i % kAhead] = v[M0 - i + NM];
    };
#pragma unroll
    for (int j = 0; j < M1 - M0; ++j) win[j] = v[M0 + j];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch(i);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        const u4 ai = aq[i % kAhead];
        if (i > 0) win[0] = lq[i % kAhead];
        win[G::CM] = hq[i % kAhead];
        fetch(i + kAhead);
        fold_align();
#pragma unroll
        for (int j = 0; j < M1 - M0; ++j) {
            if (i <= M0 + j) block4(lo[j], ai, win[j]);
            if (i >= M0 + j) block4(hi[j], ai, win[G::CM + j]);
        }
        hold(lo, hi);
#pragma unroll
        for (int j = M1 - M0 - 1; j > 0; --j) {
            win[j] = win[j - 1];
            win[G::CM + j] = win[G::CM + j - 1];
        }
    }
}

// The same columns of a square: every product i < j once with 2 a_i, the
// squares once.  Blocks (I, D) with I <= D - 2 lie wholly below the diagonal;
// in those on it the products count 0, 1 or 2 times by q (m1, m2, m3: all
// ones where q >= 1, 2, 3).
template <int CB, int WV, int W, int CM>
PMK_DEV void group_columns_sqr(uint64_t (&lo)[CM], uint64_t (&hi)[CM], const u4 *a, const u4 *v, uint32_t m1,
                               uint32_t m2, uint32_t m3) {
    using G = GroupShape<CB, WV>;
    constexpr int M0 = W * G::CM, M1 = M0 + G::CM < G::NM ? M0 + G::CM : G::NM, NM = G::NM;
    constexpr int IE = (M1 - 1 + NM) / 2;  // last I
    auto once = [&](uint32_t x) { return x + (x & m1); };             // q = 0: x, else 2 x
    auto late = [&](uint32_t x) { return (x & m2) + (x & m3); };      // q < 2: 0, q = 2: x, q = 3: 2 x
    auto add = [&](uint64_t &acc, u4 a1, u4 a2, u4 vd, int i, int d) {
        if (i <= d - 2) {
            block4(acc, a2, vd);
        } else if (i == d - 1) {
            acc += (uint64_t)a2[0] * vd[3];
            acc += (uint64_t)a2[1] * vd[2];
            acc += (uint64_t)once(a1[2]) * vd[1];
            acc += (uint64_t)late(a1[3]) * vd[0];
        } else if (i == d) {
            acc += (uint64_t)once(a1[0]) * vd[3];
            acc += (uint64_t)late(a1[1]) * vd[2];
        }
    };
    u4 win[2 * G::CM] = {}, aq[kAhead] = {}, lq[kAhead] = {}, hq[kAhead] = {};
    auto fetch = [&](int i) {
        if (i > IE) return;
        aq[i % kAhead] = a[i];
        if (i > 0 && 2 * i <= M0) lq[i % kAhead] = v[M0 - i];
        if (i >= M0) hq[i % kAhead] = v[M0 - i + NM];
    };
#pragma unroll
    for (int j = 0; j < M1 - M0; ++j) win[j] = v[M0 + j];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch(i);
#pragma unroll
    for (int i = 0; i <= IE; ++i) {
        const u4 a1 = aq[i % kAhead], a2 = a1 << 1;
        if (i > 0) win[0] = lq[i % kAhead];
        win[G::CM] = hq[i % kAhead];
        fetch(i + kAhead);
        fold_align();
#pragma unroll
        for (int j = 0; j < M1 - M0; ++j) {
            const int m = M0 + j;
            if (2 * i <= m) add(lo[j], a1, a2, win[j], i, m - i);
            if (i >= m && 2 * i <= m + NM) add(hi[j], a1, a2, win[G::CM + j], i, m - i + NM);
        }
        hold(lo, hi);
#pragma unroll
        for (int j = M1 - M0 - 1; j > 0; --j) {
            win[j] = win[j - 1];
            win[G::CM + j] = win[G::CM + j - 1];
        }
    }
}

// One block's work on (16 chunks, prime).
template <int CB, int WV>
struct Group {
    using G = GroupShape<CB, WV>;
    static constexpr int CM = G::CM, KS = G::KS, RES = G::RES;
    uint32_t *lds;
    const uint8_t *wtab;  // W of the prime
    int wave, lane, q, n, m0;
    uint32_t m1, m2, m3;
    v4i init[CM], w[CM][RES];
    uint32_t own[CM];     // limbs 4 (m0 + j) + q of the running value

    PMK_DEV int limb(int j) const { return 4 * (m0 + j) + q; }
    PMK_DEV bool skip(int j) const { return j >= G::LAST && wave == WV - 1; }  // no group j in this wave
    // the lane holding limb k of the number, k = NL - 4 + quarter
    PMK_DEV bool holds_top(int j, int quarter) const { return j == G::LAST - 1 && wave == WV - 1 && q == quarter; }

    PMK_DEV void setup(uint32_t *lds_) {
        lds = lds_;
        wave = (int)uni(threadIdx.x / 64);
        lane = threadIdx.x & 63;
        q = lane >> 4;
        n = lane & 15;
        m0 = wave * CM;
        m1 = q >= 1 ? ~0u : 0u;
        m2 = q >= 2 ? ~0u : 0u;
        m3 = q >= 3 ? ~0u : 0u;
        // zeros around the operands, digits past NL, carries into limbs 0 and 1
        for (int i = threadIdx.x; i < G::WORDS; i += 64 * WV) lds[i] = 0;
        __syncthreads();
    }
    PMK_DEV void table(const uint8_t *t) {
        wtab = t + 16 * G::NL;
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            if constexpr (RES == KS) init[j] = load_init(j);
#pragma unroll
            for (int s = 0; s < RES; ++s) w[j][s] = load_w(j, s);
        }
    }
    PMK_DEV v4i load_w(int j, int s) const {
        return *(global_v4i *)((global_u8 *)fresh(wtab + (size_t)((m0 + j) * KS + s) * 1024) + (uint32_t)lane * 16);
    }
    PMK_DEV v4i load_init(int j) const {
        return *(global_v4i *)((global_u8 *)fresh(wtab - 16 * G::NL + 64 * (m0 + j)) + (uint32_t)q * 16);
    }
    // the lane's limbs into the four copies of operand buffer `at`
    PMK_DEV void operand(int at, const uint32_t (&x)[CM]) {
        uint32_t *p = lds + at + n * G::SN + 4 * m0 + q + 3;
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
#pragma unroll
            for (int c = 0; c < 4; ++c) p[4 * j + c * (G::CP - 1)] = x[j];
        }
    }
    template <int W, bool SQR>
    PMK_DEV void columns(uint64_t (&lo)[CM], uint64_t (&hi)[CM]) {
        if constexpr (W < WV) {
            if (W == WV - 1 || wave == W) {
                const u4 *a = (const u4 *)(lds + G::X + n * G::SN + 3 * G::CP);
                const u4 *v = (const u4 *)(lds + (SQR ? G::X : G::Y) + n * G::SN + q * G::CP);
                if constexpr (W * CM < G::NM) {
                    if constexpr (SQR) group_columns_sqr<CB, WV, W>(lo, hi, a, v, m1, m2, m3);
                    else group_columns<CB, WV, W>(lo, hi, a, v);
                }
            } else {
                columns<W + 1, SQR>(lo, hi);
            }
        }
    }
    // X times Y (sqr: X squared): xl, xh = this lane's limbs of the two halves
    PMK_DEV void product(bool sqr, uint32_t (&xl)[CM], uint32_t (&xh)[CM]) {
        uint64_t lo[CM], hi[CM];
#pragma unroll
        for (int j = 0; j < CM; ++j) lo[j] = hi[j] = 0;
        if (sqr) columns<0, true>(lo, hi);
        else columns<0, false>(lo, hi);
        // a column's carries, at rows k + 2 of P: (carry to k + 1, carry to k + 2)
        uint2 *p = (uint2 *)(lds + G::P) + (4 * m0 + q + 2) * 16 + n;
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            const uint64_t cl = lo[j] >> G::LB, ch = hi[j] >> G::LB;
            p[64 * j] = make_uint2((uint32_t)cl & G::MASK, (uint32_t)(cl >> G::LB));
            p[64 * j + 16 * G::NL] =
                // the last column that has products hands all its carry to the top limb
                make_uint2((uint32_t)ch & (holds_top(j, 2) ? ~0u : G::MASK), (uint32_t)(ch >> G::LB));
        }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            xl[j] = ((uint32_t)lo[j] & G::MASK) + p[64 * j - 16].x + p[64 * j - 32].y;
            xh[j] = ((uint32_t)hi[j] & G::MASK) + p[64 * j + 16 * G::NL - 16].x + p[64 * j + 16 * G::NL - 32].y;
        }
    }
    // own = xl + 2^F xh mod m, into X as well
    PMK_DEV void fold(const uint32_t (&xl)[CM], const uint32_t (&xh)[CM]) {
        v4i acc[CM];
        uint32_t *d = lds + G::D + n * G::DS;
        auto digits = [&] {
#pragma unroll
            for (int j = 0; j < CM; ++j) {
                if (skip(j)) break;
                d[limb(j)] = (xh[j] + kDigitBias) ^ kDigitBias;
            }
        };
        auto mfma = [&](int s, auto a) {  // a(j): W's operand of row tile j, K step s
            const v4i x = *(const v4i *)(d + 16 * s + 4 * q);
#pragma unroll
            for (int j = 0; j < CM; ++j) {
                if (skip(j)) break;
                acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a(j), x, acc[j], 0, 0, 0);
            }
        };
        if constexpr (RES == KS) {
            digits();
            lds_barrier();
#pragma unroll
            for (int j = 0; j < CM; ++j) acc[j] = init[j];
#pragma unroll
            for (int s = 0; s < KS; ++s) mfma(s, [&](int j) { return w[j][s]; });
        } else {
            constexpr int CH = G::CHUNK;  // streamed K steps in flight
            v4i ws[2][CM][CH];
            auto stream = [&](int c) {  // steps RES + c CH ..
#pragma unroll
                for (int j = 0; j < CM; ++j) {
                    if (skip(j)) break;
#pragma unroll
                    for (int s = 0; s < CH; ++s)
                        if (RES + c * CH + s < KS) ws[c & 1][j][s] = load_w(j, RES + c * CH + s);
                }
            };
            stream(0);
#pragma unroll
            for (int j = 0; j < CM; ++j) {
                if (skip(j)) break;
                acc[j] = load_init(j);
            }
            digits();
            lds_barrier();
#pragma unroll
            for (int s = 0; s < RES; ++s) mfma(s, [&](int j) { return w[j][s]; });
#pragma unroll
            for (int s = 0; s < KS - RES; ++s) {
                if (s % CH == 0 && s + CH < KS - RES) stream(s / CH + 1);
                mfma(RES + s, [&](int j) { return ws[s / CH & 1][j][s % CH]; });
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        uint32_t *cr = lds + G::C + (4 * m0 + q) * 16 + n;
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            const uint32_t u = (uint32_t)acc[j][0] + ((uint32_t)acc[j][1] << 8);
            const uint32_t v = (uint32_t)acc[j][2] + ((uint32_t)acc[j][3] << 8);
            const uint64_t x = (((uint64_t)v << 16) + u) + xl[j];
            own[j] = (uint32_t)x & (holds_top(j, 3) ? ~0u : G::MASK);
            cr[64 * j + 16] = (uint32_t)(x >> G::LB);
        }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            own[j] += cr[64 * j];
        }
        operand(G::X, own);
        lds_barrier();
    }
    // table entries in global memory: [limb][16 chunks]
    PMK_DEV void store(uint32_t *t, int e, const uint32_t (&x)[CM]) const {
        global_u32 *p = (global_u32 *)fresh(t + ((size_t)e * G::NL + 4 * m0) * 16);
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            p[(uint32_t)lane + 64 * j] = x[j];
        }
    }
    PMK_DEV void load(uint32_t (&x)[CM], const uint32_t *t, int e) const {
        global_u32 *p = (global_u32 *)fresh((uint32_t *)t + ((size_t)e * G::NL + 4 * m0) * 16);
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            x[j] = p[(uint32_t)lane + 64 * j];
        }
    }
    // the same of the number of S words at src (stride kTile)
    template <int S>
    PMK_DEV void words(const uint32_t *src, uint32_t (&xl)[CM], uint32_t (&xh)[CM]) {
        auto limb_at = [&](int k) -> uint32_t {
            const int bit = G::LB * k, i = bit >> 5, sh = bit & 31;
            const uint32_t a = i < S ? src[(size_t)i * kTile] : 0u, b = i + 1 < S ? src[(size_t)(i + 1) * kTile] : 0u;
            return (uint32_t)((((uint64_t)b << 32) | a) >> sh) & G::MASK;
        };
#pragma unroll
        for (int j = 0; j < CM; ++j) {
            if (skip(j)) break;
            xl[j] = limb_at(limb(j));
            xh[j] = limb_at(G::NL + limb(j));
            __builtin_amdgcn_sched_barrier(0);  // few addresses at a time
        }
    }
};

// Job (tile, prime h), 16 chunks from `part`: r.half = c^d mod m as a fold result.
template <int CB, int WV>
PMK_DEV void halves_group_unit(Group<CB, WV> &g, const ClassRun &r, uint32_t tile, int h, int part, uint32_t *tbl) {
    using GS = GroupShape<CB, WV>;
    constexpr Geom G = make_geom(CB);
    constexpr int S = G.S, SH = G.SH;
    const int win = r.win, TH = 1 << (win - 1);
    const uint32_t key = uni(r.tile_key[tile]);
    const uint32_t *dexp = r.keys + (size_t)key * G.stride + G.off_half[0] + h * G.h_size + G.h_d;
    uint32_t xl[GS::CM], xh[GS::CM];
    g.template words<S>(r.x32 + (size_t)tile * S * kTile + 16 * part + g.n, xl, xh);
    __builtin_amdgcn_sched_barrier(0);
    g.table(r.fold + (size_t)(2 * key + h) * fold_table(CB).size + fold_table(CB).group);
    // the table's loads end here, so that waiting for them inside the loop never
    // means waiting for a window's entry
    __builtin_amdgcn_s_waitcnt(0);
    // One call site for the product and the fold.  Phases, what the pass computes:
    //   0 c mod m (entry 0)   1 x^2, the step between odd powers
    //   2 entry e = x^(2e+1)  3 the window's squares   4 times the window's entry
    int phase = 0, e = 1, sq = 0;
    uint32_t y[GS::CM];
    WinStep st = WinStep::make(0, 0u, false, -1);
    ExpWords nx{0u, 0u, 0u};
    for (;;) {
        if (phase != 0) g.product(phase == 1 || phase == 3, xl, xh);
        g.fold(xl, xh);
        if (phase == 0) {
            g.store(tbl, 0, g.own);
            phase = 1;
            continue;
        }
        if (phase == 1) {
            g.operand(GS::Y, g.own);
            g.load(g.own, tbl, 0);
            g.operand(GS::X, g.own);
            lds_barrier();
            phase = 2;
            continue;
        }
        if (phase == 2) {
            g.store(tbl, e, g.own);
            if (++e < TH) continue;
            // table complete: the first window starts at the top set bit; d = 0 gives 1
            const int top = exp_top_bit(dexp, SH);
            if (top < 0) {
#pragma unroll
                for (int j = 0; j < GS::CM; ++j) g.own[j] = g.limb(j) == 0;
                break;
            }
            st = win_first(nx, dexp, SH, top, win);
            g.load(g.own, tbl, (int)st.idx());
            g.operand(GS::X, g.own);
            lds_barrier();
            win_advance(st, nx, dexp, SH, win);
        } else if (phase == 4) {
            win_advance(st, nx, dexp, SH, win);
        }
        if (phase != 3) {  // a new step: its entry on its way while its squares run
            if (st.mul()) g.load(y, tbl, (int)st.idx());
            sq = st.nsq();
            phase = 3;
        } else {
            --sq;
        }
        if (sq == 0) {
            if (!st.mul()) break;
            g.operand(GS::Y, y);
            lds_barrier();
            phase = 4;
        }
    }
    uint32_t *dst = r.half + (size_t)(2 * tile + h) * half_stride(CB) * kTile + 16 * part + g.n;
#pragma unroll
    for (int j = 0; j < GS::CM; ++j) {
        if (g.skip(j)) break;
        dst[(size_t)g.limb(j) * kTile] = g.own[j];
    }
}

// first tile of group `first` (0: tile 0)
PMK_DEV uint32_t group_tile(const ClassRun &r, uint32_t first) {
    return first ? uni(r.groups[first]) & 0x3FFFFFFFu : 0u;
}

// Jobs (tile, h) over the tiles from that of group `first` on, each in four parts of 16
// chunks; parts without a chunk are skipped.  The grid takes a quarter of its blocks' number
// of jobs at a time, the blocks of a part one after another.  A job's parts then run
// on one die (blocks go to the eight dies by number), which keeps its table in L2
// (8192 bits, 64 keys with 64 chunks: 94 ms with the parts on four dies, 67), and where
// keys have up to 16 chunks each, and only part 0 is there, its blocks spread over all
// compute units.  A block's part turns from step to step, so that every block gets its
// share of them (256 keys with 16 chunks: 17.8 ms at 3072 bits, 31.9 at 4096 with a
// fixed part per block, 4.5 and 8.1 here).  The last step has fewer jobs.  Where tiles
// have most of their parts it takes the first blocks, which run ahead of the others and
// are spread over the compute units (18 keys with 300 chunks, 4096 bits: 13.1 ms, over all
// blocks 16.4); where they have two or less, a part stays in its quarter of the blocks,
// whose turn it is (100 keys with 25 chunks: 8.2 ms, in the first blocks 12.6).
template <int CB, int WV>
__global__ __launch_bounds__(64 * WV) __attribute__((amdgpu_waves_per_eu(fold_group_waves(CB)))) void halves_group_kernel(
    ClassRun r, uint64_t slot_words, uint32_t first) {
    __shared__ __align__(16) uint32_t lds[GroupShape<CB, WV>::WORDS];
    uint32_t *tbl = r.table + (size_t)blockIdx.x * slot_words;
    Group<CB, WV> g;
    g.setup(lds);
    const uint32_t t0 = group_tile(r, first), jobs = 2 * (r.ntiles - t0), some = gridDim.x < 4 ? 1 : gridDim.x / 4;
    const bool quarters = r.parts <= 2 * r.ntiles;
    for (uint32_t j0 = 0, k = 0; j0 < jobs; j0 += some, ++k) {  // parts turn by 0, 2, 1, 3
        const uint32_t left = (jobs - j0 + 7) & ~7u, n = left < some ? left : some;
        const uint32_t step = quarters ? some : n;
        for (uint32_t x = blockIdx.x; x < 4 * step; x += gridDim.x) {
            const uint32_t q = x / step, at = (x % step + q * (step - n)) % step;
            const uint32_t jt = j0 + at, tile = t0 + (jt >> 1);
            const int h = (int)(jt & 1), part = (int)(q + ((k & 1) << 1 | (k >> 1 & 1)) & 3);
            if (at >= n || jt >= jobs || !uni(r.desc[(size_t)tile * kTile + 16 * part].msg_len)) continue;
            halves_group_unit<CB, WV>(g, r, tile, h, part, tbl);
        }
    }
}

// Canonical halves from fold results of the 6144/8192-bit classes, whose
// numbers do not fit one lane: as fold_finish_unit, L lanes per number.
template <int CB, int L>
PMK_DEV void fold_finish_lanes_unit(const ClassRun &r, uint32_t u, uint32_t *lds) {
    constexpr Geom G = make_geom(CB);
    constexpr int FNL = fold_group(CB).nl, FLB = fold_group(CB).lb;
    constexpr int NLT = lane_limbs(G, L), K = NLT / L, LB = G.lbh, NG = 64 / L;
    constexpr int NW = (FLB * FNL + 32 + 31) / 32;  // words of a fold result
    static_assert(NW <= lds_words_lanes<CB, L>() / NG, "the words fit the staging column");
    const uint32_t jt = u / L;
    const int lane = threadIdx.x, pos = lane % L, grp = lane / L, c = (int)(u % L) * NG + grp;
    uint32_t *col = lds + grp;
    const uint32_t *hr = r.keys + (size_t)uni(r.tile_key[jt >> 1]) * G.stride + G.off_half[0] + (jt & 1) * G.h_size;
    uint32_t *io = r.half + (size_t)jt * half_stride(CB) * kTile + c;
    uint32_t n[K];
    load_limbs(n, fresh_v(hr + G.h_m + pos * K));
    const uint32_t n0 = uni(hr[G.h_m0]);
    if (pos == 0) {  // limbs into words, carries settled
        uint64_t acc = 0;
        int bits = 0, k = 0;
#pragma unroll 4
        for (int j = 0; j < FNL; ++j) {
            acc += (uint64_t)io[(size_t)j * kTile] << bits;
            bits += FLB;
            if (bits >= 32) {
                col[k++ * NG] = (uint32_t)acc;
                acc >>= 32;
                bits -= 32;
            }
        }
        for (; k < NW; ++k) {
            col[k * NG] = (uint32_t)acc;
            acc >>= 32;
        }
    }
    __syncthreads();
    uint32_t acc[K], x[K];
    limbs_from_words<K, LB>(acc, col, NG, NW, pos * K);
    limbs_from_words<K, LB>(x, col, NG, NW, NLT + pos * K);
    __syncthreads();
    stage_mem<K>(col, NG, pos, hr + lane_rr(G, L) + pos * K, 1);
#pragma unroll 1
    for (int step = 0; step < 3; ++step) {
        mont_mul_lanes<NLT, LB, L>(acc, acc, col, NG, n, n0, pos);
        if (step == 0) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t t = acc[j];
                acc[j] = x[j];
                x[j] = t;
            }
            stage_mem<K>(col, NG, pos, hr + lane_rrr(G, L) + pos * K, 1);
        } else if (step == 1) {
            uint32_t cy = 0;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t v = acc[j] + x[j] + cy;
                acc[j] = v & Radix<LB>::MASK;
                cy = v >> LB;
            }
#pragma unroll
            for (int s = 1; s < L; ++s) {
                uint32_t cin = grp_prev<L>(cy, pos);
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const uint32_t v = acc[j] + cin;
                    acc[j] = v & Radix<LB>::MASK;
                    cin = v >> LB;
                }
                cy = cin;
            }
            stage_one<K>(col, NG, pos);
        }
    }
    canonicalize_lanes<K, LB, L>(acc, n, pos);
    uint32_t *dst = io + (size_t)pos * K * kTile;
#pragma unroll
    for (int j = 0; j < K; ++j)
        if (NLT == G.nlh || pos * K + j < G.nlh) dst[(size_t)j * kTile] = acc[j];
}

// Canonical CRT halves from fold results: a block per job tile, or L blocks
// where numbers take L lanes (kFinishLanes), from the first tile of group
// `first` on, up to the tile before that of group `end` (0: the last tile).
template <int CB>
constexpr int kFinishLanes = lanes_half(CB) > 1 ? 8 : 1;
template <int CB, int FNL, int FLB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(make_geom(CB).nlh > 40 ? 1 : 2))) void fold_finish_kernel(
    ClassRun r, uint32_t first, uint32_t end) {
    const uint32_t u = blockIdx.x + 2 * kFinishLanes<CB> * group_tile(r, first);
    if (u / (2 * kFinishLanes<CB>) >= (end ? group_tile(r, end) : r.ntiles)) return;
    if constexpr (kFinishLanes<CB> > 1) {
        __shared__ uint32_t lds[lds_words_lanes<CB, kFinishLanes<CB>>()];
        fold_finish_lanes_unit<CB, kFinishLanes<CB>>(r, u, lds);
    } else {
        fold_finish_unit<CB, FNL, FLB>(r, u);
    }
}

}  // namespace pmk
