// CRT halves in the fold form with a number in one lane (fold.hpp): launches
// that fill the chip.  Included by kernels_impl.hpp after the helpers it uses.
//
// A block is two or four waves on as many tiles under one key, modulo one
// prime, sharing the prime's table in LDS (fold_lane_block).
//
// Bound by VALU issue and, at full load, by the chip's power.  2048-bit keys, the
// 12,288 jobs of the full rounds of 100 MiB: 48.3 ms, 64.4 with Montgomery
// products (2.08 against 3.80 x 10^10 VALU instructions; the matrix cores are
// 22 % busy, behind them).  16 MB: 4.9 / 4.5 ms at 1024 bits, 39.7 / 28.0 at 3072.
#pragma once

namespace pmk {

template <int CB>
struct FoldHalves {
    static constexpr FoldForm F = fold_lane(CB);
    using S = FoldShape<F.nl, F.lb>;
    static constexpr int WORDS = S::BYTES / 4;
    static constexpr int ROW4 = pad4(F.nl) * kTile;  // words of a prefetched table entry
};

// The fold of a number of 32-bit words: r = its value mod m.
template <int NL, int LB, int S32>
PMK_DEV void fold_words(uint32_t (&r)[NL], const uint32_t *w, FoldLds f, int lane) {
    using O = FoldOrder<NL, LB, true>;
    static_assert(LB * 2 * NL >= 32 * S32, "two halves hold the number");
    constexpr int PER = 2 * O::S::STEPS;  // MFMAs of a row tile
    Folder<NL, LB, O> fo(f, lane);
    static_for<0, NL>([&](auto i) { fo.template high<i()>(radix_limb_mem<S32, LB>(w, kTile, NL + i())); });
    uint64_t acc = 0;
    static_for<0, NL>([&](auto k) {
        if constexpr (k() % 8 == 0)  // the MFMAs of this limb's tile
            static_for<k() == 0 ? 0 : (k() == 8 ? 2 * PER : PER * (k() / 8)), k() == 8 ? 2 * PER : (k() == 0 ? 2 : k() / 8 + 1) * PER>(
                [&](auto n) { fo.template mfma<n()>(); });
        uint32_t u, v;
        fo.template low<k()>(u, v);
        acc += (uint64_t)v << 16;
        acc += (uint64_t)u + radix_limb_mem<S32, LB>(w, kTile, k());
        r[k()] = k() < NL - 1 ? (uint32_t)acc & Radix<LB>::MASK : (uint32_t)acc;
        acc >>= LB;
    });
}

// Job (tile, prime h): r.half = c^d mod m as a fold result, by sliding windows
// over the odd powers.  The window loop is that of halves_unit; nothing
// enters or leaves Montgomery form.
template <int CB>
PMK_DEV void halves_fold_unit(const ClassRun &r, uint32_t tile, int h, uint32_t *tbl, FoldLds f, uint32_t *lds) {
    constexpr Geom G = make_geom(CB);
    constexpr int NL = fold_lane(CB).nl, LB = fold_lane(CB).lb, S = G.S, SH = G.SH;
    const int win = r.win;
    const int lane = threadIdx.x & 63;
    const uint32_t *kr = r.keys + (size_t)uni(r.tile_key[tile]) * G.stride;  // wave-uniform
    const uint32_t *dexp = kr + G.off_half[0] + h * G.h_size + G.h_d;
    uint32_t one = 1, k16 = 1u << 16;
    asm volatile("" : "+s"(one), "+s"(k16));

    uint32_t acc[NL], b[NL], x[NL];
    fold_words<NL, LB, S>(acc, fresh_v(r.x32 + (size_t)tile * S * kTile + lane), f, lane);
    store_row4(tbl, 0, lane, acc);
#pragma unroll
    for (int j = 0; j < NL; ++j) b[j] = acc[j];
    __builtin_amdgcn_s_waitcnt(0);
    // phases: 2 x^2 (the step between odd powers), 5 entry e = x^(2e+1), 3 the windows
    const int TH = 1 << (win - 1);
    int phase = 2, e = 1, sq = 0;
    WinStep st = WinStep::make(0, 0u, false, -1);
    ExpWords nx{0u, 0u, 0u};
    for (;;) {
        if (phase == 3) {
            if (sq < st.nsq()) {
                if (fold_lane_prefetch(CB) && sq == 0 && st.mul()) prefetch_row4<NL>(lds, tbl, st.idx(), lane);
#pragma unroll
                for (int j = 0; j < NL; ++j) b[j] = acc[j] << 1;
                fold_mul<NL, LB, true>(x, acc, b, f, lane, one, k16);
#pragma unroll
                for (int j = 0; j < NL; ++j) acc[j] = x[j];
                ++sq;
                continue;
            }
            if (!st.mul()) break;
            if constexpr (fold_lane_prefetch(CB)) take_row4(b, lds, lane);
            else load_row4(b, tbl, st.idx(), lane);
        }
        fold_mul<NL, LB, false>(x, acc, b, f, lane, one, k16);
#pragma unroll
        for (int j = 0; j < NL; ++j) acc[j] = x[j];
        if (phase == 2) {
#pragma unroll
            for (int j = 0; j < NL; ++j) b[j] = acc[j];  // x^2, the multiplier of phase 5
            load_row4(acc, tbl, 0, lane);
            phase = 5;
            __builtin_amdgcn_s_waitcnt(0);
            continue;
        }
        if (phase == 5) {
            store_row4(tbl, e, lane, acc);
            ++e;
            __builtin_amdgcn_s_waitcnt(0);
            if (e < TH) continue;
            // table complete: the first window starts at the top set bit; d = 0 gives 1
            const int top = exp_top_bit(dexp, SH);
            if (top < 0) {
#pragma unroll
                for (int j = 0; j < NL; ++j) acc[j] = j == 0 ? 1u : 0u;
                st = WinStep::make(0, 0u, false, -1);
            } else {
                st = win_first(nx, dexp, SH, top, win);
                load_row4(acc, tbl, st.idx(), lane);
                win_advance(st, nx, dexp, SH, win);
            }
            __builtin_amdgcn_s_waitcnt(0);
            phase = 3;
            sq = 0;
            continue;
        }
        win_advance(st, nx, dexp, SH, win);
        sq = 0;
    }
    uint32_t *dst = r.half + ((size_t)(2 * tile + h) * half_stride(CB)) * kTile + lane;
#pragma unroll
    for (int j = 0; j < NL; ++j) dst[(size_t)j * kTile] = acc[j];
}

// a = a + R c mod m, below 2m (R = 2^(LB NL)): MM(a, R^2) + MM(c, R^3) = x R (below 4m), then a
// product by 1; one call site.
template <int NL, int LB>
PMK_DEV void reduce_two(uint32_t (&a)[NL], uint32_t (&b)[NL], uint32_t (&c)[NL], const uint32_t (&n)[NL],
                        const uint32_t *hr, int off_rr, int off_rrr, uint32_t n0) {
    load_limbs(b, hr + off_rr);
#pragma unroll 1
    for (int step = 0; step < 3; ++step) {
        mont_mul<NL, LB>(a, a, b, n, n0);
        if (step == 0) {
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const uint32_t t = a[j];
                a[j] = c[j];
                c[j] = t;
            }
            load_limbs(b, hr + off_rrr);
        } else if (step == 1) {
            uint32_t cy = 0;
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const uint32_t v = a[j] + c[j] + cy;
                a[j] = v & Radix<LB>::MASK;
                cy = v >> LB;
                b[j] = j == 0 ? 1u : 0u;
            }
        }
    }
}

// Blinded decryption, job (tile, prime h): (c*)^d c_R^(m-1-d) mod m in one
// chain, the interleaved sliding windows of halves_joint_unit on fold products.
// c* from r.x32, c_R from r.fin32 (whether m divides c_R: blind_check_kernel).
template <int CB>
PMK_DEV void halves_fold_joint_unit(const ClassRun &r, uint32_t tile, int h, uint32_t *tbl, FoldLds f, uint32_t *lds) {
    constexpr Geom G = make_geom(CB);
    constexpr int NL = fold_lane(CB).nl, LB = fold_lane(CB).lb, S = G.S, SH = G.SH;
    const int win = r.win, TH = 1 << (win - 1);  // T1 = entries [0, TH), T2 = [TH, 2 TH)
    const int lane = threadIdx.x & 63;
    const uint32_t *hr = r.keys + (size_t)uni(r.tile_key[tile]) * G.stride + G.off_half[0] + h * G.h_size;
    const uint32_t *d1 = hr + G.h_d, *d2 = hr + G.h_d2;
    uint32_t one = 1, k16 = 1u << 16;
    asm volatile("" : "+s"(one), "+s"(k16));

    uint32_t acc[NL], b[NL], x[NL];
    fold_words<NL, LB, S>(acc, fresh_v(r.x32 + (size_t)tile * S * kTile + lane), f, lane);
    store_row4(tbl, 0, lane, acc);
#pragma unroll
    for (int j = 0; j < NL; ++j) b[j] = acc[j];
    __builtin_amdgcn_s_waitcnt(0);
    // phases: 2 x^2, 3 odd powers (of c*, k = 0, then of c_R, k = 1), 5 the chain
    int phase = 2, k = 0, e = 1, sq = 0, nsq = 0, pos = 0;
    uint32_t pend = 0;
    WinStep s1 = WinStep::make(0, 0u, false, -1), s2 = s1;
    ExpWords nx1{0u, 0u, 0u}, nx2{0u, 0u, 0u};
    for (;;) {
        if (phase == 5) {
            const uint32_t ent = (pend & 1u) ? s1.idx() : TH + s2.idx();  // the event's first product
            if (sq < nsq) {
                if (fold_lane_prefetch(CB) && sq == 0 && pend) prefetch_row4<NL>(lds, tbl, ent, lane);
#pragma unroll
                for (int j = 0; j < NL; ++j) b[j] = acc[j] << 1;
                fold_mul<NL, LB, true>(x, acc, b, f, lane, one, k16);
#pragma unroll
                for (int j = 0; j < NL; ++j) acc[j] = x[j];
                ++sq;
                continue;
            }
            if (!pend) break;
            if (fold_lane_prefetch(CB) && sq == nsq) take_row4(b, lds, lane);
            else load_row4(b, tbl, sq == nsq ? ent : TH + s2.idx(), lane);  // windows of both exponents end here: T2 second
            __builtin_amdgcn_s_waitcnt(0);
            ++sq;
        }
        fold_mul<NL, LB, false>(x, acc, b, f, lane, one, k16);
#pragma unroll
        for (int j = 0; j < NL; ++j) acc[j] = x[j];
        const int base = k * TH;
        if (phase == 2) {
#pragma unroll
            for (int j = 0; j < NL; ++j) b[j] = acc[j];  // x^2, the step between odd powers
            load_row4(acc, tbl, base, lane);
            phase = 3;
            e = 1;
            __builtin_amdgcn_s_waitcnt(0);
            continue;
        }
        if (phase == 3) {
            store_row4(tbl, base + e, lane, acc);
            ++e;
            __builtin_amdgcn_s_waitcnt(0);
            if (e < TH) continue;
            if (k == 0) {  // c_R next
                k = 1;
                fold_words<NL, LB, S>(acc, fresh_v(r.fin32 + (size_t)tile * S * kTile + lane), f, lane);
                store_row4(tbl, TH, lane, acc);
#pragma unroll
                for (int j = 0; j < NL; ++j) b[j] = acc[j];
                phase = 2;
                __builtin_amdgcn_s_waitcnt(0);
                continue;
            }
            // tables complete: the chain starts from 1 above the higher top bit
#pragma unroll
            for (int j = 0; j < NL; ++j) acc[j] = j == 0 ? 1u : 0u;
            const int t1 = exp_top_bit(d1, SH), t2 = exp_top_bit(d2, SH);
            if (t1 >= 0) s1 = win_first(nx1, d1, SH, t1, win);
            if (t2 >= 0) s2 = win_first(nx2, d2, SH, t2, win);
            pos = (t1 > t2 ? t1 : t2) + 1;
            phase = 5;
        } else if (sq == nsq + 1 && pend == 3u) {
            continue;  // the T1 product is done, the T2 product of the same event follows
        } else {  // the event's products are done
            if (pend & 1u) win_advance(s1, nx1, d1, SH, win);
            if (pend & 2u) win_advance(s2, nx2, d2, SH, win);
        }
        // next event: the higher window end still pending (window [l, ...], l = next + 1)
        const int l1 = s1.mul() ? s1.next() + 1 : -1, l2 = s2.mul() ? s2.next() + 1 : -1;
        const int ev = l1 > l2 ? l1 : l2;
        pend = ev < 0 ? 0u : (l1 == ev ? 1u : 0u) | (l2 == ev ? 2u : 0u);
        nsq = pos - (ev < 0 ? 0 : ev);  // no window left: square down to bit 0
        pos = ev < 0 ? 0 : ev;
        sq = 0;
    }
    uint32_t *dst = r.half + ((size_t)(2 * tile + h) * half_stride(CB)) * kTile + lane;
#pragma unroll
    for (int j = 0; j < NL; ++j) dst[(size_t)j * kTile] = acc[j];
}

// Sets bit 1 of r.err where a prime divides a chunk's c_R (r.fin32): c_R mod m as
// fold_finish_unit computes it, 0 or m.  Block jt = job tile.
template <int CB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(make_geom(CB).nlh > 40 ? 1 : 2))) void blind_check_kernel(
    ClassRun r) {
    constexpr Geom G = make_geom(CB);
    constexpr int NL = G.nlh, LB = G.lbh, S = G.S;
    const uint32_t jt = blockIdx.x, tile = jt >> 1;
    const int lane = threadIdx.x;
    const uint32_t *hr = r.keys + (size_t)uni(r.tile_key[tile]) * G.stride + G.off_half[0] + (jt & 1) * G.h_size;
    const uint32_t *w = r.fin32 + (size_t)tile * S * kTile + lane;
    uint32_t n[NL], a[NL], b[NL], c[NL];
    load_uniform(n, hr + G.h_m);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        a[j] = radix_limb_mem<S, LB>(w, kTile, j);
        c[j] = radix_limb_mem<S, LB>(w, kTile, NL + j);
    }
    reduce_two<NL, LB>(a, b, c, n, hr, G.h_rr, G.h_rrr, uni(hr[G.h_m0]));
    uint32_t z = 0, q = 0;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        z |= a[j];
        q |= a[j] ^ n[j];
    }
    if ((z == 0 || q == 0) && r.desc[(size_t)tile * kTile + lane].msg_len) atomicOr(r.err, 2u);
}

// Units [u_begin, u_end): u = 2 group + h, one wave per tile of the group (fewer
// waves than tiles: each takes several).  split: units are single tiles instead,
// u = 2 (per group + tile of the group) + h, for blocks of one wave (launches
// that leave SIMDs idle: one-wave blocks spread over the four SIMDs of a compute
// unit, two-wave blocks were measured two deep on half of them, 5.0 against
// 3.5 us per 2048-bit square with a wave per SIMD).
template <int CB, bool JOINT = false>
PMK_DEV void halves_fold_block(const ClassRun &r, uint64_t slot_words, uint32_t u_begin, uint32_t u_end, bool split,
                               uint32_t *table, uint32_t *entry) {
    constexpr uint32_t per = fold_lane_block(CB);
    const int nw = blockDim.x / 64, wave = (int)uni(threadIdx.x / 64);
    uint32_t *tbl = r.table + ((size_t)blockIdx.x * nw + wave) * slot_words;
    for (uint32_t u = u_begin + blockIdx.x; u < u_end; u += gridDim.x) {
        const uint32_t grp = uni(r.groups[split ? (u >> 1) / per : u >> 1]), first = grp & 0x3FFFFFFFu;
        const int h = u & 1, tiles = 1 + (int)(grp >> 30), t0 = split ? (int)((u >> 1) % per) : wave;
        if (split && t0 >= tiles) continue;
        const uint4 *src = (const uint4 *)(r.fold + (size_t)(2 * uni(r.tile_key[first]) + h) * fold_table(CB).size +
                                           fold_table(CB).lane);
        __syncthreads();  // the waves still read the last unit's table
        for (int i = threadIdx.x; i < FoldHalves<CB>::WORDS / 4; i += blockDim.x) ((uint4 *)table)[i] = src[i];
        __syncthreads();
        // a wave without a tile in its block's last unit ends: its registers go to
        // other launches' waves
        if (t0 >= tiles && u + gridDim.x >= u_end) return;
        for (int t = t0; t < (split ? t0 + 1 : tiles); t += nw) {
            uint32_t *ent = entry + (fold_lane_prefetch(CB) ? wave * FoldHalves<CB>::ROW4 : 0);
            if constexpr (JOINT) halves_fold_joint_unit<CB>(r, first + t, h, tbl, FoldLds{(const uint8_t *)table}, ent);
            else halves_fold_unit<CB>(r, first + t, h, tbl, FoldLds{(const uint8_t *)table}, ent);
        }
    }
}

// Blocks of the lane form's kernel fn resident on a compute unit, by their waves:
// a block's table takes its LDS whatever its waves, and its waves their SIMDs
// together (4096 bits: 256 blocks of three waves at a time on 256 compute units,
// where 1,024 waves / 3 = 341 dealt 512 units in three rounds, 88 ms, for two).
template <int CB>
struct FoldBlocks {
    uint32_t n[fold_lane_block(CB) + 1] = {};
    explicit FoldBlocks(const void *fn) {
        for (int w = 1; w <= fold_lane_block(CB); ++w) {
            int nb = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64 * w, 0) != hipSuccess || nb < 1) nb = 1;
            n[w] = (uint32_t)nb;
        }
    }
    // blocks of nw waves, at most `waves` waves
    uint32_t resident(uint32_t nw, uint32_t waves, uint32_t cus) const {
        const uint32_t b = n[nw] * cus;
        return b < waves / nw ? b : waves / nw;
    }
};

// Launches of groups of one tile each, in blocks of one wave: one launch per round
// of a wave per SIMD (1024 bits: two), which an idle chip places evenly; in one
// launch later blocks land where one ends, some SIMDs two deep (2,048 jobs of
// 2048 bits: 12.5 ms in one launch, 8.9 here).
template <int CB, typename Launch>
int lone_rounds(uint32_t units, uint32_t grid, uint32_t cus, Launch launch) {
    const uint32_t even = (CB > 1024 ? 4 : 8) * cus, round = grid < even ? grid : even;
    int e = 0;
    for (uint32_t u = 0; u < units && !e; u += round) e = launch(u, units - u < round ? units : u + round);
    return e;
}

// The partial round after full ones, as blocks of two units (group, h): four waves,
// one on each SIMD, which blocks of one or two waves do not ensure after the full
// rounds (1,024 2048-bit jobs: 7.2 ms in blocks of one wave, some SIMDs two deep, 4.6
// ms here; 15 MB under 1024-bit keys 4.46 / 3.90 ms; from an idle chip blocks of one
// wave are as even and 3 to 7 % faster).  table and entry hold two tables and four rows,
// and fill LDS so that one block fewer fits a compute unit than the class has waves per SIMD.
template <int CB>
struct FoldQuad {
    static constexpr int WORDS = 2 * FoldHalves<CB>::WORDS;
    static constexpr int ROWS = 4 * FoldHalves<CB>::ROW4, FILL = (160 / fold_lane_waves(CB) + 1) * 256;  // words
    static constexpr int ENTRY = WORDS + ROWS > FILL ? ROWS : FILL - WORDS;
};
template <int CB, bool JOINT = false>
PMK_DEV void halves_fold_quad(const ClassRun &r, uint64_t slot_words, uint32_t u_begin, uint32_t u_end, uint32_t *table,
                              uint32_t *entry) {
    const int wave = (int)uni(threadIdx.x / 64), team = wave >> 1;
    const uint32_t u = u_begin + 2 * blockIdx.x + team;
    table += team * FoldHalves<CB>::WORDS;
    uint32_t grp = 0;
    if (u < u_end) {
        grp = uni(r.groups[u >> 1]);
        const uint4 *src = (const uint4 *)(r.fold +
                                           (size_t)(2 * uni(r.tile_key[grp & 0x3FFFFFFFu]) + (u & 1)) * fold_table(CB).size +
                                           fold_table(CB).lane);
        for (int i = threadIdx.x & 127; i < FoldHalves<CB>::WORDS / 4; i += 128) ((uint4 *)table)[i] = src[i];
    }
    __syncthreads();
    if (u >= u_end || (uint32_t)(wave & 1) > grp >> 30) return;
    const uint32_t tile = (grp & 0x3FFFFFFFu) + (wave & 1);
    uint32_t *tbl = r.table + ((size_t)blockIdx.x * 4 + wave) * slot_words, *ent = entry + wave * FoldHalves<CB>::ROW4;
    if constexpr (JOINT) halves_fold_joint_unit<CB>(r, tile, u & 1, tbl, FoldLds{(const uint8_t *)table}, ent);
    else halves_fold_unit<CB>(r, tile, u & 1, tbl, FoldLds{(const uint8_t *)table}, ent);
}
template <int CB, bool JOINT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(JOINT ? fold_joint_waves(CB) : fold_lane_waves(CB)))) void halves_quad_kernel(
    ClassRun r, uint64_t slot_words, uint32_t u_begin, uint32_t u_end) {
    __shared__ __align__(16) uint32_t table[FoldQuad<CB>::WORDS];
    __shared__ __align__(16) uint32_t entry[FoldQuad<CB>::ENTRY];
    halves_fold_quad<CB, JOINT>(r, slot_words, u_begin, u_end, table, entry);
}

// Canonical halves from fold results (nl limbs of lb bits, loose), in place.
// One lane per number.
template <int CB, int FNL, int FLB>
PMK_DEV void fold_finish_unit(const ClassRun &r, uint32_t jt) {
    constexpr Geom G = make_geom(CB);
    constexpr int NL = G.nlh, LB = G.lbh;
    const int lane = threadIdx.x;
    const uint32_t *hr = r.keys + (size_t)uni(r.tile_key[jt >> 1]) * G.stride + G.off_half[0] + (jt & 1) * G.h_size;
    uint32_t *io = r.half + (size_t)jt * half_stride(CB) * kTile + lane;
    uint32_t x[FNL + 1];
    uint32_t cy = 0;
#pragma unroll
    for (int j = 0; j < FNL; ++j) {
        const uint32_t v = io[(size_t)j * kTile] + cy;
        x[j] = v & ((1u << FLB) - 1u);
        cy = v >> FLB;
    }
    x[FNL] = cy;
    auto limb = [&](int j) -> uint32_t {
        const int at = LB * j, k = at / FLB, sh = at % FLB;
        const uint64_t lo = k <= FNL ? x[k <= FNL ? k : 0] : 0u, hi = k + 1 <= FNL ? x[k + 1 <= FNL ? k + 1 : 0] : 0u;
        return (uint32_t)((lo | hi << FLB) >> sh) & Radix<LB>::MASK;
    };
    uint32_t n[NL], a[NL], b[NL], c[NL];
    load_uniform(n, hr + G.h_m);
    const uint32_t n0 = uni(hr[G.h_m0]);
#pragma unroll
    for (int j = 0; j < NL; ++j) a[j] = limb(j);
#pragma unroll
    for (int j = 0; j < NL; ++j) c[j] = limb(NL + j);
    reduce_two<NL, LB>(a, b, c, n, hr, G.h_rr, G.h_rrr, n0);
    canonicalize<NL, LB>(a, n);
#pragma unroll
    for (int j = 0; j < NL; ++j) io[(size_t)j * kTile] = a[j];
}

}  // namespace pmk
