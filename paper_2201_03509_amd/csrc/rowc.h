// Row lengths of the FFT row pass that have kernels compiled for them, and
// the stage plan of each (host and device): three radices, chosen at compile
// time, whose product is the row length L.
//
// Stage s of a length-L Stockham FFT with radix R_s, Ns = R_0 ... R_{s-1}:
// butterfly j (j < L/R) takes x[j + t L/R], t < R, multiplies input t by
// w_{Ns R}^(t (j mod Ns)), transforms, and writes y[(j / Ns) Ns R + j mod Ns
// + t Ns].  The twiddles of the stages s >= 1 sit in one table per row length:
// stage s, entry (k, t) at stage_off(L, s) + k (R_s - 1) + t - 1, the forward
// value e^(-2 pi i t k / (Ns R_s)) (the inverse transform uses its conjugate).
#pragma once

// every 5-smooth length in [2000, 5040] (the longest row the row pass takes)
#define C3_ROWC_LIST(X)                                                                          \
    X(2000) X(2025) X(2048) X(2160) X(2187) X(2250) X(2304) X(2400) X(2430) X(2500) X(2560)     \
    X(2592) X(2700) X(2880) X(2916) X(3000) X(3072) X(3125) X(3200) X(3240) X(3375) X(3456)     \
    X(3600) X(3645) X(3750) X(3840) X(3888) X(4000) X(4050) X(4096) X(4320) X(4374) X(4500)     \
    X(4608) X(4800) X(4860) X(5000)

// FP64: every 5-smooth length in [1200, 2400], in three stages of radix at most
// 16 (a butterfly of 16 complex FP64 points takes 64 of a thread's 128 registers)
// or, where there are none, in four.  Two rows of 2400 points and the tables of
// the mode arithmetic are 80 KB, two blocks to a CU.
#define C3_ROWD_LIST(X)                                                                          \
    X(1200) X(1215) X(1250) X(1280) X(1296) X(1350) X(1440) X(1458) X(1500) X(1536) X(1600)     \
    X(1620) X(1728) X(1800) X(1875) X(1920) X(1944) X(2000) X(2025) X(2048) X(2160) X(2187)     \
    X(2250) X(2304) X(2400)

// FP64, short rows: the lengths in [160, 512] with three radices of 4 to 10, for
// segments of some thousand samples.  Long rows would leave them a handful of
// blocks (a transform of 4096 points had two, of 2048).
#define C3_ROWS_LIST(X)                                                                          \
    X(160) X(180) X(192) X(200) X(216) X(225) X(240) X(250) X(256) X(270) X(288) X(300) X(320)  \
    X(324) X(360) X(384) X(400) X(405) X(432) X(450) X(480) X(486) X(500) X(512)

namespace c3rowc {

// radices of a stage: 5-smooth, small enough that a butterfly's points fit a
// thread's registers
constexpr int kRadix[] = {4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32};
constexpr int kNRadix = sizeof(kRadix) / sizeof(kRadix[0]);

constexpr bool radix_ok(int r) {
    for (int i = 0; i < kNRadix; ++i)
        if (kRadix[i] == r) return true;
    return false;
}

struct Plan {
    int r[4];  // r[0] == 0: no plan; three stages (r[3] == 1) or four
};

// lanes of a butterfly's writes that share an LDS bank group: in the first
// stage its points lie R pairs of 32 bytes apart, and 8 pairs span the banks
constexpr int bank_share(int r) { return r % 8 == 0 ? 8 : r % 4 == 0 ? 4 : r % 2 == 0 ? 2 : 1; }

// the three-radix split of L with the smallest largest radix (ties: the
// largest smallest radix), in descending order.  FP64: radices of at most 16,
// four where no three will do, the one with the fewest lanes to a bank group
// first.
constexpr Plan plan(int L, bool f64 = false) {
    Plan best{{0, 0, 0, 1}};
    int bmax = f64 ? 17 : 1 << 30, bmin = 0;
    for (int last = 1; last <= (f64 ? 6 : 1) && best.r[0] == 0; ++last) {
        if (L % last) continue;
        for (int i = 0; i < kNRadix; ++i) {
            const int a = kRadix[i], LL = L / last;
            if (LL % a) continue;
            for (int j = 0; j < kNRadix; ++j) {
                const int b = kRadix[j];
                if ((LL / a) % b) continue;
                const int c = LL / a / b;
                if (!radix_ok(c)) continue;
                const int mx = a > b ? (a > c ? a : c) : (b > c ? b : c);
                const int mn = a < b ? (a < c ? a : c) : (b < c ? b : c);
                if (mx < bmax || (mx == bmax && mn > bmin)) {
                    bmax = mx;
                    bmin = mn;
                    const int md = a + b + c - mx - mn;
                    best = Plan{{mx, md, mn, last}};
                }
            }
        }
    }
    if (f64) {
        for (int i = 1; i < 3; ++i)
            if (bank_share(best.r[i]) < bank_share(best.r[0])) {
                const int t = best.r[0];
                best.r[0] = best.r[i];
                best.r[i] = t;
            }
    }
    return best;
}
constexpr int stages(int L, bool f64) { return plan(L, f64).r[3] > 1 ? 4 : 3; }

constexpr int row_ns(int L, int s, bool f64 = false) {
    const Plan p = plan(L, f64);
    int ns = 1;
    for (int i = 0; i < s; ++i) ns *= p.r[i];
    return ns;
}

// offset of stage s's twiddles (s >= 1) in the length's table
constexpr long stage_off(int L, int s, bool f64 = false) {
    const Plan p = plan(L, f64);
    long off = 0;
    for (int i = 1; i < s; ++i) off += (long)row_ns(L, i, f64) * (p.r[i] - 1);
    return off;
}

// lengths whose butterflies need more than 80 registers a thread (four waves per
// SIMD; the others run six)
constexpr bool wide(int L) {
    switch (L) {
    case 2500: case 3125: case 3240: case 3456: case 3888: case 4050: case 4320: case 4500: case 4608: case 4800:
    case 4860:
        return true;
    default:
        return false;
    }
}

inline bool short_row(int L) { return L <= 512; }  // FP64: C3_ROWS_LIST

inline bool compiled(int L, bool f64) {
#define C3_ROWC_CASE(LL) case LL:
    if (f64) {
        switch (L) {
            C3_ROWD_LIST(C3_ROWC_CASE)
            C3_ROWS_LIST(C3_ROWC_CASE)
            return true;
        default:
            return false;
        }
    }
    switch (L) {
        C3_ROWC_LIST(C3_ROWC_CASE)
        return true;
    default:
        return false;
    }
#undef C3_ROWC_CASE
}

}  // namespace c3rowc
