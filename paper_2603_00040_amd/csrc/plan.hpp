// How a backward is cut into workgroups: host arithmetic on the shape and the number of compute units, without the HIP runtime.
#pragma once
#include <stddef.h>

namespace aq {

// joint: both passes in one launch, the query tiles of a key tile shared by up to `splits` workgroups of `iters` query tiles whose sums
// take part_bytes; dq_first: the dQ tiles in front.
struct BwdPlan { bool joint; int splits, iters; size_t part_bytes; bool dq_first; };

// Whether a backward runs both passes in one launch, and how many query tiles a dK/dV workgroup takes.
// Joint: everything except the problems whose eight-wave workgroups (wide_workgroups) fill their rounds of the compute units to
// 97 % on average, where the halved tile copies win by 2 - 3 % (24 heads, L = 8192: 2.09 against 2.14 ms; 12 x 2 heads, L = 32760:
// 32.0 against 33.0 ms), while rounds filled to 95, 92 and 73 % lose to the joint launch by 2, 5 and 24 % (40 heads, L = 20000
// and 12000; 12 heads of 64, L = 12000).  Under a causal mask the two are even at 32768 positions (46.1 ms) and below that
// joint wins by 1 - 4 %.  (All of that at d = 128; at d = 64 bwd_plan makes the rest joint as well.)
// Pieces: time is counted in query tiles of the dK/dV pass (1.45 us); a 64-key tile of a dQ workgroup takes 1.16 of them.  With W the
// work per compute unit, pieces of 0.45 W came out best or within 10 % of it over 16 shapes (8 sizes of piece each), as long as
//   * a piece is not much shorter than the average dQ tile, which it would only have to wait for,
//   * the pieces (and, if there are few, the dQ tiles) fit the 2 workgroups per compute unit at once: a second round of
//     pieces costs more than it evens out (12 heads, L = 1560: 312 pieces 83 us, 468 pieces 107 us).
// The length of a piece grows by steps until the pieces fit.  Their number falls with it, so the step is found by bisection: every
// call makes this plan on the host, and counting the pieces walks over the key tiles (one head, L = 30000 causal: 6 us step by
// step, 1.3 us so).
inline BwdPlan plan_backward(int BHq, int BHkv, int L, int D, bool causal, int cus_)
{
    BwdPlan p{false, 1, 0, 0, false};
    const int Lp = (L + 127) / 128 * 128, nt = Lp / 128, G = BHq / BHkv, nq32 = (L + 31) / 32;
    const long long cus = cus_, n8q = (long long)BHq * ((Lp + 255) / 256), n8kv = (long long)BHkv * ((Lp + 255) / 256);
    auto fill = [&](long long n) { return (double)n / (double)((n + cus - 1) / cus * cus); };
    if (causal ? Lp >= 32768 && n8kv >= 2 * cus : n8kv >= 2 * cus && fill(n8q) + fill(n8kv) >= 2 * 0.97) return p;
    p.joint = true;
    const long long whole = (long long)nq32 * G;
    p.iters = (int)(whole < 0x7FFFFFFF ? whole : 0x7FFFFFFF);
    const double dq_longest = 1.16 * (Lp / 64), dq_mean = causal ? 0.5 * dq_longest : dq_longest;
    const double dkv_mean = (double)G * (causal ? nq32 - 2.0 * (nt - 1) : (double)nq32);
    const double W = (double)nt * (BHkv * dkv_mean + BHq * dq_mean) / (double)cus;
    double T = 0.45 * W;
    if (T < 0.6 * dq_mean) T = 0.6 * dq_mean;
    if (T < 4.0) T = 4.0;
    const long long ndq = (long long)BHq * nt, room = 2 * cus - (ndq < cus ? ndq : 0);
    if (T < (double)whole && (long long)BHkv * nt <= room) {       // (every key tile is one piece at least)
        constexpr int kSteps = 640;                                // (1.04^640 > 2^31)
        double step[kSteps];
        int n = 0;
        for (; n < kSteps && T < (double)whole; T = T * 1.04 + 1.0) step[n++] = T;
        auto fits = [&](double T_) {
            const unsigned t = (unsigned)T_;
            long long sum = 0;
            if (causal) for (int kt = 0; kt < nt; ++kt) sum += ((unsigned)(nq32 - 4 * kt) * (unsigned)G + t - 1) / t;
            else sum = (long long)nt * ((whole + t - 1) / t);
            return sum * BHkv <= room;
        };
        int lo = 0, hi = n;                                        // the first step that fits, n = none
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (fits(step[mid])) hi = mid; else lo = mid + 1;
        }
        if (lo < n) {
            p.iters = (int)step[lo];
            p.splits = (int)((whole + p.iters - 1) / p.iters);
            p.part_bytes = (size_t)BHkv * nt * p.splits * 2 * 128 * D * 4;
        }
    }
    p.dq_first = dq_longest > 1.5 * p.iters;      // (one head, L = 16000 causal, 192 pieces: 348 against 405 us)
    return p;
}

// Whether the joint launch of d = 64 keeps to two workgroups per compute unit, although three fit.  Key tiles that are not cut into pieces
// are long chains, and a third workgroup beside them slows them down; where they are one to a little over two rounds of the compute
// units, they end last and the call waits for them.  Backward with two / with three, measured over 90 shapes with 170 - 700 whole key tiles:
// without a mask, grouped heads, 257 - 384 tiles 2 - 9 % shorter (2 x 32/4 heads, L = 5000, 320 tiles 1442 / 1556 us; 16/4 heads, L = 9637,
// 304 tiles 1305 / 1432 us; 8 x 16/2 heads, L = 3000, 384 tiles even), 16/8 heads, L = 3300 x 2, 416 tiles 346 / 324 us; heads of their own up to 15 %
// longer where they are few (2 x 2 heads, L = 10205, 320 tiles).  Causal, up to 2.3 tiles per unit 0 - 9 % shorter (8 heads of 32, L = 8456, 536 tiles
// 1080 / 1162 us; 552 tiles of 12 heads, L = 5781 214 / 225 us), from 2.5 on even or longer, and so below 2048 positions (4 x 24 heads, L = 668 57 / 55 us).
inline bool joint_in_pairs(const BwdPlan& p, int BHq, int BHkv, int L, int D, bool causal, int cus)
{
    if (D != 64 || !p.joint || p.splits > 1) return false;
    const long long tiles = (long long)BHkv * ((L + 127) / 128);
    if (tiles <= cus) return false;
    return causal ? L >= 2048 && tiles * 10 <= (long long)cus * 23 : BHq > BHkv && tiles * 2 <= (long long)cus * 3;
}

// Whether the four waves of a workgroup share the tiles of 32 rows in a backward (bwd_few_kernel): up to one such group of keys or of queries per compute unit, and up to
// two under a causal mask, where most chains are short, with rows of more than four tiles.  With several query heads to a kv head a group of keys has all their
// query tiles in one chain, and the joint launch is the faster one where it may cut key tiles into pieces.  Measured over 420 shapes (L = 33 - 4000, 1 - 40 kv
// heads, 1 - 8 query heads to each, 4 - 900 groups): 7 - 90 % faster in all 288 that this rule takes but one (40 heads, L = 98, d = 128 causal, 5 % slower, which the four tiles
// leave out); beyond: no mask, 2 heads, L = 2411, d = 64, 304 groups 6 % slower, 6 heads, L = 1316, d = 128, 504 groups 17 %; causal, 4 heads, L = 2688, 672
// groups 9 %; with pieces, 8/2 heads, L = 582 causal, 190 groups 1.6 times slower, 6/3 heads, L = 575 causal, 162 groups 10 %.
inline bool few_rows(int BHq, int BHkv, int L, bool causal, bool pieces /* the joint launch would cut key tiles */, int cus)
{
    const int n32 = (L + 31) / 32;
    if (BHq != BHkv && pieces) return false;
    return (long long)(BHq + BHkv) * n32 <= (long long)cus * (causal && BHq == BHkv && n32 > 4 ? 2 : 1);
}

}  // namespace aq
