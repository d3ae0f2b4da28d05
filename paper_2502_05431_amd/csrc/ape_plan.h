// Split plans of batches whose requests have contexts of different length.  Host code without HIP in it.
//
// The even plan cuts every request into splits of the length that suits the longest one.  A batch that is dealt out has, for every
// request, as many splits as its length asks for, all of about one length, in partial results that take no more room than the even plan's.
#pragma once

#include <stdint.h>

namespace ape {

constexpr int kMaxReqPerLaunch = 32;     // requests whose descriptors travel in one kernel-argument block
constexpr int kMaxSplits = 64;           // upper bound of context splits per (request, head)

struct UnevenPlan {
    int n_splits, most, longest;         // of the launch; the most of one request; tokens of the longest
    int first[kMaxReqPerLaunch + 1], len[kMaxReqPerLaunch];
};

// What the launches of a call have in common.
struct DealRule {
    int shortest, unit;                  // tokens: what a split has at least, as in the even plan; whole stages or blocks of the kernel
    int even_splits, even_len;           // the even plan of the longest request
    long tiles;                          // workgroups of a split: KV heads x row tiles
};

inline long plan_ceil(long a, long b) { return (a + b - 1) / b; }

// Splits of nb requests of ctx(i) context tokens, `splits` of them or fewer, the longest as short as that allows.  false: one for each.
template <class Ctx>
bool deal_splits(const Ctx& ctx, int nb, long splits, const DealRule& r, UnevenPlan& p) {
    long longest = 0;
    for (int i = 0; i < nb; ++i)
        if (ctx(i) > longest) longest = ctx(i);
    auto count = [&](long len) {
        long n = 0;
        for (int i = 0; i < nb; ++i) n += plan_ceil(ctx(i), len);
        return n;
    };
    // the shortest length, in units: kMaxSplits of it hold the longest
    long lo = plan_ceil(longest, (long)r.unit * kMaxSplits), hi = plan_ceil(longest, r.unit);
    if (lo < plan_ceil(r.shortest, r.unit)) lo = plan_ceil(r.shortest, r.unit);
    while (lo < hi) {
        const long mid = (lo + hi) / 2;
        if (count(r.unit * mid) <= splits) hi = mid; else lo = mid + 1;
    }
    p.first[0] = 0; p.most = p.longest = 0;
    for (int i = 0; i < nb; ++i) {
        int n = (int)plan_ceil(ctx(i), r.unit * lo);
        p.len[i] = n > 0 ? (int)plan_ceil(ctx(i), (long)r.unit * n) * r.unit : r.unit;    // its splits are of one length
        n = (int)plan_ceil(ctx(i), p.len[i]);                                              // (no more than before)
        p.first[i + 1] = p.first[i] + n;
        if (n > p.most) p.most = n;
        if (n > 0 && p.len[i] > p.longest) p.longest = p.len[i];
    }
    p.n_splits = p.first[nb];
    static_assert(kMaxReqPerLaunch * kMaxSplits < 1 << 16, "first_split");
    return p.most > 1 && p.n_splits <= splits;
}

// ... where dealing them out gives something: shorter splits, fewer rounds of 256 workgroups (the even plan's grid holds those of splits that
// shorter requests do not have), or, with more than one workgroup to a CU, at least others.  Otherwise what the kernel looks up is all that is
// left of it (even / dealt, us: 16 steps of 3 x ~2048 tokens, 32/8 heads, the same 248 splits 77.9 / 80.9; 4 of 1 to 7 x 1000, 8/8 bf16 heads
// of 96, 25.0 / 25.9; 2 prefills of 16 rows, 6/2 of 40, 9.2 / 9.9; but the same splits in fewer rounds: 2 of 16 rows, 32/8 fp32 heads of 128,
// 31.3 / 24.2, 24 steps of ~2770 tokens, 16/2 heads, 30.6 / 20.6, and others of the same length 4 of 1 to 7 x 1000, 32/32 fp32 heads, 238 / 215).
template <class Ctx>
bool plan_uneven(const Ctx& ctx, int nb, long splits, const DealRule& r, UnevenPlan& p) {
    if (!deal_splits(ctx, nb, splits, r, p)) return false;
    if ((p.n_splits + nb) * r.tiles >= 1L << 24) return false;       // (a launch holds 2^32 work items in x, and the whole batch lies there)
    if (16L * p.longest <= 15L * r.even_len) return true;
    const long dealt = p.n_splits * r.tiles, even = (long)r.even_splits * nb * r.tiles;
    if (plan_ceil(dealt, 256) < plan_ceil(even, 256)) return true;
    if (dealt <= 256) return false;
    for (int i = 0; i < nb; ++i)
        if (plan_ceil(ctx(i), r.even_len) != p.first[i + 1] - p.first[i] || (p.first[i + 1] - p.first[i] > 1 && p.len[i] != r.even_len)) return true;
    return false;
}

// Requests per launch of an uneven batch, and the splits that a launch deals out.
struct UnevenCall {
    int per_launch;
    long splits;
};

// ... of a decode step on the flash kernels.  A launch wants 512 workgroups, all of them resident, or the next multiple that gives each of its requests
// two splits (32/8 heads, even plan | 256 / 512 / 1024 workgroups, us: 8 requests of about 4096 tokens 43.5 | 34.9 / 33.4 / 36.9; 4 of 32K 85.6 | 69.0 /
// 69.4 / 71.2; 24 of 1 to 7 x 1024 113 | 91.5 / 82.1 / 88.7; with 16 KV heads, even | 512 / two for each: 24 of 1 to 15 x 512 181 | 143 / 136, 48 of
// them 338 | 293 / 268, 64 366 | 366 / 306, 20 of 1 to 7 x 1024 134 | 119 / 130 and with 1024 workgroups 107).  Where the even plan has a single split,
// which leaves no room for that, and the longest request is far from the mean, the batch goes out in two launches, each with all of the room -- if the
// even plan gives a CU one workgroup, or the streams are long (even / halves, us: 32/8 heads, 32 of 1 to 15 x 1024 220 / 184, of 1 to 7 116 / 113; 16/16
// heads, 16 of 1 to 5 x 1024 87.4 / 78.5, 32 of 1 to 15 x 1024 402 / 345, of 1 to 7 207 / 210; 32/32 heads, 16 of 1 to 15 x 1024 415 / 382, of 1 to 5
// 134 / 141), and if every launch can then be dealt out: two even launches are never made out of one (16/16 heads, 32 of 1 to 3 x 700: 69 / 96).
template <class Ctx>
UnevenCall uneven_decode_call(const Ctx& ctx, int batch, int n_kv_heads, const DealRule& r) {
    const int per = batch < kMaxReqPerLaunch ? batch : kMaxReqPerLaunch;
    const long slots = (long)(r.even_splits + 1) * batch;      // of one request each
    auto room = [&](long workgroups, int nb) {
        const long n = plan_ceil(2L * nb * n_kv_heads, workgroups) * workgroups / n_kv_heads;
        return n < slots - nb ? n : slots - nb;
    };
    const UnevenCall one{per, room(512, per)};
    long total = 0, longest = 0;
    for (int i = 0; i < batch; ++i) {
        total += ctx(i);
        if (ctx(i) > longest) longest = ctx(i);
    }
    if (2 * one.splits >= 3L * per || 5L * longest * batch <= 8 * total || total <= ((long)batch * n_kv_heads > 256 ? 4096L : 1536L) * batch) return one;
    const UnevenCall two{(per + 1) / 2, room(256, (per + 1) / 2)};
    UnevenPlan p;
    for (int b0 = 0; b0 < batch; b0 += two.per_launch) {
        const int nb = batch - b0 < two.per_launch ? batch - b0 : two.per_launch;
        if (!plan_uneven([&](int i) { return ctx(b0 + i); }, nb, two.splits, r, p)) return one;
    }
    return two;
}

// Whether the longest request is more than an eighth longer than the mean.
template <class Ctx>
bool uneven_batch(const Ctx& ctx, int batch) {
    long total = 0, longest = 0;
    for (int i = 0; i < batch; ++i) {
        total += ctx(i);
        if (ctx(i) > longest) longest = ctx(i);
    }
    return batch > 1 && 8 * longest * batch > 9 * total;
}

}  // namespace ape
