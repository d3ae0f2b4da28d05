// Host check of csrc/ape_plan.h: random uneven batches through the plans of a call's launches.
#include "ape_plan.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

using namespace ape;

#define CHECK(x)                                                                                   \
    do {                                                                                           \
        if (!(x)) { printf("line %d: %s (case %ld)\n", __LINE__, #x, g_case); exit(1); }           \
    } while (0)

static long g_case = 0;

static long ceil_div(long a, long b) { return (a + b - 1) / b; }

// the even plan of a length: n splits at most, of whole units
static void even_plan(long longest, long n, DealRule& r) {
    r.even_len = (int)(ceil_div(ceil_div(longest, n), r.unit) * r.unit);
    r.even_splits = (int)ceil_div(longest, r.even_len);
}

// Every launch of the call: what its plan must hold.  Returns how many launches are dealt out.
static int check_call(const std::vector<long>& lens, const DealRule& r, const UnevenCall& call) {
    const int batch = (int)lens.size();
    int dealt = 0;
    CHECK(call.per_launch >= 1 && call.per_launch <= kMaxReqPerLaunch);
    for (int b0 = 0; b0 < batch; b0 += call.per_launch) {
        const int nb = std::min(batch - b0, call.per_launch);
        UnevenPlan p;
        if (!plan_uneven([&](int i) { return lens[b0 + i]; }, nb, call.splits, r, p)) continue;
        ++dealt;
        int most = 0;
        CHECK(p.first[0] == 0 && p.n_splits == p.first[nb]);
        for (int i = 0; i < nb; ++i) {
            const int n = p.first[i + 1] - p.first[i];
            CHECK(p.len[i] > 0 && p.len[i] % r.unit == 0 && n == ceil_div(lens[b0 + i], p.len[i]) && n <= kMaxSplits);
            CHECK(n < 2 || p.len[i] >= r.shortest / 2);
            most = std::max(most, n);
        }
        CHECK(most == p.most && most > 1);
        CHECK(p.n_splits + nb <= (long)(r.even_splits + 1) * batch);            // the workspace
        CHECK((p.n_splits + nb) * r.tiles < 1L << 24);
    }
    return dealt;
}

int main() {
    std::mt19937 rng(7);
    auto pick = [&](long lo, long hi) { return lo + (long)(rng() % (unsigned long)(hi - lo + 1)); };
    for (g_case = 1; g_case <= 20000; ++g_case) {
        const int batch = (int)pick(1, 80), hkv = 1 << pick(0, 6);
        const long top = 1L << pick(1, 17);
        std::vector<long> lens(batch);
        long longest = 0;
        for (long& n : lens) {
            n = pick(0, 9) == 0 ? 0 : pick(0, 3) == 0 ? pick(1, 300) : pick(1, top);
            longest = std::max(longest, n);
        }
        if (longest == 0) continue;
        const int units[] = {32, 64, 128};
        DealRule r{256, 64, 0, 0, hkv};
        even_plan(longest, pick(0, 2) ? 1L << pick(0, 6) : 1, r);
        // a decode step: never more launches than the requests ask for unless every one of them is dealt out
        const auto ctx = [&](int i) { return lens[i]; };
        const UnevenCall call = uneven_decode_call(ctx, batch, hkv, r);
        const int dealt = check_call(lens, r, call);
        const long launches = ceil_div(batch, call.per_launch), needed = ceil_div(batch, kMaxReqPerLaunch);
        CHECK(launches == needed || dealt == launches);
        // any other call
        r.unit = units[pick(0, 2)]; r.shortest = pick(0, 1) ? 64 : 128; r.tiles = hkv * pick(1, 40);
        even_plan(longest, 1L << pick(0, 6), r);
        check_call(lens, r, UnevenCall{kMaxReqPerLaunch, (long)r.even_splits * batch});
    }
    // requests of 1 .. 15 x 1024 tokens, one split each in the even plan
    for (int batch : {16, 24, 32, 64})
        for (int hkv : {8, 16, 32}) {
            g_case = 100000 + 100 * batch + hkv;
            std::vector<long> lens(batch);
            for (int b = 0; b < batch; ++b) lens[b] = 1024 * (1 + b * 7 % 15);
            DealRule r{256, 64, 0, 0, hkv};
            even_plan(15 * 1024, batch * hkv >= 256 ? 1 : 2, r);
            const UnevenCall call = uneven_decode_call([&](int i) { return lens[i]; }, batch, hkv, r);
            CHECK(check_call(lens, r, call) == ceil_div(batch, call.per_launch));
            if (batch == 32) CHECK(call.per_launch == 16 && call.splits == 32);
            if (batch == 64) CHECK(call.per_launch == 32 && call.splits >= 64);
        }
    // short contexts on many KV heads: one launch
    {
        g_case = 200000;
        std::vector<long> lens(32);
        for (int b = 0; b < 32; ++b) lens[b] = 700 * (1 + b % 3);
        DealRule r{256, 64, 0, 0, 16};
        even_plan(2100, 1, r);
        CHECK(uneven_decode_call([&](int i) { return lens[i]; }, 32, 16, r).per_launch == 32);
    }
    // a million KV heads: the batch passes what a launch holds in x (a request at a time it does not)
    {
        g_case = 250000;
        std::vector<long> lens(32);
        lens[0] = 5000; lens[1] = 700;
        DealRule r{256, 64, 0, 0, 1L << 20};
        even_plan(5000, 1, r);
        UnevenPlan p;
        const auto ctx = [&](int i) { return lens[i]; };
        CHECK(deal_splits(ctx, 32, 32, r, p) && !plan_uneven(ctx, 32, 32, r, p));
        r.tiles = 4;
        CHECK(plan_uneven(ctx, 32, 32, r, p));
    }
    // the even plan's own splits, one per CU: nothing is dealt out; one request of twice the length: it is
    {
        g_case = 300000;
        std::vector<long> lens = {1024, 4096, 2048, 512};
        DealRule r{256, 64, 0, 0, 2};
        even_plan(4096, 16, r);
        UnevenPlan p;
        const auto ctx = [&](int i) { return lens[i]; };
        CHECK(deal_splits(ctx, 4, 64, r, p) && !plan_uneven(ctx, 4, 30, r, p));
        even_plan(4096, 4, r);
        CHECK(plan_uneven(ctx, 4, 16, r, p) && p.longest < r.even_len);
    }
    printf("ok\n");
    return 0;
}
