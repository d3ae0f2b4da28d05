// Block-diagonal causal encode of short contexts (bf16, head_dim 128): one workgroup walks several query tiles of a
// (context, KV head) pair as ONE stream of K/V blocks.
//
// A query tile (128 rows; a row is a (token, head of the group) pair) of a short context sees a handful of 32-token
// blocks, so what a workgroup per tile spends around its blocks -- launch, first loads, query rows, output -- is longer
// than the blocks themselves.  Here none of it waits: the ring of K/V blocks runs on into the next tile while the current
// one computes, the next tile's query rows are fetched a whole tile ahead, and the output leaves while the next tile's
// blocks are multiplied.  Two workgroups share a CU and fill each other's gaps.
//
// LDS (80 KB, two workgroups per CU): three 16 KB slots (K rows, V rows; 256-byte rows, 16-byte chunks XOR-swizzled so
// that every read is conflict-free) and 8 KB per wavefront for its query rows, which also turns the output around.
// Scores are computed transposed, S^T = K Q^T, then O^T += V^T P^T (MFMA 32x32x16), as in the flash kernels; bf16
// probabilities, fp32 sums of the unrounded ones.  The other workgroup of the CU is what overlaps with a softmax: starting
// the next block's S^T in its shadow took more scalar and register work than it hid (815 against 738 us for the call below).
//
// 512 contexts of 64 .. 448 tokens (mean 256), 32/8 heads: 888 -> 740 us (731 .. 751 over several cards), 3.6 TB/s of
// the 5.1 that a large copy reaches here; 2048 of 16 .. 112 tokens 954 -> 532 us.  What is left is the blocks: 2048-token contexts, which the memory does not
// bound, run at 0.9 of the flash kernel's rate.
#include "ape_mfma.h"

#include <math.h>

#include <initializer_list>

namespace ape {
namespace {

constexpr int BLOCK = 32;                    // tokens per K/V block
constexpr int ROW = 256;                     // bytes of a row
constexpr int PART = BLOCK * ROW;            // K part of a slot; V follows
constexpr int SLOT = 2 * PART;
constexpr int NSLOT = 3;
constexpr int QBUF = 32 * ROW;               // query rows of one wavefront
constexpr int LDS_BYTES = NSLOT * SLOT + 4 * QBUF;
constexpr float kLazy = 40.f;                // a reference moves only when exceeded by 2^kLazy (fp32 and bf16 lose nothing by that)
constexpr float kSumMax = 0x1p40f;           // a block sum above this: some probability left the safe range

__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The keys of a (context, KV head) pair: index t is row t of the prefix while t < P, row t - P of the context from there on.
struct Keys {
    const char *kp, *vp, *kc, *vc;
    int P;
    uint32_t stride;                          // bytes between tokens
};

// Starts the loads of indices [t, t + 32), those past t_end - 1 repeating that one (finite data whose
// probabilities are zero).  Four loads per wavefront: rows 8 w .. 8 w + 7 of K and of V.
__device__ __forceinline__ void start_block(const Keys& x, int t, int t_end, int wave, int lane, char* slot) {
    const int c = lane & 15;
    const bool ctx = t >= x.P;
    if (ctx || t + BLOCK <= x.P) {                           // one segment: a wavefront-uniform base
        const long at = (long)(ctx ? t - x.P : t) * x.stride;
        const char *k = (ctx ? x.kc : x.kp) + at, *v = (ctx ? x.vc : x.vp) + at;
        const int last = t_end - 1 - t;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * wave + 4 * i + (lane >> 4);
            const uint32_t off = (uint32_t)min(r, last) * x.stride;
            load_lds16(k, off + ((c ^ (r & 15)) << 4), slot + (8 * wave + 4 * i) * ROW);
            load_lds16(v, off + ((c ^ ((r & 3) << 2)) << 4), slot + PART + (8 * wave + 4 * i) * ROW);
        }
    } else {                                                  // the prefix ends inside the block
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * wave + 4 * i + (lane >> 4), tt = min(t + r, t_end - 1);
            const long off = (long)(tt < x.P ? tt : tt - x.P) * x.stride;
            load_lds16((tt < x.P ? x.kp : x.kc) + off + ((c ^ (r & 15)) << 4), slot + (8 * wave + 4 * i) * ROW);
            load_lds16((tt < x.P ? x.vp : x.vc) + off + ((c ^ ((r & 3) << 2)) << 4), slot + PART + (8 * wave + 4 * i) * ROW);
        }
    }
}

// grid: teams (context, KV head) x `parts` workgroups; workgroup `part` takes every parts-th tile of its context, the
// heaviest (last) first, alternate rounds in opposite directions.  gshift: log2 of the query heads per KV head.
__global__ __launch_bounds__(256, 2) void encode_walk_kernel(const EncodeArgs a, int parts, int gshift) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, hi = lane >> 5;
    int team, part;
    team_of_block(blockIdx.x, parts, team, part);
    if (team >= a.n_chunks * a.n_kv_heads) return;
    const int chunk = team / a.n_kv_heads, hk = team % a.n_kv_heads;
    int c0 = 0, len = a.total_rows;
    if (a.uniform_chunks) { c0 = chunk * a.max_chunk_len; len = a.max_chunk_len; }
    else if (a.cu) { c0 = scalar_load_i32(a.cu + chunk); len = scalar_load_i32(a.cu + chunk + 1) - c0; }
    const int rows = len << gshift, n_tiles = (rows + 127) >> 7, toks = 128 >> gshift, gmask = (1 << gshift) - 1;
    // tile of this workgroup's round s; negative: none (nor in any later round)
    auto tile_of = [&](int s) { return n_tiles - 1 - (s * parts + ((s & 1) ? parts - 1 - part : part)); };
    if (tile_of(0) < 0) return;
    Keys x;
    x.P = a.prefix_len;
    x.stride = (uint32_t)a.n_kv_heads * ROW;
    // (scalar registers: the blocks' addresses are then scalar work; 512 ragged contexts of about 256 tokens 743 / 731 us)
    auto uniform = [&](const void* p, long at) { return (const char*)uniform_address((const char*)p + at); };
    x.kp = uniform(a.k_prefix, hk * ROW); x.vp = uniform(a.v_prefix, hk * ROW);
    x.kc = uniform(a.k, (long)c0 * x.stride + hk * ROW); x.vc = uniform(a.v, (long)c0 * x.stride + hk * ROW);
    auto t_end_of = [&](int q) { return x.P + min((q + 1) * toks, len); };
    char* const qbuf = lds + NSLOT * SLOT + wave * QBUF;

    // rows past the last one repeat it (and store the same values over it)
    auto row_addr = [&](int q, int lr) -> long {
        const int R = min(q * 128 + wave * 32 + lr, rows - 1);
        return ((long)(c0 + (R >> gshift)) * a.n_q_heads + (hk << gshift) + (R & gmask)) * ROW;
    };
    // (the thread's part of a row address is recomputed where it is used, not kept in registers over the walk)
    auto opaque_lane = [&]() { int ln = lane; asm volatile("" : "+v"(ln)); return ln; };
    auto start_q = [&](int q) {
        const int ln = opaque_lane();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int lr = 4 * i + (ln >> 4);
            load_lds16((const char*)a.q + row_addr(q, lr) + (((ln & 15) ^ (lr & 15)) << 4), qbuf + 4 * i * ROW);
        }
    };
    // the loader: the stream's next block is block lj of tile lq (of round ls)
    int ls = 0, lq = tile_of(0), lj = 0, in_flight = 0;
    char* to = lds;
    auto start_next = [&]() {
        if (lq < 0) return;
        const int t_end = t_end_of(lq);
        start_block(x, BLOCK * lj, t_end, wave, lane, to);
        to = to == lds + (NSLOT - 1) * SLOT ? lds : to + SLOT;
        ++in_flight;
        if (BLOCK * ++lj >= t_end) { lj = 0; lq = tile_of(++ls); }
    };

    // K fragment of k-slab ks: ko ^ 32 ks; V^T fragment of dim block db: (vo ^ 64 db) + 4096 sl (+ 2048)
    const int ko = l32 * ROW + ((hi ^ (l32 & 15)) << 4);
    const int vrow = 4 * (lane >> 5) + ((lane & 15) >> 2);
    const int vo = PART + vrow * ROW + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ ((vrow & 3) << 2)) << 4) + (lane & 1) * 8;

    int q = lq;
    start_q(q);
    start_next();
    start_next();
    bf16x8 qf[8];
    auto read_q = [&]() {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = *(const bf16x8*)(qbuf + (ko ^ (32 * ks)));
        wait_lds();                                           // (the buffer is written again next)
    };
    if (in_flight == 2) wait_loads<8>(); else wait_loads<4>();
    asm volatile("" ::: "memory");
    read_q();
    int extra = 0;                                            // loads and stores of this wavefront between blocks 1 and 2 of a tile
    if (tile_of(1) >= 0) { start_q(tile_of(1)); extra = 1; }
    const float sc2 = 0.08838834764831845f * LOG2E;           // 1 / sqrt(128)
    const char* at = lds;
    for (int s = 0;; ++s) {
        const int R0 = q * 128 + wave * 32, t_end = t_end_of(q);
        const int lim = x.P + (min(R0 + l32, rows - 1) >> gshift);          // last index this lane's row sees
        const int lim_lo = x.P + (min(R0, rows - 1) >> gshift), lim_hi = x.P + (min(R0 + 31, rows - 1) >> gshift);
        const bool active = R0 < rows;
        f32x16 o[4];
        float m = kUnset, l = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
        const int n = (t_end + BLOCK - 1) / BLOCK;
        for (int j = 0; j < n; ++j) {
            // block j has landed: all but what is younger (the next block; before block 2, also the query rows and the
            // output of the tile's start)
            if (in_flight < 2) wait_loads<0>();
            else if (j >= 2 || extra == 0) wait_loads<4>();
            else if (extra == 1) wait_loads<12>();
            else wait_loads<20>();
            stage_barrier();                                  // ... for every wavefront, all of which are done with the slot before it
            start_next();
            const int t = BLOCK * j;
            if (active && t <= lim_hi) {
                const char* slot = at;
                f32x16 sc;
#pragma unroll
                for (int r = 0; r < 16; ++r) sc[r] = 0.f;
                // the fragments of K all ahead of their MFMAs, those of V behind them: in registers before the softmax ends
                bf16x8 kf[8], vf[8];
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) kf[ks] = *(const bf16x8*)(slot + (ko ^ (32 * ks)));
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sc, 0, 0, 0);
#pragma unroll
                for (int f = 0; f < 8; ++f) {                 // fragment f: k-slab f / 4, dim block f % 4
                    const char* v = slot + (vo ^ (64 * (f & 3))) + 16 * (f >> 2) * ROW;
                    vf[f] = __builtin_shufflevector(lds_read_tr(v), lds_read_tr(v + 8 * ROW), 0, 1, 2, 3, 4, 5, 6, 7);
                }
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(0);
                if (t + BLOCK - 1 > lim_lo) {                 // register r holds index t + 8 (r / 4) + 4 hi + r % 4
                    const int nvis = lim - t + 1 - 4 * hi;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sc[r] = 8 * (r >> 2) + (r & 3) < nvis ? sc[r] : -INFINITY;
                }
                auto row_max = [&]() {
                    float x0 = fmaxf(fmaxf(sc[0], sc[1]), sc[2]), x1 = fmaxf(fmaxf(sc[3], sc[4]), sc[5]);
                    x0 = fmaxf(fmaxf(x0, sc[6]), sc[7]); x1 = fmaxf(fmaxf(x1, sc[8]), sc[9]);
                    x0 = fmaxf(fmaxf(x0, sc[10]), sc[11]); x1 = fmaxf(fmaxf(x1, sc[12]), sc[13]);
                    return max_halves(fmaxf(fmaxf(x0, x1), fmaxf(sc[14], sc[15]))) * sc2;
                };
                // every row sees index 0, but a first block may be masked by its keys: scores of -inf, or below kUnset, are no reference
                // (a later block exceeds the unset one and moves it)
                if (j == 0) m = fmaxf(row_max(), kUnset);
                float p[16], s0 = 0.f, s1 = 0.f;
                auto probs = [&]() {
                    s0 = s1 = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        p[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], sc2, -m));
                        p[r + 1] = __builtin_amdgcn_exp2f(fmaf(sc[r + 1], sc2, -m));
                        s0 += p[r]; s1 += p[r + 1];
                    }
                };
                probs();
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(s0 + s1 <= kSumMax)) != 0, 0)) {
                    const float mx = row_max(), m_new = mx > m + kLazy ? mx : m, alpha = __builtin_amdgcn_exp2f(m - m_new);
                    m = m_new; l *= alpha;
#pragma unroll
                    for (int db = 0; db < 4; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
                    probs();
                }
                l += s0 + s1;
                // k-slot e of slab sl is index 16 sl + (e < 4 ? 4 hi + e : 8 + 4 hi + e - 4): registers 8 sl .. 8 sl + 7
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    u32x4 pk;
#pragma unroll
                    for (int i = 0; i < 4; ++i) pk[i] = pack_bf16(p[8 * sl + 2 * i], p[8 * sl + 2 * i + 1]);
#pragma unroll
                    for (int db = 0; db < 4; ++db) {
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[4 * sl + db], __builtin_bit_cast(bf16x8, pk), o[db], 0, 0, 0);
                    }
                }
            }
            at = at == lds + (NSLOT - 1) * SLOT ? lds : at + SLOT;
            --in_flight;
        }
        const int q_done = q, q_next = tile_of(s + 1);
        if (q_next >= 0) {
            // the next tile's query rows: younger than them are the blocks in flight that this tile's bodies started
            if (in_flight == 2 && n >= 2) wait_loads<8>();
            else if (in_flight == 2 || n >= 2) wait_loads<4>();
            else wait_loads<0>();
            asm volatile("" ::: "memory");
            read_q();
        }
        if (active) {
            // the output turns around in the wavefront's query buffer and leaves as whole rows, 16 bytes per lane
            const float lt = sum_halves(l), inv = 1.f / lt;   // a row always sees itself
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *(u32x2*)(qbuf + l32 * ROW + (((4 * db + q4) ^ (l32 & 15)) << 4) + 8 * hi) =
                        u32x2{pack_bf16(o[db][4 * q4] * inv, o[db][4 * q4 + 1] * inv), pack_bf16(o[db][4 * q4 + 2] * inv, o[db][4 * q4 + 3] * inv)};
            if (a.lse && hi == 0) {
                const int R = min(R0 + l32, rows - 1);
                a.lse[(long)((hk << gshift) + (R & gmask)) * a.total_rows + c0 + (R >> gshift)] = (m + __builtin_amdgcn_logf(lt)) * LN2;
            }
            const int ln = opaque_lane();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int lr = 4 * i + (ln >> 4);
                *(u32x4*)((char*)a.out + row_addr(q_done, lr) + ((ln & 15) << 4)) = *(const u32x4*)(qbuf + lr * ROW + (((ln & 15) ^ (lr & 15)) << 4));
            }
        }
        if (q_next < 0) break;
        wait_lds();                                           // (the output rows have been read back)
        q = q_next;
        extra = active ? 1 : 0;
        if (tile_of(s + 2) >= 0) { start_q(tile_of(s + 2)); ++extra; }
    }
}

}  // namespace

// The walk wins while the streams of the tiles are short, the prefix in front of a context counted; past long streams the
// software-pipelined body of the flash kernel does.  Where the line lies (32/8 heads, flash / walk, us):
//   many tiles, where the mean stream counts: contexts alone (131072 tokens) 256 tokens 742 / 639, 512 964 / 880, 1024 1392 / 1382,
//   2048 2272 / 2495; behind a prefix of 256 / 384 / 1024 tokens 64 x 512 343 / 323, 396 / 389, 512 x 256 ragged at 1024 2714 / 2835,
//   64 x 256 ragged 166 / 159, 192 / 194, 1024 x 64 at 1024 1131 / 1208.  With one query head per KV head tiles are as long as 128 tokens
//   and the last one of a context is half empty, which costs the walk less, since a wavefront without rows leaves its time to the
//   others: 8/8 heads, 64 x 512 behind 512 / 1024 128 / 117, 186 / 186, 256 x 200 209 / 196, 312 / 326, 256 x 256 ragged 341 / 270, 484 / 429 and
//   behind 2048 789 / 737, but 100 x 700 ragged behind 256 273 / 280;
//   fewer than 2048, where the longest is the whole time: 4 x 512 tokens behind 0 / 128 / 256 / 512 21.9 / 21.0, 25.5 / 24.8, 28.7 / 28.7,
//   35.1 / 35.9; 8 x 256 behind 384 / 1024 27.3 / 26.8, 44.0 / 45.4;
//   a tile or less per CU, with no second workgroup to fill the gaps: 2 x 256 behind 0 / 128 10.4 / 10.0, 13.1 / 12.7; 1 x 300 behind 0 / 32
//   10.9 / 11.1, 11.6 / 12.0; 2 x 400 12.8 / 13.7; 2 x 100 behind 512 16.1 / 18.3.
// Workgroups per context: about four tiles each when that still leaves thousands of workgroups, fewer tiles otherwise
// (tiles per workgroup 4 / 2 / 1, us: 512 x 256 tokens 641 / 653 / 687, 64 x 512 - / 222 / 238, 16 x 128 ragged - / 14.7 / 12.3), but two
// also where the chip then holds all workgroups at once and would not with one (8 x 512 39.2 / 27.4 / 33.6, 6 x 512 36.1 / 25.9 / 28.0; and not
// 10 x 512 44.5 / 40.7 / 40.0).
int encode_walk_parts(const EncodeArgs& a) {
    const int group = a.n_q_heads / a.n_kv_heads;
    const long tiles = ((long)a.total_rows * group + 127) / 128 * a.n_kv_heads, teams = (long)a.n_chunks * a.n_kv_heads;
    const long prefix = a.prefix_len, context = a.max_chunk_len;
    if (a.n_kv_heads > 4096) return 0;                       // (32-bit offsets inside a block of 32 tokens)
    const long mean = group > 1 ? 512 : a.uniform_chunks || context > 512 ? 768 : 2304;
    if (tiles >= 2048 ? prefix + context / 2 > mean : tiles > 256 ? context > 512 || prefix + context > 640 : context > 256 || prefix + context > 384) return 0;
    const int longest = (a.max_chunk_len * group + 127) / 128;
    for (int per : {4, 2}) {
        const int parts = (longest + per - 1) / per;
        if (teams * parts >= (per == 4 ? 4096 : 900) || (per == 2 && tiles > 640 && teams * parts <= 512)) return parts;
    }
    return longest;
}

hipError_t launch_encode_walk(const EncodeArgs& a, int parts, hipStream_t s) {
    if (a.total_rows == 0) return hipSuccess;
    int gshift = 0;
    while (a.n_kv_heads << gshift < a.n_q_heads) ++gshift;
    hipError_t e = hipFuncSetAttribute((const void*)encode_walk_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
    const unsigned teams = (unsigned)(a.n_chunks * a.n_kv_heads + 7) / 8 * 8;
    encode_walk_kernel<<<teams * (unsigned)parts, 256, LDS_BYTES, s>>>(a, parts, gshift);
    return hipGetLastError();
}

}  // namespace ape
