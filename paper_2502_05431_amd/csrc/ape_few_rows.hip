// Matrix-core attention for a few query rows (a row is a (query token, head of the group) pair): a decode step, a query of a few tokens, and any
// query of up to 512 rows per KV head over short contexts (whole: (request, KV head, 16 rows) triples up to 256) or, while its tiles leave CUs idle, over up to 3072 tokens (split: KV heads
// times tiles of 16 rows up to 64).  bf16 of head_dims up to 256 and fp32 up to 128, any number of query heads per KV head.
//
// Math, precision and what happens to values that are not finite: as in the tile kernels (ape_tile_mfma.hip).  Errors against 64 bits likewise:
// outputs 1.6e-3 (bf16), 2e-7 to 4e-7 (fp32; relative 2-norm).
//
// Tiling.  A workgroup has 16 rows.  A wavefront takes blocks of 32 tokens past all of them, alone: K and V come through a ring of its own in LDS (five
// pieces of 16 tokens of K or of V, direct loads), it waits for its own loads by count, and there is no barrier until the
// wavefronts' results are pooled at the end.  16 rows per MFMA (16x16x32, fp32 16x16x4) are half the work of the 32 of the other kernels for
// the same tokens; S^T = K Q^T, so that the probabilities are the B operand of O^T += V^T P^T as they come.
//
// What bounds it.  A long stream: HBM, with 16 to 20 KB in flight from every wavefront.  A short one: round trips -- the arguments (0.4 us), the chunk table
// (0.5; 64 entries at once, one per lane: the search, the pointers and the next contexts cost no further trip), the first loads (1), 0.35 a block of 32
// tokens, the pooling (0.8).  A decode step of 4 x 256 tokens, 32/8 heads of 128: 5.4 us from the first instruction to the last, the flash kernel 8.1 (0.65 per block, all of them
// past one wavefront with three in flight); with launch and merge 12.6 -> 10.4 us, over 20 x 512 tokens 15.6 -> 14.0.  Where the wavefronts took a run each, one
// behind the other, ragged short contexts cost a partial block for each (100 of about 100 tokens 18.9, this 16.2, both on the 16 splits of before).
// Contexts and own tokens past wavefronts of their own at the same time: 16 fp32 rows over 4 x 32 tokens, 4/2 heads of 64, 14.6 -> 7.3 us (the tile kernel
// takes them one after the other, 6.0 + 3.5 us, two thirds of the first in looking up where its rows are).
#include "ape_exact_row.h"

namespace ape {
namespace {

template <typename T, int DP>
struct Few {
    static constexpr int PITCH = DP * (int)sizeof(T), CPR = PITCH / 16;   // bytes of a row in LDS, 16-byte chunks of it
    static constexpr int ENTRY = 16 * PITCH;                // a ring entry: 16 tokens of K or of V (or the query rows)
    static constexpr int LOADS = ENTRY / 1024, ROWS = 64 / CPR;   // load instructions of an entry, and rows of each
    static constexpr int RING = 5;
    static constexpr int WAVE = RING * ENTRY;               // LDS of a wavefront
    static constexpr int NS = PITCH / 64, NB = DP / 16;     // 64-byte slabs of Q and K, 16-dim blocks of the output
    static constexpr int BOX = 64 * DP;                     // a wavefront's result, where its ring was; references and sums follow
    static_assert(BOX + 128 <= WAVE && 4 * LOADS < 64, "sizes");
};

// One direct load of 16 bytes per lane that is not to stay in the caches (as load_lds16): a tile of 16 rows reads every byte of K and V once.  Several tiles read the same tokens each for
// itself, and carry the hint too.
__device__ __forceinline__ void load_once(const char* base, uint32_t off, const char* lds) {
    const uint32_t m0v = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1 nt" :: "v"(off), "s"(uniform_address(base)), "s"(m0v) : "m0");
}

__device__ __forceinline__ void load_once(const char* src, const char* lds) {
    const uint32_t m0v = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" :: "v"(src), "s"(m0v) : "m0");
}

// XOR swizzles of the 16-byte chunk index inside a row: 16 rows at the same chunk (K, Q), 8 rows at the same pair of chunks (V in bf16) or rows 4
// apart at the same four (V in fp32) lie in different banks.
template <int PITCH>
__device__ __forceinline__ int few_swz_k(int row) { return PITCH == 128 ? (row >> 1) & 7 : row & 15; }
template <typename T, int PITCH>
__device__ __forceinline__ int few_swz_v(int row) { return sizeof(T) == 4 ? (row >> 2 & 3) << 2 : PITCH == 128 ? ((row >> 1) & 3) << 1 : (row & 7) << 1; }

// Load i of an entry: rows i * ROWS + lane / CPR, of which the lane fetches one chunk; the swizzle's share of i is a constant.
template <typename T, int DP, bool V>
__device__ __forceinline__ uint32_t few_chunk(int i, uint32_t width) {
    using X = Few<T, DP>;
    const int lane = threadIdx.x & 63, r = lane / X::CPR;
    int c = lane % X::CPR;
    if constexpr (V && sizeof(T) == 4) c ^= 4 * (i * X::ROWS / 4 & 3);
    else c ^= X::PITCH == 128 ? (V ? r & ~1 : r >> 1 ^ 4 * i) : V ? 2 * r ^ 2 * (i * X::ROWS & 7) : r ^ i * X::ROWS;
    return 16u * c < width ? 16 * c : 0;                     // dims past head_dim: the row's first
}
// ... from the row that `first` rows are in front of: rows past the last valid one repeat it (finite data whose probabilities are zero).
template <typename T, int DP, bool V>
__device__ __forceinline__ uint32_t few_offset(int i, int first, int n_valid, uint32_t stride, uint32_t width) {
    const int row = i * Few<T, DP>::ROWS + (int)(threadIdx.x & 63) / Few<T, DP>::CPR;
    return (uint32_t)min(first + row, n_valid - 1) * stride + few_chunk<T, DP, V>(i, width);
}
template <typename T, int DP>
struct FewOffsets { uint32_t k[Few<T, DP>::LOADS], v[Few<T, DP>::LOADS]; };

// The tokens of a wavefront: blocks of 32 consecutive indices of the pooled contexts, or of the prefix and the own tokens behind it, whatever
// context they belong to; every `step`-th token's block, so that the wavefronts of a workgroup read one run of memory together.
struct FewWalk {
    int t, step, t1;                 // the next block's first index; the stream's end
    long stride, head;
    const int32_t* cu;               // NULL: prefix + own tokens, their K rows at ka + i * stride below np, at kb + i * stride from there on
    const void* const* kt;
    const void* const* vt;
    int n_chunks, base;              // contexts base .. base + 63 are in the lanes
    int c0, c1, end;                 // the lane's context; the last one's end
    uint64_t kp, vp;
    const char *ka, *va, *kb, *vb;
    int np;
    uint64_t kr, vr;                 // a block with tokens of more than one segment: the rows of its token lane & 31

    __device__ __forceinline__ void read_table() {
        const int c = min(base + (int)(threadIdx.x & 63), n_chunks - 1);
        c0 = cu[c]; c1 = cu[c + 1];
        kp = (uint64_t)kt[c]; vp = (uint64_t)vt[c];
    }
    // The lane of the context that holds index i (i < cu[n_chunks]): the first one that ends behind it (empty ones never do).
    __device__ __forceinline__ int context_of(int i) {
        uint64_t there;
        while ((there = __builtin_amdgcn_ballot_w64(c1 > i)) == 0) { base += 64; read_table(); }
        return __builtin_ctzll(there);
    }
    __device__ __forceinline__ void init_ctx(const KvView& kv, int t0, int t1_, int wave, int waves, long stride_, long head_) {
        stride = stride_; head = head_; cu = kv.cu; kt = kv.k_chunks; vt = kv.v_chunks; n_chunks = kv.n_chunks;
        t = t0 + 32 * wave; step = 32 * waves; np = 0; ka = va = kb = vb = nullptr;
        base = n_chunks <= 64 ? 0 : find_chunk(cu, n_chunks, t);
        t1 = t1_;
        end = cu[n_chunks];
        read_table();
    }
    // (after init_ctx, when its loads have come back) stay inside the table whatever the caller says
    __device__ __forceinline__ void clamp() { if (cu) t1 = min(t1, __builtin_amdgcn_readfirstlane(end)); }
    __device__ __forceinline__ void init_seq(const KvView& kv, int n, int wave, int waves, long stride_, long head_) {
        stride = stride_; head = head_; cu = nullptr; kt = vt = nullptr; n_chunks = base = 0; c0 = c1 = end = 0; kp = vp = 0;
        t = 32 * wave; step = 32 * waves; t1 = n; np = kv.prefix_len;
        ka = (const char*)kv.k_prefix + head; va = (const char*)kv.v_prefix + head;
        kb = (const char*)kv.k_self + head - np * stride; vb = (const char*)kv.v_self + head - np * stride;
    }
};

// A block of n tokens from index t on (0: none).
struct FewBlock {
    const char *k, *v;               // the row of the first; NULL: the walk's rows
    int n, t;
};
__device__ __forceinline__ FewBlock take(FewWalk& w) {
    FewBlock b{nullptr, nullptr, max(min(w.t1 - w.t, 32), 0), w.t};
    if (b.n == 0) return b;
    w.t += w.step;
    const int last = b.t + b.n - 1, tt = min(b.t + (int)(threadIdx.x & 31), last);
    if (w.cu) {
        int l = w.context_of(b.t);
        int from = __builtin_amdgcn_readlane(w.c0, l), to = __builtin_amdgcn_readlane(w.c1, l);
        uint64_t k = lane_u64(w.kp, l) + w.head, v = lane_u64(w.vp, l) + w.head;
        if (__builtin_expect(last < to, 1)) {
            b.k = (const char*)k + (long)(b.t - from) * w.stride; b.v = (const char*)v + (long)(b.t - from) * w.stride;
            return b;
        }
        for (;;) {
            if (tt >= from) { w.kr = k + (long)(tt - from) * w.stride; w.vr = v + (long)(tt - from) * w.stride; }
            if (last < to) return b;
            l = w.context_of(to);
            from = __builtin_amdgcn_readlane(w.c0, l); to = __builtin_amdgcn_readlane(w.c1, l);
            k = lane_u64(w.kp, l) + w.head; v = lane_u64(w.vp, l) + w.head;
        }
    }
    if (last < w.np || b.t >= w.np) {
        b.k = (last < w.np ? w.ka : w.kb) + b.t * w.stride; b.v = (last < w.np ? w.va : w.vb) + b.t * w.stride;
    } else {
        w.kr = (uint64_t)((tt < w.np ? w.ka : w.kb) + tt * w.stride); w.vr = (uint64_t)((tt < w.np ? w.va : w.vb) + tt * w.stride);
    }
    return b;
}

// Starts the loads of entry E (K tokens 0..15, K 16..31, V 0..15, V 16..31) of the block that was taken last.
template <typename T, int DP, int E>
__device__ __forceinline__ void start_entry(const FewBlock& b, const FewWalk& w, uint32_t width, const FewOffsets<T, DP>& full, const char* slot) {
    using X = Few<T, DP>;
    constexpr bool V = E >= 2;
    constexpr int first = 16 * (E & 1);
    const char* p = V ? b.v : b.k;
    if (__builtin_expect(p != nullptr && b.n == 32, 1)) {
        p += first * w.stride;
#pragma unroll
        for (int i = 0; i < X::LOADS; ++i) load_once(p, V ? full.v[i] : full.k[i], slot + 1024 * i);
    } else if (p != nullptr) {
#pragma unroll
        for (int i = 0; i < X::LOADS; ++i) load_once(p, few_offset<T, DP, V>(i, first, b.n, (uint32_t)w.stride, width), slot + 1024 * i);
    } else {
        const uint64_t r = V ? w.vr : w.kr;
#pragma unroll
        for (int i = 0; i < X::LOADS; ++i) {
            const int from = first + i * X::ROWS + (int)(threadIdx.x & 63) / X::CPR;
            const uint64_t at = (uint64_t)(uint32_t)__shfl((int)(uint32_t)(r >> 32), from) << 32 | (uint32_t)__shfl((int)(uint32_t)r, from);
            load_once((const char*)at + few_chunk<T, DP, V>(i, width), slot + 1024 * i);
        }
    }
}

// All but the youngest N entries have landed in the wavefront's ring.
template <typename T, int DP, int N>
__device__ __forceinline__ void wait_entries() {
    wait_loads<N * Few<T, DP>::LOADS>();
    asm volatile("" ::: "memory");
}
// The LDS reads so far are done: what they read may be written over.
__device__ __forceinline__ void reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ float max_groups(float x) {
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max_halves(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_groups(float x) {
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return sum_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Row = lane & 15; the four groups of 16 lanes share its tokens (scores: token 4 group + r of 16) and its dims (output: the same).
template <typename T, int DP>
struct FewRows {
    u32x4 q[Few<T, DP>::NS];         // chunk 4 s + group of the row
    float m, l;                      // softmax reference (units of ScoreScale) and this lane's share of the sum
    f32x4 o[Few<T, DP>::NB];
};

// S^T = K Q^T of an entry.  fp32 scores are summed in four chains, as in the tile kernels.
template <typename T, int DP>
__device__ __forceinline__ f32x4 few_scores(const char* slot, int koff, const FewRows<T, DP>& st) {
    f32x4 s[sizeof(T)] = {};
#pragma unroll
    for (int i = 0; i < Few<T, DP>::NS; ++i) {
        const u32x4 a = *(const u32x4*)(slot + (koff ^ (64 * i)));
        if constexpr (sizeof(T) == 2) {
            s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, st.q[i]), s[0], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(st.q[i][e]), s[e], 0, 0, 0);
        }
    }
    if constexpr (sizeof(T) == 4) return (s[0] + s[1]) + (s[2] + s[3]);
    return s[0];
}

// The probabilities of a block's scores.  nvis: how many of its tokens this lane's row sees.
template <typename T, int DP>
__device__ __forceinline__ void few_softmax(const f32x4& s0, const f32x4& s1, int nvis, const ScoreScale<T>& sc, FewRows<T, DP>& st, float (&p)[8]) {
    const int group = (threadIdx.x & 63) >> 4;
    float s[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
    const bool masked = __builtin_amdgcn_ballot_w64(nvis < 32) != 0;
    if (masked) {
#pragma unroll
        for (int r = 0; r < 8; ++r) s[r] = 16 * (r >> 2) + (r & 3) + 4 * group < nvis ? s[r] : -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 8; ++r) mx = fmaxf(mx, s[r]);
    mx = max_groups(mx) * sc.hi;                             // -inf: the row sees nothing here
    if (__builtin_amdgcn_ballot_w64(mx > st.m + kSlack) != 0) {
        const float m_new = mx > st.m + kSlack ? mx : st.m, alpha = ScoreScale<T>::exp_of(st.m - m_new);
        st.m = m_new;
        st.l *= alpha;
#pragma unroll
        for (int b = 0; b < Few<T, DP>::NB; ++b) st.o[b] *= alpha;
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) p[r] = sc.prob(s[r], st.m);
    // (fp32: a score of -inf times the scale's remainder need not be -inf, see the tile kernels)
    auto drop = [&]() {
#pragma unroll
        for (int r = 0; r < 8; ++r) p[r] = __float_as_uint(s[r]) == 0xff800000u ? 0.f : p[r];
    };
    auto sum = [&]() { return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])); };
    if (sizeof(T) == 4 && masked) drop();
    float x = sum();
    if constexpr (sizeof(T) == 4) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!finite(x)) != 0, 0)) { drop(); x = sum(); }
    }
    st.l += x;
}

// O^T += V^T P^T over 16 tokens of fp32 values.
template <int DP>
__device__ __forceinline__ void few_values(const char* slot, int voff, const float* p, FewRows<float, DP>& st) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < DP / 16; ++b)
            st.o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(*(const float*)(slot + (voff ^ (64 * b)) + r * 4 * DP), p[r], st.o[b], 0, 0, 0);
}

// Streams the walk's tokens past the rows.  The query rows' loads are the first entry, in slot 0, and started by the caller.
template <typename T, int DP>
__device__ __forceinline__ void few_stream(FewWalk& walk, const FewOffsets<T, DP>& full, uint32_t width, int d, float temperature, int lim, char* ring, FewRows<T, DP>& st) {
    using X = Few<T, DP>;
    const int lane = threadIdx.x & 63, row = lane & 15, group = lane >> 4;
    FewBlock cur = take(walk);
    if (cur.n == 0) return;
    int o[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) o[i] = (i + 1) % 5 * X::ENTRY;
    start_entry<T, DP, 0>(cur, walk, width, full, ring + o[0]);
    start_entry<T, DP, 1>(cur, walk, width, full, ring + o[1]);
    start_entry<T, DP, 2>(cur, walk, width, full, ring + o[2]);
    start_entry<T, DP, 3>(cur, walk, width, full, ring + o[3]);
    const int koff = row * X::PITCH + ((group ^ few_swz_k<X::PITCH>(row)) << 4);
    // V, bf16: the transposing read's token 4 group + row / 4, 8 bytes; fp32: token 4 group (+ r), dim row
    const int vrow = 4 * group + (sizeof(T) == 2 ? row >> 2 : 0), vchunk = (sizeof(T) == 2 ? (row & 3) >> 1 : row >> 2) ^ few_swz_v<T, X::PITCH>(vrow);
    const int voff = vrow * X::PITCH + (vchunk << 4) + (sizeof(T) == 2 ? (row & 1) * 8 : (row & 3) * 4);
    asm volatile("" : "+v"(temperature));                   // (the division is for the loads to hide)
    const ScoreScale<T> sc(d, temperature);
    wait_entries<T, DP, 4>();
#pragma unroll
    for (int i = 0; i < X::NS; ++i) {
        st.q[i] = *(const u32x4*)(ring + (koff ^ (64 * i)));
#pragma unroll
        for (int e = 0; e < 4; ++e) st.q[i][e] = 64u * i + 16u * group < width ? st.q[i][e] : 0u;      // zeros beyond head_dim
    }
    reads_done();
    FewBlock next = take(walk);
    if (next.n > 0) start_entry<T, DP, 0>(next, walk, width, full, ring + o[4]);
    for (;;) {
        const bool more = next.n > 0;
        if (more) wait_entries<T, DP, 4>(); else wait_entries<T, DP, 3>();
        const f32x4 s0 = few_scores<T, DP>(ring + o[0], koff, st);
        reads_done();
        if (more) { start_entry<T, DP, 1>(next, walk, width, full, ring + o[0]); wait_entries<T, DP, 4>(); } else wait_entries<T, DP, 2>();
        const f32x4 s1 = few_scores<T, DP>(ring + o[1], koff, st);
        reads_done();
        if (more) start_entry<T, DP, 2>(next, walk, width, full, ring + o[1]);
        FewBlock after{nullptr, nullptr, 0, 0};
        const int nvis = min(cur.n, lim - cur.t + 1);
        float p[8];
        if constexpr (sizeof(T) == 2) {
            if (more) wait_entries<T, DP, 3>(); else wait_entries<T, DP, 0>();
            bf16x4 v0[X::NB], v1[X::NB];
#pragma unroll
            for (int b = 0; b < X::NB; ++b) { v0[b] = lds_read_tr(ring + o[2] + (voff ^ (32 * b))); v1[b] = lds_read_tr(ring + o[3] + (voff ^ (32 * b))); }
            few_softmax<T, DP>(s0, s1, nvis, sc, st, p);
            u32x4 h, l;                                      // probabilities as the sum of two bf16 values
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = pack_bf16(p[2 * i], p[2 * i + 1]);
                l[i] = pack_bf16(p[2 * i] - __uint_as_float(h[i] << 16), p[2 * i + 1] - __uint_as_float(h[i] & 0xffff0000u));
            }
            reads_done();
            if (more) {
                start_entry<T, DP, 3>(next, walk, width, full, ring + o[2]);
                after = take(walk);
                if (after.n > 0) start_entry<T, DP, 0>(after, walk, width, full, ring + o[3]);
            }
#pragma unroll
            for (int b = 0; b < X::NB; ++b) {
                const bf16x8 a = __builtin_shufflevector(v0[b], v1[b], 0, 1, 2, 3, 4, 5, 6, 7);
                st.o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, h), st.o[b], 0, 0, 0);
                st.o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, l), st.o[b], 0, 0, 0);
            }
        } else {
            few_softmax<T, DP>(s0, s1, nvis, sc, st, p);
            if (more) wait_entries<T, DP, 4>(); else wait_entries<T, DP, 1>();
            few_values<DP>(ring + o[2], voff, p, st);
            reads_done();
            if (more) { start_entry<T, DP, 3>(next, walk, width, full, ring + o[2]); wait_entries<T, DP, 4>(); } else wait_entries<T, DP, 0>();
            few_values<DP>(ring + o[3], voff, p + 4, st);
            reads_done();
            if (more) {
                after = take(walk);
                if (after.n > 0) start_entry<T, DP, 0>(after, walk, width, full, ring + o[3]);
            }
        }
        if (!more) break;
        cur = next; next = after;
        const int o4 = o[4];
        o[4] = o[3]; o[3] = o[2]; o[2] = o[1]; o[1] = o[0]; o[0] = o4;
    }
}

// r / group as (r * inverse) >> kFewShift, the inverse rounded up: exact as long as r * group < 2^kFewShift, and both are 512 or less.
constexpr int kFewShift = 20;

// A split's workgroup writes a partial result.  WHOLE: one workgroup per (request, KV head), with wavefronts of their own for the contexts and for the
// prefix and own tokens, whose results make the output.
template <typename T, typename Args, int DP, int W, bool WHOLE>
__global__ __launch_bounds__(64 * W) void few_rows_kernel(const Args a, const int group, const uint32_t group_inv) {
    using X = Few<T, DP>;
    constexpr bool ONE = Args::kRequests == 1;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), row = lane & 15;
    const int d = a.head_dim, hq = a.n_q_heads, hkv = a.n_kv_heads, G = group, q_len = a.q_len;
    // grid: x = KV head (the heads of a token's row are read at about the same time), y = the splits of all requests, then the short prefix +
    // own streams, z = rows.
    const int hk = blockIdx.x, y = blockIdx.y, n_splits = WHOLE ? 0 : (ONE ? 1 : a.n_req) * a.n_ctx_splits;
    int rq = ONE ? 0 : y - n_splits, split = a.n_ctx_splits;
    const bool own = y >= n_splits;
    if (!own) {
        if constexpr (ONE) split = y;
        else { rq = y / a.n_ctx_splits; split = y - rq * a.n_ctx_splits; }
    }
    const KvView kv = load_view<Args>(rq);
    const long stride = (long)hkv * d * sizeof(T), head = (long)hk * d * sizeof(T);
    const uint32_t width = (uint32_t)sizeof(T) * d;
    const int rows = q_len * G, R0 = 16 * blockIdx.z, R = min(R0 + row, rows - 1);
    auto token_of = [&](int r) { return (int)(r * group_inv >> kFewShift); };   // r / G
    const int tok = token_of(R);

    // the wavefront's stream, which it shares with `waves` others: tokens [t0, t1) of the contexts (from_ctx), or the prefix and the own tokens
    long t0 = 0, t1 = 0;
    const int off = kv.prefix_len + kv.self_len - q_len, n_seq = off + token_of(min(R0 + 15, rows - 1)) + 1;   // (index of query token 0; what the rows see)
    int n_ctx_waves = W, w0 = wave, waves = W;               // the first n_ctx_waves wavefronts have contexts
    bool from_ctx = !own;
    if constexpr (WHOLE) {
        t1 = kv.total_ctx;
        const int cu = (int)((t1 + 31) / 32), su = (n_seq + 31) / 32;
        n_ctx_waves = cu == 0 ? 0 : min(max((int)(W * (float)cu * __builtin_amdgcn_rcpf((float)(cu + su)) + 0.5f), 1), W - 1);
        n_ctx_waves = __builtin_amdgcn_readfirstlane(n_ctx_waves);
        from_ctx = wave < n_ctx_waves;
        waves = from_ctx ? n_ctx_waves : W - n_ctx_waves; w0 = from_ctx ? wave : wave - n_ctx_waves;
    } else if (!own) {
        ctx_split_range(a, kv, split, t0, t1);
        if (t0 >= t1) return;                                // an empty split: the merge never looks at it
    }

    char* const ring = lds + wave * X::WAVE;
    FewRows<T, DP> st;
    st.m = kNone; st.l = 0.f;
#pragma unroll
    for (int b = 0; b < X::NB; ++b) st.o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (32 * w0 < (from_ctx ? (int)(t1 - t0) : n_seq)) {
        FewWalk walk;
        if (from_ctx) walk.init_ctx(kv, (int)t0, (int)t1, w0, waves, stride, head); else walk.init_seq(kv, n_seq, w0, waves, stride, head);
        const char* q = (const char*)a.q + ((long)rq * q_len * hq + hk * G) * width;
#pragma unroll
        for (int i = 0; i < X::LOADS; ++i) {
            const int r = min(R0 + i * X::ROWS + lane / X::CPR, rows - 1);
            load_lds16(q, (uint32_t)(token_of(r) * (hq - G) + r) * width + few_chunk<T, DP, false>(i, width), ring + 1024 * i);
        }
        FewOffsets<T, DP> full;
        const uint32_t down = lane / X::CPR * (uint32_t)stride;
#pragma unroll
        for (int i = 0; i < X::LOADS; ++i) {
            full.k[i] = down + i * X::ROWS * (uint32_t)stride + few_chunk<T, DP, false>(i, width);
            full.v[i] = down + i * X::ROWS * (uint32_t)stride + few_chunk<T, DP, true>(i, width);
        }
        walk.clamp();
        few_stream<T, DP>(walk, full, width, d, from_ctx ? kv.temperature : 1.f, from_ctx ? INT32_MAX - 1 : off + tok, ring, st);
        wait_loads<0>();                                     // (the query rows of a walk without a token)
    }

    // The wavefronts' results are pooled: each puts its own where its ring was, then takes its share of the dims of all rows.
#pragma unroll
    for (int b = 0; b < X::NB; ++b) *(f32x4*)(ring + 1024 * b + 16 * lane) = st.o[b];
    const float sum = sum_groups(st.l);
    if (lane < 16) *(f32x2*)(ring + X::BOX + 8 * row) = f32x2{st.m, sum};
    __syncthreads();
    constexpr int SHARE = (X::NB + W - 1) / W;
    const int b0 = wave * SHARE;
    if (b0 >= X::NB) return;
    f32x2 ml[W];
#pragma unroll
    for (int w = 0; w < W; ++w) ml[w] = *(const f32x2*)(lds + w * X::WAVE + X::BOX + 8 * row);
    bool far = false;
    float mc = kNone, ms = kNone, lc = 0.f, ls = 0.f;        // contexts (or the split); prefix and own tokens
#pragma unroll
    for (int w = 0; w < W; ++w) {
        far |= fabsf(ml[w][0]) > kFar && ml[w][0] > kNone;
        if (w < n_ctx_waves) mc = fmaxf(mc, ml[w][0]); else ms = fmaxf(ms, ml[w][0]);
    }
    float f[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        f[w] = ScoreScale<T>::exp_of(ml[w][0] - (w < n_ctx_waves ? mc : ms));
        if (w < n_ctx_waves) lc = fmaf(ml[w][1], f[w], lc); else ls = fmaf(ml[w][1], f[w], ls);
    }
    float m = mc, l = lc;
    if constexpr (WHOLE) {
        // contexts: weight S times their LogSumExp, values normalised (Appendix C.3/C.4)
        const bool any = seen(lc);
        const float nat = kv.scale * ScoreScale<T>::lse(mc, lc), ac = !any ? kNone : sizeof(T) == 4 ? nat : nat * LOG2E;
        m = fmaxf(ac, ms);
        const float wc = any ? ScoreScale<T>::exp_of(ac - m) : 0.f, ws = ScoreScale<T>::exp_of(ms - m);
        l = fmaf(ls, ws, wc);
        const float fc = any ? wc / (lc * l) : 0.f, fs = ws / l;
#pragma unroll
        for (int w = 0; w < W; ++w) f[w] *= w < n_ctx_waves ? fc : fs;
    } else {
        const float inv = seen(l) ? 1.f / l : 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) f[w] *= inv;
    }
    const bool valid = R0 + row < rows;
    const int h = hk * G + R - tok * G;
    const long unit = ((long)(a.req_base + rq) * q_len + tok) * hq + h;
    const long part0 = (long)split * a.units_total + (long)(a.req_base + rq) * q_len * hq;
    f32x4 out[SHARE];
    bool odd = far || !finite(l);
#pragma unroll
    for (int b = 0; b < SHARE; ++b) {
        out[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const f32x4 x = *(const f32x4*)(lds + w * X::WAVE + 1024 * (b0 + b) + 16 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) out[b][e] = fmaf(x[e], f[w], out[b][e]);
        }
        if (16 * (b0 + b) + 4 * (lane >> 4) < d)             // (values beyond head_dim are the row's first dims again)
#pragma unroll
            for (int e = 0; e < 4; ++e) odd |= !finite(out[b][e]);
    }
    const uint64_t odd_lanes = __builtin_amdgcn_ballot_w64(valid && odd);
    uint32_t redo = (uint32_t)odd_lanes | (uint32_t)(odd_lanes >> 32);
    redo = (redo | redo >> 16) & 0xffff;
    if (valid && !(redo >> row & 1)) {
        const long slot = part0 + (long)tok * hq + h;
#pragma unroll
        for (int b = 0; b < SHARE; ++b) {
            const int c = 16 * (b0 + b) + 4 * (lane >> 4);
            const float x[4] = {out[b][0], out[b][1], out[b][2], out[b][3]};
            if (c < d) { if constexpr (WHOLE) store4((T*)a.out + unit * d + c, x); else store4(a.part_o + slot * d + c, x); }
        }
        if (wave == 0 && lane < 16) {
            const float lse = seen(l) ? ScoreScale<T>::lse(m, l) : -INFINITY;
            if constexpr (!WHOLE) a.part_lse[slot] = lse;
            else if (a.lse_out) a.lse_out[a.lse_head_major ? ((long)(a.req_base + rq) * hq + h) * q_len + tok : unit] = lse;
        }
    }
    if (__builtin_expect(redo != 0, 0))
        redo_query_rows<T>(kernarg_again<Args>(), rq, hk, part0, (int)t0, (int)t1, own, WHOLE, R0, redo, 16 * b0, 16 * (b0 + SHARE));
}

template <typename T, typename Args, int DP, int W, bool WHOLE>
hipError_t few_as(const QueryArgs& q, hipStream_t s) {
    const Args a(q);
    auto kernel = few_rows_kernel<T, Args, DP, W, WHOLE>;
    const int splits = WHOLE ? 0 : q.n_req * q.n_ctx_splits, group = q.n_q_heads / q.n_kv_heads, lds = W * Few<T, DP>::WAVE;
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    kernel<<<dim3((unsigned)q.n_kv_heads, (unsigned)(splits + q.n_req), (unsigned)((q.q_len * group + 15) / 16)), 64 * W, lds, s>>>
        (a, group, (uint32_t)(((1 << kFewShift) + group - 1) / group));
    return hipGetLastError();
}
template <typename T, int DP>
hipError_t few_with(const QueryArgs& a, FewForm form, hipStream_t s) {
    constexpr int W = 160 * 1024 / Few<T, DP>::WAVE;
    const bool one = OneQuery::holds(a);
    if (form == FewForm::whole) return one ? few_as<T, OneQuery, DP, W, true>(a, s) : few_as<T, QueryArgs, DP, W, true>(a, s);
    if (form == FewForm::full) return one ? few_as<T, OneQuery, DP, W, false>(a, s) : few_as<T, QueryArgs, DP, W, false>(a, s);
    return one ? few_as<T, OneQuery, DP, W / 2, false>(a, s) : few_as<T, QueryArgs, DP, W / 2, false>(a, s);
}
template <typename T>
hipError_t few_of(const QueryArgs& a, FewForm form, hipStream_t s) {
    if constexpr (sizeof(T) == 2)
        if (a.head_dim > 128) return few_with<T, 256>(a, form, s);
    return a.head_dim <= 64 ? few_with<T, 64>(a, form, s) : few_with<T, 128>(a, form, s);
}

}  // namespace

hipError_t launch_few_rows(const QueryArgs& a, int dtype, FewForm form, hipStream_t s) {
    return dtype == APE_F32 ? few_of<float>(a, form, s) : few_of<__bf16>(a, form, s);
}

}  // namespace ape
