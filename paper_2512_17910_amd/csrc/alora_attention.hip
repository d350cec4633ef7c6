// Reader of the paged K/V cache: causal softmax attention of query rows over the cached keys and
// values of their sequences (Sec. 2.1; formula and layout in alora_attention.h).
//
// One workgroup (4 wavefronts) per (query row, K/V head); the G = n_q_heads / n_kv_heads query heads
// that share the K/V head are processed together, so every cached byte is loaded once per row.
// The work is a stream of K and V rows (2 * head_dim elements per context position and K/V head)
// against 4 * G * head_dim flops: memory-bound, so plain fp32 vector arithmetic, no LDS staging and
// no matrix instructions.  Contexts of a decode batch, which differ, are started longest first (see
// longest_first) and in bf16, where no other row reads them too, with non-temporal loads (contexts_read_once): equal contexts come at 6.2 TB/s, where a plain
// read of a large buffer reaches 6.3 with ordinary and 7.05 with non-temporal loads (ordinary loads here: 5.6).
//
// Lane layout: head_dim / 8 lanes share one context position, 8 consecutive elements (16 bytes of
// bf16) each, so a wavefront's load instruction covers 64 / (head_dim / 8) positions with whole
// contiguous head rows.  The partial dot products are summed over those lanes with DPP adds
// (quad swaps, then half-row and row mirrors: every lane ends with the same bits).  Each lane
// group keeps its own running (max, sum, weighted V) -- 16 or 32 independent streams per
// workgroup -- rescaled once per U positions; the streams are merged in a fixed order at the end
// (lane groups by shuffles, wavefronts through LDS), so the result does not depend on timing.
#include "alora_internal.h"
#include "alora_attention.h"
#include <type_traits>
#include "alora_attention_internal.h"
#include <new>
#include <algorithm>
#include <vector>

namespace alora {


template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true);
    return v + __int_as_float(o);
}

// sum over the LPP lanes that share a position; all of them receive it
template <int LPP>
__device__ __forceinline__ float group_sum(float v)
{
    v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);   // row_half_mirror: the other quad of the 8 lanes
    if (LPP == 16) v = dpp_add<0x140>(v);   // row_mirror: the other half of the 16 lanes
    return v;
}

// 8 consecutive elements of a cache or query row, as loaded
template <bool BF16> struct Raw8;
template <> struct Raw8<true> {
    u32x4 v;
    __device__ __forceinline__ void zero() { v = u32x4{0u, 0u, 0u, 0u}; }
    template <bool STREAM = false>
    __device__ __forceinline__ void load(const void *base, size_t elem)
    {
        const u32x4 *p = (const u32x4 *)((const bf16_t *)base + elem);
        v = STREAM ? __builtin_nontemporal_load(p) : *p;
    }
    __device__ __forceinline__ void widen(float f[8]) const
    {
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
        f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
        f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
    }
};
template <> struct Raw8<false> {
    f32x4 a, b;
    __device__ __forceinline__ void zero() { a = f32x4{0.f, 0.f, 0.f, 0.f}; b = a; }
    template <bool = false>    // (always ordinary loads)
    __device__ __forceinline__ void load(const void *base, size_t elem)
    {
        a = *(const f32x4 *)((const float *)base + elem);
        b = *(const f32x4 *)((const float *)base + elem + 4);
    }
    __device__ __forceinline__ void widen(float f[8]) const
    {
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
        f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
};

constexpr float NEG_INF = -__builtin_inff();

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// <q chunk, k chunk> over 8 elements.  bf16: four packed two-element dot products on the stored bits
// (fp32 accumulate); fp32: eight FMAs.  The pairs are taken with shufflevector on the 8-element vector:
// bit casts of the single 32-bit words were compiled into four uses of the first word by this toolchain.
__device__ __forceinline__ float dot8(const Raw8<true> &q, const Raw8<true> &k)
{
    const bf16x8 qv = __builtin_bit_cast(bf16x8, q.v), kv = __builtin_bit_cast(bf16x8, k.v);
    float d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(qv, qv, 0, 1), __builtin_shufflevector(kv, kv, 0, 1), 0.f, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(qv, qv, 2, 3), __builtin_shufflevector(kv, kv, 2, 3), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(qv, qv, 4, 5), __builtin_shufflevector(kv, kv, 4, 5), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(qv, qv, 6, 7), __builtin_shufflevector(kv, kv, 6, 7), d, false);
    return d;
}
__device__ __forceinline__ float dot8(const Raw8<false> &q, const Raw8<false> &k)
{
    float d = q.a.x * k.a.x;
    d = fmaf(q.a.y, k.a.y, d); d = fmaf(q.a.z, k.a.z, d); d = fmaf(q.a.w, k.a.w, d);
    d = fmaf(q.b.x, k.b.x, d); d = fmaf(q.b.y, k.b.y, d); d = fmaf(q.b.z, k.b.z, d); d = fmaf(q.b.w, k.b.w, d);
    return d;
}

// The running maximum starts at a large negative FINITE number: differences with it stay finite, so the
// softmax needs no "nothing seen yet" cases (a position that is left out scores -inf and weighs
// exp2(-inf) = 0).  Scores below it are treated like -inf.
constexpr float M_FLOOR = -1.0e30f;

// What is known of a call's contexts: nothing, that there are no more rows than sequences (see contexts_read_once), or that there are several turns
// of workgroups of them besides, which take the longest first: whole contexts (in runs of `sorted` batch rows), or some in more parts than others.
enum Contexts { ANY, READ_ONCE, LONGEST_FIRST, IN_PARTS };

// Which row, K/V head and part of the context workgroup b is for when the longest contexts go first; of 256 threads.  Lengths count in
// steps of an eighth (128 of them from 16 positions to a million), rows of one step in batch order: every workgroup finds the same
// order, and each row once.  Where no context is longer than SHORT_CONTEXT, or rows read together (see there), it is the batch's order.  Without parts the order is that
// of every `sorted` rows (at most 256).  In parts there are no more rows than that; those of a.splits parts (see parts_of) come first, where there are
// none the batch's order stays, and the last workgroups find nothing to do (t = -1).  scr: ORDER_SCRATCH ints of LDS.  near: this thread's row.
// GROUPS: look for rows that read together.
struct Turn { int t, seq, pos, hk, part; };
struct Near { int t, seq, n_ctx; };   // a row, its sequence and context (0: none)
constexpr int ORDER_SCRATCH = 128 + 8 + 2;
constexpr int SHORT_CONTEXT = 512;
constexpr int LONG_PART = 512;      // positions per part from which a context is cut into the larger number of parts
__device__ __forceinline__ int parts_of(const AttnArgs &a, int n_ctx) { return n_ctx < a.splits * LONG_PART ? a.short_splits : a.splits; }
template <bool PARTS, bool GROUPS>
__device__ __forceinline__ Turn longest_first(const AttnArgs &a, int sorted, int b, int *scr, Near &near, bool &together)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned long long *const masks = (unsigned long long *)(scr + 128);
    const int first = PARTS ? 0 : b / a.Hkv / sorted * sorted, rows = min(sorted, a.T - first);
    int key = -1, n_ctx = 0, sq = -1, p = -1;
    bool more = false;
    if (tid < rows) {
        sq = a.seq[first + tid], p = a.pos[first + tid];
        if (sq >= 0 && sq < a.n_seqs && p >= 0) n_ctx = (int)min(p + 1ll, (long long)a.max_blocks * a.bs);
        key = 127 - min(max((int)(__float_as_uint((float)n_ctx) >> 20) - ((127 + 4) << 3), 0), 127);
        more = PARTS && parts_of(a, n_ctx) > a.short_splits;
        if (PARTS) key = (more ? 0 : 64) + (key >> 1);   // (steps of a quarter)
    }
    near = {first + tid, sq, n_ctx};
    if (tid < 128) scr[tid] = 0;
    b -= first * a.Hkv;
    int rank, unit, parts = PARTS ? a.short_splits : 1;
    bool ordered = n_ctx > SHORT_CONTEXT;
    if (PARTS) {
        const int n_more = __syncthreads_count(more), in_more = n_more * a.splits * a.Hkv;
        ordered = n_more > 0;
        if (b < in_more) parts = a.splits;
        else b -= in_more;
        unit = parts * a.Hkv;
        rank = b / unit;
        b -= rank * unit;
        if (parts == a.short_splits) rank += n_more;
        if (rank >= rows) return {-1, -1, -1, 0, 0};
    } else {
        unit = a.Hkv;
        rank = b / unit;
        b -= rank * unit;
    }
    const int hk = b / parts, part = b - hk * parts;
    if (tid == rank) scr[136] = sq, scr[137] = p;
    // Groups of rows that read one context: a row goes with the one before it in the batch if both read the same cache block half way through
    // the shorter of the two.  Where three quarters of the rows are in groups, of eight on average or fewer, the batch's order stays, in which a group
    // reads its context together, with ordinary loads.  us, longest first | batch order: 200 rows that share 1024 of 1075 to 1625 positions in pairs, 8/8
    // heads 184 | 152, 16/8 185 | 155, 32/8 195 | 170 (64/8 265 | 272: not looked for), in fours 8/8 175 | 127, 32/8 186 | 160, in eights 158 | 114 and 171 | 157;
    // half of the rows in pairs 243 | 257 and 260 | 279; a chunk of 144 rows beside 56 others 308 | 333; one prefix for all 196 | 207.
    bool same = false;
    if (GROUPS && tid > 0 && tid < rows) {
        const int sq1 = a.seq[first + tid - 1], half = min(n_ctx, a.pos[first + tid - 1] + 1) >> 1;
        if (half > SHORT_CONTEXT / 2 && sq1 >= 0 && sq1 < a.n_seqs) {
            const int at = a.bs_shift >= 0 ? half >> a.bs_shift : half / a.bs;
            same = a.bt[(size_t)sq * a.max_blocks + at] == a.bt[(size_t)sq1 * a.max_blocks + at];
        }
    }
    const unsigned long long with_last = __builtin_amdgcn_ballot_w64(same);
    const int begin = (int)__builtin_popcountll(with_last & ~(with_last << 1)), in_groups = begin + (int)__builtin_popcountll(with_last);
    if (lane == 0) scr[128 + w] = (__builtin_amdgcn_ballot_w64(ordered) ? 1 << 24 : 0) + (begin << 12) + in_groups;   // (64 and 128 at most)
    __syncthreads();
    const int all = scr[128] + scr[129] + scr[130] + scr[131];
    together = GROUPS && 8 * ((all >> 12) & 0xfff) >= rows && 4 * (all & 0xfff) >= 3 * rows;
    if (all < 1 << 24 || together) return {first + rank, scr[136], scr[137], hk, part};
    if (key >= 0) atomicAdd(&scr[key], 1);   // counts only: their values do not depend on the order
    __syncthreads();
    const int h0 = scr[2 * lane], h1 = scr[2 * lane + 1], upto = sum_upto64(h0 + h1);
    const int at = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(rank < upto));   // (rank < rows, the last lane's)
    int n = rank - __builtin_amdgcn_readlane(upto - h0 - h1, at);
    const int even = __builtin_amdgcn_readlane(h0, at), step = 2 * at + (n >= even ? 1 : 0);
    if (n >= even) n -= even;
    const unsigned long long mine = __builtin_amdgcn_ballot_w64(key == step);
    if (lane == 0) masks[w] = mine;
    __syncthreads();
    // the n-th of the step's rows: its thread says which it is
    int before = 0;
    for (int i = 0; i < w; ++i) before += (int)__builtin_popcountll(masks[i]);
    before += __builtin_amdgcn_mbcnt_hi((unsigned)(mine >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mine, 0u));
    if (key == step && before == n) scr[0] = first + tid, scr[136] = sq, scr[137] = p;
    __syncthreads();
    return {scr[0], scr[136], scr[137], hk, part};
}

template <int D, int G, bool BF16, bool POW2, Contexts CONTEXTS>
__global__ __launch_bounds__(256, G == 4 ? 3 : 1) void paged_attention_kernel(AttnArgs a, int sorted)
{
    constexpr int LPP = D / 8;         // lanes per context position
    constexpr int PPW = 64 / LPP;      // positions per wavefront and step
    constexpr int PPI = 4 * PPW;       // positions per workgroup and step
    constexpr int U = BF16 ? 4 : 2;    // steps per block: loaded together, one rescale of the running sums
    constexpr int BLK = PPI * U;       // positions per workgroup and block
    constexpr bool ORDERED = CONTEXTS == LONGEST_FIRST || CONTEXTS == IN_PARTS;
    constexpr bool STREAMED = BF16 && CONTEXTS != ANY;   // (see contexts_read_once)
    constexpr bool GROUPS = CONTEXTS == LONGEST_FIRST && G <= 4, LOOK = STREAMED && (CONTEXTS == IN_PARTS || (CONTEXTS == LONGEST_FIRST && G <= 2));   // (see there)
    constexpr bool MAY_SHARE = STREAMED && (GROUPS || LOOK);

    __shared__ float sm[4][G], sl[4][G];
    __shared__ float sacc[4][G][D];

    // workgroup -> (row, K/V head, part of the context)
    int t, sq, p, hk, sp;
    Near near = {-1, -1, 0};
    bool shared = false;      // contexts that rows of the call share
    if constexpr (ORDERED) {
        __shared__ __attribute__((aligned(8))) int order[ORDER_SCRATCH];
        const Turn turn = longest_first<CONTEXTS == IN_PARTS, GROUPS>(a, sorted, (int)blockIdx.x, order, near, shared);
        shared = __builtin_amdgcn_readfirstlane(shared);
        t = __builtin_amdgcn_readfirstlane(turn.t), sq = __builtin_amdgcn_readfirstlane(turn.seq), p = __builtin_amdgcn_readfirstlane(turn.pos);
        hk = turn.hk, sp = turn.part;
        if (t < 0) return;
    } else {
        const int rh = (int)blockIdx.x / a.splits;
        sp = (int)blockIdx.x - rh * a.splits;
        t = rh / a.Hkv, hk = rh % a.Hkv;
        sq = a.seq[t], p = a.pos[t];
    }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int grp = lane / LPP, c = lane % LPP;

    const long long cap = (long long)a.max_blocks * a.bs;
    int n_ctx = 0;
    if (sq >= 0 && sq < a.n_seqs && p >= 0) n_ctx = (int)(p + 1ll < cap ? p + 1ll : cap);
    const int32_t *bt = a.bt + (size_t)(n_ctx ? sq : 0) * a.max_blocks;
    // this workgroup's part of the context: whole blocks of BLK positions, the same number for every part
    int jbeg = 0;
    int parts = a.splits;
    if (a.splits > 1) {
        if constexpr (CONTEXTS == IN_PARTS) parts = parts_of(a, n_ctx);
        const int per = ((n_ctx + parts * BLK - 1) / (parts * BLK)) * BLK;
        jbeg = min(n_ctx, sp * per);
        n_ctx = min(n_ctx, jbeg + per);
    }
    // A part that another row of the run reads as well (the same cache block half way through it) takes ordinary loads: requests over one
    // cached prefix, adapters evaluated on one conversation.  us, non-temporal | ordinary, and in brackets all rows in batch order and fewer parts, 8/8
    // heads: 12 rows sharing 16K positions 126 | 97 (81), 100 sharing 2K, in parts 91 | 80 (96), 200 in 50 groups sharing 2K 306 | 277 (297); 32/8
    // heads, in parts: 12 sharing 16K 137 | 128 (126), 12 in pairs 148 | 135 (145), 8 sharing 32K 197 | 174 (190).  What the look costs is under the first loads:
    // 256 rows of 2 to 2047 positions, 8/8 heads 179.6 | 180.0, 40 in parts at 4 to 5K 123.5 | 123.9.  Batches of whole contexts and more heads take the same time either way.
    int half_here = -1, half_near = -2;
    if (LOOK && n_ctx > jbeg) {
        const int half = (jbeg + n_ctx) >> 1, at = POW2 ? (half >> a.bs_shift) : (half / a.bs);
        half_here = bt[at];
        if (near.t != t && near.n_ctx > half) half_near = a.bt[(size_t)near.seq * a.max_blocks + at];
    }
    const int Nkv = a.Hkv * D;
    const int col = hk * D + 8 * c;
    const int jl = wave * PPW + grp;   // this lane group's position inside a step
    const long long n_blocks = a.n_slots / a.bs;

    Raw8<BF16> qr[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qr[g].load(a.q, ((size_t)t * a.Hq + (size_t)hk * G + g) * D + 8 * c);

    float m[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = M_FLOOR;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    }

    // block-table entries of the block starting at j0 (-1 past the context).  Only the loads are issued
    // here: the entries are first looked at one block later, in fetch, so their latency is covered.
    auto lookup = [&](int j0, int (&blk)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * PPI + jl;
            blk[u] = -1;
            if (j < n_ctx) blk[u] = bt[POW2 ? (j >> a.bs_shift) : (j / a.bs)];
        }
    };
    // K and V chunks of the block starting at j0, through table entries looked up earlier; a position past
    // the context or with a table entry outside the cache is left out (zero chunks, validity bit clear).
    // Returns the validity of this lane's positions, one bit per step.
    auto fetch_as = [&](auto streamed, int j0, const int (&blk)[U], Raw8<BF16> (&kr)[U], Raw8<BF16> (&vr)[U]) {
        unsigned ok = 0;
        if (MAY_SHARE && decltype(streamed)::value) asm volatile("");   // (keeps the compiler from making one of the two kinds of load)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * PPI + jl;
            const bool have = blk[u] >= 0 && blk[u] < n_blocks;   // blk is -1 past the context
            ok |= (unsigned)have << u;
            kr[u].zero();
            vr[u].zero();
            if (have) {
                const int off = POW2 ? (j & (a.bs - 1)) : (j % a.bs);
                const size_t at = ((size_t)blk[u] * a.bs + off) * Nkv + col;
                kr[u].template load<decltype(streamed)::value>(a.kc, at);
                vr[u].template load<decltype(streamed)::value>(a.vc, at);
            }
        }
        if (MAY_SHARE && decltype(streamed)::value) asm volatile("");
        return ok;
    };
    auto fetch = [&](int j0, const int (&blk)[U], Raw8<BF16> (&kr)[U], Raw8<BF16> (&vr)[U]) {
        if constexpr (MAY_SHARE)
            if (shared) return fetch_as(std::false_type{}, j0, blk, kr, vr);
        return fetch_as(std::bool_constant<STREAMED>{}, j0, blk, kr, vr);
    };
    // scores, running softmax (rescaled once per block) and weighted sum of V for one block
    auto consume = [&](const Raw8<BF16> (&kr)[U], const Raw8<BF16> (&vr)[U], unsigned ok) {
        float s[U][G];   // in units of log2
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) s[u][g] = dot8(qr[g], kr[u]);
        // the sums over the lanes of a position, one reduction step at a time over all scores: consecutive
        // DPP instructions then work on different registers
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) s[u][g] = dpp_add<0xB1>(s[u][g]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) s[u][g] = dpp_add<0x4E>(s[u][g]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) s[u][g] = dpp_add<0x141>(s[u][g]);
        if (LPP == 16) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int g = 0; g < G; ++g) s[u][g] = dpp_add<0x140>(s[u][g]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) s[u][g] = ((ok >> u) & 1u) ? s[u][g] * a.scale_log2e : NEG_INF;
        float pw[U][G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mx = s[0][g];
#pragma unroll
            for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u][g]);
            const float mn = fmaxf(m[g], mx);
            const float corr = __builtin_amdgcn_exp2f(m[g] - mn);
            m[g] = mn;
            float ls = l[g] * corr;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pw[u][g] = __builtin_amdgcn_exp2f(s[u][g] - mn);
                ls += pw[u][g];
            }
            l[g] = ls;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] *= corr;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float vf[8];
            vr[u].widen(vf);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(pw[u][g], vf[e], acc[g][e]);
        }
    };

    // Two register sets: while one block is consumed the next block's K/V loads and the table entries of
    // the block after it are in flight.
    int blkA[U], blkB[U];
    Raw8<BF16> krA[U], vrA[U], krB[U], vrB[U];
    lookup(jbeg, blkA);
    unsigned okA = fetch(jbeg, blkA, krA, vrA), okB;
    lookup(jbeg + BLK, blkB);
    if constexpr (LOOK) {
        asm volatile("" : "+v"(half_here), "+v"(half_near));   // (looked at here, not where they are requested)
        shared = __builtin_amdgcn_readfirstlane(__syncthreads_or(half_here == half_near));
    }
    for (int j0 = jbeg; j0 < n_ctx; j0 += 2 * BLK) {
        okB = fetch(j0 + BLK, blkB, krB, vrB);
        lookup(j0 + 2 * BLK, blkA);
        consume(krA, vrA, okA);
        if (j0 + BLK < n_ctx) {
            okA = fetch(j0 + 2 * BLK, blkA, krA, vrA);
            lookup(j0 + 3 * BLK, blkB);
            consume(krB, vrB, okB);
        }
    }

    // merge the lane groups of a wavefront (same chunk c, different positions)
#pragma unroll
    for (int off = LPP; off < 64; off <<= 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float mo = __shfl_xor(m[g], off), lo = __shfl_xor(l[g], off);
            const float mn = fmaxf(m[g], mo);
            const float ca = __builtin_amdgcn_exp2f(m[g] - mn), cb = __builtin_amdgcn_exp2f(mo - mn);
            l[g] = l[g] * ca + lo * cb;
            m[g] = mn;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float ao = __shfl_xor(acc[g][e], off);
                acc[g][e] = acc[g][e] * ca + ao * cb;
            }
        }
    }
    if (grp == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (c == 0) { sm[wave][g] = m[g]; sl[wave][g] = l[g]; }
#pragma unroll
            for (int e = 0; e < 8; ++e) sacc[wave][g][8 * c + e] = acc[g][e];
        }
    }
    __syncthreads();

    // merge the four wavefronts in fixed order and store
    for (int idx = tid; idx < G * D; idx += 256) {
        const int g = idx / D, dd = idx % D;
        float M = sm[0][g];
#pragma unroll
        for (int w = 1; w < 4; ++w) M = fmaxf(M, sm[w][g]);
        float L = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = __builtin_amdgcn_exp2f(sm[w][g] - M);
            L += sl[w][g] * f;
            o += sacc[w][g][dd] * f;
        }
        if (a.splits > 1) {   // this part's (maximum, sum, unnormalised output); the merge kernel finishes
            float *const p0 = a.part + ((size_t)t * a.Hq + (size_t)hk * G + g) * a.splits * (D + 2), *pp = p0 + (size_t)sp * (D + 2);
            if (dd == 0) { pp[0] = M; pp[1] = L; }
            // fewer parts than there is room for: the last place tells how many (a sum of weights is never negative)
            if (CONTEXTS == IN_PARTS && dd == 0 && sp == 0 && parts < a.splits) *(f32x2 *)(p0 + (size_t)(a.splits - 1) * (D + 2)) = (f32x2){(float)parts, -1.f};
            pp[2 + dd] = o;
            continue;
        }
        const float y = L > 0.f ? o / L : 0.f;
        const size_t at = ((size_t)t * a.Hq + (size_t)hk * G + g) * D + dd;
        if (BF16) ((bf16_t *)a.out)[at] = (bf16_t)f32_to_bf16_bits(y);
        else ((float *)a.out)[at] = y;
    }
}

// Second pass of a split call: the parts of a (row, query head) are combined in a fixed order.  The pass is a
// few round trips to memory long and little else, so a workgroup requests everything it needs at once: D / 2
// lanes take one part (two elements each), 512 / D groups of them every NG-th part.  Measured (32/8 heads of 128): 8 rows in
// 16 parts 16.0 us with one part after the other, 5.0 us now; 256 rows in 8 parts (34 MB) 17.0 -> 9.0 us.
// COUNTED: the last part's place may hold how many there are instead, (number, -1); what lies between is not read.
template <int D, bool BF16, bool COUNTED>
__global__ __launch_bounds__(256) void paged_attention_merge_kernel(const float *__restrict__ part, void *__restrict__ out, int splits)
{
    constexpr int LP = D / 2, NG = 256 / LP, PER = MAX_PARTS / NG;
    __shared__ float gm[NG], gl[NG];
    __shared__ f32x2 go[NG][LP];
    const size_t rh = blockIdx.x;   // row * Hq + query head
    const int dd = threadIdx.x % LP, grp = threadIdx.x / LP;
    const float *pp = part + rh * splits * (D + 2);
    f32x2 ml[PER], ov[PER];
    auto load = [&](int i, bool there) {
        const int s2 = grp + NG * i;
        ml[i] = (f32x2){M_FLOOR, 0.f};
        ov[i] = (f32x2){0.f, 0.f};
        if (there) {
            ml[i] = *(const f32x2 *)(pp + (size_t)s2 * (D + 2));
            ov[i] = *(const f32x2 *)(pp + (size_t)s2 * (D + 2) + 2 + 2 * dd);
        }
    };
    constexpr int AHEAD = COUNTED ? 2 : PER;   // requested before it is known how many there are
    const int room = splits;
    f32x2 last = {};
    if (COUNTED) last = *(const f32x2 *)(pp + (size_t)(room - 1) * (D + 2));
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load(i, grp + NG * i < room);
    float M = M_FLOOR, L = 0.f;
    f32x2 o = {0.f, 0.f};
    auto combine = [&](auto n) {
#pragma unroll
        for (int i = 0; i < decltype(n)::value; ++i) M = fmaxf(M, ml[i].x);
#pragma unroll
        for (int i = 0; i < decltype(n)::value; ++i) {
            const float f = __builtin_amdgcn_exp2f(ml[i].x - M);
            L += ml[i].y * f;
            o.x += ov[i].x * f;
            o.y += ov[i].y * f;
        }
    };
    if (COUNTED) {
        splits = __builtin_amdgcn_readfirstlane(last.y < 0.f ? (int)last.x : room);
        if (room > AHEAD * NG) {
#pragma unroll
            for (int i = AHEAD; i < PER; ++i) load(i, grp + NG * i < splits);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (grp + NG * i >= splits) {      // (whatever the workspace held)
                ml[i] = (f32x2){M_FLOOR, 0.f};
                ov[i] = (f32x2){0.f, 0.f};
            }
        // (Where there is room for no more than these, the instructions of the others are left out: 21 thousand rows and heads in 3 parts
        // 15.2 us as a call without counted parts, 17.3 with and all the instructions, now 11.7.)
        if (room > AHEAD * NG) combine(std::integral_constant<int, PER>{});
        else combine(std::integral_constant<int, AHEAD>{});
    } else {
        combine(std::integral_constant<int, PER>{});
    }
    if (dd == 0) { gm[grp] = M; gl[grp] = L; }
    go[grp][dd] = o;
    __syncthreads();
    if (grp != 0) return;
    float Ma = gm[0];
#pragma unroll
    for (int g = 1; g < NG; ++g) Ma = fmaxf(Ma, gm[g]);
    float La = 0.f;
    f32x2 oa = {0.f, 0.f};
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const float f = __builtin_amdgcn_exp2f(gm[g] - Ma);
        La += gl[g] * f;
        oa.x += go[g][dd].x * f;
        oa.y += go[g][dd].y * f;
    }
    const float y0 = La > 0.f ? oa.x / La : 0.f, y1 = La > 0.f ? oa.y / La : 0.f;
    if (BF16) *(uint32_t *)((bf16_t *)out + rh * D + 2 * dd) = f32_to_bf16_bits(y0) | (f32_to_bf16_bits(y1) << 16);
    else *(f32x2 *)((float *)out + rh * D + 2 * dd) = (f32x2){y0, y1};
}

// Non-temporal loads where it may be assumed that a context is read once per head (no more rows than sequences; rows that share cache
// blocks all the same are found by the kernels that fill the chip) and the memory-side cache would not
// keep this layer's K and V until they are read again (its pool is taken for what is read: with the caches of twelve layers in turn, 39 MB read from each of 1 GB,
// 18.1 | 17.3; of three, which are still there the next time, 16.3 | 17.1).  us, ordinary | non-temporal loads, 32/8 heads, three layers' caches in turn:
// 64 rows of equal contexts, 500 MB 100.8 | 91.4, 200 MB 45.2 | 40.9, 100 MB 25.9 | 24.6, 64 MB 16.9 | 17.4; 256 rows of 10 to
// 100 positions, 66 MB 25.5 | 26.5; one cache over and over, 200 MB 38.5 | 40.4.  Not of fp32, whose positions take two loads per lane that share their lines:
// 16 rows at 500 to 1500 positions, 8/8 heads, twelve layers 57.7 | 72.9, 100 rows 145.7 | 165.8, head size 64, 8/4 heads 49.0 | 62.1, in parts 4 at 5000 to
// 9000 46.5 | 48.4 (the longest first, or in more parts, they go all the same: 100 rows 152.9 | 145.7, 12 in parts at 8000 to 14000 206 | 200).
static bool contexts_read_once(const alora_attn_dims *d)
{
    return d->n_tokens <= d->n_seqs && outgrows_cache(d->n_slots, d->n_kv_heads, d->head_dim, d->dtype == ALORA_BF16);
}

template <int D, int G>
static void launch_dg(const AttnArgs &a, bool bf16, hipStream_t st)
{
    const dim3 grid((unsigned)a.T * (unsigned)a.Hkv * (unsigned)a.splits);
    const bool pow2 = a.bs_shift >= 0;
    // The longest contexts first where workgroups take several turns on the chip (three per compute unit fit) and contexts can be
    // long: one of 2000 positions that starts last is half the call's length.  us, in batch order | longest first (non-temporal both): 256 rows of 2 to
    // 2047 positions 210 | 185, 100 of 300 to 3000 147 | 134, 250 of 100 to 4000, 64/8 heads 554 | 478.  Contexts of at most SHORT_CONTEXT
    // keep their order: finding it would be 2 of 25 us (256 rows of 10 to 100).  Of contexts in parts only where some are long enough for
    // the larger number (12 rows of 10K to 30K 196 | 169 with it; 7 of 3000 to 9000 43.4 | 44.9 by their order alone).
    const bool longest = a.once && a.T > 1 && (a.splits == 1 || a.short_splits < a.splits) && (long long)a.T * a.Hkv * a.splits > 512 && (long long)a.max_blocks * a.bs > SHORT_CONTEXT;
    const int runs = (a.T + 255) / 256, sorted = (a.T + runs - 1) / runs;
    auto launch = [&](auto is_bf16, auto is_pow2, auto contexts) {
        launch_kernel((paged_attention_kernel<D, G, decltype(is_bf16)::value, decltype(is_pow2)::value, decltype(contexts)::value>), grid, dim3(256), 0, st, a, sorted);
    };
    auto choose = [&](auto is_bf16, auto is_pow2) {
        if (longest && a.splits > 1) launch(is_bf16, is_pow2, std::integral_constant<Contexts, IN_PARTS>{});
        else if (longest) launch(is_bf16, is_pow2, std::integral_constant<Contexts, LONGEST_FIRST>{});
        else if (a.once && decltype(is_bf16)::value) launch(is_bf16, is_pow2, std::integral_constant<Contexts, decltype(is_bf16)::value ? READ_ONCE : ANY>{});
        else launch(is_bf16, is_pow2, std::integral_constant<Contexts, ANY>{});
    };
    if (bf16 && pow2) choose(std::true_type{}, std::true_type{});
    else if (bf16) choose(std::true_type{}, std::false_type{});
    else if (pow2) choose(std::false_type{}, std::true_type{});
    else choose(std::false_type{}, std::false_type{});
    if (a.splits > 1) {
        const dim3 mgrid((unsigned)a.T * (unsigned)a.Hq);
        const bool counted = a.short_splits < a.splits;
        if (bf16 && counted) launch_kernel((paged_attention_merge_kernel<D, true, true>), mgrid, dim3(256), 0, st, a.part, a.out, a.splits);
        else if (bf16) launch_kernel((paged_attention_merge_kernel<D, true, false>), mgrid, dim3(256), 0, st, a.part, a.out, a.splits);
        else if (counted) launch_kernel((paged_attention_merge_kernel<D, false, true>), mgrid, dim3(256), 0, st, a.part, a.out, a.splits);
        else launch_kernel((paged_attention_merge_kernel<D, false, false>), mgrid, dim3(256), 0, st, a.part, a.out, a.splits);
    }
}

template <int D>
static bool launch_d(const AttnArgs &a, int G, bool bf16, hipStream_t st)
{
    switch (G) {
    case 1: launch_dg<D, 1>(a, bf16, st); return true;
    case 2: launch_dg<D, 2>(a, bf16, st); return true;
    case 4: launch_dg<D, 4>(a, bf16, st); return true;
    case 8: launch_dg<D, 8>(a, bf16, st); return true;
    }
    return false;
}

static int check_dims(const alora_attn_dims *d)
{
    if (!d) return ALORA_EINVAL;
    if (d->dtype != ALORA_F32 && d->dtype != ALORA_BF16) return ALORA_EINVAL;
    if (d->n_tokens < 0 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_seqs < 0 || d->max_blocks < 0 ||
        d->block_size < 1 || d->n_slots < 0 || !(d->scale >= 0.f))
        return ALORA_EINVAL;
    if (d->head_dim != 64 && d->head_dim != 128) return ALORA_ESHAPE;
    if (d->n_q_heads % d->n_kv_heads) return ALORA_ESHAPE;
    const int G = d->n_q_heads / d->n_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return ALORA_ESHAPE;
    if ((long long)d->n_tokens * d->n_kv_heads > 0x7fffffffll || d->n_slots > 0x7fffffffll) return ALORA_ESHAPE;
    return ALORA_OK;
}

// Parts a row's context is cut into so that a small batch still fills the chip: about 1024 workgroups,
// at most 32 parts, one part when (rows x K/V heads) already gives that many.
static int parts_for(const alora_attn_dims *d, int workgroups)
{
    const long long wgs = (long long)d->n_tokens * d->n_kv_heads;
    if (wgs <= 0 || wgs >= 1024) return 1;
    return (int)std::min<long long>(MAX_PARTS, (workgroups + wgs - 1) / wgs);
}
static int plan_short_splits(const alora_attn_dims *d) { return parts_for(d, 1024); }
// About 2048 for contexts of LONG_PART positions and more in each part then, if the block tables have room for any and the longest go first: the chip holds 768
// workgroups (four query heads per K/V head), and what starts last should be small; of short contexts more parts are only more to
// combine.  us, 1024 | 1536 | 2048 for all: 8 rows of 32K to 64K positions 273 | 257 | 258, 12 of 10K to 30K 196 | 171 | 166, 5 with 64/8 heads
// 122 | 113 | 115; 6 of 1000 to 3000 20.0 | 23.1 | 23.3, 7 of 3000 to 9000 43.4 | 45.1 | 47.2.
static int plan_splits(const alora_attn_dims *d)
{
    const int parts = parts_for(d, 2048);
    const bool room = (long long)d->max_blocks * d->block_size >= (long long)parts * LONG_PART && contexts_read_once(d) && d->n_tokens > 1 && d->n_tokens <= 256;
    return room ? parts : plan_short_splits(d);
}

// The same for the row-block kernel, whose unit of work is a block of rows.
static BlockPlan block_plan(const alora_attn_dims *d, bool parts)
{
    return plan_blocks(d->n_tokens, d->n_seqs, d->n_kv_heads, d->n_q_heads / d->n_kv_heads, parts);
}

static size_t block_split_bytes(const alora_attn_dims *d)
{
    const int sp = block_plan(d, true).splits;
    if (sp <= 1) return 0;
    return (size_t)d->n_tokens * d->n_q_heads * sp * (d->head_dim + 2) * sizeof(float);
}

static size_t split_bytes(const alora_attn_dims *d, int sp)
{
    if (sp <= 1) return 0;
    return (size_t)d->n_tokens * d->n_q_heads * sp * (d->head_dim + 2) * sizeof(float);
}

// which kernel an entry point asks for
enum Reader { PER_ROW, PER_ROW_SPLIT, ROW_BLOCKS, ROW_BLOCKS_SPLIT };

static int run(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
               const int32_t *token_seq_ids, const int32_t *token_positions, void *out, const alora_attn_dims *dims,
               void *workspace, size_t workspace_bytes, Reader mode, void *hip_stream);

}  // namespace alora

extern "C" {

int alora_paged_attention_workspace_bytes(const alora_attn_dims *dims, size_t *out_bytes)
{
    using namespace alora;
    if (!out_bytes) return ALORA_EINVAL;
    const int st = check_dims(dims);
    if (st) return st;
    *out_bytes = split_bytes(dims, plan_splits(dims));
    return ALORA_OK;
}

int alora_paged_attention_split(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                                const int32_t *token_seq_ids, const int32_t *token_positions, void *out,
                                const alora_attn_dims *dims, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return alora::run(q, k_cache, v_cache, block_tables, token_seq_ids, token_positions, out, dims, workspace,
                      workspace_bytes, alora::PER_ROW_SPLIT, hip_stream);
}

int alora_paged_attention_suffix(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                                 const int32_t *token_seq_ids, const int32_t *token_positions, void *out,
                                 const alora_attn_dims *dims, void *hip_stream)
{
    return alora::run(q, k_cache, v_cache, block_tables, token_seq_ids, token_positions, out, dims, nullptr, 0,
                      alora::ROW_BLOCKS, hip_stream);
}

int alora_paged_attention_suffix_workspace_bytes(const alora_attn_dims *dims, size_t *out_bytes)
{
    using namespace alora;
    if (!out_bytes) return ALORA_EINVAL;
    const int st = check_dims(dims);
    if (st) return st;
    if (dims->dtype != ALORA_BF16 || dims->head_dim != 128) return ALORA_ESHAPE;
    *out_bytes = block_split_bytes(dims);
    return ALORA_OK;
}

int alora_paged_attention_suffix_split(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                                       const int32_t *token_seq_ids, const int32_t *token_positions, void *out,
                                       const alora_attn_dims *dims, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return alora::run(q, k_cache, v_cache, block_tables, token_seq_ids, token_positions, out, dims, workspace,
                      workspace_bytes, alora::ROW_BLOCKS_SPLIT, hip_stream);
}

int alora_paged_attention(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                          const int32_t *token_seq_ids, const int32_t *token_positions, void *out,
                          const alora_attn_dims *dims, void *hip_stream)
{
    return alora::run(q, k_cache, v_cache, block_tables, token_seq_ids, token_positions, out, dims, nullptr, 0,
                      alora::PER_ROW, hip_stream);
}

}  // extern "C"

namespace alora {

static int run(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
               const int32_t *token_seq_ids, const int32_t *token_positions, void *out, const alora_attn_dims *dims,
               void *workspace, size_t workspace_bytes, Reader mode, void *hip_stream)
{
    const int st = check_dims(dims);
    if (st) return st;
    const bool blocks_asked = mode == ROW_BLOCKS || mode == ROW_BLOCKS_SPLIT;
    if (blocks_asked && (dims->dtype != ALORA_BF16 || dims->head_dim != 128)) return ALORA_ESHAPE;
    // (the row-block kernel reads one table entry per four aligned positions; other block sizes, and a call
    // without table or cache, take the per-row kernel)
    const bool row_blocks = blocks_asked && dims->block_size % 4 == 0 && dims->n_seqs >= 1 && dims->max_blocks >= 1 &&
                            dims->n_slots >= dims->block_size;
    int splits = mode == PER_ROW_SPLIT ? plan_splits(dims) : (mode == ROW_BLOCKS_SPLIT && row_blocks) ? block_plan(dims, true).splits : 1;
    // (by rows: a workspace that holds the fewer parts is enough)
    if (mode == PER_ROW_SPLIT && workspace_bytes < split_bytes(dims, splits)) splits = plan_short_splits(dims);
    const size_t need = mode == PER_ROW_SPLIT ? split_bytes(dims, splits) : mode == ROW_BLOCKS_SPLIT ? block_split_bytes(dims) : 0;
    if (splits > 1 && (!workspace || ((uintptr_t)workspace & 15) || workspace_bytes < need)) return ALORA_EWORKSPACE;
    if (dims->n_tokens == 0) return ALORA_OK;
    if (!q || !k_cache || !v_cache || !block_tables || !token_seq_ids || !token_positions || !out) return ALORA_EINVAL;
    if (((uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)out) & 15) return ALORA_EINVAL;
    if (((uintptr_t)block_tables | (uintptr_t)token_seq_ids | (uintptr_t)token_positions) & 3) return ALORA_EINVAL;
    AttnArgs a;
    a.q = q; a.kc = k_cache; a.vc = v_cache;
    a.bt = block_tables; a.seq = token_seq_ids; a.pos = token_positions;
    a.out = out;
    a.T = dims->n_tokens; a.Hq = dims->n_q_heads; a.Hkv = dims->n_kv_heads;
    a.n_seqs = dims->n_seqs; a.max_blocks = dims->max_blocks; a.bs = dims->block_size;
    a.bs_shift = -1;
    for (int sft = 0; sft < 31; ++sft)
        if ((1 << sft) == dims->block_size) a.bs_shift = sft;
    a.n_slots = dims->n_slots;
    a.splits = splits;
    a.short_splits = mode == PER_ROW_SPLIT ? plan_short_splits(dims) : splits;
    a.once = contexts_read_once(dims);
    a.part = (float *)workspace;
    const float scale = dims->scale > 0.f ? dims->scale : 1.0f / sqrtf((float)dims->head_dim);
    a.scale_log2e = scale * 1.4426950408889634f;
    const bool bf16 = dims->dtype == ALORA_BF16;
    const int G = dims->n_q_heads / dims->n_kv_heads;
    if (row_blocks) {
        const BlockPlan plan = block_plan(dims, mode == ROW_BLOCKS_SPLIT);
        const int e2 = launch_attention_blocks(a, G, plan, (hipStream_t)hip_stream);
        if (e2) { note_hip_error(e2); return ALORA_EHIP; }
        if (splits > 1) {
            const dim3 grid((unsigned)a.T * (unsigned)a.Hq);
            if (plan.count) launch_kernel((paged_attention_merge_kernel<128, true, true>), grid, dim3(256), 0, (hipStream_t)hip_stream, a.part, a.out, a.splits);
            else launch_kernel((paged_attention_merge_kernel<128, true, false>), grid, dim3(256), 0, (hipStream_t)hip_stream, a.part, a.out, a.splits);
            const int e3 = launch_status();
            if (e3) { note_hip_error(e3); return ALORA_EHIP; }
        }
        return ALORA_OK;
    }
    const bool launched = dims->head_dim == 128 ? launch_d<128>(a, G, bf16, (hipStream_t)hip_stream)
                                                : launch_d<64>(a, G, bf16, (hipStream_t)hip_stream);
    if (!launched) return ALORA_ESHAPE;
    const int e = launch_status();
    if (e) { note_hip_error(e); return ALORA_EHIP; }
    return ALORA_OK;
}

}  // namespace alora

extern "C" {

int alora_paged_attention_validate(const int32_t *block_tables, const int32_t *token_seq_ids,
                                   const int32_t *token_positions, const alora_attn_dims *dims)
{
    using namespace alora;
    const int st = check_dims(dims);
    if (st) return st;
    if (dims->n_tokens == 0) return ALORA_OK;
    if (!block_tables || !token_seq_ids || !token_positions) return ALORA_EINVAL;
    const size_t T = (size_t)dims->n_tokens, nt = (size_t)dims->n_seqs * (size_t)dims->max_blocks;
    try {
    std::vector<int32_t> seq(T), pos(T), bt(nt);
    hipError_t e = hipDeviceSynchronize();
    if (!e) e = hipMemcpy(seq.data(), token_seq_ids, T * sizeof(int32_t), hipMemcpyDeviceToHost);
    if (!e) e = hipMemcpy(pos.data(), token_positions, T * sizeof(int32_t), hipMemcpyDeviceToHost);
    if (!e && nt) e = hipMemcpy(bt.data(), block_tables, nt * sizeof(int32_t), hipMemcpyDeviceToHost);
    if (e) { note_hip_error((int)e); return ALORA_EHIP; }
    const long long cap = (long long)dims->max_blocks * dims->block_size;
    const long long n_blocks = dims->n_slots / dims->block_size;
    std::vector<long long> reach((size_t)dims->n_seqs, -1);   // furthest position any row of the sequence reads
    for (size_t t = 0; t < T; ++t) {
        if (seq[t] < 0 || seq[t] >= dims->n_seqs) return ALORA_EDATA;
        if (pos[t] < 0 || pos[t] >= cap) return ALORA_EDATA;
        if (pos[t] > reach[(size_t)seq[t]]) reach[(size_t)seq[t]] = pos[t];
    }
    for (int s = 0; s < dims->n_seqs; ++s) {
        if (reach[(size_t)s] < 0) continue;
        const long long last = reach[(size_t)s] / dims->block_size;
        for (long long b = 0; b <= last; ++b) {
            const int32_t blk = bt[(size_t)s * dims->max_blocks + (size_t)b];
            if (blk < 0 || blk >= n_blocks) return ALORA_EDATA;
        }
    }
    return ALORA_OK;
    } catch (const std::bad_alloc &) {
        return ALORA_ENOMEM;
    }
}

}  // extern "C"
