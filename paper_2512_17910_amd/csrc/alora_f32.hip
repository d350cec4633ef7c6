// fp32 path (fp32 operands and fp32 accumulate throughout): the small-layer / reference-precision variant
// of the masked multi-adapter QKV projection.  Three kernels:
//   shrink_f32 : S[t,:] = x[t,:] . A[a]   for adapted rows only, one workgroup per row; for batches of at
//                most 256 rows the workgroups behind those do the grouping step (alora_group_small.h)
//   gemm_f32   : y = x . W on fp32 MFMA, then for adapted rows y += S[t,:] . B[a], the rotation where heads lie inside a tile of 64
//                features, then the q_out store and the paged K/V store; of small layers with few adapters the whole call
//   rope_f32   : the rotation of other heads, in place
// Pre-activation and base-model rows never read S, A or B (Sec. 2.3: they are the base model's).
//
// Such calls are small, so what bounds them is the number of dependent round trips to memory and of launches,
// not arithmetic: every wavefront requests all it needs before it multiplies.  Measured at 64 rows, hidden 256,
// 512 features, rank 8 (profiler): as three launches with a 64 x 64 LDS tile and a serial loop per rank column, grouping,
// shrink and projection took 4.4 + 8.4 + 23.1 us; shrink with grouping and projection 4.1 + 5.9; all in one launch 7.4 (the
// turn of projection and attention 38.5 -> 21.0 -> 12.2 us).  Error against fp64 2.7e-7 -> 1.5e-7.
#include "alora_internal.h"
#include "alora_group_small.h"

namespace alora {

constexpr int F32_THREADS = 256;

// One workgroup per token row.  Thread = (slice of the hidden dimension, rank column): consecutive threads read
// consecutive elements of A, eight rows per thread are requested at once, the slices are added in fixed order.
// The classification is worked out from the row's own metadata (no wait for a grouping kernel).
__global__ __launch_bounds__(F32_THREADS) void shrink_f32_kernel(const float *__restrict__ x, PtrTable A, RankTable ranks,
                                                                 GroupSmallArgs ga, int T, int L, int H, int r,
                                                                 float *__restrict__ S)
{
    __shared__ int scr[GROUP_SMALL_SCRATCH];
    if ((int)blockIdx.x >= T) {   // grouping of a batch of at most 256 rows, one block-table entry per workgroup
        int grp, cnt;
        group_small(ga, T, L, (int)blockIdx.x - T, true, scr, grp, cnt);
        return;
    }
    static_assert(GROUP_SMALL_SCRATCH >= F32_THREADS, "reduction array");
    float *red = (float *)scr;
    const int t = blockIdx.x;
    const int a = effective_adapter(ga.aid, ga.seg, ga.pos, ga.start, t);
    if (a < 0 || a >= L) return;
    const float *xr = x + (size_t)t * H;
    const float *Aa = (const float *)A.p[a];
    const int ra = ranks.r[a];   // this adapter's rank: A_a is [H, ra]; S keeps the common row pitch r
    const int slices = F32_THREADS / ra;          // ra <= 64: at least four
    const int tid = threadIdx.x, sl = tid / ra, j = tid - sl * ra;
    float acc = 0.f;
    if (sl < slices) {
        constexpr int U = 8;
        int k = sl;
        for (; k + (U - 1) * slices < H; k += U * slices) {
            float xv[U], av[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                xv[u] = xr[k + u * slices];
                av[u] = Aa[(size_t)(k + u * slices) * ra + j];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc = fmaf(xv[u], av[u], acc);
        }
        for (; k < H; k += slices) acc = fmaf(xr[k], Aa[(size_t)k * ra + j], acc);
    }
    red[tid] = acc;
    __syncthreads();
    if (tid < ra) {
        float s = 0.f;
        for (int i = 0; i < slices; ++i) s += red[i * ra + tid];
        S[(size_t)t * r + tid] = s;
    }
}

// Tile: 16 * MT token rows x 64 features, one workgroup; the four wavefronts take a quarter of the hidden
// dimension each, operands go from memory straight into the registers of 16x16x4 fp32 MFMAs.  The order of k
// inside a block of 16 is free as long as both operands agree: lane (c, g) = (lane % 16, lane / 16) holds
// x[row c][4g .. 4g+3] (one 16-byte load) and W[4g+j][4c .. 4c+3], j = 0..3; multiplication j of feature tile e
// takes element j of the former and element e of load j of the latter, so the 64 features of the tile are
// 4c + e.  Partial sums of the wavefronts meet in LDS and are added in fixed order.
// MT = 1 for small calls, as long as their chain of round trips: many short workgroups.  MT = 4 where the products count: a weight
// element serves 64 rows, but 64 KB of partial sums leave a CU two workgroups.  MT = 2 between (see launch_gemm_f32).
//
// Whole: the call's only launch.  A wavefront's quarter of its 16 token rows is in registers after one round trip, and one more product,
// with the rows of A, gives it S as well: every workgroup works S out for itself, which saves a launch and its 4.3 us where that is little
// work: hidden dimension at most 256, rank at most 16 (one tile of columns), at most four adapters (all of A requested together; one
// after the other, 16 adapters of a decode batch made a call 35 us of 21).  The grouping of at most 256 rows is done by workgroups behind
// the projection's.  us, shrink and projection | one launch, 256 -> 512: turn of 64 rows, rank 8 14.7 | 11.8, of 4 x 1 rows, rank 16, four
// adapters, rotation 17.4 | 16.0, 4 x 32 rows with rotation 24.0 | 17.9, 4 x 128 35.8 | 31.0; two layers of 256 rows 23.8 | 18.0.
constexpr int WHOLE_HIDDEN = 256, WHOLE_RANK = 16, WHOLE_ADAPTERS = 4;
struct RopeF32 { const float *cs, *sn; int n_pos, half; };   // cs null: no rotation in the store
// (Whole's further arguments are a type's, so that the other kernels are launched without them: 1.5 KB of tables more to write are 0.4 us a launch,
// four layers of 940 -> 6144 at five rows 70.9 without, 73.5 with)
struct Projection { static constexpr bool whole = false; struct More {}; };
struct Whole { static constexpr bool whole = true; struct More { PtrTable A; GroupSmallArgs group; }; };
template <int MT, typename CALL>
__global__ __launch_bounds__(F32_THREADS) void gemm_f32_kernel(
    const float *__restrict__ x, const float *__restrict__ W, const float *__restrict__ bias, PtrTable B,
    RankTable ranks, const float *__restrict__ S,
    const int32_t *__restrict__ aid, const int32_t *__restrict__ seg, const int32_t *__restrict__ pos,
    const int32_t *__restrict__ start, const int64_t *__restrict__ slot, float *__restrict__ q,
    float *__restrict__ kc, float *__restrict__ vc, int T, int H, int Nq, int Nkv, int r, RopeF32 rope, int L, typename CALL::More more)
{
    constexpr bool WHOLE = CALL::whole;
    static_assert(!WHOLE || MT == 1, "one row tile");
    __shared__ __attribute__((aligned(16))) float red[4][16 * MT][64];
    __shared__ float s_red[WHOLE ? 4 : 1][16][WHOLE_RANK + 1], s_sum[WHOLE ? 16 : 1][WHOLE_RANK];
    const int N = Nq + 2 * Nkv;
    const int m0 = blockIdx.y * (16 * MT), n0 = blockIdx.x * 64;
    if constexpr (WHOLE) {
        if (m0 >= T) {   // grouping of a batch of at most 256 rows, one block-table entry per workgroup
            static_assert(sizeof(red) >= GROUP_SMALL_SCRATCH * 4, "scratch");
            const int e = (blockIdx.y - (T + 15) / 16) * gridDim.x + blockIdx.x;
            int grp, cnt;
            if (e < more.group.n_blocks) group_small(more.group, T, L, e, true, (int *)red, grp, cnt);
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    f32x4 acc[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[m][e] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // classification of the rows whose outputs this thread stores: requested ahead of the products (WHOLE: of row c of the tile by
    // every wavefront, in three steps, see below)
    const int nn = n0 + 4 * (tid & 15);
    int a_of[MT];
    int aid_c = -1, seg_c = 0, pos_c = 0;
    if constexpr (WHOLE) {
        if (m0 + c < T) aid_c = aid[m0 + c], seg_c = seg[m0 + c], pos_c = pos[m0 + c];
    } else {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int t = m0 + 16 * m + (tid >> 4);
            a_of[m] = t < T ? effective_adapter(aid, seg, pos, start, t) : -1;
            if (a_of[m] >= L) a_of[m] = -1;
        }
    }

    const int KB = (H + 15) >> 4, per = (KB + 3) >> 2;   // blocks of 16, per wavefront
    const int kb0 = min(KB, w * per), kb1 = min(KB, kb0 + per);
    const int n_l = n0 + 4 * c;
    constexpr int D = MT == 1 ? 4 : 2;                   // blocks requested together
    static_assert(!WHOLE || 4 * 16 * D >= WHOLE_HIDDEN, "the quarter of a row a wavefront takes is requested at once");
    f32x4 xv[D][MT], wv[D][4];
    auto request = [&](int kb) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int k = 16 * (kb + d) + 4 * g;         // H is a multiple of 4: all four or none
            const bool k_ok = (kb + d < kb1) & (k < H);  // (no && here and below: a branch for each half makes four layers of 1000 -> 768 at three rows 57.8 us of 54.6)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                xv[d][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (k_ok & (m0 + 16 * m + c < T)) xv[d][m] = *(const f32x4 *)(x + (size_t)(m0 + 16 * m + c) * H + k);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                wv[d][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (k_ok & (n_l < N)) wv[d][j] = *(const f32x4 *)(W + (size_t)(k + j) * N + n_l);
            }
        }
    };
    auto multiply = [&]() {
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[m][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[d][m][j], wv[d][j][e], acc[m][e], 0, 0, 0);
    };
    f32x4 b8[8];     // WHOLE: the first rows of B_a for the row this thread stores, on their way beside those of A
    if constexpr (WHOLE) {
        request(kb0);
        int a_c = -1;
        if (aid_c >= 0 && aid_c < L && pos_c >= start[seg_c]) a_c = aid_c;
        a_of[0] = __shfl(a_c, 4 * w + g);
        // (the adapters' tables by constant index: a load that waits for the index is another 0.6 us)
        const void *Ba = nullptr;
        int ra = 1;
#pragma unroll
        for (int i = 0; i < WHOLE_ADAPTERS; ++i)
            if (a_of[0] == i) Ba = B.p[i], ra = ranks.r[i];
        if (a_of[0] >= 0 && nn < N) {
#pragma unroll
            for (int j = 0; j < 8; ++j) b8[j] = *(const f32x4 *)((const float *)Ba + nn + (size_t)min(j, ra - 1) * N);
        }
        // what lies past A_a (rows past the hidden dimension, columns past the rank) reads as zero
        unsigned rows[WHOLE_ADAPTERS];
        float av[WHOLE_ADAPTERS][D][4];
#pragma unroll
        for (int i = 0; i < WHOLE_ADAPTERS; ++i) {
            rows[i] = (unsigned)__builtin_amdgcn_ballot_w64(a_c == i) & 0xffffu;
            if (!rows[i]) continue;
            const int ri = ranks.r[i];
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)more.A.p[i], 0, H * ri * 4, 0x00020000);
            const uint32_t at = c < ri ? (uint32_t)((16 * kb0 + 4 * g) * ri + c) * 4u : 0x80000000u;
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    av[i][d][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, at + (uint32_t)((16 * d + j) * ri) * 4u, 0, 0));
        }
        multiply();
#pragma unroll
        for (int i = 0; i < WHOLE_ADAPTERS; ++i) {
            if (!rows[i]) continue;
            f32x4 sa[D];     // (a sum for every 16 of the hidden dimension: one after the other the error was 1.06 times the separate shrink's)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                sa[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (kb0 + d < kb1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) sa[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[d][0][j], av[i][d][j], sa[d], 0, 0, 0);
                }
            }
            static_assert(D == 4 || !WHOLE, "four sums");
            sa[0] = (sa[0] + sa[1]) + (sa[D - 2] + sa[D - 1]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((rows[i] >> (4 * g + e)) & 1u) s_red[w][4 * g + e][c] = sa[0][e];   // (a wavefront without a share of the hidden dimension: zeros)
        }
    } else {
        for (int kb = kb0; kb < kb1; kb += D) {
            request(kb);
            multiply();
        }
    }
    // D[row 4g + i][feature tile e, column c]: register i
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(f32x4 *)&red[w][16 * m + 4 * g + i][4 * c] = (f32x4){acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]};
    __syncthreads();
    if constexpr (WHOLE) {
        const int row = tid >> 4, j = tid & 15;
        if (a_of[0] >= 0) s_sum[row][j] = (s_red[0][row][j] + s_red[1][row][j]) + (s_red[2][row][j] + s_red[3][row][j]);
        __syncthreads();
    }
    if (nn >= N) return;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = 16 * m + (tid >> 4), t = m0 + row;
        if (t >= T) continue;
        int64_t s_at = -1;
        int p = 0;
        if (nn >= Nq) s_at = slot[t];
        const bool turned = rope.cs && nn < Nq + Nkv;
        if (turned) p = min(max(pos[t], 0), rope.n_pos - 1);
        f32x4 y = *(const f32x4 *)&red[0][row][4 * (tid & 15)];
#pragma unroll
        for (int ww = 1; ww < 4; ++ww) y += *(const f32x4 *)&red[ww][row][4 * (tid & 15)];
        if (bias) y += *(const f32x4 *)(bias + nn);   // part of the base output of every row
        const int a = a_of[m];
        if (a >= 0) {
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            const float *Ba = (const float *)B.p[a] + nn;
            const float *Sr = WHOLE ? s_sum[row] : S + (size_t)t * r;
            const int ra = ranks.r[a];
            if constexpr (WHOLE) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[e] = j < ra ? fmaf(Sr[j], b8[j][e], d[e]) : d[e];
            }
#pragma unroll 8
            for (int j = WHOLE ? 8 : 0; j < ra; ++j) {
                const float s = Sr[j];
                const f32x4 b4 = *(const f32x4 *)(Ba + (size_t)j * N);
                d.x = fmaf(s, b4.x, d.x); d.y = fmaf(s, b4.y, d.y);
                d.z = fmaf(s, b4.z, d.z); d.w = fmaf(s, b4.w, d.w);
            }
            y += d;
        }
        if (rope.cs) {
            // heads of 8, 16, 32 or 64: the partner features i +- half are the lane's half / 4 further on or back, of the same tile and row
            f32x4 other;
#pragma unroll
            for (int e = 0; e < 4; ++e) other[e] = __shfl_xor(y[e], rope.half >> 2);
            if (turned) {
                const bool first = !(nn & rope.half);
                const size_t at = (size_t)p * rope.half + (nn & (rope.half - 1));
                const f32x4 cv = *(const f32x4 *)(rope.cs + at), sv = *(const f32x4 *)(rope.sn + at);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = first ? y[e] * cv[e] - other[e] * sv[e] : y[e] * cv[e] + other[e] * sv[e];
            }
        }
        if (nn < Nq) {
            *(f32x4 *)(q + (size_t)t * Nq + nn) = y;
        } else if (s_at >= 0) {
            if (nn < Nq + Nkv) *(f32x4 *)(kc + (size_t)s_at * Nkv + (nn - Nq)) = y;
            else *(f32x4 *)(vc + (size_t)s_at * Nkv + (nn - Nq - Nkv)) = y;
        }
    }
}

// Rotary embedding on the fp32 path: the q_out rows and the K slots this call wrote, turned in place.  The
// stored values are the unrounded fp32 outputs, so this equals a rotation fused into the store.  One
// workgroup per token row; a thread takes the pairs (i, i + D/2) of the q heads and then of the k heads.
__global__ __launch_bounds__(256) void rope_f32_kernel(float *__restrict__ q, float *__restrict__ kc,
                                                       const int64_t *__restrict__ slot, const int32_t *__restrict__ pos,
                                                       const float *__restrict__ cs, const float *__restrict__ sn,
                                                       int n_pos, int Nq, int Nkv, int D)
{
    const int t = blockIdx.x, half = D / 2;
    const int p = min(max(pos[t], 0), n_pos - 1);
    const int64_t sl = slot[t];
    const int pairs = (Nq + Nkv) / 2;
    for (int idx = threadIdx.x; idx < pairs; idx += 256) {
        const int h = idx / half, i = idx % half;
        float *row;
        if (h * D < Nq) row = q + (size_t)t * Nq + h * D;
        else if (sl >= 0) row = kc + (size_t)sl * Nkv + (h * D - Nq);
        else continue;
        const float c = cs[(size_t)p * half + i], s = sn[(size_t)p * half + i];
        const float a = row[i], b = row[i + half];
        row[i] = a * c - b * s;
        row[i + half] = b * c + a * s;
    }
}

// Heads that lie inside a 64-feature tile of the projection are turned in its store.  (The tables are read 16 bytes at a time: half a
// multiple of four.)
static bool rope_in_store_f32(const Fwd &f) { return f.D == 8 || f.D == 16 || f.D == 32 || f.D == 64; }

int launch_rope_f32(const Fwd &f)
{
    if (f.T == 0 || rope_in_store_f32(f)) return 0;
    launch_kernel(rope_f32_kernel, dim3(f.T), dim3(256), 0, f.stream, (float *)f.q, (float *)f.kc, f.slot, f.pos,
                       f.rope_cos, f.rope_sin, f.rope_positions, f.Nq, f.Nkv, f.D);
    return launch_status();
}

// The grouping step of a small batch rides in the shrink's launch (its results are the caller's to read; the
// fp32 kernels themselves classify a row from its metadata).
bool group_in_shrink_f32(const Fwd &f) { return f.dtype == ALORA_F32 && f.L > 0 && f.T <= GROUP_SMALL_ROWS; }

static int rows_of_tile_f32(const Fwd &f)
{
    const long long tiles = (f.N + 63) / 64, tiles32 = (f.T + 31) / 32 * tiles, tiles64 = (f.T + 63) / 64 * tiles;
    if (tiles64 >= 768 && f.H >= 1024 && tiles64 * f.H >= 5ll << 18) return 64;
    return tiles32 >= 400 ? 32 : 16;
}

// One launch as long as its workgroups, of which a compute unit holds two, are on the chip together; more of them take turns, each as long as its chain
// of round trips.  us, two | one, four layers: 48 -> 1536, 400 rows (600 workgroups) 49.6 | 56.3, 48 -> 3072, 186 rows (576) 46.7 | 57.1, 256 -> 3072 59.2 | 60.7;
// 256 -> 6144, 64 rows (384) 47.7 | 43.7, 48 -> 384, 1000 rows (378) 45.2 | 42.7, 256 -> 1536, 186 rows (288) 48.2 | 41.1.
constexpr long long WHOLE_WORKGROUPS = 512;
static bool whole_call_f32(const Fwd &f)
{
    const long long workgroups = (long long)((f.N + 63) / 64) * ((f.T + 15) / 16);
    return f.L > 0 && f.L <= WHOLE_ADAPTERS && f.H <= WHOLE_HIDDEN && f.r <= WHOLE_RANK && rows_of_tile_f32(f) == 16 && workgroups <= WHOLE_WORKGROUPS;
}

int launch_shrink_f32(const Fwd &f, const PtrTable &A, bool reuse_grouping)
{
    if (f.T == 0 || f.L == 0 || whole_call_f32(f)) return 0;
    const GroupSmallArgs ga = {f.aid, f.seg, f.pos, f.start, f.active, f.aeff, f.perm, f.offsets, f.blocktab, f.n_blocks, nullptr};
    const int group_wgs = group_in_shrink_f32(f) && !reuse_grouping ? f.n_blocks : 0;
    launch_kernel(shrink_f32_kernel, dim3(f.T + group_wgs), dim3(F32_THREADS), 0, f.stream, (const float *)f.x, A, f.ranks, ga,
                       f.T, f.L, f.H, f.r, (float *)f.S);
    return launch_status();
}

int launch_gemm_f32(const Fwd &f, const PtrTable &B, const PtrTable &A, bool reuse_grouping)
{
    if (f.T == 0) return 0;
    // us for 16 | 32 | 64 rows a tile (and the 64 x 64 LDS tile before them): 256 -> 512, two layers, 1500 rows 28 | 30 | 33 (49), 2048 rows 32 | 31 |
    // 33 (49), 6000 rows 69 | 70 | 81 (73), 16384 rows 148 | 137 | 154 (145); 1024 -> 1536, two layers, 512 rows 61 | 62 | 65 (141), 1024
    // rows 115 | 95 | 115 (158), 4096 rows 385 | 322 | 309 (366); 4096 -> 6144, 100 rows 102 | 94 | 108 (281), 256 rows 214 | 147 | 174
    // (286), 512 rows 437 | 338 | 323 (386), 2048 rows 1822 | 1212 | 973 (1308).
    const int rows = rows_of_tile_f32(f);
    const bool whole = whole_call_f32(f);
    RopeF32 rope = {};
    if (f.rope_cos && rope_in_store_f32(f)) rope = RopeF32{f.rope_cos, f.rope_sin, f.rope_positions, f.D / 2};
    const GroupSmallArgs group = {f.aid, f.seg, f.pos, f.start, f.active, f.aeff, f.perm, f.offsets, f.blocktab, f.n_blocks, nullptr};
    dim3 grid((f.N + 63) / 64, (f.T + rows - 1) / rows);
    if (whole && group_in_shrink_f32(f) && !reuse_grouping) grid.y += (f.n_blocks + grid.x - 1) / grid.x;
    auto launch = [&](auto kernel, auto more) {
        launch_kernel(kernel, grid, dim3(F32_THREADS), 0, f.stream, (const float *)f.x, (const float *)f.W, (const float *)f.bias, B, f.ranks,
                      (const float *)f.S, f.aid, f.seg, f.pos, f.start, f.slot, (float *)f.q, (float *)f.kc, (float *)f.vc, f.T, f.H, f.Nq, f.Nkv,
                      f.r, rope, f.L, more);
    };
    if (rows == 64) launch(gemm_f32_kernel<4, Projection>, Projection::More{});
    else if (rows == 32) launch(gemm_f32_kernel<2, Projection>, Projection::More{});
    else if (whole) launch(gemm_f32_kernel<1, Whole>, Whole::More{A, group});
    else launch(gemm_f32_kernel<1, Projection>, Projection::More{});
    return launch_status();
}

}  // namespace alora
