// fp32 path (fp32 operands and fp32 accumulate throughout): the small-layer / reference-precision variant
// of the masked multi-adapter QKV projection.  Two kernels:
//   shrink_f32 : S[t,:] = x[t,:] . A[a]   for adapted rows only, one workgroup per row; for batches of at
//                most 256 rows the workgroups behind those do the grouping step (alora_group_small.h)
//   gemm_f32   : y = x . W on fp32 MFMA, then for adapted rows y += S[t,:] . B[a], then the q_out store and
//                the paged K/V store.
// Pre-activation and base-model rows never read S, A or B (Sec. 2.3: they are the base model's).
//
// Such calls are small, so what bounds them is the number of dependent round trips to memory and of launches,
// not arithmetic: every wavefront requests all it needs before it multiplies.  Measured at 64 rows, hidden 256,
// 512 features, rank 8: as three launches with a 64 x 64 LDS tile and a serial loop per rank column, grouping,
// shrink and projection took 4.4 + 8.4 + 23.1 us; shrink with grouping and projection now take 4.6 + 6.2 us (the
// turn of projection and attention 38.5 -> 21.0 us).  Error against fp64 2.7e-7 -> 1.5e-7.
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
template <int MT>
__global__ __launch_bounds__(F32_THREADS) void gemm_f32_kernel(
    const float *__restrict__ x, const float *__restrict__ W, const float *__restrict__ bias, PtrTable B,
    RankTable ranks, const float *__restrict__ S,
    const int32_t *__restrict__ aid, const int32_t *__restrict__ seg, const int32_t *__restrict__ pos,
    const int32_t *__restrict__ start, const int64_t *__restrict__ slot, float *__restrict__ q,
    float *__restrict__ kc, float *__restrict__ vc, int T, int H, int Nq, int Nkv, int r)
{
    __shared__ __attribute__((aligned(16))) float red[4][16 * MT][64];
    const int N = Nq + 2 * Nkv;
    const int m0 = blockIdx.y * (16 * MT), n0 = blockIdx.x * 64;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    f32x4 acc[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[m][e] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // classification of the row whose outputs this thread stores first: requested ahead of the products
    const int nn = n0 + 4 * (tid & 15);
    int a_of[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int t = m0 + 16 * m + (tid >> 4);
        a_of[m] = t < T ? effective_adapter(aid, seg, pos, start, t) : -1;
    }

    const int KB = (H + 15) >> 4, per = (KB + 3) >> 2;   // blocks of 16, per wavefront
    const int kb0 = min(KB, w * per), kb1 = min(KB, kb0 + per);
    const int n_l = n0 + 4 * c;
    constexpr int D = MT == 1 ? 4 : 2;                   // blocks requested together
    for (int kb = kb0; kb < kb1; kb += D) {
        f32x4 xv[D][MT], wv[D][4];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int k = 16 * (kb + d) + 4 * g;         // H is a multiple of 4: all four or none
            const bool k_ok = kb + d < kb1 && k < H;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                xv[d][m] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (k_ok && m0 + 16 * m + c < T) xv[d][m] = *(const f32x4 *)(x + (size_t)(m0 + 16 * m + c) * H + k);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                wv[d][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (k_ok && n_l < N) wv[d][j] = *(const f32x4 *)(W + (size_t)(k + j) * N + n_l);
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[m][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[d][m][j], wv[d][j][e], acc[m][e], 0, 0, 0);
    }
    // D[row 4g + i][feature tile e, column c]: register i
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(f32x4 *)&red[w][16 * m + 4 * g + i][4 * c] = (f32x4){acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]};
    __syncthreads();
    if (nn >= N) return;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = 16 * m + (tid >> 4), t = m0 + row;
        if (t >= T) continue;
        f32x4 y = *(const f32x4 *)&red[0][row][4 * (tid & 15)];
#pragma unroll
        for (int ww = 1; ww < 4; ++ww) y += *(const f32x4 *)&red[ww][row][4 * (tid & 15)];
        if (bias) y += *(const f32x4 *)(bias + nn);   // part of the base output of every row
        const int a = a_of[m];
        if (a >= 0) {
            const float *Ba = (const float *)B.p[a] + nn;
            const float *Sr = S + (size_t)t * r;
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            const int ra = ranks.r[a];
#pragma unroll 8
            for (int j = 0; j < ra; ++j) {
                const float s = Sr[j];
                const f32x4 b4 = *(const f32x4 *)(Ba + (size_t)j * N);
                d.x = fmaf(s, b4.x, d.x); d.y = fmaf(s, b4.y, d.y);
                d.z = fmaf(s, b4.z, d.z); d.w = fmaf(s, b4.w, d.w);
            }
            y += d;
        }
        if (nn < Nq) {
            *(f32x4 *)(q + (size_t)t * Nq + nn) = y;
        } else {
            const int64_t s = slot[t];
            if (s < 0) continue;
            if (nn < Nq + Nkv) *(f32x4 *)(kc + (size_t)s * Nkv + (nn - Nq)) = y;
            else *(f32x4 *)(vc + (size_t)s * Nkv + (nn - Nq - Nkv)) = y;
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

int launch_rope_f32(const Fwd &f)
{
    if (f.T == 0) return 0;
    launch_kernel(rope_f32_kernel, dim3(f.T), dim3(256), 0, f.stream, (float *)f.q, (float *)f.kc, f.slot, f.pos,
                       f.rope_cos, f.rope_sin, f.rope_positions, f.Nq, f.Nkv, f.D);
    return launch_status();
}

// The grouping step of a small batch rides in the shrink's launch (its results are the caller's to read; the
// fp32 kernels themselves classify a row from its metadata).
bool group_in_shrink_f32(const Fwd &f) { return f.dtype == ALORA_F32 && f.L > 0 && f.T <= GROUP_SMALL_ROWS; }

int launch_shrink_f32(const Fwd &f, const PtrTable &A, bool reuse_grouping)
{
    if (f.T == 0 || f.L == 0) return 0;
    const GroupSmallArgs ga = {f.aid, f.seg, f.pos, f.start, f.active, f.aeff, f.perm, f.offsets, f.blocktab, f.n_blocks, nullptr};
    const int group_wgs = group_in_shrink_f32(f) && !reuse_grouping ? f.n_blocks : 0;
    launch_kernel(shrink_f32_kernel, dim3(f.T + group_wgs), dim3(F32_THREADS), 0, f.stream, (const float *)f.x, A, f.ranks, ga,
                       f.T, f.L, f.H, f.r, (float *)f.S);
    return launch_status();
}

template <int MT>
static void launch_gemm_f32_rows(const Fwd &f, const PtrTable &B)
{
    launch_kernel(gemm_f32_kernel<MT>, dim3((f.N + 63) / 64, (f.T + 16 * MT - 1) / (16 * MT)), dim3(F32_THREADS), 0, f.stream,
                       (const float *)f.x, (const float *)f.W, (const float *)f.bias, B, f.ranks, (const float *)f.S, f.aid, f.seg,
                       f.pos, f.start, f.slot, (float *)f.q, (float *)f.kc, (float *)f.vc, f.T, f.H, f.Nq, f.Nkv, f.r);
}

int launch_gemm_f32(const Fwd &f, const PtrTable &B)
{
    if (f.T == 0) return 0;
    // us for MT = 1 | 2 | 4 (and the 64 x 64 LDS tile before them): 256 -> 512, two layers, 1500 rows 28 | 30 | 33 (49), 2048 rows 32 | 31 |
    // 33 (49), 6000 rows 69 | 70 | 81 (73), 16384 rows 148 | 137 | 154 (145); 1024 -> 1536, two layers, 512 rows 61 | 62 | 65 (141), 1024
    // rows 115 | 95 | 115 (158), 4096 rows 385 | 322 | 309 (366); 4096 -> 6144, 100 rows 102 | 94 | 108 (281), 256 rows 214 | 147 | 174
    // (286), 512 rows 437 | 338 | 323 (386), 2048 rows 1822 | 1212 | 973 (1308).
    const long long tiles = (f.N + 63) / 64, tiles32 = (f.T + 31) / 32 * tiles, tiles64 = (f.T + 63) / 64 * tiles;
    if (tiles64 >= 768 && f.H >= 1024 && tiles64 * f.H >= 5ll << 18) launch_gemm_f32_rows<4>(f, B);
    else if (tiles32 >= 400) launch_gemm_f32_rows<2>(f, B);
    else launch_gemm_f32_rows<1>(f, B);
    return launch_status();
}

}  // namespace alora
