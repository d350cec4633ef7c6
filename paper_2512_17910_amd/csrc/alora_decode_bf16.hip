// Projection of bf16 batches of a few token rows (decode of a quiet server: at most 64): fp32 partial products of x . W over ranges
// of the hidden dimension, with classification, grouping and shrink of the batch on workgroups of their own in
// the same launch.  The finishing kernel adds the ranges, the low-rank term, rounds and stores.
//
// Such a call is as long as W takes to arrive, so the kernel is built around requesting W early and once:
//   - an element of W passes through no LDS on its way to the matrix unit.  W is stored k-major while an MFMA
//     operand wants eight consecutive k of one feature per lane: a lane loads 16 bytes (eight features) of eight
//     consecutive rows and turns the 8 x 8 block around in registers (one v_perm per two elements), so that
//     MFMA f of eight takes feature 8 * (lane % 16) + f.
//   - the wavefronts of a workgroup take different ranges of the hidden dimension (no element of W is loaded
//     twice for a token tile, no barrier in the loop) and keep the next 64 of the hidden dimension in flight in registers;
//     their sums meet in LDS at the end and are added in fixed order.
//   - the ends of a wavefront's range are the ends of its buffer descriptors: slices past them are requested
//     like any other and come back as zeros without memory traffic, so the loop has no tail.
//   - x arrives in whole 128-byte lines, eight lanes to a token's piece, and becomes operands (eight consecutive k of
//     one token per lane) through LDS that a wavefront shares with no other.  (Loaded as the operand wants it,
//     neighbouring lanes would read different rows: 16 bytes per clock and compute unit, measured, against 43 for
//     the line pattern.)
// Token tiles of 16, 32, 48 or 64 rows: no matrix work is spent on rows a small batch does not have.
// Measured, 4096 -> 6144 with 50 MB of W from memory: 16.0 us for the 256-row tile of the projection kernel at one
// row, 11.5 us here (4.4 TB/s over the whole kernel; non-temporal loads of W included, 78.7 -> 71.0 us for four
// layers); 8192 -> 10240, four layers at eight rows, 235 -> 160 us.  64 rows, four adapters, twelve layers (nothing of
// W in the memory-side cache), 311 -> 287 us.  With four layers, which that cache holds, the projection kernel's 256-row tile was the faster from
// 41 rows on (64 rows 88 us, here 89.3).  From 65 rows on W would be read once per token tile: that kernel is the better one, in
// tiles of 128 rows up to 128 (65 rows 95 us, 128 rows 117), of 256 above (256 rows 163 against 200 us here).
#include <algorithm>
#include "alora_internal.h"
#include "alora_group_small.h"

namespace alora {

constexpr int DEC_FEATURES = 128;             // features per workgroup
constexpr int DEC_WAVES = 4;
constexpr int DEC_THREADS = 64 * DEC_WAVES;
constexpr int DEC_ROWS = 64;                  // most token rows of a call on this path
constexpr int DEC_STREAM = 2;                 // cache policy of the loads of W: non-temporal
constexpr int DEC_PITCH = DEC_FEATURES + 4;   // floats per token row of the reduction array
constexpr uint32_t DEC_OOR = 0x80000000u;     // past the end of every descriptor (operands are smaller than 2 GiB)

struct DecodeArgs {
    const bf16_t *x, *W;
    int T, H, N, L, r;
    int ntiles, splits;           // projection workgroups: ntiles * splits, padded to a multiple of 8
    int units_per_split;          // 64-wide slices of the hidden dimension per split
    int prep_wgs, prep_ranges, prep_units;   // workgroups of the grouping and shrink, ranges per block-table entry and their 64-wide slices
    float *partial;               // [splits][T][N]
    float *S;                     // [prep_ranges][T][r]
    GroupSmallArgs group;
    RankTable ranks;
};

// acc[nt][f] += (rows of x) . (columns of M) over slices u0 .. u1 - 1 of the hidden dimension (64 wide).  M is
// [H, n_cols], this lane's eight columns start at col (past n_cols: zeros).  row_at(i): where token i of the tile
// starts in x, in bytes (DEC_OOR: no such token).  xs: LDS of this wavefront alone (in order, no barriers).
// Result: lane (c, g) holds, for token nt * 16 + c, columns 32 g + 8 i + f of the tile in register i of acc[nt][f].
template <int NTT, int NT, typename RowAt>
__device__ __forceinline__ void decode_products(const bf16_t *x, uint32_t x_bytes, RowAt row_at, const bf16_t *M, int n_cols, int col,
                                                int u0, int u1, unsigned char *xs, f32x4 (&acc)[NTT][8])
{
    const int lane = threadIdx.x & 63, c = lane & 15, g4 = lane >> 4;
    const int n_units = max(u1 - u0, 0);
    const uint32_t pitch = (uint32_t)n_cols * 2u, half_bytes = 32u * pitch;
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc((void *)(M + (size_t)u0 * 64 * n_cols), 0, (int)(n_units * 2u * half_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, (int)x_bytes, 0x00020000);
    const uint32_t m_at = (uint32_t)(8 * g4) * pitch + (uint32_t)col * 2u;
    // x: load q of a slice covers tokens 8q .. 8q+7, eight lanes to a token's 128 bytes
    uint32_t x_at[2 * NTT];
#pragma unroll
    for (int q = 0; q < 2 * NTT; ++q) x_at[q] = row_at(8 * q + (lane >> 3));
    // Slices in flight: one (two halves, each requested again as soon as it is multiplied).  With two the loop is twice as long and takes 212 and 256
    // registers for 16 and 32 rows instead of 170 (a unit holds as many workgroups either way): four layers of 4096 -> 6144, two | one in flight,
    // us: one row 64.6 | 63.2, 24 rows 73.3 | 72.0, 64 rows 92.1 | 89.3, 8192 -> 10240 at two rows 151 | 149; three or four 70.4 at one row.
    constexpr int DEPTH = 1;
    u32x4 mv[2 * DEPTH][8], xv[DEPTH][2 * NTT];
    auto request_m = [&](int d, int h) {   // half slice h of the range; streamed: no other workgroup reads it
        const uint32_t mo = h < 2 * n_units && col < n_cols ? m_at + (uint32_t)h * half_bytes : DEC_OOR;
#pragma unroll
        for (int j = 0; j < 8; ++j) mv[d][j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rm, mo + (uint32_t)j * pitch, 0, NT));
    };
    auto request_x = [&](int d, int u) {
        const uint32_t ko = (uint32_t)((u0 + u) * 128 + 16 * (lane & 7));
#pragma unroll
        for (int q = 0; q < 2 * NTT; ++q)
            xv[d][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, u < n_units && x_at[q] != DEC_OOR ? x_at[q] + ko : DEC_OOR, 0, 0));
    };
    // token row r: 128 bytes, its eight 16-byte chunks XOR-swizzled by r % 8
    auto park_x = [&](int d) {
#pragma unroll
        for (int q = 0; q < 2 * NTT; ++q)
            *(u32x4 *)(xs + (8 * q + (lane >> 3)) * 128 + (((lane & 7) ^ (lane >> 3)) << 4)) = xv[d][q];
    };
    auto multiply = [&](int d) {
        bf16x8 xf[NTT];
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt) xf[nt] = *(const bf16x8 *)(xs + (16 * nt + c) * 128 + (((4 * (d & 1) + g4) ^ (c & 7)) << 4));
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            u32x4 a;   // k pairs (0,1) (2,3) (4,5) (6,7) of feature f of this lane's eight
#pragma unroll
            for (int p = 0; p < 4; ++p)
                a[p] = __builtin_amdgcn_perm(mv[d][2 * p + 1][f >> 1], mv[d][2 * p][f >> 1], (f & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt)
                acc[nt][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), xf[nt], acc[nt][f], 0, 0, 0);
        }
    };
#pragma unroll
    for (int d = 0; d < 2 * DEPTH; ++d) {
        if (!(d & 1)) request_x(d / 2, d / 2);
        request_m(d, d);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int b = 0; b < n_units; b += DEPTH) {
#pragma unroll
        for (int d = 0; d < 2 * DEPTH; ++d) {
            // (kept in this order: hoisting the arithmetic of later slices would wait for their loads first)
            if (!(d & 1)) {
                park_x(d / 2);
                request_x(d / 2, b + DEPTH + d / 2);
            }
            multiply(d);
            __builtin_amdgcn_sched_barrier(0);
            request_m(d, 2 * (b + DEPTH) + d);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The wavefronts' sums meet in LDS, all token tiles at once (one after the other, with two barriers each: 90.0 against
// 88.3 us for four layers at 37 rows), and are added in fixed order; thread -> four consecutive columns of a token.
// Calls out(token, column, value) for every four elements of the tile.
template <int NTT, typename Out>
__device__ __forceinline__ void decode_reduce(float *red, const f32x4 (&acc)[NTT][8], Out out)
{
    constexpr int ROWS = 16 * NTT;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        float *mine = red + (w * ROWS + 16 * nt + c) * DEC_PITCH + 32 * g4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *(f32x4 *)(mine + 8 * i) = (f32x4){acc[nt][0][i], acc[nt][1][i], acc[nt][2][i], acc[nt][3][i]};
            *(f32x4 *)(mine + 8 * i + 4) = (f32x4){acc[nt][4][i], acc[nt][5][i], acc[nt][6][i], acc[nt][7][i]};
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < ROWS * DEC_FEATURES / 4 / DEC_THREADS; ++h) {
        const int idx = h * DEC_THREADS + tid, tok = idx / (DEC_FEATURES / 4), cc = (idx % (DEC_FEATURES / 4)) * 4;
        f32x4 s = *(const f32x4 *)(red + tok * DEC_PITCH + cc);
#pragma unroll
        for (int ww = 1; ww < DEC_WAVES; ++ww) s += *(const f32x4 *)(red + (ww * ROWS + tok) * DEC_PITCH + cc);
        out(tok, cc, s);
    }
}

template <int NTT>
__global__ __launch_bounds__(DEC_THREADS, NTT > 2 ? 1 : 2) void decode_projection_kernel(DecodeArgs g, PtrTable A)
{
    constexpr int XS_TILES = NTT < 2 ? 2 : NTT, RED_BYTES = DEC_WAVES * 16 * XS_TILES * DEC_PITCH * 4, XS_BYTES = XS_TILES * 2048;   // (the shrink takes two tiles)
    __shared__ __attribute__((aligned(16))) unsigned char lds[RED_BYTES > DEC_WAVES * XS_BYTES ? RED_BYTES : DEC_WAVES * XS_BYTES];
    __shared__ int scr[GROUP_SMALL_SCRATCH];
    float *const red = (float *)lds;
    const int lane = threadIdx.x & 63, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char *const xs = lds + w * XS_BYTES;
    const uint32_t x_bytes = (uint32_t)g.T * (uint32_t)g.H * 2u;
    const int units = g.H >> 6;

    // The grouping and shrink workgroups come first: their chain of dependent steps is the longer one.
    if ((int)blockIdx.x < g.prep_wgs) {
        // prep_ranges workgroups per entry of the 32-row block table, one per range of the hidden dimension; each
        // works the grouping out for itself, the first of them writes the entry's share of its results
        const int e = (int)blockIdx.x / g.prep_ranges, range = (int)blockIdx.x - e * g.prep_ranges;
        int grp, cnt;
        if (e == 0 && range == 0)   // entries no workgroup stands for
            for (int i = g.prep_wgs / g.prep_ranges + threadIdx.x; i < g.group.n_blocks; i += DEC_THREADS) g.group.blocktab[i] = make_int4(-1, 0, 0, 0);
        const int *rows = group_small(g.group, g.T, g.L, e, range == 0, scr, grp, cnt);
        if (grp < 0 || grp >= g.L) return;   // unused entry or the rows that keep the base output
        const int rk = g.ranks.r[grp];
        auto row_at = [&](int i) { const int t = rows[i]; return t >= 0 ? (uint32_t)t * (uint32_t)g.H * 2u : DEC_OOR; };
        const int r0 = min(units, range * g.prep_units), n_u = min(units, r0 + g.prep_units) - r0;
        f32x4 acc[2][8] = {};
        decode_products<2, 0>(g.x, x_bytes, row_at, (const bf16_t *)A.p[grp], rk, 8 * c, r0 + n_u * w / DEC_WAVES, r0 + n_u * (w + 1) / DEC_WAVES, xs, acc);
        __syncthreads();   // the reduction works where the wavefronts parked their tokens
        float *S = g.S + (size_t)range * g.T * g.r;
        decode_reduce<2>(red, acc, [&](int tok, int cc, f32x4 s) {
            const int t = rows[tok];
            if (t >= 0 && cc < rk) *(f32x4 *)(S + (size_t)t * g.r + cc) = s;
        });
        return;
    }

    // Workgroups go to the 8 XCDs in turn; an XCD takes a contiguous range of (split, feature tile): neighbouring
    // pieces of W's rows.
    const int b = (int)blockIdx.x - g.prep_wgs, total = g.ntiles * g.splits, chunk = (total + 7) >> 3;
    const int l = (b & 7) * chunk + (b >> 3);
    if ((b >> 3) >= chunk || l >= total) return;
    const int split = l / g.ntiles, n0 = (l - split * g.ntiles) * DEC_FEATURES;
    auto row_at = [&](int i) { return i < g.T ? (uint32_t)i * (uint32_t)g.H * 2u : DEC_OOR; };
    const int r0 = min(units, split * g.units_per_split), n_u = min(units, r0 + g.units_per_split) - r0;
    f32x4 acc[NTT][8] = {};
    decode_products<NTT, DEC_STREAM>(g.x, x_bytes, row_at, g.W, g.N, n0 + 8 * c, r0 + n_u * w / DEC_WAVES, r0 + n_u * (w + 1) / DEC_WAVES, xs, acc);
    __syncthreads();   // the reduction works where the wavefronts parked their tokens
    float *out = g.partial + (size_t)split * g.T * g.N;
    decode_reduce<NTT>(red, acc, [&](int tok, int cc, f32x4 s) {
        const int n = n0 + cc;
        if (tok < g.T && n < g.N) *(f32x4 *)(out + (size_t)tok * g.N + n) = s;
    });
}

// ---- host side: how a call of given sizes is cut, from (T, hidden, N) alone (see plan_gemm) -------------------
bool few_rows_call(const Fwd &f)
{
    if (f.dtype != ALORA_BF16 || f.T <= 0 || f.T > DEC_ROWS) return false;
    // room for the partials; descriptors of x, W and A below 2 GiB (a masked lane's offset is past all of them)
    return gemm_partial_bytes(f.T, f.H, f.N) && (long long)f.T * f.H * 2 < (1ll << 31) && (long long)f.H * ALORA_MAX_RANK * 2 < (1ll << 31);
}

int launch_decode_bf16(const Fwd &f, const PtrTable &B, const PtrTable &A, hipEvent_t after_projection)
{
    DecodeArgs g;
    g.x = (const bf16_t *)f.x; g.W = (const bf16_t *)f.W;
    g.T = f.T; g.H = f.H; g.N = f.N; g.L = f.L; g.r = f.r;
    const int units = f.H / 64;
    g.ntiles = (f.N + DEC_FEATURES - 1) / DEC_FEATURES;
    // One workgroup per compute unit, shrink workgroups of a few adapters included (a unit that got two took twice as long),
    // hence 200 for the projection.  (The shrink has two for every 32 rows of an adapter, at most two per row, and its workgroups come
    // first: 64 rows of 32 adapters each get to 262 in all.)  Four layers of 4096 -> 6144 at one row, us: 144 workgroups 80, 192 73, 240 81, 384 78;
    // 3072 -> 5120 at eight rows: 160 67, 200 65, 240 70; 8192 -> 10240: 80 251, 160 160, 240 159, 320 174.
    // The fewest splits that leave a wavefront the least (3072 -> 5120 at 48 rows, five 74.6, four 71.9).  Of a few rows the shrink's
    // workgroups are few for certain, and the projection takes the rest where that saves a wavefront two slices and more (8192 -> 10240, two | three
    // splits: one row 148.4 | 132.3, eight 153.9 | 136.5; 3072 -> 5120 at two rows, one slice less, four splits 57.9, six 59.0).
    auto share = [&](int splits) { return ((units + splits - 1) / splits + DEC_WAVES - 1) / DEC_WAVES; };
    auto splits_of = [&](int workgroups) {
        int best = 1;
        for (int s = 2; s <= std::min(std::min(8, units / DEC_WAVES), workgroups / g.ntiles); ++s)   // (a slice per wavefront at least)
            if (share(s) < share(best)) best = s;
        return best;
    };
    g.splits = splits_of(200);
    const int more = splits_of(256 - 2 * f.T);
    if (share(more) + 2 <= share(g.splits)) g.splits = more;
    g.units_per_split = (units + g.splits - 1) / g.splits;
    g.splits = (units + g.units_per_split - 1) / g.units_per_split;
    // Two ranges of the hidden dimension for the shrink (one: 88 against 73 us, four and eight: no gain); without
    // adapters the grouping alone.
    const int ranges = f.L > 0 && units >= 2 ? 2 : 1;
    g.prep_units = (units + ranges - 1) / ranges;
    g.prep_ranges = (units + g.prep_units - 1) / g.prep_units;
    g.prep_wgs = used_blocks(f) * g.prep_ranges;
    g.partial = f.partial; g.S = (float *)f.S;
    g.group = GroupSmallArgs{f.aid, f.seg, f.pos, f.start, f.active, f.aeff, f.perm, f.offsets, f.blocktab, f.n_blocks, f.block_rows};
    g.ranks = f.ranks;
    const dim3 grid((g.ntiles * g.splits + 7) / 8 * 8 + g.prep_wgs), block(DEC_THREADS);
    if (f.T <= 16) launch_kernel((decode_projection_kernel<1>), grid, block, 0, f.stream, g, A);
    else if (f.T <= 32) launch_kernel((decode_projection_kernel<2>), grid, block, 0, f.stream, g, A);
    else if (f.T <= 48) launch_kernel((decode_projection_kernel<3>), grid, block, 0, f.stream, g, A);
    else launch_kernel((decode_projection_kernel<4>), grid, block, 0, f.stream, g, A);
    int e = launch_status();
    if (!e && after_projection) e = (int)hipEventRecord(after_projection, f.stream);
    if (e) return e;
    return launch_finish_bf16(f, B, g.splits, g.prep_ranges, f.block_rows, true);
}

}  // namespace alora
