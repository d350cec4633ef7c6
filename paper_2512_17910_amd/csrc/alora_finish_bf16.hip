// Finishing kernel of the small-batch (decode-sized) bf16 path.
//
// With few token rows the projection is cut along the hidden dimension so that every compute unit
// streams a share of W; the splits leave fp32 partial products P[s][t][:].  This kernel walks the
// grouped row list (half an entry of the block table, 16 rows of one adapter or of the base group, per workgroup and
// 256 features) and produces the final rows:
//     y[t,:] = sum_s P[s][t,:]  (fixed split order)   [+ S[t,:] . B[a]  for rows of adapter a]
// rounds once to bf16 and stores q_out / the paged K and V slots.  Rows of the base group never
// touch S or B, and their arithmetic does not depend on which rows are adapted: they come out
// bit-identical to a call without adapters.
//
// The low-rank term runs on bf16 MFMA without giving up a bit of S: the fp32 shrink result (the fixed-order sum of the
// shrink's partials, or hi + lo of the bf16 pair it stored) is cut into three bf16 that add up to it exactly, B is
// bf16 as it is, every product is exact in the fp32 accumulator; sums that are not finite are done again the plain way.  (As fp32 multiply-adds, rank x 8 per thread, it was what
// bounded the kernel: a vector instruction takes four cycles, 640 of them per wavefront at rank 32.)
//
// What bounds it is a chain of dependent round trips, and for larger batches the partials' way in (25 MB at 256 rows and
// four splits).  So there are few round trips: table entry and row ids, then (adapted rows, which wait for them in the shadow of all other loads) the adapters'
// tables, a lane per adapter; all splits' partials, the S row, slot and position, and the B slice; then the angles.  And workgroups are small: of 32 rows and
// 1024 threads one fits a CU (106 registers), and the 12 rows an adapter has in a decode batch leave two thirds of
// it idle while it loads its slice of B; of 16 rows two fit.
// Measured, us: one row 5.7 -> 4.5, 256 rows of 16 adapters, rank 32 11.9 -> 9.3 (32 rows per workgroup 12.0), 777 rows in two splits 17.7 -> 13.0 (48 MB: 3.7 TB/s), 256 base rows 6.0 -> 6.2
// (6.4 with the tables in front of the row ids), 1024 in three splits beside adapters of rank 64 13.7 -> 14.4 (15.5 with S . B in LDS of its own);
// the whole call of 256 rows at rank 64 54.4 -> 47.5.
#include <type_traits>
#include "alora_internal.h"

namespace alora {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

constexpr int FIN_COLS = 256;  // features per workgroup: 32 threads x 8 features per row
constexpr int FIN_ROWS = 16;   // rows per workgroup: half an entry of the block table (blockIdx.z)
constexpr int FIN_THREADS = 32 * FIN_ROWS;

// An fp32 number as three bf16 whose sum it is, exactly: 8 significant bits each, cut off rather than rounded (no part
// can overflow).  Infinities and NaN travel in the first part alone.
__device__ __forceinline__ void split3(float v, bf16_t &p0, bf16_t &p1, bf16_t &p2)
{
    const uint32_t u = __float_as_uint(v);
    if ((u & 0x7f800000u) == 0x7f800000u) {
        p0 = (bf16_t)((u >> 16) | ((u & 0x007fffffu) ? 0x40u : 0u));
        p1 = p2 = 0;
        return;
    }
    const float r1 = v - __uint_as_float(u & 0xffff0000u);
    const uint32_t u1 = __float_as_uint(r1);
    const float r2 = r1 - __uint_as_float(u1 & 0xffff0000u);
    p0 = (bf16_t)(u >> 16);
    p1 = (bf16_t)(u1 >> 16);
    p2 = (bf16_t)(__float_as_uint(r2) >> 16);
}

// RT: 32-wide rank tiles (1 for rank <= 32, else 2)
template <int SPLITS, int RT>
__global__ __launch_bounds__(FIN_THREADS) void finish_bf16_kernel(const float *__restrict__ partial,
                                                           const void *__restrict__ S_any, int s_splits, bool s_f32, PtrTable B,
                                                           RankTable ranks, const bf16_t *__restrict__ bias,
                                                           const int32_t *__restrict__ perm,
                                                           const int32_t *__restrict__ block_rows,
                                                           const int4 *__restrict__ blocktab,
                                                           const int64_t *__restrict__ slot, bf16_t *__restrict__ q,
                                                           bf16_t *__restrict__ kc, bf16_t *__restrict__ vc, int T, int Nq,
                                                           int Nkv, int L, int r, const float *__restrict__ rope_cos,
                                                           const float *__restrict__ rope_sin, const int32_t *__restrict__ pos,
                                                           int rope_positions)
{
    constexpr int K = 32 * RT;
    constexpr int B_PITCH = FIN_COLS * 2 + 32;      // bytes per rank row of B (the transposing read takes 16 rows at once: 8 banks further each)
    constexpr int S_PITCH = 3 * K * 2 + 16;         // bytes per row of S: the three parts, K each
    constexpr int D_PITCH = FIN_COLS + 4;           // floats per row of S . B
    // Two rank tiles: S . B takes the place of B, whose columns 32w .. 32w+31 are wavefront w's alone (row r, features 16h .. 16h+15 in
    // row 2r + h), so that three workgroups fit a CU's LDS instead of two: 777 rows in two splits at rank 64 122.8 us a call, now 119.3,
    // 1000 rows 136.8 and 134.7; one rank tile gains no place by it, and decode batches lose 1 %.
    constexpr bool IN_B = RT == 2;
    __shared__ __attribute__((aligned(16))) unsigned char b_lds[K * B_PITCH], s_lds[FIN_ROWS * S_PITCH];
    __shared__ __attribute__((aligned(16))) float d_lds[IN_B ? 4 : FIN_ROWS * D_PITCH];

    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = tid >> 5, c = tid & 31, n0 = blockIdx.y * FIN_COLS, n = n0 + 8 * c;
    const int half = FIN_ROWS * blockIdx.z;
    const int4 entry = blocktab[blockIdx.x];
    // row ids straight from the per-entry list when there is one: the load does not wait for the entry
    int t = -1;
    if (block_rows) t = block_rows[32 * blockIdx.x + half + i];
    const int a = __builtin_amdgcn_readfirstlane(entry.x), j0 = entry.y, cnt = entry.z;
    if (a < 0 || cnt <= half) return;  // unused table entry, or no rows in this half; uniform across the workgroup
    if (a > L || j0 < 0 || cnt > 32 || j0 + cnt > T) return;   // not a table of this batch
    const int N = Nq + 2 * Nkv;
    const bool adapted = a < L;
    if (!block_rows && half + i < cnt) t = perm[j0 + half + i];
    // The adapters' tables, a lane per adapter, on the way together with the row ids and behind them: rows of the base group do not wait for them.
    uint64_t bp0 = 0, bp1 = 0;
    int rk = 0;
    if (adapted) {
        bp0 = (uint64_t)B.p[lane], bp1 = (uint64_t)B.p[64 + lane];
        rk = ranks.r[lane] | ranks.r[64 + lane] << 8;
    }
    if (half + i >= cnt || t >= T) t = -1;
    const bool live = t >= 0 && n < N;

    // everything that depends on the row id, issued together (the position first: the angles wait for it)
    const bool turned = rope_cos && n < Nq + Nkv;
    int p = 0;
    int64_t sl = -1;
    f32x4 plo[SPLITS], phi[SPLITS];
    if (live) {
        if (turned) p = pos[t];
        if (n >= Nq) sl = slot[t];
    }
    float sj[RT] = {};
    u32x4 bv[2 * RT] = {};
    if (adapted) {
        const int a6 = a & 63;
        const int ra = (__builtin_amdgcn_readlane(rk, a6) >> (a < 64 ? 0 : 8)) & 0xff;   // this group's rank; S and B_a rows beyond it do not exist
        const uint32_t plow = a < 64 ? __builtin_amdgcn_readlane((uint32_t)bp0, a6) : __builtin_amdgcn_readlane((uint32_t)bp1, a6);
        const uint32_t phigh = a < 64 ? __builtin_amdgcn_readlane((uint32_t)(bp0 >> 32), a6) : __builtin_amdgcn_readlane((uint32_t)(bp1 >> 32), a6);
        const bf16_t *Ba = (const bf16_t *)((uint64_t)phigh << 32 | plow);
        // B[a][:, n0 : n0+256]: K rank rows (zeros past the rank) x 32 chunks of 8 features
#pragma unroll
        for (int u = 0; u < 2 * RT; ++u)
            if (16 * u + i < ra && n < N) bv[u] = *(const u32x4 *)(Ba + (size_t)(16 * u + i) * N + n);
        // S of row i, rank columns c, c+32
        if (t >= 0) {
#pragma unroll
            for (int u = 0; u < RT; ++u) {
                const int j = 32 * u + c;
                if (j >= ra) continue;
                if (s_f32) {
                    // all ranges' loads first, then the sum in range order (absent ranges add +0)
                    const float *S_part = (const float *)S_any;
                    float sp[ALORA_SHRINK_MAX_SPLITS];
#pragma unroll
                    for (int ks = 0; ks < ALORA_SHRINK_MAX_SPLITS; ++ks)
                        sp[ks] = ks < s_splits ? S_part[((size_t)ks * T + t) * r + j] : 0.f;
#pragma unroll
                    for (int ks = 0; ks < ALORA_SHRINK_MAX_SPLITS; ++ks) sj[u] += sp[ks];
                } else {
                    const bf16_t *row = (const bf16_t *)S_any + (size_t)t * 2 * r;
                    sj[u] = bf16_bits_to_f32(row[j]) + bf16_bits_to_f32(row[r + j]);
                }
            }
        }
    }
    u32x4 bias4 = {0u, 0u, 0u, 0u};
    f32x4 c0 = {}, c1 = {}, s0 = {}, s1 = {};
    if (live) {
#pragma unroll
        for (int s = 0; s < SPLITS; ++s) {
            const float *pp = partial + ((size_t)s * T + t) * N + n;
            plo[s] = *(const f32x4 *)pp;
            phi[s] = *(const f32x4 *)(pp + 4);
        }
        if (bias) bias4 = *(const u32x4 *)(bias + n);
        if (turned) {
            const size_t at = (size_t)min(max(p, 0), rope_positions - 1) * 64 + (n & 63);
            c0 = *(const f32x4 *)(rope_cos + at), c1 = *(const f32x4 *)(rope_cos + at + 4);
            s0 = *(const f32x4 *)(rope_sin + at), s1 = *(const f32x4 *)(rope_sin + at + 4);
        }
    }

    float d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (adapted) {
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            *(u32x4 *)(b_lds + (32 * u + i) * B_PITCH + 16 * c) = bv[2 * u];
            *(u32x4 *)(b_lds + (32 * u + 16 + i) * B_PITCH + 16 * c) = bv[2 * u + 1];
            bf16_t *sr = (bf16_t *)(s_lds + i * S_PITCH) + 32 * u + c;
            split3(sj[u], sr[0], sr[K], sr[2 * K]);
        }
        __syncthreads();
        // wavefront w: features 32w .. 32w+31 of all rows
        const int c16 = lane & 15, g4 = lane >> 4;
        f32x4 acc[2] = {};
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            bf16x8 bf[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const lds_byte *bp = (const lds_byte *)b_lds + (32 * u + 8 * g4 + (c16 >> 2)) * B_PITCH + 64 * w + 32 * h + 8 * (c16 & 3);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)bp);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(bp + 4 * B_PITCH));
                bf[h] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
            for (int part = 2; part >= 0; --part) {
                const bf16x8 sf = *(const bf16x8 *)(s_lds + c16 * S_PITCH + (part * K + 32 * u + 8 * g4) * 2);
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[h], sf, acc[h], 0, 0, 0);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *(f32x4 *)(IN_B ? (float *)(b_lds + (2 * c16 + h) * B_PITCH + 64 * w + 16 * g4) : d_lds + c16 * D_PITCH + 32 * w + 16 * h + 4 * g4) = acc[h];
        __syncthreads();
        float *const dl = IN_B ? (float *)(b_lds + (2 * i + (c >> 1 & 1)) * B_PITCH + 64 * (c >> 2) + 32 * (c & 1)) : d_lds + i * D_PITCH + 8 * c;
        f32x4 d0 = *(const f32x4 *)dl, d1 = *(const f32x4 *)(dl + 4);
        // An infinite element of B times S is +-inf, but times a part of S that is zero, as the third one mostly is, NaN: a sum that is
        // not finite is done again with S whole, product by product.  (0 times such a sum is NaN, 0 times all others 0.)
        float none = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) none = fmaf(0.f, d0[e], fmaf(0.f, d1[e], none));
        if (none != 0.f) {
            const int a6 = a & 63, ra = (__builtin_amdgcn_readlane(rk, a6) >> (a < 64 ? 0 : 8)) & 0xff;
            const bf16_t *const Ba = (const bf16_t *)B.p[a];
#pragma unroll 1
            for (int e = 0; e < 8; ++e) {
                if (fabsf(dl[e]) < __builtin_inff() || n >= N) continue;
                float sum = 0.f;
#pragma unroll 1
                for (int j = 0; j < ra; ++j) {
                    const bf16_t *sr = (const bf16_t *)(s_lds + i * S_PITCH) + j;
                    const float s = bf16_bits_to_f32(sr[0]) + (bf16_bits_to_f32(sr[K]) + bf16_bits_to_f32(sr[2 * K]));   // exact
                    sum = fmaf(s, bf16_bits_to_f32(Ba[(size_t)j * N + n + e]), sum);
                }
                dl[e] = sum;
            }
            d0 = *(const f32x4 *)dl, d1 = *(const f32x4 *)(dl + 4);
        }
        d[0] = d0.x; d[1] = d0.y; d[2] = d0.z; d[3] = d0.w;
        d[4] = d1.x; d[5] = d1.y; d[6] = d1.z; d[7] = d1.w;
    }
    if (!live) return;

    float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) {
        y[0] += plo[s].x; y[1] += plo[s].y; y[2] += plo[s].z; y[3] += plo[s].w;
        y[4] += phi[s].x; y[5] += phi[s].y; y[6] += phi[s].z; y[7] += phi[s].w;
    }
    if (bias) {   // part of the base output of every row
        y[0] += __uint_as_float(bias4.x << 16); y[1] += __uint_as_float(bias4.x & 0xffff0000u);
        y[2] += __uint_as_float(bias4.y << 16); y[3] += __uint_as_float(bias4.y & 0xffff0000u);
        y[4] += __uint_as_float(bias4.z << 16); y[5] += __uint_as_float(bias4.z & 0xffff0000u);
        y[6] += __uint_as_float(bias4.w << 16); y[7] += __uint_as_float(bias4.w & 0xffff0000u);
    }
    if (adapted) {
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] += d[e];
    }
    if (rope_cos) {
        // Rotary embedding on the unrounded row (heads of 128): the partner features i +- 64 are held by the
        // thread 8 lanes away, which is live whenever this one is (heads never straddle N).  Every live lane
        // takes part in the exchange; lanes of the v part keep their values.
        float other[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) other[e] = __shfl_xor(y[e], 8);
        if (turned) {
            const float cc[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            const float ss[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
            const float sign = (n & 127) < 64 ? -1.f : 1.f;     // first half: y cos - partner sin; second half: y cos + partner sin
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = y[e] * cc[e] + sign * (other[e] * ss[e]);
        }
    }
    u32x4 out;
    {
        const f32x2 p0 = {y[0], y[1]}, p1 = {y[2], y[3]}, p2 = {y[4], y[5]}, p3 = {y[6], y[7]};
        out.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(p0, bf16x2));
        out.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(p1, bf16x2));
        out.z = __builtin_bit_cast(uint32_t, __builtin_convertvector(p2, bf16x2));
        out.w = __builtin_bit_cast(uint32_t, __builtin_convertvector(p3, bf16x2));
    }
    if (n < Nq) {
        *(u32x4 *)(q + (size_t)t * Nq + n) = out;
    } else if (sl >= 0) {
        if (n < Nq + Nkv) *(u32x4 *)(kc + (size_t)sl * Nkv + (n - Nq)) = out;
        else *(u32x4 *)(vc + (size_t)sl * Nkv + (n - Nq - Nkv)) = out;
    }
}

template <int SPLITS>
static void launch_finish(const Fwd &f, const PtrTable &B, int s_splits, const int32_t *block_rows, bool s_f32)
{
    const dim3 grid(used_blocks(f), (f.N + FIN_COLS - 1) / FIN_COLS, f.T > FIN_ROWS ? 2 : 1);
    auto launch = [&](auto rank_tiles) {
        launch_kernel((finish_bf16_kernel<SPLITS, decltype(rank_tiles)::value>), grid, dim3(FIN_THREADS), 0, f.stream, (const float *)f.partial,
                           f.S, s_splits, s_f32, B, f.ranks, (const bf16_t *)f.bias, f.perm, block_rows, f.blocktab, f.slot, (bf16_t *)f.q, (bf16_t *)f.kc,
                           (bf16_t *)f.vc, f.T, f.Nq, f.Nkv, f.L, f.r, f.rope_cos, f.rope_sin, f.pos, f.rope_positions);
    };
    if (f.r <= 32) launch(std::integral_constant<int, 1>{});
    else launch(std::integral_constant<int, 2>{});
}

int launch_finish_bf16(const Fwd &f, const PtrTable &B, int splits, int s_splits, const int32_t *block_rows, bool s_f32)
{
    switch (splits) {
    case 1: launch_finish<1>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 2: launch_finish<2>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 3: launch_finish<3>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 4: launch_finish<4>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 5: launch_finish<5>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 6: launch_finish<6>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 7: launch_finish<7>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    case 8: launch_finish<8>(f, B, s_splits, block_rows, s_f32 || s_splits > 1); break;
    default: return (int)hipErrorInvalidValue;
    }
    return launch_status();
}

}  // namespace alora
