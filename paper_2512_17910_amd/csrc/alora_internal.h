// Internal declarations shared by the HIP translation units of libalora_qkv (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "alora_qkv.h"

namespace alora {

typedef uint16_t bf16_t;  // raw bf16 bit pattern

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Device pointers of the adapters' factors, passed to kernels by value.
struct PtrTable {
    const void *p[ALORA_MAX_ADAPTERS];
};

// Rank of every adapter (A_i is [hidden, r_i], B_i is [r_i, N]), passed to kernels by value.
struct RankTable {
    uint8_t r[ALORA_MAX_ADAPTERS];
};

struct GemmPlan {
    int ntw;     // 32-wide feature tiles per wavefront (tile width 64 * ntw)
    int splits;  // 1: fused kernel; > 1: split hidden dimension + finishing kernel
    int kps;     // 64-wide K-slices per split
    int panels;  // 256-row tiles; the rows behind them, if any, in tiles of 128 x 128 (fused kernel)
};
struct ShrinkPlan {
    int splits;  // ranges of the hidden dimension; the shrink result is the fixed-order sum of their partials
    int kper;    // width of one range (multiple of 64)
    // Prefill-sized batches: the number of ranges is chosen on the device, per call, from the number of
    // adapted 32-row blocks (at most `splits`); the last range of a block to finish adds the partials in
    // fixed order and stores the (hi, lo) form.  The shrink then walks Fwd::items.
    bool combine;
};
// Which kernels a bf16 call takes and how they are cut.  Decided once per call (plan_call), from its sizes, from whether it rotates and
// from ONE reading of the tuning override: every launch of the call follows it, so that an override set by another
// host thread meanwhile cannot give one call the launches of two different paths.
struct Route {
    GemmPlan gemm;
    ShrinkPlan shrink;
    bool few_rows;      // at most 64 rows: the projection kernel of alora_decode_bf16.hip
    bool prep_inside;   // grouping and shrink run inside the projection kernel
};

// Everything one forward call needs, resolved on the host.
struct Fwd {
    int dtype, T, H, Nq, Nkv, N, L, r, G;
    long long n_slots;
    int block_size;
    const void *x, *W;
    const void *bias;    // [N] or null: added to the base output of every row (Algorithm 1, l.apply(x, b))
    RankTable ranks;     // per adapter, <= r
    const float *rope_cos, *rope_sin;   // [rope_positions][D / 2] or null: rotary embedding fused into the store
    int rope_positions, D;              // D = head_dim
    const int32_t *aid, *seg, *pos, *start;
    const int64_t *slot;
    void *q, *kc, *vc;
    // workspace regions
    uint8_t *active;
    int8_t *aeff;        // [T] adapter id of adapted rows, -1 for rows that keep the base output
    int32_t *perm, *offsets;
    void *S;          // shrink result.  f32 path: [T][r] fp32.  bf16 path: [T][2r] bf16 (hi | lo halves of the fp32
                      // result), or with several shrink ranges (see plan_shrink) fp32 partials [ranges][T][r]
    float *partial;      // small-batch path: fp32 partial products [splits][T][N]
    int32_t *hist;       // large batches: rows per (2048-row slice, group), see the grouping kernels
    int4 *blocktab;      // shrink: (adapter, first perm index, rows, 0) per 32-row block; adapter -1 = unused
    int n_blocks;        // entries in blocktab (upper bound on 32-row blocks)
    // prefill-sized bf16 batches: the shrink's work list, one item per (32-row block of an adapter, range
    // of the hidden dimension), written by the grouping step from the number of adapted blocks it finds;
    // null when the shrink walks blocktab instead
    int4 *items;         // (adapter, first perm index, rows | range width/64 << 8, range | ranges << 4 | block << 8)
    int32_t *counters;   // per block: ranges that have stored their partial (zeroed by the grouping step)
    int n_items;
    int32_t *block_rows;  // decode-sized bf16 batches: the row ids of every block-table entry, 32 per entry, -1 padded
                          // (the finishing kernel then needs no look-up through perm)
    Route route;          // bf16 calls
    hipStream_t stream;
};

// fp32 -> bf16 bits, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// App. B mask negated and combined with "row has an adapter": -1 when the row keeps the base
// output, else its adapter id.  seg/pos/start are only read for rows that have an adapter.
__device__ __forceinline__ int effective_adapter(const int32_t *aid, const int32_t *seg, const int32_t *pos,
                                                 const int32_t *start, int t)
{
    int a = aid[t];
    if (a < 0) return -1;
    return (pos[t] >= start[seg[t]]) ? a : -1;
}

// remember a failed HIP call for alora_last_hip_error() (per host thread)
void note_hip_error(int hip_error);

// Launches, and the first failure among those since the last look.  The launch's own status, not hipGetLastError's: that holds what any
// earlier call of the program left behind, which is neither this library's failure nor its to take away.
inline thread_local int first_launch_error = 0;
template <typename... P>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t stream, typename std::common_type<P>::type... args)
{
    void *at[] = {(void *)&args...};
    const int e = (int)hipLaunchKernel((const void *)kernel, grid, block, at, lds_bytes, stream);
    if (!e) return;
    (void)hipGetLastError();   // reported from here
    if (!first_launch_error) first_launch_error = e;
}
inline int launch_status()
{
    const int e = first_launch_error;
    first_launch_error = 0;
    return e;
}

// launches (each returns the hipError_t of its launch as int)
int launch_classify_group(const Fwd &f);
int launch_shrink_f32(const Fwd &f, const PtrTable &A, bool reuse_grouping);
bool group_in_shrink_f32(const Fwd &f);   // the grouping runs on workgroups of the fp32 shrink or, where that has no launch of its own, projection
int launch_gemm_f32(const Fwd &f, const PtrTable &B, const PtrTable &A, bool reuse_grouping);
int launch_shrink_bf16(const Fwd &f, const PtrTable &A);
int launch_gemm_bf16(const Fwd &f, const PtrTable &B, const PtrTable &A, hipEvent_t after_projection);
int launch_finish_bf16(const Fwd &f, const PtrTable &B, int splits, int s_splits, const int32_t *block_rows, bool s_f32);
void plan_call(Fwd &f);   // fills f.route (f holds the sizes, block_rows and rope_cos)
bool few_rows_call(const Fwd &f);   // a batch of a few rows (alora_decode_bf16.hip), from its sizes alone
int launch_decode_bf16(const Fwd &f, const PtrTable &B, const PtrTable &A, hipEvent_t after_projection);
size_t gemm_partial_bytes(int T, int H, int N);
void set_gemm_tuning(int ntw, int splits);
int group_blocks(int T, int L);
// Block-table entries that can be in use: they come first in the table, and each holds a row.  (Workgroups for all entries, two and
// N / 256 of K4 for every adapter of the server, 4096 -> 6144 with 32 adapters, four layers: one row 84 us, now 73; eight rows 88, 73.)
inline int used_blocks(const Fwd &f) { return f.n_blocks < f.T ? f.n_blocks : f.T; }
size_t group_hist_bytes(int T);
constexpr int ALORA_SHRINK_MAX_SPLITS = 8;
constexpr int ALORA_SHRINK_TARGET_WGS = 256;   // workgroups the prefill-sized shrink aims for (one per compute unit)
// what the grouping kernels need to write the shrink's work list
struct ShrinkWork {
    int4 *items;
    int32_t *counters;
    int n_items, k64, rmax;
};
int shrink_items(int T, int L);   // entries of the work list
ShrinkPlan plan_shrink(const GemmPlan &gemm, int T, int H, int L, int r);
int launch_rope_f32(const Fwd &f);   // fp32 path: rotation of the stored q and k rows in place

}  // namespace alora
