// Declarations shared by the translation units of the paged-cache reader.
#pragma once
#include "alora_internal.h"
#include "alora_attention.h"

namespace alora {

struct AttnArgs {
    const void *q, *kc, *vc;
    const int32_t *bt, *seq, *pos;
    void *out;
    int T, Hq, Hkv, n_seqs, max_blocks, bs, bs_shift;
    long long n_slots;
    float scale_log2e;   // scale * log2(e): the softmax runs on powers of two
    int splits;          // parts a row's context is cut into (one workgroup each); > 1: partials go to `part`
    int short_splits;    // per-row kernel: parts of a context too short for that many
    bool once;           // per-row kernel: see contexts_read_once
    float *part;         // [T][Hq][splits][D + 2]: running maximum, sum of weights, unnormalised weighted V
};

constexpr int MAX_PARTS = 32;   // of a row's context

// A layer's K and V that the memory-side cache (256 MB) would not keep until they are read again.
inline bool outgrows_cache(long long n_slots, int Hkv, int D, bool bf16) { return n_slots * Hkv * D * (bf16 ? 4 : 8) > 96ll << 20; }

// sums over lanes 0 .. lane (row_shr:1, 2, 4, 8, then row_bcast:15 and 31 into the rows above)
__device__ __forceinline__ int sum_upto64(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    return x + __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
}
constexpr int LOOKED_OVER = 256;   // batch rows per wavefront of which a row-block workgroup finds those that lead a block

// How the row-block kernel cuts a batch: wavefronts per workgroup (row blocks of 32 * waves / G rows), batch rows per
// range (a multiple of 64), workgroups that share a range's row blocks (per K/V head and part), parts of every block's context.
struct BlockPlan {
    int waves, range, wgs, splits;
    bool count;          // the kernel settles the number of parts (at most splits) once it sees the row blocks
};
BlockPlan plan_blocks(int T, int n_seqs, int Hkv, int G, bool parts);

// Row-block kernel (bf16, head_dim 128): rows of one sequence that follow each other in the batch share
// the loads of their context.  Returns the hipError_t of its launch.
int launch_attention_blocks(const AttnArgs &a, int G, const BlockPlan &p, hipStream_t stream);

}  // namespace alora
