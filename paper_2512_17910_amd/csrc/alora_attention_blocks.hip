// Reader of the paged K/V cache for query rows that share a context: consecutive rows of one sequence
// (a projected suffix attending over a cached prefix, Sec. 2.3 / 4.2) are handled by ONE workgroup per
// K/V head, which loads every cached row once for all of them.  bf16, head_dim 128, on bf16 MFMA.
//
// A wavefront owns 32 columns (query row, query head of the K/V head's group): 32 / G rows; the wavefronts of a
// workgroup (eight, or four) consecutive rows, which share the K and V tiles of 32 context positions through LDS:
// every cached row is loaded once per 256 / G (128 / G) query rows.  Row blocks are cut at multiples of that number
// of the POSITION, so whether a batch row leads a block is decided from the row before it alone.
// The workgroups of a range of batch rows look the whole range over for leading rows and take them in turn: how many
// there are, a few of a prompt chunk or every row of a decode batch, is known on the device only.
//
// For batches with few row blocks the context of every block is cut into parts, one workgroup each, which
// leave (running maximum, weight sum, unnormalised output) per column for the kernel that combines them; how many,
// the kernel settles from the blocks it finds, within what the workspace was sized for.
//
// Per 32 context positions a wavefront runs two sets of 32x32x16 MFMAs that keep every column in the same
// two lanes (c, c+32) from the scores to the output:
//   scores^T [position x column] = K [position x d] . Q^T [d x column]   K rows from the LDS tile into the A operand
//       (a lane holds 8 consecutive d of one position), Q in registers;
//   online softmax down each column: 16 accumulator registers per lane, in most blocks no exchange between
//       lanes (none brings a new maximum) and no masking arithmetic where every column of the wavefront sees
//       the whole block;
//   out^T [d x column] += V^T [d x position] . P [position x column]   four tiles of 32 d; V comes back from LDS with
//       the transposing load, whose two halves are taken eight rows apart: that hands a lane exactly the
//       positions its score registers hold, so P is the score accumulator itself, rounded to bf16.
// K and V rows go from global memory straight into LDS (no registers in between), two blocks of 32 positions per
// barrier; the block-table entries of 64 blocks sit in an LDS window.  An assembly statement never reads a register
// an MFMA writes (the compiler cannot place the wait states for it); the copies and their wait counts are assembly
// because the compiler's own bookkeeping would wait for all of them.
//
// Measured, 4 x 2048 rows over 16K positions, 32/8 heads (2.06 TFLOP): 16 columns per wavefront on 16x16x32 MFMAs 2640 us
// (each byte read from LDS fed 16 columns, every block exchanged its maximum between four lanes); 32 columns, four
// wavefronts, with a maximum that lags (see the softmax), 2270, of it 440 for the copies; eight (half the copies per score), two blocks per
// barrier 2220 us = 0.93 PFLOP/s, where a large bf16 matrix product reaches 1.2 on the same card.  What is left: matrix
// unit 38 % and vector unit 42 % of the cycles, which add up more than they overlap, and the copies.  Running the
// scores of the next block and the output of the one before it between the vector instructions of the softmax
// (three blocks in flight, one matrix product per four vector instructions) was built and measured: 2470 us.
#include <numeric>
#include "alora_attention_internal.h"

namespace alora {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

constexpr float AB_NEG_INF = -__builtin_inff();
constexpr float AB_M_FLOOR = -1.0e30f;   // finite floor of the running maximum (scores below it weigh nothing)

// four k of this lane's column, then the four that lie eight rows further on
__device__ __forceinline__ bf16x8 read_tr_frag(const lds_byte *p, int pitch)
{
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 8 * pitch));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// 16 bytes straight from global memory into LDS at lds_addr + 16 * lane.  An assembly statement: the
// kernel orders these copies against its LDS reads itself (wait counts and barriers in the main loop).
__device__ __forceinline__ void load_lds16(uint32_t lds_addr, const void *p)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(p) : "memory");
}
// the same with a scalar base address and a 32-bit byte offset per lane; ONCE: no other workgroup will read these bytes
template <bool ONCE>
__device__ __forceinline__ void load_lds16(uint32_t lds_addr, const void *base, uint32_t voffset)
{
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(lds_addr), "v"(voffset), "s"(base) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voffset), "s"(base) : "memory");
}
// Exchange between the two lanes of a column (lanes c, c+32), as an assembly statement (the builtin returned its
// first result twice) with wait states on both sides, which the compiler cannot place for an instruction it does
// not see.  Checked with an in-bounds probe:
//   v_permlane32_swap on two copies of x: lo <- x of the lower 32 lanes, hi <- the upper 32 lanes'
__device__ __forceinline__ void both_halves(float x, float &lo, float &hi)
{
    lo = x, hi = x;
    asm("s_nop 3\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 3" : "+v"(lo), "+v"(hi));
}
// sums of floats, and largest from 0 on, over lanes 0 .. lane
__device__ __forceinline__ float sum_upto64(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x142, 0xa, 0xf, false));
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x143, 0xc, 0xf, false));
}
__device__ __forceinline__ int max_upto64(int x)
{
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
    return max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
}
// what a lane loads for a position that is not part of the context (the weighted sum multiplies it by 0)
__device__ const uint32_t ab_zero_chunk[4] = {0u, 0u, 0u, 0u};

// whether the kernel settles the number of parts (a kernel of its own: what the counting adds costs 2 x 2 rows at 2000 positions 1.3 of 13 us)
struct AsPlanned { static constexpr bool count = false, once = false; };
struct Counted { static constexpr bool count = true, once = false; };
// and contexts of which most are read once per head (see launch_attention_blocks); which, the kernel finds out
struct AsPlannedOnce { static constexpr bool count = false, once = true; };
struct CountedOnce { static constexpr bool count = true, once = true; };

// NW: wavefronts per workgroup; POW2: the block size is a power of two (shifts instead of divisions)
template <int G, int NW, bool POW2, typename PARTS>
__global__ __launch_bounds__(64 * NW, 2) void paged_attention_blocks_kernel(AttnArgs a, int range, int wgs)
{
    constexpr bool count = PARTS::count;
    constexpr int D = 128;
    constexpr int GPW = 8 / NW;       // groups of four positions a wavefront copies per block of 32
    constexpr int PLACES = NW == 8 ? 256 : 512;   // workgroups the chip holds at once
    constexpr int RBW = 32 / G;       // query rows per wavefront (32 columns = rows x heads of the group)
    constexpr int RBG = NW * RBW;     // query rows per workgroup
    constexpr int PITCH = 256;        // bytes per position row of the K and V tiles in LDS
    constexpr int TILE = 32 * PITCH;  // one tile: 32 positions
    constexpr int NB = NW == 8 ? 6 : 4;   // (K, V) tile pairs, taken two at a time (four wavefronts: two workgroups share a CU's LDS)
    __shared__ __attribute__((aligned(1024))) unsigned char tiles[NB * 2 * TILE];
    __shared__ __attribute__((aligned(16))) unsigned char ok_bytes[NB][8];     // byte i: validity of positions 4i .. 4i+3 of a pair
    constexpr int LOOK = LOOKED_OVER * NW, SCANS = LOOKED_OVER / 64;   // batch rows a workgroup looks over, and each of its threads
    __shared__ unsigned long long lead_mask[LOOK / 64];          // bit i of word j: row 64 j + i from the range's first leads a block
    __shared__ int32_t row_seq[LOOK], row_pos[LOOK];
    __shared__ u32x4 wave_found[NW];      // last position of a row, leading rows, what they cost in us (see there)
    // what 64 positions of a row block cost, us, and what every row of it adds (for the number of parts, see there)
    constexpr float US_BLOCK = NW == 8 ? 1.4f : 1.8f, US_ROW = NW == 8 ? .6f / RBG : 0.f;
    constexpr int WIN = 64;            // blocks of 32 positions whose table entries the window below holds
    __shared__ int32_t window[WIN * 32 / 4 + 2];   // block sizes are multiples of 4

    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4, li = lane & 31, lh = lane >> 5;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    // grid: (range of batch rows, workgroup of the range, K/V head, part of the context); a.splits parts, 1 = the whole context
    // (counted parts: one range, and the workgroups are dealt out once the row blocks are known)
    int splits = a.splits, part = 0, hk = 0, which = 0, r_begin = 0, r_end = a.T;
    if constexpr (!count) {
        part = (int)blockIdx.x % splits;
        const int bid = (int)blockIdx.x / splits;
        hk = bid % a.Hkv, which = bid / a.Hkv % wgs;
        r_begin = bid / a.Hkv / wgs * range, r_end = min(a.T, r_begin + range);
    }
    // ---- the rows of the range that lead a block (range <= LOOK - RBG: the RBG rows behind it say where its last block ends) ----
    // A row does unless the row before it in the batch is the same sequence's previous position and the position
    // is not a multiple of RBG (then an earlier row leads).  The workgroups of a range take them in turn: the leading rows
    // of a long run are RBG rows apart, those of a decode batch next to each other, and how they lie is known here only.
    {
        int sq[SCANS], p0[SCANS], sq1[SCANS], p1[SCANS];
#pragma unroll
        for (int i = 0; i < SCANS; ++i) {
            const int t = r_begin + i * 64 * NW + tid;
            sq[i] = sq1[i] = p0[i] = p1[i] = -1;
            if (t < a.T && t < r_end + RBG) {
                sq[i] = a.seq[t];
                p0[i] = a.pos[t];
                if (t > 0) { sq1[i] = a.seq[t - 1]; p1[i] = a.pos[t - 1]; }
            }
        }
        int furthest = 0, blocks = 0;          // last position of a row; leading rows
        float us = 0.f;                        // all their positions cost
#pragma unroll
        for (int i = 0; i < SCANS; ++i) {
            const bool ok = sq[i] >= 0 && sq[i] < a.n_seqs && p0[i] >= 0;
            const bool lead = !(ok && (p0[i] % RBG) != 0 && sq1[i] == sq[i] && p1[i] == p0[i] - 1);   // (row 0 has none before it)
            const unsigned long long mk = __builtin_amdgcn_ballot_w64(lead);
            if (lane == 0) lead_mask[i * NW + w] = mk;
            row_seq[i * 64 * NW + tid] = sq[i];
            row_pos[i * 64 * NW + tid] = p0[i];
            if (count && ok && i * 64 * NW + tid < a.T) {
                furthest = max(furthest, p0[i]);
                us += (float)p0[i] * (1.f / 64) * (lead ? US_BLOCK + US_ROW : US_ROW);
            }
            const int own = min(64, a.T - 64 * (i * NW + wu));     // rows of the word that are the batch's
            if (count && own > 0) blocks += (int)__builtin_popcountll(mk << (64 - own));
        }
        if constexpr (count) {
            wave_found[w] = (u32x4){(unsigned)__builtin_amdgcn_readlane(max_upto64(furthest), 63), (unsigned)blocks,   // (every lane writes the same)
                                    (unsigned)__builtin_amdgcn_readlane(__float_as_int(sum_upto64(us)), 63), 0u};
        }
        __syncthreads();
    }
    // n-th leading row of the range (counted from its first row; -1: it has not as many) and the rows of its block, up to the next
    // leading row or the end of the batch.  Lane j counts word j.
    struct Block { int at, rows; };
    auto block_of = [&](int n) -> Block {
        static_assert(LOOK / 64 <= 32, "a lane per word, two rows of lanes");
        const unsigned long long mk = lane < LOOK / 64 ? lead_mask[lane] : 0ull;
        const int own = min(64, r_end - r_begin - 64 * lane);      // rows of the word that are the range's
        const int c = own > 0 ? __builtin_popcountll(mk << (64 - own)) : 0;
        const int upto = sum_upto64(c);                            // leading rows in words 0 .. lane
        if (n >= __builtin_amdgcn_readlane(upto, 31)) return {-1, 0};
        auto word_of = [&](int j) {
            const unsigned lo = __builtin_amdgcn_readlane((unsigned)mk, j), hi = __builtin_amdgcn_readlane((unsigned)(mk >> 32), j);
            return ((unsigned long long)hi << 32) | lo;
        };
        const int word = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(n < upto));
        n -= __builtin_amdgcn_readlane(upto - c, word);
        const unsigned long long m = word_of(word);
        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));   // set bits below this lane's
        const int bit = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(((m >> lane) & 1ull) && before == n));
        const unsigned long long rest = m & (~1ull << bit), later = __builtin_amdgcn_ballot_w64(mk != 0ull) & (~1ull << word);
        int end = LOOK;
        if (rest) end = 64 * word + (int)__builtin_ctzll(rest);
        else if (later) { const int j = (int)__builtin_ctzll(later); end = 64 * j + (int)__builtin_ctzll(word_of(j)); }
        return {64 * word + bit, end - 64 * word - bit};
    };
    // ---- parts of every context, at most a.splits: what the partial sums have room for, and right only if rows fill their blocks and
    // nothing is cut off at a block's end.  How many blocks there are and how long the contexts is known here: lane i prices i + 1
    // parts, in us.  A workgroup takes START and US_BLOCK for 64 positions, and with eight wavefronts, which share a CU's matrix units, US_ROW
    // for every row besides.  As many as the chip has places for last as long as the longest one; more of them whole turns of it if
    // all are alike, and the more they differ the work there is and the end of a long one: a place whose part is short takes another.  A part's
    // sums are written and read at about 5 TB/s.  10 us of the call depend on none of it, and fewer parts have to promise 5 %.
    // Fitted to 1000 calls, and measured against always a.splits parts on 540 (1 to 64 sequences of 1 to 256 rows at 256 to 32K positions, 8 to
    // 64 heads): 1.15 times as fast on average, five calls under 0.97 (the counting takes up to 1 us; the worst, 0.87 and 0.89, are
    // 3 x 39 rows at 14-28K, 64/8 heads, 158 and 181 us, and 12 x 18 at 2-5.5K, 70 and 79).  With one length for all contexts and 8 us for a
    // start, which are the call's: 1.11 times, one call in 30 under 0.97.  us, always a.splits parts | priced like that | now, 32/8 heads: 4 x 16
    // rows over 2-3K positions 39.4 | 26.8 | 25.8, 8 x 7 over 1-4K 50.0 | 33.9 | 31.7, 32 single rows at 500-2000 88 | 48.9 | 45.5, 64 at 2-8K 325 |
    // 254 | 247, 2 x 200 rows at 7-9K 136 | 98 | 95, 4 x 60 at 9-16K 130 | 116 | 115, 8 x 30 at 6-12K 111 | 107 | 105, 3 x 155 at 1-3K
    // 47 | 54 | 44; 8/8 heads 3 x 212 at 3-10K 63 | 69 | 64; 64/8 heads 4 x 241 at 500-1600 113 | 125 | 112.
    // (What the counting itself took was a workgroup's start longer by 1 to 2 us, two of them in a row in a call of two turns: every value
    // of every wavefront added up in turn, and the plan's divisions twice.)
    if constexpr (count) {
        const u32x4 found = wave_found[lane % NW];        // (quad_perm with the neighbour and with the other pair, then the row's other quad)
        int longest = (int)found.x, blocks = (int)found.y;
        float total = __uint_as_float(found.z);
#define AB_MEET(CTRL)                                                                                             \
        longest = max(longest, __builtin_amdgcn_update_dpp(0, longest, CTRL, 0xf, 0xf, false));                   \
        blocks += __builtin_amdgcn_update_dpp(0, blocks, CTRL, 0xf, 0xf, false);                                  \
        total += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(total), CTRL, 0xf, 0xf, false))
        AB_MEET(0xb1);
        AB_MEET(0x4e);
        if (NW == 8) { AB_MEET(0x141); }
#undef AB_MEET
        constexpr float START = NW == 8 ? 2.f : 3.f, SUMS = NW == 8 ? 1.6e-4f : 2.4e-4f;
        const int parts = lane + 1, items = blocks * a.Hkv * parts;
        const float share = __builtin_amdgcn_rcpf((float)parts), turns = (float)((items + PLACES - 1) / PLACES);
        const float each = __builtin_amdgcn_rcpf((float)blocks);
        const float one = START + (US_BLOCK + US_ROW * (float)a.T * each) * (1.f / 64) * (float)longest * share, mean = START + total * each * share;
        float us = turns * one;
        if (turns > 1.f) {
            const float differ = fminf(fmaxf(4.f - 4.f * mean * __builtin_amdgcn_rcpf(one), 0.f), 1.f);
            us += differ * fminf((float)items * (1.f / PLACES) * mean + (NW == 8 ? .35f : .5f) * one - us, 0.f);
        }
        us += 10.f + (float)a.T * (float)a.Hq * (float)parts * SUMS;
        if (parts == splits) us *= .95f;
        unsigned key = parts <= splits ? (unsigned)fminf(us * 8.f, 1.0e8f) << 5 | (unsigned)lane : ~0u;
        static_assert(MAX_PARTS <= 32, "five bits, two rows of lanes");
        key = min(key, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)key, 0x111, 0xf, 0xf, false));
        key = min(key, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)key, 0x112, 0xf, 0xf, false));
        key = min(key, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)key, 0x114, 0xf, 0xf, false));
        key = min(key, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)key, 0x118, 0xf, 0xf, false));
        key = min(key, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)key, 0x142, 0xa, 0xf, false));
        splits = (int)(__builtin_amdgcn_readlane(key, 31) & 31u) + 1;
        // the grid's workgroups, dealt out (quotients of numbers far below 2^21, half way between two whole ones at the nearest)
        auto over = [](int x, float each) { return __builtin_amdgcn_readfirstlane((int)(((float)x + .5f) * each)); };
        const float part_each = __builtin_amdgcn_rcpf((float)splits), head_each = __builtin_amdgcn_rcpf((float)a.Hkv);
        const int bid = over((int)blockIdx.x, part_each);
        part = (int)blockIdx.x - bid * splits;
        which = over(bid, head_each);
        hk = bid - which * a.Hkv;
        wgs = over(over((int)gridDim.x, part_each), head_each);
        if (which >= wgs) return;
    }
    const int Nkv = a.Hkv * D;
    const long long n_blocks = a.n_slots / a.bs;
    const long long cap = (long long)a.max_blocks * a.bs;
    const uint32_t tiles_at = (uint32_t)(uintptr_t)(lds_byte *)tiles;
    const uint32_t row_bytes = (uint32_t)Nkv * 2u, head_bytes = (uint32_t)hk * D * 2u;
    const unsigned n_blocks_u = (unsigned)(n_blocks < 0x7fffffffll ? n_blocks : 0x7fffffffll);
    // ---- copies global -> LDS: wavefront w fills positions 4w .. 4w+3 of a block of 32 (of four wavefronts: and 16 further
    // on) with one K and one V instruction each (one cache block: block sizes are multiples of 4, so its table entry
    // is a scalar); lane -> position + lane / 16, physical 16-byte chunk lane % 16.
    // K tile: row = position, the physical chunk holds logical chunk XOR (row % 16) (the score product reads one
    // logical chunk of 32 rows).  V tile: row = position, XOR 4 * (row % 4) (the transposing read takes four chunks of
    // four rows per 32 lanes).
    const uint32_t row_off = (uint32_t)g4 * (uint32_t)Nkv * 2u;
    const uint32_t k_off = row_off + (uint32_t)((c16 ^ ((4 * wu + g4) & 15)) << 4);
    const uint32_t v_off = row_off + (uint32_t)((c16 ^ (g4 << 2)) << 4);
    // K fragment of k step ks (16 d): row li, chunk 2ks + lh -> k_base ^ (ks << 5)
    const uint32_t k_base = (uint32_t)li * PITCH + (uint32_t)((lh ^ (li & 15)) << 4);
    // V fragment of d tile dt (32 d) and positions 16s ..: rows 16s + 4lh + j (then eight further on), j = c16 / 4; the 8
    // bytes of d = 32dt + 16 * (lane / 16 % 2) + 4(c16 % 4) .. -> (v_base ^ (dt << 6)) + s * 16 * PITCH
    uint32_t v_base;
    {
        const int j = c16 >> 2, vrow = 4 * lh + j;
        v_base = (uint32_t)vrow * PITCH + (uint32_t)(((2 * (g4 & 1) + ((c16 & 3) >> 1)) ^ (j << 2)) << 4) + (uint32_t)((c16 & 1) << 3);
    }

  for (int turn = which;; turn += wgs) {
    const Block block = block_of(turn);
    if (block.at < 0) break;
    if (turn != which) __syncthreads();      // everyone is done with the tiles of the block before
    const int t0 = r_begin + block.at, nrows = block.rows;
    const int sq = __builtin_amdgcn_readfirstlane(row_seq[block.at]), p0 = __builtin_amdgcn_readfirstlane(row_pos[block.at]);
    int near_seq[2] = {-1, -1}, near_pos[2] = {-1, -1};      // rows before and behind the block
    if constexpr (PARTS::once) {
        const int before = max(block.at - 1, 0), behind = min(block.at + nrows, LOOK - 1);
        near_seq[0] = block.at > 0 ? row_seq[before] : -1, near_pos[0] = row_pos[before];
        near_seq[1] = block.at + nrows < LOOK ? row_seq[behind] : -1, near_pos[1] = row_pos[behind];
    }
    const bool row_ok = sq >= 0 && sq < a.n_seqs && p0 >= 0;
    int n_ctx = 0;
    if (row_ok) n_ctx = (int)((long long)p0 + nrows < cap ? (long long)p0 + nrows : cap);
    // this workgroup's part of the context: blocks c_lo .. c_hi - 1 of 32 positions (all of them without parts)
    int c_lo = 0, c_hi = (n_ctx + 31) >> 5;
    if (a.splits > 1) {
        const int per = (c_hi + splits - 1) / splits;
        c_lo = min(part * per, c_hi);
        c_hi = min(c_lo + per, c_hi);
        n_ctx = min(n_ctx, 32 * c_hi);                 // positions past the part are not loaded
    }
    const int n_chunks = c_hi;
    const int32_t *bt = a.bt + (size_t)(row_ok ? sq : 0) * a.max_blocks;

    // this lane's column: query row r_j of the block (rows w*RBW .. of this wavefront), query head g_j
    const int r_j = w * RBW + li / G, g_j = li % G;
    const bool col_ok = row_ok && r_j < nrows;
    const int lim_j = col_ok ? p0 + r_j : -1;                        // last position the column attends to
    const int lim_w = (row_ok && wu * RBW < nrows) ? p0 + min((wu + 1) * RBW, nrows) - 1 : -1;   // ... and any column of this wavefront
    const int lim_first = p0 + wu * RBW;                             // ... and the wavefront's first column
    const size_t q_at = ((size_t)(t0 + (col_ok ? r_j : 0)) * a.Hq + (size_t)hk * G + g_j) * D;
    bf16x8 qf[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (col_ok) v = *(const u32x4 *)((const bf16_t *)a.q + q_at + 16 * s + 8 * lh);
        qf[s] = __builtin_bit_cast(bf16x8, v);
    }
    f32x16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    float m = AB_M_FLOOR, l = 0.f;

    // Table entries come from a window in LDS that holds those of WIN blocks of 32 positions and is refilled
    // by the whole workgroup when the lookups reach its end (the index of four aligned positions is the same
    // in every lane); an entry past the context reads as -1.
    auto entry_of = [&](int pu) { return POW2 ? (pu >> a.bs_shift) : (pu / a.bs); };
    int win_first = 0, win_block = 0;        // table index of window[0]; first block the window covers
    auto refill = [&](int cw) {              // entries of blocks cw .. cw + WIN - 1; all wavefronts call it together
        win_block = cw;
        win_first = entry_of(32 * cw);
        const int last = entry_of(min(32 * (cw + WIN), n_ctx) - 1);      // n_ctx > 32 * cw whenever this is called
        __syncthreads();
        for (int i = tid; win_first + i <= last; i += 64 * NW) window[i] = bt[win_first + i];
        __syncthreads();
    };
    // Which cache block is half way through this part, and, where the batch rows before and behind this row block reach as far, in their contexts: the
    // same one if they are of the same run, or of a sequence over the same cached prefix.  Then this part is not read once, and its copies are ordinary
    // ones.  Known before the loop, which is there twice (a branch at every copy costs a call 3 to 6 %; a look at all rows of the range 1 us a block).
    // us, non-temporal | by what is found, and in brackets ordinary, 32/8 heads: a chunk of 2048 rows at 16K positions under a block table of 256 rows
    // 628 | 603 (607), of 1024 beside 255 single rows 354 | 350 (353), 16 x 8 rows in parts, each four sequences over one prefix of 8K, 100.0 | 96.4 (94.5), 20 x 4 at 3 to
    // 6K, some in two row blocks, 91.4 | 84.8 (91.7); 64 single rows over one prefix of 4K in parts 138.8 | 142.6 (139.6); nothing shared: 64 at 4096 169.4 | 169.6
    // (186.9), in parts 100 at 500 to 4000 179.2 | 180.4 (200.8).
    int half_here = -1, half_near[2] = {-2, -2};
    auto look_around = [&]() {
        const int half = min(16 * (c_lo + c_hi), n_ctx - 1), at = entry_of(half);
        half_here = bt[at];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int s2 = __builtin_amdgcn_readfirstlane(near_seq[i]);
            if (s2 >= 0 && s2 < a.n_seqs && __builtin_amdgcn_readfirstlane(near_pos[i]) >= half) half_near[i] = a.bt[(size_t)s2 * a.max_blocks + at];
        }
    };
    // table entry of this wavefront's four positions pu .. of a block (the same value in every lane; made a scalar
    // where it is used, a step later, so that nothing waits for the read here)
    auto lookup = [&](int pu) { return pu < n_ctx ? window[entry_of(pu) - win_first] : -1; };
    // (the scalar unit of a CU serves all its wavefronts: what a wavefront computes per step besides the
    // matrix and vector work is kept to a few instructions)
    auto issue4 = [&](auto once, int slot_pair, int c, int grp, int entry) {
        const int pu = 32 * c + 4 * grp, blk = __builtin_amdgcn_readfirstlane(entry);
        const uint32_t k_to = tiles_at + (uint32_t)slot_pair * (2 * TILE) + ((uint32_t)grp << 10), v_to = k_to + TILE;
        static_assert(4 * PITCH == 1 << 10, "tile geometry");
        unsigned okb = 0xfu;
        if ((unsigned)blk < n_blocks_u && pu + 4 <= n_ctx) {   // the usual case: scalar base, the lane's constant offset
            const unsigned slot = (POW2 ? ((unsigned)blk << a.bs_shift) : (unsigned)blk * (unsigned)a.bs) + (unsigned)(POW2 ? (pu & (a.bs - 1)) : (pu % a.bs));
            const unsigned long long at = (unsigned long long)slot * row_bytes + head_bytes;   // first of the four cache rows
            load_lds16<decltype(once)::value>(k_to, (const char *)a.kc + at, k_off);
            load_lds16<decltype(once)::value>(v_to, (const char *)a.vc + at, v_off);
        } else {           // rows that are not part of the context read 16 zero bytes
            const bool blk_ok = (unsigned)blk < n_blocks_u;
            const int n_ok = blk_ok ? max(0, min(4, n_ctx - pu)) : 0;
            okb = (1u << n_ok) - 1u;
            const unsigned slot = (blk_ok ? (unsigned)blk * (unsigned)a.bs : 0u) + (unsigned)(pu % a.bs);
            const unsigned long long at = (unsigned long long)slot * row_bytes + head_bytes;
            const bool have = g4 < n_ok;
            const void *kp = have ? (const void *)((const char *)a.kc + at + k_off) : (const void *)ab_zero_chunk;
            const void *vp = have ? (const void *)((const char *)a.vc + at + v_off) : (const void *)ab_zero_chunk;
            load_lds16(k_to, kp);
            load_lds16(v_to, vp);
        }
        ok_bytes[slot_pair][grp] = (unsigned char)okb;      // (every lane writes the same byte)
    };
    auto issue = [&](auto once, int slot_pair, int c, const int (&entry)[GPW]) {
#pragma unroll
        for (int h = 0; h < GPW; ++h) issue4(once, slot_pair, c, wu + NW * h, entry[h]);
    };
    // ---- scores^T = K . Q^T -------------------------------------------------------------------------
    auto scores = [&](int slot_pair) {
        const lds_byte *kb = (const lds_byte *)tiles + slot_pair * (2 * TILE);
        f32x16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
        bf16x8 kf[8];     // (all requested ahead of the products: a pair at a time would wait for LDS four times)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kf[ks] = *(const __attribute__((address_space(3))) bf16x8 *)(kb + (k_base ^ (uint32_t)(ks << 5)));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sc, 0, 0, 0);
        return sc;
    };
    auto consume = [&](int c, int slot_pair, f32x16 sc) {
        const int cb = 32 * c;
        const lds_byte *vb = (const lds_byte *)tiles + slot_pair * (2 * TILE) + TILE;
        const u32x2 ob = *(const u32x2 *)ok_bytes[slot_pair];
        bf16x8 vf[2][4];      // requested ahead of the softmax, which covers their way
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) vf[s][t] = read_tr_frag(vb + (v_base ^ (uint32_t)(t << 6)) + s * 16 * PITCH, PITCH);
        __builtin_amdgcn_sched_barrier(0);
        // ---- softmax down this lane's column (its 32 positions sit in two lanes) ---------------------
        __builtin_amdgcn_s_setprio(2);   // the vector arithmetic of this wavefront goes ahead of wavefronts waiting for the matrix unit
        const unsigned ok_lo = __builtin_amdgcn_readfirstlane(ob.x), ok_hi = __builtin_amdgcn_readfirstlane(ob.y);
        if (!((ok_lo & ok_hi) == 0x0f0f0f0fu && cb + 31 <= lim_first)) {   // a block that every column of the wavefront sees whole needs no mask
            auto nibbles = [](unsigned x) { x |= x >> 4; return (x & 0xffu) | ((x >> 8) & 0xff00u); };
            const unsigned okmask = nibbles(ok_lo) | (nibbles(ok_hi) << 16);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int idx = 8 * (v >> 2) + 4 * lh + (v & 3);
                const bool on = ((okmask >> idx) & 1u) && cb + idx <= lim_j;
                sc[v] = on ? sc[v] : AB_NEG_INF;
            }
        }
        float mx = fmaxf(sc[0], sc[1]);
#pragma unroll
        for (int v = 2; v < 16; v += 2) mx = fmaxf(fmaxf(mx, sc[v]), sc[v + 1]);
        // The running maximum moves (and everything summed so far with it) only where some column of the wavefront has a
        // larger score, which its two lanes then settle between them; long before the end of a long context most
        // blocks bring none.  (Letting it lag by up to a factor 2^8 in weight takes 4 % off a call of 4 x 2048 rows, but
        // then the largest weight is no longer exactly 1 in bf16: error against fp64 2.31e-3 -> 2.34e-3 there, 2.01e-3 ->
        // 2.28e-3 on peaked scores.)
        if (__builtin_amdgcn_ballot_w64(mx * a.scale_log2e > m)) {
            float lo, hi;
            both_halves(mx, lo, hi);
            const float mn = fmaxf(m, fmaxf(lo, hi) * a.scale_log2e);
            const float corr = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= corr;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[t][e] *= corr;
        }
        float ps = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            sc[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[v], a.scale_log2e, -m));
            ps += sc[v];
        }
        l += ps;
        // ---- out^T += V^T . P : P straight from the score registers (k step s: positions 16s + 4lh .. +3 and eight
        // further on) -------------------------------------------------------------------------------------
        u32x4 pv[2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
            pv[s] = (u32x4){pack_bf16(sc[8 * s], sc[8 * s + 1]), pack_bf16(sc[8 * s + 2], sc[8 * s + 3]), pack_bf16(sc[8 * s + 4], sc[8 * s + 5]),
                            pack_bf16(sc[8 * s + 6], sc[8 * s + 7])};
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s][t], __builtin_bit_cast(bf16x8, pv[s]), acc[t], 0, 0, 0);
    };

    // ---- the context, two blocks of 32 positions at a time: all wavefronts share the tiles ----------
    // Block c_lo + i lives in tile pair i % NB.  A step takes blocks c and c+1: every wavefront waits for its own copies
    // of them (those of the NB - 4 blocks after them stay in flight), the barrier makes that hold for all of them
    // and tells that blocks c-2 and c-1 have been multiplied by everyone; their pairs then take the copies of the
    // next two blocks, whose table entries were looked up a step earlier.  Blocks past the context are copied
    // too (all zeros, from one 16-byte constant), which keeps the count of copies in flight the same in every step.
    {
        bool once = PARTS::once;
        if (n_chunks > c_lo) {
            if (PARTS::once) look_around();
            refill(c_lo);
            if (PARTS::once) {
                asm volatile("" : "+v"(half_here), "+v"(half_near[0]), "+v"(half_near[1]));   // (looked at here, not where they are requested)
                once = __builtin_amdgcn_readfirstlane(half_here != half_near[0] && half_here != half_near[1]);
            }
        }
        // (a use of the query registers ahead of the loop: the compiler places its wait for these loads here, behind that for the
        // table entries, and not in front of the first MFMA of every step, where it would also wait for the copies in flight)
#pragma unroll
        for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[s]));
        auto entries = [&](int cb, int (&e)[GPW]) {
#pragma unroll
            for (int h = 0; h < GPW; ++h) e[h] = lookup(32 * cb + 4 * (wu + NW * h));
        };
        int b0[GPW], b1[GPW];
        int cur = 0, nxt = NB - 2;           // tile pairs of block c and of block c + NB - 2
        auto start = [&](auto once) {
#pragma unroll
            for (int kk = 0; kk < NB - 2; ++kk) {
                entries(c_lo + kk, b0);
                issue(once, kk, c_lo + kk, b0);
            }
            entries(c_lo + NB - 2, b0);
            entries(c_lo + NB - 1, b1);
        };
        auto step = [&](auto once, int c) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * GPW * (NB - 4)) : "memory");
            issue(once, nxt, c + NB - 2, b0);
            issue(once, nxt + 1, c + NB - 1, b1);
            const int cn = c + NB;
            if (cn == win_block + WIN && 32 * cn < n_ctx) refill(cn);
            entries(cn, b0);
            entries(cn + 1, b1);
        };
        auto advance = [&]() { cur = cur + 2 == NB ? 0 : cur + 2; nxt = nxt + 2 == NB ? 0 : nxt + 2; };
        // (two loops: the accumulators live in the first only)
        const int n_chunks_w = lim_w >= 0 ? min((lim_w >> 5) + 1, n_chunks) : 0;
        int c = c_lo;
        // (the loop on a line of the instruction cache: 8 single rows at 16K positions 398 us without, 393 with, twice in a kernel 336 and 329; 4 x 1024 rows at
        // 8192, 594 and 581)
#define AB_CONTEXT(ONCE)                                                                                                                           \
        start(ONCE{});                                                                                                                             \
        if (ONCE::value) asm volatile(".p2align 6" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])); /* (cleared ahead of the line) */    \
        else asm volatile(".p2align 6");                                                                                                           \
        for (; c < n_chunks_w; c += 2) {                                                                                                           \
            step(ONCE{}, c);                                                                                                                       \
            consume(c, cur, scores(cur));                                                                                                          \
            if (c + 1 < n_chunks_w) consume(c + 1, cur + 1, scores(cur + 1));                                                                      \
            advance();                                                                                                                             \
        }                                                                                                                                          \
        asm volatile(".p2align 6");                                                                                                                \
        for (; c < n_chunks; c += 2) {                                                                                                             \
            step(ONCE{}, c);                                                                                                                       \
            advance();                                                                                                                             \
        }
        // (a macro: as a function object it changes the registers of the kernels that have one loop only, and costs them 1 to 2 %)
        if (PARTS::once && once) { AB_CONTEXT(std::bool_constant<PARTS::once>) }
        else { AB_CONTEXT(std::false_type) }
#undef AB_CONTEXT
        // nothing may be on its way into LDS when the workgroup gives it back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }

    // ---- the two lanes of a column add their weight sums; normalise and store -----------------------
    {
        float lo, hi;
        both_halves(l, lo, hi);
        l = lo + hi;
    }
    if (a.splits > 1) {
        // this part's (running maximum, weight sum, unnormalised output) of every column, for the kernel that
        // combines the parts of a (row, query head) in part order
        if (col_ok || (!row_ok && w == 0 && li < G)) {
            float *p0 = a.part + ((size_t)(t0 + (col_ok ? r_j : 0)) * a.Hq + (size_t)hk * G + g_j) * a.splits * (D + 2), *pp = p0 + part * (D + 2);
            if (lh == 0) *(f32x2 *)pp = (f32x2){m, l};
            // fewer parts than there is room for: the last place tells how many (a sum of weights is never negative)
            if (count && lh == 0 && part == 0 && splits < a.splits) *(f32x2 *)(p0 + (a.splits - 1) * (D + 2)) = (f32x2){(float)splits, -1.f};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 16; v += 4) {
                    *(f32x2 *)(pp + 2 + 32 * t + 2 * v + 4 * lh) = (f32x2){acc[t][v], acc[t][v + 1]};
                    *(f32x2 *)(pp + 2 + 32 * t + 2 * v + 4 * lh + 2) = (f32x2){acc[t][v + 2], acc[t][v + 3]};
                }
        }
        continue;
    }
    // Columns are rows of the result: a wavefront turns its 32 around through LDS, in the tiles nobody reads any more, so that a store
    // instruction writes four pieces of 256 bytes.  (Straight from the registers it would be 8 bytes of 32 rows: one
    // run of 300 rows at 2048 positions 85.1 us, now 83.6; the sums of parts, few columns to a workgroup, go straight: through LDS
    // one row at 1000 positions pays 0.5 of 9 us.)
    __syncthreads();
    lds_byte *strip = (lds_byte *)tiles + wu * (int)(sizeof(tiles) / NW);
    constexpr int SP = 256 + 16;             // bytes per column of 128 bf16
    static_assert(32 * SP <= sizeof(tiles) / NW, "a strip per wavefront");
    auto column_ok = [&](int c) { return row_ok ? wu * RBW + c / G < nrows : wu == 0 && c < G; };   // a row that is not valid leads a block of its own
    auto result_at = [&](int c) { return (size_t)(t0 + wu * RBW + c / G) * a.Hq + (size_t)hk * G + c % G; };   // (row, query head) of column c
    // a row that is not valid gets zeros
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; v += 4)       // d = 32 t + 8 (v / 4) + 4 lh ..
            *(__attribute__((address_space(3))) u32x2 *)(strip + li * SP + (32 * t + 2 * v + 4 * lh) * 2) =
                (u32x2){pack_bf16(acc[t][v] * inv, acc[t][v + 1] * inv), pack_bf16(acc[t][v + 2] * inv, acc[t][v + 3] * inv)};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = 4 * i + g4;
        const u32x4 o = *(const __attribute__((address_space(3))) u32x4 *)(strip + c * SP + 16 * c16);
        if (column_ok(c)) *(u32x4 *)((bf16_t *)a.out + result_at(c) * D + 8 * c16) = o;
    }
  }
}

// How a batch is cut, from its sizes alone.
// Eight wavefronts share a context's copies among twice the rows and keep six tile pairs in LDS where four keep four, but a CU holds
// one such workgroup: nothing covers its start and its stores.  They take
//   - runs of 1024 rows on average, where that gives two workgroups per CU: the copies count, starts do not;
//   - few short blocks, at most one per CU and all of them at once: only the depth of the copies counts;
//   - long runs whose contexts are cut into parts.
// us, eight | four wavefronts: 4 x 2048 rows at 16K positions, 32/8 heads 2211 | 2337, 4 x 1024 at 8192 591 | 619, 3 x 1300 at 5-6K 510 |
// 510, 12 x 700 at 3K 537 | 525, 30 prompts of 200-600 153 | 140, 100 of 128 117 | 97, 200 of 30-90 107 | 88; 8 single rows at 16K
// 330 | 390, 32 at 300 37 | 42, 4 x 64 rows at 16K, 8/8 heads 357 | 414; in parts, 4 x 64 rows over 16K 108 | 123, 4 x 32 104 | 78.
BlockPlan plan_blocks(int T, int n_seqs, int Hkv, int G, bool parts)
{
    BlockPlan p = {4, 64, 1, 1, false};
    if (T <= 0) return p;
    const bool long_runs = (long long)T * G > 128ll * n_seqs;   // longer than a block of four wavefronts
    if (long_runs) {
        if (parts || (T >= 1024ll * n_seqs && (long long)T * G / 256 * Hkv >= 512)) p.waves = 8;
    } else if (!parts) {
        const long long blocks8 = n_seqs + 2 * (((long long)T * G + 255) / 256);   // (a run of r rows lies in two with a chance of r G / 256)
        if ((blocks8 < T ? blocks8 : T) * Hkv <= 256) p.waves = 8;
    }
    const int rbg = 32 * p.waves / G;
    if (parts) {
        // parts of every block's context, one workgroup each, until there is one per CU (two of four wavefronts); the kernel
        // takes fewer where there turn out to be more than T / rbg blocks
        const long long wgs = (long long)((T + rbg - 1) / rbg) * Hkv, want = p.waves == 8 ? 256 : 512;
        if (wgs < want) p.splits = (int)((want + wgs - 1) / wgs < MAX_PARTS ? (want + wgs - 1) / wgs : MAX_PARTS);
        if (p.splits == 1) return plan_blocks(T, n_seqs, Hkv, G, false);   // nothing is cut: the call is the one without parts
    }
    // Ranges as long as a workgroup looks over at once, each with a workgroup per row block it can hold: T / rbg of long runs and
    // two more for every sequence (its first and its last block; one where there are several ranges, since few sequences start in
    // each), as far as 2048 workgroups allow; where there are more blocks than that, a workgroup takes several.  In parts, where a
    // workgroup per rbg rows fills the chip and one that finds no block waits for a place on it: one more for every sequence unless
    // T is whole blocks for each, and 4096 in all.  (us, in parts, without | with one more: 3 x 150 rows at 9000, 8/8 heads 83 | 73,
    // 5 x 200 at 30K 430 | 341, 1024 and 16 single rows at 8192, 32/8 heads 375 | 310; 4 x 64 at 4096 42.5 | 44.1.)
    // How rows lie is not known here, and one workgroup with several blocks is the whole call's length: with ranges of at most a
    // block's rows, each shared by one or two workgroups, decode rows beside a prompt chunk were up to 16 contexts in a row.
    // us, 32/8 heads, such ranges | the ranges before them (128 / G rows, halved until 2048 workgroups) | now: 2048 rows and 32 single
    // rows at 4096 positions 1690 | 825 | 274, 1024 and 16 at 8192 1635 | 800 | 317, 4 x 512 and 32 at 4096 1730 | 905 | 299, in
    // parts 1490 | 904 | 291; 5 x 61 rows at 8190 442 | 325 | 229; equal runs the same (4 x 1024 rows at 8192 622 | 1280 | 584).
    const int most = LOOKED_OVER * p.waves - (rbg + 63) / 64 * 64;   // (they look rbg rows further)
    int ranges = (T + most - 1) / most;
    const int unit = rbg > 64 ? rbg : 64;
    p.range = ((T + ranges - 1) / ranges + unit - 1) / unit * unit;
    ranges = (T + p.range - 1) / p.range;
    const int rows = p.range < T ? p.range : T;
    const long long blocks = (rows + rbg - 1) / rbg, heads = (long long)ranges * Hkv * p.splits;
    const bool whole = n_seqs > 0 && T % n_seqs == 0 && T / n_seqs % rbg == 0;   // every sequence may bring whole blocks
    long long ends = p.splits > 1 ? (whole ? 0 : n_seqs) : ranges > 1 ? n_seqs + 1ll : 2ll * n_seqs, spare = p.splits > 1 ? 4096 / heads - blocks : 2048 / heads;
    if (ranges > 1) {
        // Workgroups go to the eight XCDs in turn, and on each to its four shader engines; one whose engine is full holds up all
        // behind it.  Between the blocks of one range and the next, workgroups without any in other than whole turns leave places
        // empty for as long as a block takes: 4 x 2048 rows at 16K positions, five ranges, 5 of them 2530 us, 8 of them 2216; 4 x 1024
        // at 8192 813 and 591.  (Ranges are whole blocks for the same reason.)
        const long long m = 32 / std::gcd(32, Hkv * p.splits);
        ends = (ends + m - 1) / m * m;
        spare = spare / m * m;
    }
    const long long wgs = blocks + (spare < 0 ? 0 : spare < ends ? spare : ends);
    p.wgs = (int)(wgs < rows ? wgs : rows);
    // Parts counted by the kernel (one range: every workgroup sees all blocks) where as many blocks as runs that start anywhere
    // make on average would not fit the chip at once: a call that fits pays 1 us for nothing (2 x 2 rows at 2000 positions 12.8 us,
    // counted 14.1).  And where there are four parts to choose from: of 54 calls cut into two or three, 26 lost more than they gained
    // (3 x 222 rows at 1-4K 68.5 us, counted 71.4; 4 x 241, 64/8 heads, at 500-1600 114 and 125), six gained 3 to 9 %.
    const long long n = n_seqs < T ? n_seqs : T, likely = whole ? T / rbg : n + (T - n) / rbg;
    p.count = p.splits > 1 && ranges == 1 && likely * Hkv * p.splits > (p.waves == 8 ? 256 : 512);
    return p;
}

int launch_attention_blocks(const AttnArgs &a, int G, const BlockPlan &p, hipStream_t stream)
{
    const int ranges = (a.T + p.range - 1) / p.range;
    const dim3 grid((unsigned)ranges * (unsigned)p.wgs * (unsigned)a.Hkv * (unsigned)a.splits), block(64 * p.waves);
    const bool pow2 = a.bs_shift >= 0;
#define AB_LAUNCH_AS(GG, NW, POW2, PARTS) launch_kernel((paged_attention_blocks_kernel<GG, NW, POW2, PARTS>), grid, block, 0, stream, a, p.range, p.wgs)
    // A kernel that streams what is read once where a sequence brings a quarter of a row block on average (then few runs lie in two blocks, which would both read the
    // context; the rows of the block table are taken for the call's sequences, of which there may be fewer) and the memory-side cache would not keep K and V.
    // us, ordinary | non-temporal, 32/8 heads: 64 single rows at 4096
    // positions 187 | 169, in parts 100 at 500 to 4000 201 | 179, 6 at 10K to 30K 110 | 100, 40 x 6 rows at 2K to 5K 148 | 144; 4 x 11 at
    // 16K to 20K 75 | 74, 4 x 24 98 | 103, 40 x 20 at 2K to 5K 188 | 197, 8/8 heads 6 x 40 at 10K to 30K 143 | 153.
    const bool once = pow2 && (long long)a.T * G <= 32ll * a.n_seqs && outgrows_cache(a.n_slots, a.Hkv, 128, true);
#define AB_LAUNCH(GG, NW) \
    if (once && p.count && NW == 4) AB_LAUNCH_AS(GG, 4, true, CountedOnce); \
    else if (once && !p.count) AB_LAUNCH_AS(GG, NW, true, AsPlannedOnce); \
    else if (p.count && pow2) AB_LAUNCH_AS(GG, NW, true, Counted); \
    else if (p.count) AB_LAUNCH_AS(GG, NW, false, Counted); \
    else if (pow2) AB_LAUNCH_AS(GG, NW, true, AsPlanned); \
    else AB_LAUNCH_AS(GG, NW, false, AsPlanned)
    switch (G * 16 + p.waves) {
    case 16 + 8: AB_LAUNCH(1, 8); break;
    case 32 + 8: AB_LAUNCH(2, 8); break;
    case 64 + 8: AB_LAUNCH(4, 8); break;
    case 128 + 8: AB_LAUNCH(8, 8); break;
    case 16 + 4: AB_LAUNCH(1, 4); break;
    case 32 + 4: AB_LAUNCH(2, 4); break;
    case 64 + 4: AB_LAUNCH(4, 4); break;
    case 128 + 4: AB_LAUNCH(8, 4); break;
    default: return (int)hipErrorInvalidValue;
    }
#undef AB_LAUNCH
#undef AB_LAUNCH_AS
    return launch_status();
}

}  // namespace alora
