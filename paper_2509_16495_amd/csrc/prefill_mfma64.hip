// Causal prefill attention of the local head shard over the paged KV cache (Algorithm 1, boxed attention line,
// prefill rows; chunked prefill continues a cached context): the wide-tile kernel.  bf16 tensors, fp32
// accumulation, head_dim 128, bf16 cache.
//
// One wavefront per SIMD, 64 columns per wavefront.  A workgroup is four wavefronts and owns a tile of 256
// "columns"; a column is one (new token, query head) pair, the G query heads that share a KV head lying next to
// each other (column = token * G + head, any G up to 256), so one K/V tile serves the whole GQA group.  All four
// wavefronts walk the same keys, 32 at a time (two cache blocks), and share every K and V^T tile through LDS:
// against a 128-column tile with 32-column wavefronts this halves the bytes that go from the cache into LDS per
// MFMA, halves the operand bytes read from LDS per MFMA (an operand read feeds two MFMAs, one per 32-column
// block) and halves the barriers per SIMD.  The price is registers - Q^T (64), O^T (128), two S^T tiles (64) and
// two P^T tiles (32) per lane - which is why only one wavefront fits a SIMD; the matrix pipe and the vector ALU
// then overlap inside the one instruction stream, which is written out slot by slot (one MFMA, the softmax work
// of one logit, a share of the operand reads).
//
// Math per key tile, transposed so that P never leaves registers (as in the 128-column kernel):
//   S^T[key][col]  = K[key][:] . Q^T[:][col]      32x32x16 bf16 MFMA, A = K rows from LDS, B = Q^T in registers
//   O^T[d][col]   += V^T[d][key] . P^T[key][col]  A = V^T rows from LDS, B = P^T straight from the softmax
// with bits 2 and 3 of the K row index swapped in the MFMA row assignment, so that the keys a lane holds are runs
// of eight consecutive tokens (one 16-byte piece of a dimension-major V row).
//
// Softmax against a reference that lags.  Softmax does not care which reference its exponentials are shifted by as long
// as nothing leaves the range of bf16 and the fp32 sums.  The first attempt at a pass takes the reference from the
// column's first visible key tile, or the first two (whose maximum then gets P = 1 exactly: a row with few keys, all in
// those, comes out as exactly as the careful way would give it) and follows no maximum behind it: a fused multiply-add, an
// exponential and the row sum per logit, one packing per two, is all the loop spends on the softmax.  Real logits stay
// within 2^100 of their first tile's maximum, and P up to 2^100 is held by bf16 and the fp32 sums without loss; a column
// whose sum ends beyond that flags the pass, which is then run again the careful way: the exponentials of a tile are
// taken against the column's reference maximum as it stood when the tile began (so they do not wait for the tile's own
// maximum and spread evenly over the MFMA slots), the tile's maximum is collected on the side and checked against the
// reference (slack 2^32): a column that has no sums yet takes a new reference and recomputes the tile's P from the S^T
// values it still holds, one that has sums flags the pass once more, and the third attempt starts from references
// within the slack of every column's true maximum.  O^T is never rescaled inside the loop.
// A process-wide switch (off by default) makes the first attempt cheaper still: Q^T is multiplied by the softmax scale
// when the tile fetches it and rounded to bf16 again, the logits leave the MFMAs in exp2 units, and P is the exp2 of
// the logit itself, with no reference at all (sums must end inside [2^-40, 2^40]).  A logit then moves by up to 2^-9 of
// its value and the largest P is no longer exactly 1, which can put an output of magnitude 2 or more one bf16 step from
// the correctly rounded value; a pass that is flagged fetches Q^T again as given.
//
// Pipeline of iteration j: S^T of tile j+1 (16 MFMAs), softmax of tile j, O^T += V^T P^T of tile j-1 (16 MFMAs).
// LDS holds a ring of four stages of K (32 keys) + V^T (32 keys), tile t in stage t%4, so that the four iterations of a
// trip of the loop read and fill stages known at compile time.  During iteration j wavefronts 0 and 1 bring K of tile j+4
// (one cache block each) and wavefronts 2 and 3 V^T of tile j+2, by direct-to-LDS loads; what iteration j reads was loaded
// three iterations earlier and made visible by the barrier of the iteration before, so operand reads and MFMAs run on
// across the one barrier per iteration.
//
// What bounds the loop.  A lone wavefront issues an instruction about every four clocks (an exponential takes eight, a
// v_readlane nine), a 32x32x16 MFMA occupies the matrix pipe for 32: the pipe stays busy if every slot - an MFMA and what
// follows it - asks for no more than 28 clocks besides, and if an operand read follows the MFMA of its slot instead of
// standing in front of it (32.1 against 37.1 clocks a slot, everything else alike).  So the work is dealt to the slots
// evenly, the addresses of the loads are kept ready in a vector register pair, and nothing is moved between register files.
// MFMA pipe busy 60 -> 69 % of a launch's SIMD-clocks (81 % of those with a wavefront resident; 2048 tokens on 131072 cached); what
// is left is the power limit, the clock settles at 1.76 instead of 2.05 GHz:
// 16384 tokens of 8 heads 464 -> 424 us, 2048 tokens on 131072 cached with 64 decodes 957 -> 882.
//
// Two groups (kG = 2).  The same wavefronts on a tile of 128 columns: wavefronts 0 and 1 walk the even key tiles, 2 and 3 the odd
// ones, each pair with a ring of its own and a first-tile reference of its own, and the groups merge through LDS at the end, each
// finishing one half of the head dimension.  Twice the bytes into LDS per MFMA, half the length of a pass: what batches take whose
// 256-column tiles would not fill the chip.  4 x 4096 tokens of 4 heads: 73.2 us in the 128-column kernel of eight 32-column
// wavefronts, 85 in tiles of 256 columns, 67.6 here.
//
// Scheduling: tiles of a sequence are processed in pairs (heaviest with lightest) by one workgroup; a short chunk on a
// long context is taken one tile per workgroup, its keys split into ranges merged by launch_combine.
#include "decode_body.h"
#include "tile_order.h"

#include <utility>

namespace shiftattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;
constexpr int kThreads = 256;
constexpr int kCols = 256;                     // columns of a workgroup tile
constexpr int kKv = 32;                        // keys per iteration
constexpr int kKBytes = kKv * kD * 2;          // 8192: K tile, 32 rows of 256 B
constexpr int kVBytes = kD * kKv * 2;          // 8192: V^T tile, 2 blocks of [128 rows][32 B]
constexpr int kStageBytes = kKBytes + kVBytes; // 16384
constexpr int kRingBytes = 4 * kStageBytes;    // 65536
constexpr int kBlockBytes = kBlockSize * kD * 2;  // 4096: K (or V^T) of one cache block and head
constexpr int kPitch = 272;                    // row pitch of the output staging tile (256 + 16 bytes)
constexpr int kFlagBytes = 16;                 // one redo flag per wavefront
constexpr int kFlagsAt = kRingBytes + kCols * kPitch;
constexpr int kIdsAt = kFlagsAt + kFlagBytes;  // two windows of 64 block ids per wavefront
constexpr int kLdsBytes = kIdsAt + kPrefill64Waves * 2 * 64 * 4;  // 137232
// Two groups: a ring each; when the key loops are over the same bytes hold what the groups exchange - parked accumulators, one
// (reference, sum) pair per column block and lane - and the staged rows.
constexpr int kParkBytes = kPrefill64Waves * 64 * 64 * 4;                        // 65536
constexpr int kMlAt = kParkBytes, kStagedAt = kMlAt + kPrefill64Waves * 2 * 64 * 8;  // 69632
static_assert(2 * kRingBytes <= kFlagsAt && kStagedAt + kCols / 2 * kPitch <= 2 * kRingBytes);
// A column's reference maximum may lag its true running maximum by this much (exp2 units): P reaches 2^32 at most, far
// inside what bf16 and the fp32 sums hold (their relative precision does not depend on magnitude); O^T overflows only
// for |V| beyond 2^70.
constexpr float kRefSlack = 32.0f;
// The first attempt on scaled Q^T uses no reference (see the top of the file): the sum of a column that sees keys must end
// inside this range - its largest P then lies within a factor "number of keys" of the sum, far from bf16's denormals and
// from overflow (O^T overflows only for |V| beyond 2^87), and every logit that matters lies within 40 + log2(keys) of
// zero (which also bounds what a second rounding of Q^T can move).  An infinity or a NaN fails the test.
constexpr float kFreeSumLo = 0x1p-40f, kFreeSumHi = 0x1p40f;
// The default first attempt keeps the reference the column's first key tiles left and follows no maximum behind it: P may
// then reach 2^100 (still far inside bf16 and fp32 range; O^T overflows only for |V| beyond 2^27), and a sum beyond that
// sends the pass to the attempts that do follow the maximum.
constexpr float kKeepSumBound = 0x1p100f;

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

template <int kV>
struct IC {
    static constexpr int value = kV;
};

#define SHIFTATTN_INLINE __attribute__((always_inline))
#define SHIFTATTN_FORCE_INLINE inline __attribute__((always_inline))

// s_waitcnt vmcnt(0) with the other counters left alone (gfx9 encoding)
__device__ inline void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The matrix instructions are written as assembly to fix where their accumulators live: S^T in ordinary vector
// registers (the softmax reads every element with the vector ALU), O^T in accumulation registers (touched by
// nothing but MFMAs in the steady state), Q^T (a B operand) in accumulation registers as well.  Left to itself the
// compiler gives all MFMA results of a function to one register file and copies S^T across, one extra vector
// instruction per logit.  The compiler does not see that these statements are MFMAs, so it inserts none of the wait
// states a reader of their result needs (11 for an 8-pass MFMA): every place where compiler-generated code reads
// such a result sits behind at least that many instructions, and mfma_settle() is put where that is not evident.
// The same blindness works the other way: where the compiler itself writes an MFMA source right in front of such a
// statement (it moves accumulators between registers where differently allocated copies of the loop body meet) it adds
// no wait state either, and the MFMA reads a stale register.  kGuard puts the wait states into the statement; every
// MFMA outside the steady-state loop is guarded, the loop itself has no such writes (its accumulators never move).
template <bool kGuard>
__device__ SHIFTATTN_FORCE_INLINE void mfma_s_first(f32x16& d, u32x4 a, bf16x8 b) {
    if constexpr (kGuard) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
}
template <bool kGuard>
__device__ SHIFTATTN_FORCE_INLINE void mfma_s_acc(f32x16& d, u32x4 a, bf16x8 b) {
    if constexpr (kGuard) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
template <bool kGuard>
__device__ SHIFTATTN_FORCE_INLINE void mfma_o_acc(f32x16& d, u32x4 a, u32x4 b) {
    if constexpr (kGuard) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
// Wait states in front of compiler-generated reads of accumulators (and of anything else in their registers): the
// statement takes the accumulators as operands, so that they are read, or their registers used again, behind it only.
__device__ SHIFTATTN_FORCE_INLINE void mfma_settle(f32x16 (&d)[2]) { asm volatile("s_nop 7\n\ts_nop 7" : "+v"(d[0]), "+v"(d[1])); }
__device__ SHIFTATTN_FORCE_INLINE void mfma_settle(f32x16 (&d)[2][4]) {
    asm volatile("s_nop 7\n\ts_nop 7" : "+a"(d[0][0]), "+a"(d[0][1]), "+a"(d[0][2]), "+a"(d[0][3]), "+a"(d[1][0]), "+a"(d[1][1]), "+a"(d[1][2]), "+a"(d[1][3]));
}

// Q^T of a lane - eight 16-byte pieces for each of its two column blocks, 32 bytes apart - from global memory straight
// into accumulation registers, where the MFMAs take it as their B operand (a value that is born in ordinary registers
// and only used from accumulation registers is copied across at every use).  One statement with its own wait: the
// compiler does not know these are loads, so the registers must hold their values when the statement ends.
__device__ SHIFTATTN_FORCE_INLINE void load_q_to_acc(bf16x8 (&q0)[8], bf16x8 (&q1)[8], const void* p0, const void* p1) {
    asm volatile(
        "global_load_dwordx4 %0, %16, off\n\tglobal_load_dwordx4 %1, %16, off offset:32\n\t"
        "global_load_dwordx4 %2, %16, off offset:64\n\tglobal_load_dwordx4 %3, %16, off offset:96\n\t"
        "global_load_dwordx4 %4, %16, off offset:128\n\tglobal_load_dwordx4 %5, %16, off offset:160\n\t"
        "global_load_dwordx4 %6, %16, off offset:192\n\tglobal_load_dwordx4 %7, %16, off offset:224\n\t"
        "global_load_dwordx4 %8, %17, off\n\tglobal_load_dwordx4 %9, %17, off offset:32\n\t"
        "global_load_dwordx4 %10, %17, off offset:64\n\tglobal_load_dwordx4 %11, %17, off offset:96\n\t"
        "global_load_dwordx4 %12, %17, off offset:128\n\tglobal_load_dwordx4 %13, %17, off offset:160\n\t"
        "global_load_dwordx4 %14, %17, off offset:192\n\tglobal_load_dwordx4 %15, %17, off offset:224\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&a"(q0[0]), "=&a"(q0[1]), "=&a"(q0[2]), "=&a"(q0[3]), "=&a"(q0[4]), "=&a"(q0[5]), "=&a"(q0[6]), "=&a"(q0[7]),
          "=&a"(q1[0]), "=&a"(q1[1]), "=&a"(q1[2]), "=&a"(q1[3]), "=&a"(q1[4]), "=&a"(q1[5]), "=&a"(q1[6]), "=&a"(q1[7])
        : "v"(p0), "v"(p1)
        : "memory");
}

// block tables are read through the constant address space: with a wavefront-uniform index the compiler then issues
// scalar loads (and places the waits itself)
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
// operand reads take their LDS address as a plain 32-bit number (formed once from the array's base): indexing the
// shared array with a register costs a vector addition of the base per read
typedef const __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
__device__ SHIFTATTN_FORCE_INLINE u32x4 lds_read16(int addr) {
    return *(lds_u32x4_ptr)(uintptr_t)(uint32_t)addr;
}

struct Prefill64Params {
    const uint16_t* __restrict__ q;
    const uint16_t* __restrict__ cache;
    const int32_t* __restrict__ block_table;
    const int32_t* __restrict__ cu_seqlens_q;
    const int32_t* __restrict__ seq_lens;
    uint16_t* __restrict__ out;
    float* __restrict__ o_part;
    float* __restrict__ ml_part;
    int64_t q_stride, out_stride;
    int num_seqs, total_q, hq_l, hkv_l, G;
    int tile_tokens;  // columns of a tile / G
    int g_magic;      // 2^20 / G rounded up: x * g_magic >> 20 is x / G for the columns x < 256 of a tile
    int n_splits;     // key ranges per tile
    int paired;       // tiles of a sequence taken two per workgroup (see prefill_mfma64_plan)
    int rotate;       // the (sequence, KV head) index is rotated by the (tile rank, key range) index (see internal.h)
    int max_blocks;
    float c;          // softmax_scale * log2(e) (times k_scale for a cache widened from FP8)
    float out_scale;  // multiplies the normalised output: v_scale of an FP8 cache, else 1
    // launches that carry decode rows
    int ranks;        // tiles per sequence at most
    float range_div;  // a tile's keys are cut into ranges of 1 / range_div of them, the last one what remains
};

static_assert(kThreads == 64 * kPrefill64Waves && decode_flat::kRoleLdsBytes<kPrefill64Waves> <= kLdsBytes);

// kDecode: 0 = prefill only; 1, 2 = the first workgroups take decode rows over a bf16 (1) or FP8 (2) cache
// kScaledQ: the first attempt at a pass works on Q^T times the softmax scale, rounded to bf16 again
// kG: groups of wavefronts.  1: a tile of 256 columns, all four wavefronts on the same keys.  2: a tile of 128 columns, wavefronts
// 0 and 1 on the even key tiles, 2 and 3 on the odd ones, merged through LDS at the end
template <int kDecode, bool kScaledQ, int kG>
__global__ __launch_bounds__(kThreads, 1) void prefill64_kernel(Prefill64Params p, DecodeRole dec) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if constexpr (kDecode != 0) {
        if (static_cast<int>(blockIdx.x) < dec.n_wg) {   // uniform
            decode_flat::decode_role<kDecode == 2, kPrefill64Waves>(dec, p.q_stride, p.hq_l, p.hkv_l, lds, blockIdx.x);
            return;
        }
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = kG == 1 ? 0 : wave >> 1, wcol = kG == 1 ? wave : wave & 1;   // group; 64-column block of the tile
    constexpr int kGroupThreads = kThreads / kG;
    const int gtid = tid & (kGroupThreads - 1);

    // ---- which (pair rank, key split, sequence, KV head) is this workgroup --------------------------------------
    const int n_sg = p.num_seqs * p.hkv_l;
    const TileItem ti = tile_item(blockIdx.x, kDecode == 0 ? 0 : dec.n_wg, n_sg, p.ranks, p.n_splits, kDecode != 0, p.rotate != 0);
    const int rank = ti.rank, split = ti.split;
    const int s = ti.sh / p.hkv_l;
    const int g = ti.sh - s * p.hkv_l;

    const int q_begin = p.cu_seqlens_q[s];
    const int q_len = p.cu_seqlens_q[s + 1] - q_begin;
    const int ctx = p.seq_lens[s];
    const int tile_tokens = p.tile_tokens;
    const int cols_used = tile_tokens * p.G;
    // token and head of a column of the tile (a division costs some thirty instructions, and a pass has forty of them: 2 us)
    auto token_of = [&](int col) SHIFTATTN_INLINE -> int { return static_cast<int>(static_cast<uint32_t>(col * p.g_magic) >> 20); };
    auto head_of = [&](int col) SHIFTATTN_INLINE -> int { return g * p.G + col - token_of(col) * p.G; };
    const int n_tiles = (q_len + tile_tokens - 1) / tile_tokens;
    // paired: the workgroup takes tile n_tiles - 1 - rank and then tile rank (heaviest with lightest); else the former
    // alone - workgroups start in the order of their index, so the heaviest tiles of all sequences go first and the light
    // ones fill the compute units that fall free
    const int hi_tile = n_tiles - 1 - rank;
    if (p.paired ? rank > hi_tile : hi_tile < 0) return;  // uniform
    const int n_pass = (!p.paired || hi_tile == rank) ? 1 : 2;
    const int32_t* table = p.block_table + static_cast<size_t>(s) * p.max_blocks;
    const int last_block = (ctx - 1) / kBlockSize;

    // In the key loop of one group wavefronts 0 and 1 bring K (cache block 0 / 1 of a tile), wavefronts 2 and 3 V^T; of two groups
    // either wavefront brings K and V^T of its cache block.
    const bool is_k = kG == 2 || wave < 2;
    const int ld_blk = wave & 1;
    // LDS address of this wavefront's u-th load: ld_dst for u % 4 = 0, ld_dst2 for 2, one stage further for 1 and 3.  (Of two groups
    // that is K's; V^T goes kKBytes further, to the stage two before.)
    const int lds_at = static_cast<int>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)lds)) + grp * kRingBytes;
    const int ld_dst = __builtin_amdgcn_readfirstlane(lds_at + (is_k ? 0 : 2 * kStageBytes + kKBytes) + ld_blk * kBlockBytes);
    const int ld_dst2 = __builtin_amdgcn_readfirstlane(lds_at + (is_k ? 2 * kStageBytes : kKBytes) + ld_blk * kBlockBytes);
    // a wavefront-uniform pointer, said explicitly to be in scalar registers
    auto uniform_ptr = [](const unsigned char* ptr) SHIFTATTN_INLINE -> const unsigned char* {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
        return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
    };
    const unsigned char* cache_g =
        uniform_ptr(reinterpret_cast<const unsigned char*>(p.cache) + static_cast<size_t>(g) * 2 * kBlockBytes);
    // 4 KiB from src (uniform, scalar registers) + a 32-bit byte offset per lane and load into LDS at dst (uniform).
    // Written as assembly so that the address is formed by the load itself (scalar base + vector offset) instead of a
    // 64-bit vector addition per load.  The LDS destination goes through M0; the compiler treats M0 as reserved (it
    // sets it right before each use of its own and keeps no value in it), so writing it here needs no clobber.  The
    // compiler does not count these loads: around the key loop they are waited for with vmcnt(0) (wait_vm0), in the loop
    // with a count of the newest ones (see the barrier there).
    auto dma_4k = [&](const unsigned char* src, const int (&off)[4], int m0v) SHIFTATTN_INLINE {
        asm volatile(
            "s_mov_b32 m0, %0\n\ts_nop 4\n\t"
            "global_load_lds_dwordx4 %1, %5\n\t"
            "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
            "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
            "global_load_lds_dwordx4 %4, %5 offset:3072"
            :: "s"(m0v), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(src) : "memory");
    };


    for (int pass = 0; pass < n_pass; ++pass) {
        const int tile = pass == 0 ? hi_tile : rank;
        const int tok0 = tile * tile_tokens;
        // ---- LDS addressing (derived from an opaque copy of the lane index in every pass: as loop invariants of the
        // whole kernel these would be kept in registers through the key loop) -------------------------------------
        int lane_p = lane;
        asm volatile("" : "+v"(lane_p));
        const int l32 = lane_p & 31, half = lane_p >> 5;
        const int lds_base = lds_at;
        // K operand of MFMA row l32 is K row tau (bits 2 and 3 swapped); piece c of row r sits at c ^ (r & 15)
        const int tau = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
        int k_rd[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) k_rd[ks] = lds_base + tau * 256 + (((2 * ks + half) ^ (tau & 15)) << 4);
        // V^T operand: block-major [2][128 rows][32 B]; the two 16-byte halves of a row are swapped in every other run
        // of eight rows
        const int v_rd = lds_base + kKBytes + l32 * 32 + ((half ^ ((l32 >> 3) & 1)) << 4);
        // Direct-to-LDS loads: one cache block (K or V^T, 4 KiB) per wavefront and iteration as four 1-KiB loads, LDS
        // side contiguous in lane order (the swizzle is applied to the global address).  The loads' immediate offsets
        // (0, 1024, 2048, 3072) move source and destination together, the per-lane offsets carry the rest:
        // K block, load x: rows 4 x + lane / 16, piece lane % 16 of a row stored at (lane % 16) ^ row;
        // V^T block, load x: rows 32 x + lane / 2 (same per-lane offset for every x).
        int k_ld[4];
    #pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int r0 = lane_p >> 4;
            k_ld[x] = r0 * 256 + (((lane_p & 15) ^ r0 ^ (4 * x)) << 4);
        }
        const int v_ld = kBlockBytes + (lane_p >> 1) * 32 + (((lane_p & 1) ^ ((lane_p >> 4) & 1)) << 4);
        const int v_off[4] = {v_ld, v_ld, v_ld, v_ld};
        int ld_off[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) ld_off[x] = is_k ? k_ld[x] : v_ld;   // (two groups: K's, V^T's is v_ld)
        int pos_col[2];
        bf16x8 qf[2][8];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int cw = wcol * 64 + cb * 32 + l32;
            const int tok = tok0 + token_of(cw);
            const bool valid = cw < cols_used && tok < q_len;
            pos_col[cb] = valid ? ctx - q_len + tok : -1;
        }
        // Q^T of this lane's columns into the accumulation registers.  with_scale: multiplied by the softmax scale (times
        // log2 e, times k_scale of a cache widened from FP8) and rounded to bf16 again, for the attempt that follows no
        // reference: its logits then leave the MFMAs in exp2 units and its loop spends no instruction on scaling them.
        // (the addresses are formed here and not kept: a second fetch is rare)
        auto fetch_q = [&](auto with_scale) SHIFTATTN_INLINE {
            int lane_q = lane;
            asm volatile("" : "+v"(lane_q));
            const uint16_t* q_ptr[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int cw = wcol * 64 + cb * 32 + (lane_q & 31);
                // a column beyond the tile's or the sequence's end reads the row of the nearest real one: every one of
                // its logits is masked (position -1) or its results are dropped, and columns do not mix
                const int cw_r = min(cw, cols_used - 1);
                const int tok_r = min(tok0 + token_of(cw_r), q_len - 1);
                q_ptr[cb] = p.q + static_cast<size_t>(q_begin + tok_r) * p.q_stride + head_of(cw_r) * kD + (lane_q >> 5) * 8;
            }
            load_q_to_acc(qf[0], qf[1], q_ptr[0], q_ptr[1]);
            if constexpr (decltype(with_scale)::value != 0) {
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        bf16x8 v = qf[cb][ks];
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = static_cast<__bf16>(static_cast<float>(v[e]) * p.c);
                        qf[cb][ks] = v;
                        // (the scaled value is made to look born in accumulation registers, as the loaded one was)
                        asm volatile("" : "+a"(qf[cb][ks]));
                    }
            }
        };
        // ---- key tiles of this (column tile, split) -------------------------------------------------------
        const int tile_pos_max = ctx - q_len + min(tok0 + tile_tokens, q_len) - 1;
        // First position of this wavefront's columns.  One that has no column at all (behind the end of a ragged tile, which is the
        // heaviest of its sequence) computes the nearest real one's once more and takes part to the end of the tile's keys, without the
        // selects of the masked tiles: with those in every iteration it held up the others (three tokens of eight heads on 20000 keys, one
        // workgroup: 245 us where sixteen tokens take 182, now 177; two prompts of 3747 tokens in two groups 78 -> 68).
        const int w_tok_first = tok0 + token_of(wcol * 64);
        const int w_pos_min = __builtin_amdgcn_readfirstlane(wcol * 64 < cols_used && w_tok_first < q_len ? ctx - q_len + w_tok_first : tile_pos_max);
        const int kv_tiles = tile_pos_max / kKv + 1;
        const int per_split = kDecode == 0 ? (kv_tiles + p.n_splits - 1) / p.n_splits : static_cast<int>(ceilf(kv_tiles / p.range_div));
        const int kt_begin = __builtin_amdgcn_readfirstlane(split * per_split);
        const int kt_end = kDecode != 0 && split == p.n_splits - 1 ? kv_tiles : min(kv_tiles, kt_begin + per_split);
        const int n_all = __builtin_amdgcn_readfirstlane(max(kt_end - kt_begin, 0));
        // this group's tiles: kt_first + kG j, j < n (the first group has as many or one more)
        const int n = (n_all + kG - 1 - grp) / kG;
        const int kt_first = kt_begin + grp;
        // the tile that reaches past the context (if any) holds unwritten V slots: cleared in LDS before use
        // (asked where it is needed: kept through the key loop it would cost scalar registers)
        auto is_ragged = [&]() SHIFTATTN_INLINE -> bool { return n_all > 0 && kt_end * kKv > ctx; };

        f32x16 oacc[2][4];
        f32x16 sbuf[2][2];          // [parity][column block]
        u32x4 pw[2][2][2];          // [parity][column block][16-key slice]: four registers of packed P each
        // per column block: reference maximum, its product with the scale (0 while there is none), the largest logit
        // the reference covers (reference + slack), running sum
        float m_used[2] = {-INFINITY, -INFINITY}, mc[2] = {0.f, 0.f}, bound[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
        int redo = 0;               // uniform: a column of this wavefront needed a rescaling the key loop does not do
        float m_rep[2] = {-INFINITY, -INFINITY};
        const float thr = kRefSlack / p.c;  // how far a logit may exceed the reference (attempts that follow the maximum)

        // Ring of four LDS stages: K of tile t and V^T of tile t live in stage t % 4.  Iteration j reads K of tile j + 1 and V^T
        // of tile j - 1 and loads K of tile j + 4 and V^T of tile j + 2, whose stages were read for the last time in iteration
        // j - 1.  What an iteration reads was loaded three iterations before and complete before the barrier of the iteration
        // before, so operand reads run on across the barrier and loads have two iterations to land.
        u32x4 pre_a = {0u, 0u, 0u, 0u}, pre_c = pre_a;  // first K and first V^T operand of the coming iteration

        // Where this wavefront's loads come from.  Its u-th load is K of tile u (wavefronts 0, 1) or V^T of tile u - 2
        // (2, 3); lanes hold the byte addresses of the loads of a window of 64, lane 0 the next one's: an iteration reads lane 0 and
        // moves the others down by one, instead of loading a block id, waiting for it and multiplying it out with a dozen scalar
        // instructions.  The ids of the window after come straight into LDS meanwhile.
        const int ld_ahead = __builtin_amdgcn_readfirstlane(is_k ? 0 : 2);
        uint32_t a_lo = 0, a_hi = 0;
        int u_left = 0, window = 0;   // loads left in the window; its number
        int* my_ids = reinterpret_cast<int*>(lds + kIdsAt) + __builtin_amdgcn_readfirstlane(wave * 128);
        auto block_index = [&](int w) SHIFTATTN_INLINE -> int {
            return min(2 * (kt_first + kG * max(64 * w + lane_p - ld_ahead, 0)) + ld_blk, last_block);
        };
        auto take_window = [&](int id) SHIFTATTN_INLINE {   // ids are those of blocks that exist: not negative
            const uint64_t a = reinterpret_cast<uint64_t>(cache_g) + static_cast<uint64_t>(static_cast<uint32_t>(id)) * static_cast<uint32_t>(p.hkv_l * 2 * kBlockBytes);
            a_lo = static_cast<uint32_t>(a);
            a_hi = static_cast<uint32_t>(a >> 32);
        };
        auto request_window = [&](int w) SHIFTATTN_INLINE {
            const uint32_t m0v = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(my_ids + (w & 1) * 64));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2"
                         :: "s"(m0v), "v"(block_index(w) * 4), "s"(uniform_ptr(reinterpret_cast<const unsigned char*>(table))) : "memory");
        };
        auto join = [](uint32_t lo, uint32_t hi) SHIFTATTN_INLINE -> const unsigned char* {
            return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
        };
        auto lane_above = [](uint32_t v) SHIFTATTN_INLINE -> uint32_t {   // wave_rol:1, lane i takes lane i + 1's
            v = __builtin_amdgcn_update_dpp(v, v, 0x134, 0xf, 0xf, false);
            asm volatile("" : "+v"(v));
            return v;
        };

        // logits of keys beyond a column's position in the tile that begins at key0
        auto mask_tile = [&](f32x16 (&sv)[2], int key0) SHIFTATTN_INLINE {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                int left = pos_col[cb] - key0 - 8 * half;   // (formed here: kept from outside the loop it would cost registers)
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    sv[cb][r] = 16 * (r >> 3) + (r & 7) > left ? -INFINITY : sv[cb][r];
            }
        };
        // first iteration whose tile holds keys beyond the first column's position
        const int j_diag = __builtin_amdgcn_readfirstlane(((w_pos_min - (kKv - 1) - kt_first * kKv) >> (4 + kG)) + 1);

        // zero the V^T entries of keys at or past the context in the given stage (tile kt)
        auto clear_ragged_v = [&](int kt, int stage_off) SHIFTATTN_INLINE {
            const int h = gtid & 1;
#pragma unroll
            for (int bi = 0; bi < 2; ++bi) {
                const int n_valid = ctx - (kt * kKv + bi * 16 + h * 8);
#pragma unroll
                for (int d0 = 0; d0 < kD; d0 += kGroupThreads / 2)
                if (n_valid < 8) {
                    const int d = d0 + (gtid >> 1);
                    u32x4* ptr = reinterpret_cast<u32x4*>(lds + grp * kRingBytes + stage_off + kKBytes + bi * kBlockBytes + d * 32 +
                                                          ((h ^ ((d >> 3) & 1)) << 4));
                    u32x4 v = *ptr;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        v[w] &= n_valid > 2 * w + 1 ? 0xFFFFFFFFu : (n_valid > 2 * w ? 0x0000FFFFu : 0u);
                    *ptr = v;
                }
            }
        };

        // One iteration on tile j.  PH = j % 4: selects the stages and, by its parity, the register sets at compile time.
        // track_c: 1 = the maximum is followed (TRACK); 2 = the reference the column's first key tiles left is kept and no
        // maximum followed (KEEP); 0 = no reference at all, on logits that arrive in exp2 units (Q^T carries the scale)
        // s_lo, s_hi: addresses of the last four loads of K (two groups: V^T's is K's of two iterations before)
        auto body = [&](auto ph_c, auto guard_c, auto track_c, int j, uint32_t (&s_lo)[4], uint32_t (&s_hi)[4]) SHIFTATTN_INLINE {
            constexpr int PH = decltype(ph_c)::value, PAR = PH & 1;
            constexpr bool GUARD = decltype(guard_c)::value != 0;  // outside the steady-state loop
            constexpr bool TRACK = decltype(track_c)::value == 1;
            constexpr bool KEEP = decltype(track_c)::value == 2;
            f32x16(&s_cur)[2] = sbuf[PAR];
            f32x16(&s_nxt)[2] = sbuf[1 - PAR];
            u32x4(&p_cur)[2][2] = pw[PAR];
            u32x4(&p_prv)[2][2] = pw[1 - PAR];

            if (j >= j_diag) {  // tile crosses the diagonal of this wavefront: uniform
                // (a real branch: the selects below take their inputs from a statement that cannot be moved out of it)
                asm volatile("; keys beyond a column's position" : "+v"(s_cur[0]), "+v"(s_cur[1]));
                mask_tile(s_cur, (kt_first + kG * j) * kKv);
            }

            // operand reads: op o feeds the two MFMAs (column blocks 0 and 1) of slots 2 o and 2 o + 1: even ops K of tile j + 1,
            // odd ones V^T of tile j - 1.  Ops 16 and 17 are the first two of the next iteration.
            u32x4 opnd[18];
            opnd[0] = pre_a;
            opnd[1] = pre_c;
            auto op_read = [&](auto oc) SHIFTATTN_INLINE -> u32x4 {
                constexpr int o = decltype(oc)::value, of = o / 16, idx = (o % 16) / 2;   // of: of the next iteration
                if constexpr (o % 2 == 0) return lds_read16(k_rd[idx] + ((PH + 1 + of) & 3) * kStageBytes);
                else return lds_read16(v_rd + ((PH + 3 + of) & 3) * kStageBytes + (idx / 4) * kBlockBytes + (idx % 4) * 1024);
            };
            // ---- interleaved block ------------------------------------------------------------------------
            float mx[2] = {-INFINITY, -INFINITY};
            // chunk v (0..31): the logit of column block v / 16, accumulator register v % 16.  Slot v takes the exponential of
            // logit v and adds logit v - 2 to the row sum; odd slots pack logits v - 3 and v - 2, even ones issue an operand read:
            // no slot then asks for more issue time than its MFMA takes.  No instruction of a slot reads an exponential issued last.
            // (the empty asm statements pin results to their slots: left free they drift together)
            float ev[32];
            auto sum_up = [&](auto vc) SHIFTATTN_INLINE {
                constexpr int v = decltype(vc)::value;
                l_run[v / 16] += ev[v];
                asm volatile("" : "+v"(l_run[v / 16]));
            };
            auto pack = [&](auto vc) SHIFTATTN_INLINE {   // logits v, v + 1
                constexpr int v = decltype(vc)::value, cb = v / 16, r = v % 16;
                bf16x2 t;
                t[0] = static_cast<__bf16>(ev[v]);
                t[1] = static_cast<__bf16>(ev[v + 1]);
                uint32_t w = __builtin_bit_cast(uint32_t, t);
                if constexpr (!TRACK) asm volatile("" : "+v"(w));
                p_cur[cb][r >> 3][(r & 7) >> 1] = w;
            };
            auto chunk = [&](auto vc) SHIFTATTN_INLINE {
                constexpr int v = decltype(vc)::value;
                constexpr int cb = v / 16, r = v % 16;
                // (no reference followed: Q^T carries the scale, the logit arrives in exp2 units)
                const float x = TRACK || KEEP ? fmaf(s_cur[cb][r], p.c, -mc[cb]) : s_cur[cb][r];
                ev[v] = __builtin_amdgcn_exp2f(x);
                if constexpr (!TRACK) asm volatile("" : "+v"(ev[v]));
                if constexpr (v >= 2) sum_up(IC<v - 2>{});
                if constexpr (v >= 3 && v % 2 == 1) pack(IC<v - 3>{});
                if constexpr (TRACK && r % 2 == 1) {
                    mx[cb] = fmaxf(fmaxf(mx[cb], s_cur[cb][r - 1]), s_cur[cb][r]);
                    asm volatile("" : "+v"(mx[cb]));
                }
                if constexpr (v == 31) {
                    sum_up(IC<30>{});
                    sum_up(IC<31>{});
                    pack(IC<30>{});
                }
            };
            auto op_mfma = [&](auto tc, u32x4 a) SHIFTATTN_INLINE {
                constexpr int t = decltype(tc)::value;
                constexpr int o = t / 2, cb = t % 2, idx = o / 2;
                if constexpr (o % 2 == 0) {
                    if constexpr (idx == 0) mfma_s_first<GUARD>(s_nxt[cb], a, qf[cb][idx]);
                    else mfma_s_acc<GUARD>(s_nxt[cb], a, qf[cb][idx]);
                } else {
                    mfma_o_acc<GUARD>(oacc[cb][idx % 4], a, p_prv[cb][idx / 4]);
                }
            };
            // What runs once per iteration besides, spread over the odd slots: the address of this iteration's loads (slots 1 and 3),
            // the barrier (slot 2) with the wait for the loads of the iteration before last in front, the address of the next one's
            // (slots 5 and 7), now and then the next window of them (slot 7), and the loads into the stage nobody reads any more
            // (slots 9 to 15): all four right behind the barrier hold up the matrix pipe (2048 tokens on 131072 cached beside 64
            // decodes: 3 % of the launch).  Loads beyond the last tile are made all the same (of the context's last block at most):
            // the count that the wait relies on then always holds.
            auto next_window = [&]() SHIFTATTN_INLINE {
                if (--u_left == 0) {
                    take_window(my_ids[(window & 1) * 64 + lane_p]);
                    request_window(++window);
                    u_left = 64;
                }
            };
            uint32_t& src_lo = s_lo[PH];
            uint32_t& src_hi = s_hi[PH];
            auto housekeeping = [&](auto tc) SHIFTATTN_INLINE {
                constexpr int t = decltype(tc)::value;
                if constexpr (t == 1) {
                    src_lo = __builtin_amdgcn_readfirstlane(a_lo);
                    asm volatile("" : "+s"(src_lo));
                } else if constexpr (t == 2) {
                    // a bare barrier: __syncthreads() would first drain every outstanding LDS read.  What has to be complete
                    // is this wavefront's loads of the iteration before last - all but the newest four, or eight of two groups,
                    // which are the tile loads of the iteration before: nothing else may be issued behind those, so a request
                    // for the next window of block ids stays in front of its iteration's (slots 7 and 8) and no spill may load
                    // in here - and its reads of the stages about to be overwritten (their data went into MFMAs in the
                    // iteration before).
                    if constexpr (kG == 1) asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
                } else if constexpr (t == 3) {
                    src_hi = __builtin_amdgcn_readfirstlane(a_hi);
                    asm volatile("" : "+s"(src_hi));
                } else if constexpr (t == 5) {
                    a_lo = lane_above(a_lo);
                } else if constexpr (t == 7) {
                    a_hi = lane_above(a_hi);
                    if constexpr (!(kG == 2 && TRACK)) next_window();
                } else if constexpr (t == 8) {
                    // (two groups, the rare attempts that follow the maximum: a scalar register too few, kept in a vector lane)
                    if constexpr (kG == 2 && TRACK) next_window();
                } else if constexpr (t == 9) {
                    asm volatile("s_add_i32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                                 :: "s"(PH < 2 ? ld_dst : ld_dst2), "v"(ld_off[0]), "s"(join(src_lo, src_hi)), "n"((PH & 1) * kStageBytes) : "memory", "scc");
                } else if constexpr (t == 11 || t == 13 || t == 15) {
                    constexpr int x = (t - 9) / 2;
                    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(ld_off[x]), "s"(join(src_lo, src_hi)), "n"(1024 * x) : "memory");
                } else if constexpr (kG == 2 && (t == 17 || t == 19 || t == 21 || t == 23)) {   // V^T of tile j + 2
                    constexpr int x = (t - 17) / 2, v2 = (PH + 2) & 3;
                    const int off = v_off[x], dst = PH < 2 ? ld_dst2 : ld_dst;
                    const unsigned char* v_src = join(s_lo[v2], s_hi[v2]);
                    if constexpr (x == 0)
                        asm volatile("s_add_i32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                                     :: "s"(dst), "v"(off), "s"(v_src), "n"((PH & 1) * kStageBytes + kKBytes) : "memory", "scc");
                    else
                        asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(off), "s"(v_src), "n"(1024 * x) : "memory");
                }
            };
            [&]<int... T>(std::integer_sequence<int, T...>) SHIFTATTN_INLINE {
                (([&]() SHIFTATTN_INLINE {
                     op_mfma(IC<T>{}, opnd[T / 2]);
                     __builtin_amdgcn_sched_barrier(0);  // the rest of the slot goes behind its MFMA
                     if constexpr (T % 2 == 0) {
                         opnd[T / 2 + 2] = op_read(IC<T / 2 + 2>{});
                         __builtin_amdgcn_sched_barrier(0);
                     }
                     housekeeping(IC<T>{});
                     chunk(IC<T>{});
                     __builtin_amdgcn_sched_barrier(0);
                 }()),
                 ...);
            }
            (std::make_integer_sequence<int, 32>{});
            pre_a = opnd[16];
            pre_c = opnd[17];

            // ---- the tile's maximum against what the reference covers: rarely, a new reference ------------------
            if constexpr (TRACK)
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx[0] > bound[0] || mx[1] > bound[1]) != 0, 0)) {
                // A column that meets its first visible keys has no sums yet (O^T = 0, l = 0): its reference is set and
                // the tile's P recomputed, nothing else.  A column that already holds sums would need them rescaled;
                // O^T is not touched by the vector ALU inside this loop (that would pull it out of the accumulation
                // registers), so such a tile only flags the pass, which is then run a second time from the reference
                // this attempt ends with.
                bool bad = false;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    // both lanes of a column (its two halves of the keys) must take the same decision
                    const float mo = __shfl_xor(mx[cb], 32);
                    const float mfull = fmaxf(mx[cb], mo);
                    const bool grow = mfull > bound[cb];
                    bad = bad || (grow && m_used[cb] != -INFINITY);
                    if (grow) {
                        m_used[cb] = mfull;
                        mc[cb] = mfull * p.c;
                        bound[cb] = mfull + thr;
                    }
                    float ps = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        const float e0 = __builtin_amdgcn_exp2f(fmaf(s_cur[cb][r], p.c, -mc[cb]));
                        const float e1 = __builtin_amdgcn_exp2f(fmaf(s_cur[cb][r + 1], p.c, -mc[cb]));
                        bf16x2 t;
                        t[0] = static_cast<__bf16>(e0);
                        t[1] = static_cast<__bf16>(e1);
                        ps += e0;
                        ps += e1;
                        p_cur[cb][r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, t);
                    }
                    if (grow) l_run[cb] = ps;  // (a column that keeps its reference has just recomputed what it had)
                }
                redo = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_ballot_w64(bad) ? 1 : redo);
            }
        };

        // prologue loads: K of the first four tiles, V^T of the first two
        auto issue_prologue = [&]() SHIFTATTN_INLINE {
            take_window(table[block_index(0)]);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const unsigned char* from = join(__builtin_amdgcn_readfirstlane(a_lo), __builtin_amdgcn_readfirstlane(a_hi));
                const int dst = ((x & 2) ? ld_dst2 : ld_dst) + (x & 1) * kStageBytes;
                if (is_k || x >= 2) dma_4k(from, ld_off, dst);
                if constexpr (kG == 2)
                    if (x < 2) dma_4k(from, v_off, dst + kKBytes);
                a_lo = lane_above(a_lo);
                a_hi = lane_above(a_hi);
            }
            request_window(1);
            window = 1;
            u_left = 60;
        };
        // The first attempt's go out in front of the fetch of Q^T, whose wait then covers both.
        if (n > 0) issue_prologue();
        fetch_q(IC<kScaledQ ? 1 : 0>{});

        // Up to three attempts at the pass.  The first follows no maximum behind the first key tile or two (its steady-state
        // bodies save the instruction per two logits that would collect it; real logits stay within 2^100 of their
        // first tiles' maximum).  If some wavefront flags it (behind its key loop), the second starts over and
        // follows the maximum tile by tile; it can end flagged itself (a column outgrew its reference after it had sums),
        // and then holds, for every column, a reference within the slack of the true maximum: the third attempt starts
        // from that and is not flagged.
        auto reset_sums = [&]() SHIFTATTN_INLINE {
            redo = 0;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                l_run[cb] = 0.f;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[cb][mt][r] = 0.f;
            }
        };
        auto key_loop = [&](auto track_c) SHIFTATTN_INLINE {
            // prologue: S^T of the first tile (the loads are on their way).  Iteration 0 multiplies V^T "of tile -1" (stage 3) by
            // P = 0: zeros, so that no product of it is a NaN.
#pragma unroll
            for (int x = 0; x < 2 * kG; ++x)
                *reinterpret_cast<u32x4*>(lds + grp * kRingBytes + 3 * kStageBytes + kKBytes + (x * kGroupThreads + gtid) * 16) = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int ks2 = 0; ks2 < 2; ++ks2) pw[1][cb][ks2] = u32x4{0u, 0u, 0u, 0u};
            wait_vm0();
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const u32x4 a = lds_read16(k_rd[ks]);
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    if (ks == 0) mfma_s_first<true>(sbuf[0][cb], a, qf[cb][ks]);
                    else mfma_s_acc<true>(sbuf[0][cb], a, qf[cb][ks]);
                }
            }
            pre_a = lds_read16(k_rd[0] + kStageBytes);
            pre_c = lds_read16(v_rd + 3 * kStageBytes);
            mfma_settle(sbuf[0]);
            if constexpr (decltype(track_c)::value == 2) {   // the reference that is kept: the first tile's maximum, or the first two's
                // (Keys that are their column's reference have P = 1, exact in bf16, and the heaviest keys carry most of the rounding
                // error: where rows of less than 1000 keys are among the columns, the second tile's keys take part.  Prompts of
                // 4096 tokens, 2-norm of the error of rows 128 to 256 3.8 % larger without.)
                const bool second = n > 1 && (kG == 2 || w_pos_min < kt_first * kKv + 1000);
                if (j_diag <= 0) mask_tile(sbuf[0], kt_first * kKv);
                if (second) {
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        const u32x4 a = lds_read16(k_rd[ks] + kStageBytes);
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) {
                            if (ks == 0) mfma_s_first<true>(sbuf[1][cb], a, qf[cb][ks]);
                            else mfma_s_acc<true>(sbuf[1][cb], a, qf[cb][ks]);
                        }
                    }
                    mfma_settle(sbuf[1]);
                    if (j_diag <= 1) mask_tile(sbuf[1], (kt_first + kG) * kKv);
                }
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sbuf[0][cb][r]);
                    if (second)
#pragma unroll
                        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sbuf[1][cb][r]);
                    mx = fmaxf(mx, __shfl_xor(mx, 32));
                    if (mx > -INFINITY) m_used[cb] = mx, mc[cb] = mx * p.c;
                }
                // The loop sums P as it was before the rounding to bf16.  Rows of few keys are what that tells on (their outputs are
                // the large ones): where there are some, the sums begin with what rounding adds to the first tile's P, so that
                // those rows divide by the sum of what they multiply (2-norm of the error of prompts of 4096 tokens 1.3 %
                // larger without).
                if (w_pos_min < kt_first * kKv + 128) {
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const float e = __builtin_amdgcn_exp2f(fmaf(sbuf[0][cb][r], p.c, -mc[cb]));
                            l_run[cb] += static_cast<float>(static_cast<__bf16>(e)) - e;
                        }
                }
            }
            // four tiles per trip, so that the stages and the register sets are fixed at compile time
            uint32_t s_lo[4], s_hi[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {   // (the prologue's four addresses have gone round to the last lanes)
                s_lo[x] = __builtin_amdgcn_readlane(a_lo, 60 + x);
                s_hi[x] = __builtin_amdgcn_readlane(a_hi, 60 + x);
            }
            int j = 0;
            for (; j + 4 <= n; j += 4) {
                body(IC<0>{}, IC<0>{}, track_c, j, s_lo, s_hi);
                body(IC<1>{}, IC<0>{}, track_c, j + 1, s_lo, s_hi);
                body(IC<2>{}, IC<0>{}, track_c, j + 2, s_lo, s_hi);
                body(IC<3>{}, IC<0>{}, track_c, j + 3, s_lo, s_hi);
            }
            if (j < n) {
                body(IC<0>{}, IC<1>{}, track_c, j, s_lo, s_hi);
                if (j + 1 < n) {
                    body(IC<1>{}, IC<1>{}, track_c, j + 1, s_lo, s_hi);
                    if (j + 2 < n) body(IC<2>{}, IC<1>{}, track_c, j + 2, s_lo, s_hi);
                }
            }
            // (the S^T of the tile beyond the last is nobody's: its registers are free behind its MFMAs only)
            asm volatile("s_nop 7\n\ts_nop 3" :: "v"(sbuf[0][0]), "v"(sbuf[0][1]), "v"(sbuf[1][0]), "v"(sbuf[1][1]));
            // epilogue: O^T += V^T P^T of the last tile (in its stage since the barrier of the last iteration)
            const int last_stage = ((n - 1) & 3) * kStageBytes;
            if (kG == 2 && n < (n_all + kG - 1) / kG) asm volatile("s_barrier" ::: "memory");   // (the other group's last iteration)
            if (is_ragged()) {
                if (kG == 1 || ((n_all - 1) & 1) == grp) clear_ragged_v(kt_end - 1, last_stage);
                __syncthreads();
            }
            const bool odd = ((n - 1) & 1) != 0;
#pragma unroll
            for (int ks2 = 0; ks2 < 2; ++ks2) {
                u32x4 p_last[2];
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) p_last[cb] = odd ? pw[1][cb][ks2] : pw[0][cb][ks2];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const u32x4 a = lds_read16(last_stage + v_rd + ks2 * kBlockBytes + mt * 1024);
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) mfma_o_acc<true>(oacc[cb][mt], a, p_last[cb]);
                }
            }
            mfma_settle(oacc);
            wait_vm0();   // loads that nobody needs any more may still be on their way into LDS
        };
        // Does a wavefront of the workgroup ask for another attempt?  Behind its barrier every wavefront has left its last operand
        // reads behind and its own loads have landed (wait_vm0): only then may the ring's bytes be written by anything but loads.
        auto vote = [&]() SHIFTATTN_INLINE -> bool {
            int* flags = reinterpret_cast<int*>(lds + kFlagsAt);
            if (lane == 0) flags[wave] = redo;
            __syncthreads();
            const u32x4 all = *reinterpret_cast<const u32x4*>(flags);
            return __builtin_amdgcn_readfirstlane(all[0] | all[1] | all[2] | all[3]) != 0;
        };
        // a group without tiles beside one that has some (one tile in all): its barriers
        auto idle_group = [&]() SHIFTATTN_INLINE {
            for (int b = (n_all + kG - 1) / kG + 1 + (is_ragged() ? 1 : 0); b > 0; --b) asm volatile("s_barrier" ::: "memory");
        };
        reset_sums();
        if (n > 0) key_loop(IC<kScaledQ ? 0 : 2>{});
        else if (kG == 2 && n_all > 0) idle_group();
        // The first attempt followed no maximum.  That is exact as long as nothing left the range bf16 and the fp32 sums hold
        // without loss.  With the first tile's reference kept: a column's sum must not exceed 2^100 (P then stays below it;
        // what underflows is negligible beside the first tile's keys).  With no reference at all: a column that sees keys of
        // this range must end with a sum inside [2^-40, 2^40].  An infinity or a NaN fails either test; the pass is then flagged.
        // So is one with a column that sees keys but got no reference, every logit of its first tile or two being -inf: what it
        // summed behind them would be merged as a range without keys.
        bool out_of_range = false;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const float l_tot = l_run[cb] + __shfl_xor(l_run[cb], 32);
            const bool sees = n > 0 && pos_col[cb] >= kt_first * kKv;
            if constexpr (kScaledQ) {
                if (sees && !(l_tot >= kFreeSumLo && l_tot <= kFreeSumHi)) out_of_range = true;
                m_rep[cb] = sees ? 0.f : -INFINITY;   // what a partial result reports as its reference (exp2 units)
            } else {
                if (!(l_tot <= kKeepSumBound) || (sees && m_used[cb] == -INFINITY)) out_of_range = true;
                m_rep[cb] = m_used[cb] * p.c;
            }
        }
        redo = __builtin_amdgcn_ballot_w64(out_of_range) != 0 ? 1 : 0;
        if (__builtin_expect(vote(), 0)) {   // start over without references, on Q^T as given, and follow the maximum
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) m_used[cb] = -INFINITY, mc[cb] = 0.f, bound[cb] = -INFINITY;
            for (int attempt = 1;; ++attempt) {
                if (n > 0) issue_prologue();
                fetch_q(IC<0>{});
                reset_sums();
                if (n > 0) key_loop(IC<1>{});
                else if (kG == 2 && n_all > 0) idle_group();
                // (the vote's barrier is asked for behind the last attempt too: what follows writes into the ring of two groups)
                if (!vote() || attempt == 2) break;
            }
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) m_rep[cb] = m_used[cb] * p.c;
        }

        // ---- results of the pass ----------------------------------------------------------------------------
        // the lane index is read through an opaque copy: addresses derived from the plain value are loop invariants
        // that the optimiser computes before the key loop and then keeps in registers through it
        int lane_m = lane;
        asm volatile("" : "+v"(lane_m));
        const int l32_m = lane_m & 31, half_m = lane_m >> 5;
        if constexpr (kG == 2) {
            // Each group finishes one half of the head dimension (group 0 rows 0..63, group 1 rows 64..127): it parks the other
            // half of its accumulators for the other group, (reference, sum) beside them, and folds in what that group parked.
            float* ml = reinterpret_cast<float*>(lds + kMlAt);
            float l_tot[2];
            auto park_half = [&](auto g_c) SHIFTATTN_INLINE {
                constexpr int GRP = decltype(g_c)::value;
                unsigned char* mine = lds + (GRP * 2 + wcol) * (64 * 64 * 4) + lane_m * 16;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4) {
                            f32x4 v;
#pragma unroll
                            for (int x = 0; x < 4; ++x) v[x] = oacc[cb][2 * (1 - GRP) + k][r4 * 4 + x];
                            *reinterpret_cast<f32x4*>(mine + ((cb * 2 + k) * 4 + r4) * 1024) = v;
                        }
            };
            if (grp == 0) park_half(IC<0>{});
            else park_half(IC<1>{});
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                l_tot[cb] = l_run[cb] + __shfl_xor(l_run[cb], 32);
                ml[((wave * 2 + cb) * 2 + 0) * 64 + lane_m] = m_rep[cb];
                ml[((wave * 2 + cb) * 2 + 1) * 64 + lane_m] = l_tot[cb];
            }
            __syncthreads();
            const bool whole = p.n_splits == 1;
            auto finish_half = [&](auto g_c) SHIFTATTN_INLINE {
                constexpr int GRP = decltype(g_c)::value;
                const unsigned char* theirs = lds + ((1 - GRP) * 2 + wcol) * (64 * 64 * 4) + lane_m * 16;
                const int other = wave ^ 2;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const float m_o = ml[((other * 2 + cb) * 2 + 0) * 64 + lane_m], l_o = ml[((other * 2 + cb) * 2 + 1) * 64 + lane_m];
                    const float m_star = fmaxf(m_rep[cb], m_o);
                    const float w_me = m_rep[cb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_rep[cb] - m_star);
                    const float w_o = m_o == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_o - m_star);
                    const float l_all = l_tot[cb] * w_me + l_o * w_o;
                    const int cw = wcol * 64 + cb * 32 + l32_m;
                    // accumulator register r of row tile mt is head-dim 32*mt + 8*(r/4) + 4*half + r%4
                    auto folded = [&](int k, int r4, float a_me, float a_o) SHIFTATTN_INLINE -> f32x4 {
                        const f32x4 o = *reinterpret_cast<const f32x4*>(theirs + ((cb * 2 + k) * 4 + r4) * 1024);
                        f32x4 v;
#pragma unroll
                        for (int x = 0; x < 4; ++x) v[x] = oacc[cb][2 * GRP + k][r4 * 4 + x] * a_me + o[x] * a_o;
                        return v;
                    };
                    if (whole) {
                        const float inv = l_all > 0.f ? p.out_scale / l_all : 0.f;
                        unsigned char* srow = lds + kStagedAt + cw * kPitch + (64 * GRP + 4 * half_m) * 2;
#pragma unroll
                        for (int k = 0; k < 2; ++k)
#pragma unroll
                            for (int r4 = 0; r4 < 4; ++r4) {
                                const f32x4 v = folded(k, r4, w_me * inv, w_o * inv);
                                bf16x4 h;
#pragma unroll
                                for (int x = 0; x < 4; ++x) h[x] = static_cast<__bf16>(v[x]);
                                *reinterpret_cast<u32x2*>(srow + (32 * k + 8 * r4) * 2) = __builtin_bit_cast(u32x2, h);
                            }
                    } else if (pos_col[cb] >= 0) {
                        const size_t prow = (static_cast<size_t>(split) * p.total_q + q_begin + tok0 + token_of(cw)) * p.hq_l + head_of(cw);
                        float* op = p.o_part + prow * kD + 64 * GRP + 4 * half_m;
#pragma unroll
                        for (int k = 0; k < 2; ++k)
#pragma unroll
                            for (int r4 = 0; r4 < 4; ++r4) *reinterpret_cast<f32x4*>(op + 32 * k + 8 * r4) = folded(k, r4, w_me, w_o);
                        if (GRP == 0 && half_m == 0) {
                            p.ml_part[prow * 2] = m_star;  // -inf when this key range held no visible key
                            p.ml_part[prow * 2 + 1] = l_all;
                        }
                    }
                }
            };
            if (grp == 0) finish_half(IC<0>{});
            else finish_half(IC<1>{});
            if (whole) {
                __syncthreads();
                int tid_m = tid;
                asm volatile("" : "+v"(tid_m));
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int col = (tid_m >> 4) + 16 * i, piece = tid_m & 15;
                    const int tok_c = tok0 + token_of(col);
                    if (col < cols_used && tok_c < q_len) {
                        const u32x4 v = *reinterpret_cast<const u32x4*>(lds + kStagedAt + col * kPitch + piece * 16);
                        uint16_t* op = p.out + static_cast<size_t>(q_begin + tok_c) * p.out_stride + head_of(col) * kD + piece * 8;
                        *reinterpret_cast<u32x4*>(op) = v;
                    }
                }
            }
        } else if (p.n_splits == 1) {
            // normalise, put bf16 rows into this wavefront's part of the staging tile, then write them out in whole
            // 256-byte rows (one 16-byte piece per lane, 1 KiB of consecutive output per 4 rows)
            unsigned char* stage = lds + kRingBytes + wave * 64 * kPitch;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const float l_tot = l_run[cb] + __shfl_xor(l_run[cb], 32);
                const float inv = l_tot > 0.f ? p.out_scale / l_tot : 0.f;
                unsigned char* srow = stage + (cb * 32 + l32_m) * kPitch + 8 * half_m;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        // accumulator register r of row tile mt is head-dim 32*mt + 8*(r/4) + 4*half + r%4
                        bf16x4 v;
#pragma unroll
                        for (int x = 0; x < 4; ++x) v[x] = static_cast<__bf16>(oacc[cb][mt][r4 * 4 + x] * inv);
                        *reinterpret_cast<u32x2*>(srow + (32 * mt + 8 * r4) * 2) = __builtin_bit_cast(u32x2, v);
                    }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int col = 4 * i + (lane_m >> 4), piece = lane_m & 15;
                const int cw = wave * 64 + col;
                const int tok_c = tok0 + token_of(cw);
                if (cw < cols_used && tok_c < q_len) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + col * kPitch + piece * 16);
                    uint16_t* op = p.out + static_cast<size_t>(q_begin + tok_c) * p.out_stride + head_of(cw) * kD + piece * 8;
                    *reinterpret_cast<u32x4*>(op) = v;
                }
            }
        } else {
            // key ranges split over workgroups: the un-normalised partial of this range
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const float l_tot = l_run[cb] + __shfl_xor(l_run[cb], 32);
                if (pos_col[cb] >= 0) {
                    const int cw = wcol * 64 + cb * 32 + l32_m;
                    const int row_col = q_begin + tok0 + token_of(cw);
                    const int head_col = head_of(cw);
                    const size_t prow = (static_cast<size_t>(split) * p.total_q + row_col) * p.hq_l + head_col;
                    float* op = p.o_part + prow * kD + 4 * half_m;
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                        for (int r4 = 0; r4 < 4; ++r4) {
                            f32x4 v;
#pragma unroll
                            for (int x = 0; x < 4; ++x) v[x] = oacc[cb][mt][r4 * 4 + x];
                            *reinterpret_cast<f32x4*>(op + 32 * mt + 8 * r4) = v;
                        }
                    if (half_m == 0) {
                        p.ml_part[prow * 2] = m_rep[cb];  // exp2 units; -inf when this key range held no visible key
                        p.ml_part[prow * 2 + 1] = l_tot;
                    }
                }
            }
        }
        // The next pass reuses the ring, the flags and the staging tile: every wavefront must have left this pass's last
        // LDS reads behind.  A bare barrier: __syncthreads() would also wait for the output stores just issued (several
        // microseconds until the last is acknowledged); nothing in the next pass depends on them, and its first loads
        // overlap them.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

}  // namespace

bool prefill_mfma64_supported(const AttnShape& a) {
    return a.elem == 2 && a.D == kD && !a.kv_fp8() && a.hq_l % a.hkv_l == 0 && a.hq_l / a.hkv_l <= kCols;
}

Prefill64Plan prefill_mfma64_plan(int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a,
                                  int forced_splits) {
    Prefill64Plan pl;
    const int G = a.hq_l / a.hkv_l;
    pl.groups = 1;
    pl.tile_tokens = kCols / G;
    const int tiles = (max_q_len + pl.tile_tokens - 1) / pl.tile_tokens;
    // Causal tiles differ in work (tile i sees i + 1 tiles' worth of keys).  Two ways to level it: a workgroup takes the
    // heaviest tile left together with the lightest (equal workgroups, one round when the pairs fit the chip), or one
    // tile per workgroup, heaviest first, the light ones filling the compute units that fall free (any number of tiles
    // levels out, but a tile is never shorter than its keys: it wants key ranges when the heaviest outweighs a compute
    // unit's share).  A short chunk behind a long context has nothing to level - its tiles all walk the context - and
    // pairing only makes every workgroup pay set-up, first tile and write-out twice.  Both are priced with the same rough
    // model (plus kPassSeconds per pass a compute unit makes) over the key ranges per tile - a workgroup's time falls with
    // the ranges, every range adds a partial result per (token, head) that the merge kernel writes and reads back - and
    // the cheaper plan is taken.
    constexpr double kPassSeconds = 15e-6;  // set-up, Q fetch, first and last tiles, write-out: what a pass costs around its loop
    const double seqs_equiv = longest_chunk_equivalents(num_seqs, total_q, max_q_len);
    const int by_len = max_seq_len / (32 * kKv);  // at least 32 key tiles per range
    struct Cand {
        int splits;
        double seconds, with_passes;
    };
    auto best_of = [&](auto model) {  // model(splits) -> {seconds, passes per compute unit}
        Cand best = {0, 0.0, 0.0};
        auto take = [&](int sp) {
            const auto [t, passes] = model(sp);
            const Cand c = {sp, t, t + passes * kPassSeconds};
            if (best.splits == 0 || c.with_passes < best.with_passes * 0.97) best = c;  // a further range must pay for itself
        };
        if (forced_splits > 0) take(forced_splits);
        else
            for (int cand = 1; cand <= 16 && (cand == 1 || cand <= by_len); ++cand) take(cand);
        return best;
    };
    const int pair_ranks = (tiles + 1) / 2;
    const Cand paired = best_of([&](int sp) {
        const long wgs = static_cast<long>(pair_ranks) * num_seqs * a.hkv_l;
        const double rounds = static_cast<double>((wgs * sp + 255) / 256);
        return std::pair<double, double>(
            launch_model_seconds(wgs, sp, kCols, total_q, max_seq_len, a.hq_l, paired_walks(max_q_len, max_seq_len)), 2.0 * rounds);
    });
    const Cand single = best_of([&](int sp) {
        // tile i of a sequence walks (S - Q + (i + 1) tile_tokens) / S of the longest context S
        const double S = max_seq_len > 0 ? max_seq_len : 1, Q = max_q_len < max_seq_len ? max_q_len : max_seq_len;
        const double unit = 4.0 * 128 * kCols * S / 3.9e12, merge = 2.0 * total_q * a.hq_l * 130 * 4 / 4.0e12;
        const double base = (S - Q) / S, step = pl.tile_tokens / S;
        const double seqs = seqs_equiv;
        const double total = (tiles * base + step * tiles * (tiles + 1) / 2.0) * seqs * a.hkv_l;
        const double heaviest = (base + step * tiles < 1.0 ? base + step * tiles : 1.0) / sp;
        const long items = static_cast<long>(tiles * seqs * a.hkv_l * sp + 0.5);
        const double share = 1.03 * total / 256.0;  // a compute unit's share of all the work, filled by ever lighter tiles
        const double span = items <= 256 ? heaviest : (heaviest > share ? heaviest : share);
        return std::pair<double, double>(span * unit + (sp > 1 ? sp * merge + 5.0e-6 : 0.0), static_cast<double>((items + 255) / 256));
    });
    const int forced_pairing = option_prefill_pairing();
    pl.paired = forced_pairing == 1 || (forced_pairing == 0 && paired.with_passes <= single.with_passes);
    pl.pair_ranks = pl.paired ? pair_ranks : tiles;
    int splits = pl.paired ? paired.splits : single.splits;
    pl.model_seconds = pl.paired ? paired.seconds : single.seconds;
    pl.model_with_passes = pl.paired ? paired.with_passes : single.with_passes;
    if (splits < 1) splits = 1;
    if (splits > 64) splits = 64;
    pl.n_splits = splits;
    pl.rotate = rotate_sequences_over_dies(num_seqs, a.hkv_l, total_q, max_q_len);
    pl.workgroups = static_cast<long>(pl.pair_ranks) * splits * num_seqs * a.hkv_l;
    return pl;
}

size_t prefill_mfma64_workspace(int total_q, const Prefill64Plan& pl, const AttnShape& a) {
    return pl.n_splits == 1 ? 0 : static_cast<size_t>(pl.n_splits) * total_q * a.hq_l * (kD + 2) * sizeof(float);
}

hipError_t prefill_mfma64_init() {
    for (const void* kernel :
         {reinterpret_cast<const void*>(&prefill64_kernel<0, false, 1>), reinterpret_cast<const void*>(&prefill64_kernel<1, false, 1>),
          reinterpret_cast<const void*>(&prefill64_kernel<2, false, 1>), reinterpret_cast<const void*>(&prefill64_kernel<0, true, 1>),
          reinterpret_cast<const void*>(&prefill64_kernel<1, true, 1>), reinterpret_cast<const void*>(&prefill64_kernel<2, true, 1>),
          reinterpret_cast<const void*>(&prefill64_kernel<0, false, 2>), reinterpret_cast<const void*>(&prefill64_kernel<1, false, 2>),
          reinterpret_cast<const void*>(&prefill64_kernel<2, false, 2>)})
        if (hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes); e != hipSuccess) return e;
    return hipSuccess;
}

namespace {

template <int kDecode>
void enqueue(unsigned grid, int groups, const Prefill64Params& p, const DecodeRole& dec, hipStream_t st) {
    if (groups == 2) prefill64_kernel<kDecode, false, 2><<<grid, kThreads, kLdsBytes, st>>>(p, dec);
    else if (option_prefill_scaled_q()) prefill64_kernel<kDecode, true, 1><<<grid, kThreads, kLdsBytes, st>>>(p, dec);
    else prefill64_kernel<kDecode, false, 1><<<grid, kThreads, kLdsBytes, st>>>(p, dec);
}

Prefill64Params wide_params(const void* q, const void* cache, const int32_t* block_table, int max_blocks, const int32_t* cu_seqlens_q,
                            const int32_t* seq_lens, int num_seqs, int total_q, const Prefill64Plan& pl, void* out, void* workspace,
                            const AttnShape& a, float c, float out_scale) {
    Prefill64Params p;
    p.q = static_cast<const uint16_t*>(q);
    p.cache = static_cast<const uint16_t*>(cache);
    p.block_table = block_table;
    p.cu_seqlens_q = cu_seqlens_q;
    p.seq_lens = seq_lens;
    p.out = static_cast<uint16_t*>(out);
    const size_t part_rows = static_cast<size_t>(pl.n_splits) * total_q * a.hq_l;
    p.o_part = static_cast<float*>(workspace);
    p.ml_part = pl.n_splits > 1 ? p.o_part + part_rows * kD : nullptr;
    p.q_stride = a.q_stride;
    p.out_stride = a.out_stride;
    p.num_seqs = num_seqs;
    p.total_q = total_q;
    p.hq_l = a.hq_l;
    p.hkv_l = a.hkv_l;
    p.G = a.hq_l / a.hkv_l;
    p.g_magic = ((1 << 20) + p.G - 1) / p.G;
    p.tile_tokens = pl.tile_tokens;
    p.n_splits = pl.n_splits;
    p.paired = pl.paired ? 1 : 0;
    p.rotate = pl.rotate ? 1 : 0;
    p.max_blocks = max_blocks;
    p.c = c;
    p.out_scale = out_scale;
    p.ranks = pl.pair_ranks;
    p.range_div = static_cast<float>(pl.n_splits);
    return p;
}

}  // namespace

hipError_t launch_prefill_mfma64(const void* q, const void* cache, const int32_t* block_table, int max_blocks,
                                 const int32_t* cu_seqlens_q, const int32_t* seq_lens, int num_seqs, int total_q,
                                 const Prefill64Plan& pl, void* out, void* workspace, const AttnShape& a, float c,
                                 float out_scale, hipStream_t st) {
    const Prefill64Params p = wide_params(q, cache, block_table, max_blocks, cu_seqlens_q, seq_lens, num_seqs, total_q, pl, out, workspace, a,
                                          c, out_scale);
    enqueue<0>(static_cast<unsigned>(pl.workgroups), pl.groups, p, DecodeRole{}, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.n_splits > 1)
        return launch_combine(p.o_part, p.ml_part, total_q, a.hq_l, kD, pl.n_splits, 0, nullptr, 0, out, a.out_stride, a.elem,
                              out_scale, st);
    return hipSuccess;
}

hipError_t launch_prefill64_and_decode(const void* q, const void* cache, const int32_t* block_table, int max_blocks,
                                       const int32_t* cu_seqlens_q, const int32_t* seq_lens, int num_seqs, int total_q,
                                       const Prefill64Plan& pl, float range_div, const DecodeRole& dec, void* out, void* workspace,
                                       const AttnShape& a, float c, float out_scale, hipStream_t st) {
    Prefill64Params p = wide_params(q, cache, block_table, max_blocks, cu_seqlens_q, seq_lens, num_seqs, total_q, pl, out, workspace, a, c, out_scale);
    p.range_div = range_div;
    const unsigned grid = static_cast<unsigned>(pl.workgroups + dec.n_wg);
    if (a.kv_fp8()) enqueue<2>(grid, pl.groups, p, dec, st);
    else enqueue<1>(grid, pl.groups, p, dec, st);
    return hipGetLastError();
}

}  // namespace shiftattn
