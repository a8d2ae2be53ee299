// Causal prefill attention of the local head shard over the paged KV cache (Algorithm 1, boxed
// attention line, prefill rows; chunked prefill continues a cached context).  bf16 tensors, fp32
// accumulation, head_dim 128.
//
// Tiling.  A workgroup owns a tile of 128 "columns"; a column is one (new token, query head) pair.
// The query heads that share a KV head are stacked next to each other in the column index (GS heads
// per token), so one K/V tile serves the whole GQA group and the causal diagonal of a tile spans
// only 128/GS tokens.  The workgroup has eight wavefronts in two groups of four: a wavefront owns 32
// columns, and the two groups split the key tiles (64 keys = four cache blocks each) of the column
// tile between them - group 0 takes the even tiles, group 1 the odd ones - and merge their
// partial results through LDS at the end.  That puts two wavefronts of the same workgroup on every
// SIMD (the matrix pipe and the vector ALUs only overlap across wavefronts: a lone wavefront hides
// about six vector instructions under one MFMA, measured) while the tile stays small enough that a
// 4 x 4096-token batch still yields one equal-work workgroup per compute unit.
//
// Math per key tile, transposed so that P never leaves registers:
//   S^T[key][col]  = K[key][:] . Q^T[:][col]     32x32x16 bf16 MFMA, A = K rows from LDS,
//                                                 B = Q^T held in registers for the whole tile
//   softmax down each column: a lane holds 32 keys of one column, the other 32 sit in lane+32, so
//   the column max costs one v_permlane32_swap
//   O^T[d][col]   += V^T[d][key] . P^T[key][col]  A = V^T rows from LDS, B = P^T straight from the
//                                                 softmax registers
// K rows are assigned to MFMA rows with bits 2 and 3 of the row index swapped; with that
// assignment the keys a lane holds are runs of eight consecutive tokens, matching one 16-byte piece
// of a dimension-major V row in the cache.
//
// Pipeline.  In iteration i a wavefront issues, interleaved in one instruction stream,
//   A(i+1): S^T of its next tile (16 MFMAs), B(i): softmax of the current tile (vector ALU),
//   C(i-1): O^T += V^T P^T of the previous tile (16 MFMAs),
// one MFMA, the LDS read of the operand two MFMAs ahead and a few softmax instructions at a time.
// Rescaling of O is lazy: a column's reference maximum only moves when the tile maximum exceeds it
// by more than 2^8 (in exp2 units), so `O *= alpha` is a rare wavefront-uniform branch; P then ranges
// up to 2^8, which bf16 and the fp32 sums hold without loss.
//
// Memory.  K and V^T tiles go from the cache to LDS with direct-to-LDS loads (no registers, no
// LDS store instructions), issued one iteration ahead of their use; a wavefront loads "its" cache
// block of the tile with eight 1-KiB loads that are contiguous in HBM.  LDS is not padded; bank
// conflicts are avoided by XOR-swizzling 16-byte pieces, applied on the global-address side of
// the load.  Stage `par` of a group is filled during an iteration of parity `par` and read during
// the next one; one barrier per iteration.
//
// Scheduling.  Either tiles of a sequence are processed in pairs (heaviest with lightest) by one
// workgroup, so that every workgroup of a causal prefill does the same amount of work, or one tile
// per workgroup, heaviest first: half the latency where the tiles do not fill the chip (eleven
// prompts of 149 to 1097 tokens, 5 heads: 34.6 -> 28.2 us a call).  The long contexts of chunked
// prefill are additionally split into key ranges whose partial results are merged by launch_combine.
// plan_within() below prices the plans of both prefill kernels.
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
constexpr int kThreads = 512;
constexpr int kKvTile = kPrefillKvTile;        // 64 keys
constexpr int kKBytes = kKvTile * kD * 2;      // 16384: K tile, 64 rows of 256 B
constexpr int kVBytes = kD * kKvTile * 2;      // 16384: V^T tile, 4 blocks of [128 rows][32 B]
constexpr int kStageBytes = kKBytes + kVBytes; // 32768
constexpr int kGroupBytes = 2 * kStageBytes;   // two stages per wavefront group
// The merge of the two groups at the end of a pass: parked accumulators, the staged rows and the (max, sum) pairs lie
// beside stage 0 of K of both groups, which the next pass's first tiles are loaded into meanwhile.
constexpr int kPitch = 272;                    // staging row pitch in bytes (256 + 16)
constexpr int kStagedAt = kKBytes;             // [128 columns][kPitch], then [2 groups][2][256] floats
constexpr int kParkAt = kGroupBytes + kKBytes; // [2 groups][32 values][256 lanes] floats
constexpr int kLdsBytes = kParkAt + 2 * 32 * 256 * 4;  // 147456
static_assert(kStagedAt + 128 * kPitch + 2 * 2 * 256 * 4 <= kGroupBytes && kLdsBytes >= 2 * kGroupBytes);
constexpr int kBlockBytes = kBlockSize * kD * 2;  // 4096: K (or V^T) of one cache block and head

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

template <int kV>
struct IC {
    static constexpr int value = kV;
};

#define SHIFTATTN_INLINE __attribute__((always_inline))

// s_waitcnt vmcnt(0) with the other counters left alone (gfx9 encoding)
__device__ inline void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }

struct PrefillParams {
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
    int gs_log2;      // log2 of heads stacked per token in the column index
    int head_slots;   // hq_l >> gs_log2
    int n_splits;     // key ranges per tile
    int paired;       // tiles of a sequence taken two per workgroup (heaviest with lightest), else one
    int rotate;       // the (sequence, head slot) index is rotated by the (pair rank, key range) index (see internal.h)
    int max_blocks;
    float c;          // softmax_scale * log2(e) (times k_scale for a cache widened from FP8)
    float out_scale;  // multiplies the normalised output: v_scale of an FP8 cache, else 1
    // launches that carry decode rows (see launch_prefill_and_decode)
    int ranks;        // tiles per sequence at most
    float range_div;  // a tile's keys are cut into ranges of 1 / range_div of them, the last one what remains
};

constexpr int kDecodeWaves = kThreads / 64;
constexpr int kLdsBytesBoth = decode_flat::kRoleLdsBytes<kDecodeWaves> > kLdsBytes ? decode_flat::kRoleLdsBytes<kDecodeWaves> : kLdsBytes;

// kDecode: 0 = prefill only; 1, 2 = the first workgroups take decode rows over a bf16 (1) or FP8 (2) cache
template <int kDecode>
__global__ __launch_bounds__(kThreads, 2) void prefill_kernel(PrefillParams p, DecodeRole dec) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int kCols = 128;
    if constexpr (kDecode != 0) {
        if (static_cast<int>(blockIdx.x) < dec.n_wg) {   // uniform
            decode_flat::decode_role<kDecode == 2, kDecodeWaves>(dec, p.q_stride, p.hq_l, p.hq_l / p.G, lds, blockIdx.x);
            return;
        }
    }

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int grp = wave >> 2;  // key-tile parity this wavefront works on
    const int wg = wave & 3;    // column block of the wavefront; also the cache block of a tile it loads
    const int l32 = lane & 31, half = lane >> 5;

    // ---- which (pair rank, key split, sequence, head slot) is this workgroup -----------------------
    const int tile_tokens = kCols >> p.gs_log2;
    const int gs_mask = (1 << p.gs_log2) - 1;
    // a pass of this workgroup: the key tiles [kt_begin, kt_end) of a tile
    struct Part {
        int tile, kt_begin, kt_end;
    };
    const int n_sh = p.num_seqs * p.head_slots;
    const TileItem ti = tile_item(blockIdx.x, kDecode == 0 ? 0 : dec.n_wg, n_sh, p.ranks, p.n_splits, kDecode != 0, p.rotate != 0);
    const int rank = ti.rank, split = ti.split;
    const int s = ti.sh / p.head_slots;
    const int hs = ti.sh - s * p.head_slots;
    // (uniform values, said so: kept in vector registers through the key loop they would be spilled)
    const int q_begin = __builtin_amdgcn_readfirstlane(p.cu_seqlens_q[s]);
    const int q_len = __builtin_amdgcn_readfirstlane(p.cu_seqlens_q[s + 1]) - q_begin;
    const int ctx = __builtin_amdgcn_readfirstlane(p.seq_lens[s]);
    const int n_tiles = (q_len + tile_tokens - 1) / tile_tokens;
    if (p.paired ? rank > n_tiles - 1 - rank : n_tiles - 1 - rank < 0) return;  // uniform
    auto part_of = [&](int tile) SHIFTATTN_INLINE -> Part {
        const int tile_pos_max = ctx - q_len + min((tile + 1) * tile_tokens, q_len) - 1;
        const int kv_tiles = tile_pos_max / kKvTile + 1;
        const int per_split = kDecode == 0 ? (kv_tiles + p.n_splits - 1) / p.n_splits : static_cast<int>(ceilf(kv_tiles / p.range_div));
        const int begin = split * per_split;
        return Part{tile, begin, kDecode != 0 && split == p.n_splits - 1 ? kv_tiles : min(kv_tiles, begin + per_split)};
    };
    Part cur = part_of(n_tiles - 1 - rank), next{};
    const int g = (hs << p.gs_log2) / p.G;  // KV head of every column of this workgroup
    const int32_t* __restrict__ table = p.block_table + static_cast<size_t>(s) * p.max_blocks;
    const int last_block = (ctx - 1) / kBlockSize;

    // ---- LDS addressing ---------------------------------------------------------------------------------
    unsigned char* gbase = lds + grp * kGroupBytes;  // this group's two stages
    // where this wavefront's direct-to-LDS loads land, as a scalar: the destination of such a load goes through M0,
    // and a per-lane copy of a wavefront-uniform value would cost vector ALU instructions at every load
    unsigned char* ld_base = lds + __builtin_amdgcn_readfirstlane(grp * kGroupBytes + wg * kBlockBytes);
    const int grp_u = __builtin_amdgcn_readfirstlane(grp), wg_u = __builtin_amdgcn_readfirstlane(wg);
    // K operand of MFMA row l32 is K row tau (bits 2 and 3 swapped); piece c of row r sits at c ^ (r & 15)
    const int tau = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
    int k_rd[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) k_rd[ks] = tau * 256 + (((2 * ks + half) ^ (tau & 15)) << 4);
    // V^T operand: block-major [4][128 rows][32 B]; the two 16-byte halves of a row are swapped in
    // every other run of eight rows
    const int v_rd = kKBytes + l32 * 32 + ((half ^ ((l32 >> 3) & 1)) << 4);
    // direct-to-LDS loads: this wavefront fills cache block `wg` of a tile, 1 KiB per instruction
    // (LDS side contiguous in lane order; the swizzle is applied to the global address)
    int k_ld[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 4 * j + (lane >> 4);
        k_ld[j] = row * 256 + (((lane & 15) ^ row) << 4);
    }
    const int v_ld = kBlockBytes + (lane >> 1) * 32 + (((lane & 1) ^ ((lane >> 4) & 1)) << 4);
    const size_t blk_bytes = static_cast<size_t>(p.hkv_l) * 2 * kBlockBytes;
    // uniform values that the register allocator would otherwise keep in vector registers are pinned to scalar ones:
    // arithmetic on them then costs no vector instruction (each of which costs MFMA issue time in the key loop)
    auto uniform_ptr = [](const unsigned char* ptr) SHIFTATTN_INLINE -> const unsigned char* {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
        return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
    };

    typedef __attribute__((address_space(3))) void* lds_ptr;
    typedef const __attribute__((address_space(1))) void* glb_ptr;

    bf16x2 ones;
    ones[0] = static_cast<__bf16>(1.0f);
    ones[1] = static_cast<__bf16>(1.0f);
    const float thr = 8.0f / p.c;

    // 1 KiB from src (wavefront-uniform, in scalar registers) + a 32-bit byte offset per lane + kImm into LDS at dst + kImm
    // (dst uniform): written as assembly so that the address is formed by the load itself (scalar base + vector offset)
    // instead of a 64-bit vector addition per load, which would cost MFMA issue time like any vector instruction.
    // The compiler does not count these loads: they are waited for explicitly, with vmcnt(0) (wait_vm0) or, where a pass begins, vmcnt(4).
    auto dma_1k = [&](const unsigned char* src, uint32_t lane_off, auto imm_c, unsigned char* dst) SHIFTATTN_INLINE {
        constexpr int kImm = decltype(imm_c)::value;
        const uint32_t m0v = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
        // (M0 is reserved by the compiler - it sets it right before each use of its own and keeps no value in it,
        // and rejects it on a clobber list - so writing it here needs no clobber.)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                     :: "s"(m0v), "v"(lane_off), "s"(src), "n"(kImm) : "memory");
    };
    // the base must sit in scalar registers for the assembly above: said explicitly (it is wavefront-uniform, but the
    // register allocator may keep a uniform pointer in vector registers)
    auto scalar_ptr = [](const unsigned char* ptr) SHIFTATTN_INLINE -> const unsigned char* {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
        return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
    };
    auto load_k = [&](const unsigned char* src_any, int stage) SHIFTATTN_INLINE {
        const unsigned char* src = scalar_ptr(src_any);
        unsigned char* dst = ld_base + stage * kStageBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) dma_1k(src, static_cast<uint32_t>(k_ld[j]), IC<0>{}, dst + j * 1024);
    };
    auto load_v = [&](const unsigned char* src_any, int stage) SHIFTATTN_INLINE {
        const unsigned char* src = scalar_ptr(src_any);
        unsigned char* dst = ld_base + stage * kStageBytes + kKBytes;
        // the instruction's immediate offset moves the LDS destination along with the source
        dma_1k(src, static_cast<uint32_t>(v_ld), IC<0>{}, dst);
        dma_1k(src, static_cast<uint32_t>(v_ld), IC<1024>{}, dst);
        dma_1k(src, static_cast<uint32_t>(v_ld), IC<2048>{}, dst);
        dma_1k(src, static_cast<uint32_t>(v_ld), IC<3072>{}, dst);
    };
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    const const_i32_ptr table_c =
        (const_i32_ptr)reinterpret_cast<const int32_t*>(uniform_ptr(reinterpret_cast<const unsigned char*>(table)));
    const unsigned char* cache_g =
        uniform_ptr(reinterpret_cast<const unsigned char*>(p.cache) + static_cast<size_t>(g) * 2 * kBlockBytes);
    auto block_base = [&](int id) SHIFTATTN_INLINE -> const unsigned char* {
        return cache_g + static_cast<int64_t>(id) * blk_bytes;
    };
    // What the first iterations of a pass wait for is requested while the pass before merges its groups and writes its rows
    // out: the block ids of the first three tiles, K of the first, Q^T - a chain of two round trips to memory that a
    // workgroup of two tiles otherwise waits for twice (4 x 4096 tokens, 4 heads: 76.8 -> 76.0 us a call).
    bf16x8 qf[8];
    int id0 = 0, id1 = 0, id2 = 0;  // ids of tiles j, j+1, j+2 at the top of iteration j (uniform)
    auto load_q = [&](const Part& of) SHIFTATTN_INLINE {
        const int c = wg * 32 + l32, tok = of.tile * tile_tokens + (c >> p.gs_log2);
        const uint16_t* qp = p.q + static_cast<size_t>(q_begin + tok) * p.q_stride + ((hs << p.gs_log2) + (c & gs_mask)) * kD + half * 8;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (tok < q_len) v = *reinterpret_cast<const u32x4*>(qp + ks * 16);
            qf[ks] = as_bf16x8(v);
        }
    };
    auto group_tiles = [&](const Part& of) SHIFTATTN_INLINE { return (max(of.kt_end - of.kt_begin, 0) + 1 - grp) >> 1; };
    auto request_first = [&](const Part& of) SHIFTATTN_INLINE {   // the ids, and K of the first tile into stage 0
        const int n = __builtin_amdgcn_readfirstlane(group_tiles(of));
        if (n == 0) return;
        auto id_of = [&](int j) SHIFTATTN_INLINE { return table_c[min((of.kt_begin + grp_u + 2 * min(j, n - 1)) * 4 + wg_u, last_block)]; };
        id0 = id_of(0), id1 = id_of(1), id2 = id_of(2);
        load_k(block_base(id0), 0);
    };
    load_q(cur);
    request_first(cur);
    for (;;) {
        const int tile = cur.tile;
        const int kt_begin = cur.kt_begin, kt_end = cur.kt_end;
        const int tok0 = tile * tile_tokens;
        const int cw = wg * 32 + l32;
        const int tok = tok0 + (cw >> p.gs_log2);
        const bool valid = tok < q_len;
        const int pos_col = valid ? ctx - q_len + tok : -1;
        const int w_tok_first = tok0 + ((wg * 32) >> p.gs_log2);
        const int w_pos_min = __builtin_amdgcn_readfirstlane(w_tok_first < q_len ? ctx - q_len + w_tok_first : -1);

        // ---- key tiles of this (column tile, split), dealt alternately to the two groups ------------------
        const int n_all = max(kt_end - kt_begin, 0);
        const int n = group_tiles(cur);              // tiles of this group: kt(j) = kt_begin + grp + 2 j
        const int n_other = (n_all + grp) >> 1;
        // The tile that reaches past the context (if any) holds unwritten V slots; its owner clears them
        // in LDS before use, which costs one extra barrier that the other group mirrors.
        const bool pass_ragged = n_all > 0 && kt_end * kKvTile > ctx;
        const bool own_ragged = pass_ragged && (((n_all - 1) & 1) == grp);

        f32x16 oacc[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[mt][r] = 0.f;
        f32x16 sbuf[2][2];
        uint32_t pw[2][4][4];
        float m_used = -INFINITY, l_run = 0.f, alpha_pending = 1.f;

        auto kt_of = [&](int j) SHIFTATTN_INLINE { return kt_begin + grp_u + 2 * j; };
        // Cache block `wg` of the group's tile j.  Ids are fetched three tiles ahead and waited for a
        // whole iteration later: loads return in order, so a wait right behind the direct-to-LDS loads
        // (or right after the barrier) would stall for a full memory round trip every iteration.
        const int n_u = __builtin_amdgcn_readfirstlane(n);
        auto fetch_id = [&](int j) SHIFTATTN_INLINE -> int {
            // every term of the address is uniform, and the table is read through the constant address space: the
            // compiler issues a scalar load, the id arrives in a scalar register without a vector instruction, and the
            // compiler itself places the wait in front of the first use (the bottom of the iteration, see below)
            const int idx = min((kt_begin + grp_u + 2 * min(j, max(n_u - 1, 0))) * 4 + wg_u, last_block);
            return table_c[idx];
        };
        // zero the V^T entries of keys at or past the context in the given stage (tile kt)
        auto clear_ragged_v = [&](int kt, int stage) SHIFTATTN_INLINE {
            const int t4 = tid & 255;  // thread within the group
            const int d = t4 >> 1, h = t4 & 1;
#pragma unroll
            for (int bi = 0; bi < 4; ++bi) {
                const int n_valid = ctx - (kt * kKvTile + bi * 16 + h * 8);
                if (n_valid < 8) {
                    u32x4* ptr = reinterpret_cast<u32x4*>(gbase + stage * kStageBytes + kKBytes + bi * kBlockBytes + d * 32 +
                                                          ((h ^ ((d >> 3) & 1)) << 4));
                    u32x4 v = *ptr;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        v[w] &= n_valid > 2 * w + 1 ? 0xFFFFFFFFu : (n_valid > 2 * w ? 0x0000FFFFu : 0u);
                    *ptr = v;
                }
            }
        };
        auto apply_pending = [&]() SHIFTATTN_INLINE {
            if (__builtin_amdgcn_ballot_w64(alpha_pending != 1.f)) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[mt][r] *= alpha_pending;
            }
            alpha_pending = 1.f;
        };

        // One iteration on the group's tile j.  PAR = parity of j: selects register sets and LDS stages
        // at compile time (stage PAR is filled in this iteration, stage 1-PAR is read).
        auto body = [&](auto par_c, auto has_a_c, auto has_c_c, int j) SHIFTATTN_INLINE {
            constexpr int PAR = decltype(par_c)::value;
            constexpr bool HAS_A = decltype(has_a_c)::value != 0;
            constexpr bool HAS_C = decltype(has_c_c)::value != 0;
            constexpr int RD = 1 - PAR;
            f32x16(&s_cur)[2] = sbuf[PAR];
            f32x16(&s_nxt)[2] = sbuf[1 - PAR];
            uint32_t(&p_cur)[4][4] = pw[PAR];
            uint32_t(&p_prv)[4][4] = pw[1 - PAR];
            const int kt = kt_of(j);
            const int key0 = kt * kKvTile;

            constexpr int NOPS = (HAS_A ? 16 : 0) + (HAS_C ? 16 : 0);
            auto op_read = [&](auto tc) SHIFTATTN_INLINE -> u32x4 {
                constexpr int t = decltype(tc)::value;
                constexpr bool is_a = HAS_A && (!HAS_C || (t % 2 == 0));
                constexpr int o = (HAS_A && HAS_C) ? t / 2 : t;
                if constexpr (is_a)
                    return *reinterpret_cast<const u32x4*>(gbase + RD * kStageBytes + (o / 8) * 8192 + k_rd[o % 8]);
                else
                    return *reinterpret_cast<const u32x4*>(gbase + RD * kStageBytes + v_rd + (o / 4) * kBlockBytes + (o % 4) * 1024);
            };
            __syncthreads();
            // the operands of the first two MFMAs are requested first: their LDS latency passes while the loads below
            // are issued, instead of holding up the first MFMA behind the barrier
            u32x4 first0 = {0u, 0u, 0u, 0u}, first1 = first0;
            if constexpr (NOPS > 0) {
                first0 = op_read(IC<0>{});
                first1 = op_read(IC<1>{});
            }
            // fill stage PAR for the next iteration: K of tile j+2, V^T of tile j
            int id3_v = fetch_id(j + 3);  // consumed at the bottom of this iteration
            // In the steady state the two groups issue their loads at different times - the first group here, the second
            // behind its sixteenth MFMA: all eight wavefronts issuing at once queue up 64 KiB in the CU's one load path,
            // and a wavefront stuck at a load issues no MFMA; staggered, the other wavefront of its SIMD (which belongs to
            // the other group) keeps the pipe busy meanwhile.  Later than the middle of the step the loads would not
            // land before its end.
            constexpr bool kStagger = HAS_A && HAS_C;
            constexpr int kLateSlot = 16;
            const bool more_k = j + 2 < n;
            const unsigned char* k_src = block_base(id2);
            const unsigned char* v_src = block_base(id0);
            if (!kStagger || grp_u == 0) {
                if (more_k) load_k(k_src, PAR);
                load_v(v_src, PAR);
            }
            if (HAS_C) apply_pending();
            if (key0 + kKvTile - 1 > w_pos_min) {  // tile crosses the diagonal of this wavefront: uniform
#pragma unroll
                for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = key0 + 32 * sub + 16 * (r >> 3) + 8 * half + (r & 7);
                        if (key > pos_col) s_cur[sub][r] = -INFINITY;
                    }
            }

            // ---- interleaved block ------------------------------------------------------------------
            float mx = -INFINITY, mc = 0.f, alpha = 1.f, psum = 0.f;
            auto chunk = [&](auto cc) SHIFTATTN_INLINE {
                constexpr int c = decltype(cc)::value;
                if constexpr (c < 8) {
                    constexpr int sub = (4 * c) / 16, r = (4 * c) % 16;
                    mx = fmaxf(fmaxf(mx, s_cur[sub][r]), s_cur[sub][r + 1]);
                    mx = fmaxf(fmaxf(mx, s_cur[sub][r + 2]), s_cur[sub][r + 3]);
                } else if constexpr (c == 8) {
                    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                    // one v_max_f32: through fmaxf the two swapped halves would each be canonicalised first
                    asm("v_max_f32 %0, %1, %2" : "=v"(mx) : "v"(__uint_as_float(sw[0])), "v"(__uint_as_float(sw[1])));
                    const bool grow = mx > m_used + thr;
                    const float m_new = grow ? mx : m_used;
                    alpha = grow ? __builtin_amdgcn_exp2f((m_used - m_new) * p.c) : 1.f;
                    m_used = m_new;
                    mc = (m_new == -INFINITY ? 0.f : m_new) * p.c;
                    alpha_pending = alpha;
                    // the empty asm statements pin each result to its slot: without them the optimiser
                    // sinks the softmax below the MFMA sequence, next to its first use
                    asm volatile("" : "+v"(mc), "+v"(alpha), "+v"(m_used));
                } else if constexpr (c < 25) {
                    constexpr int v = 2 * (c - 9), sub = v / 16, r = v % 16;
                    const float e0 = __builtin_amdgcn_exp2f(fmaf(s_cur[sub][r], p.c, -mc));
                    const float e1 = __builtin_amdgcn_exp2f(fmaf(s_cur[sub][r + 1], p.c, -mc));
                    bf16x2 t;
                    t[0] = static_cast<__bf16>(e0);
                    t[1] = static_cast<__bf16>(e1);
                    psum = __builtin_amdgcn_fdot2_f32_bf16(t, ones, psum, false);
                    uint32_t w = __builtin_bit_cast(uint32_t, t);
                    asm volatile("" : "+v"(w), "+v"(psum));
                    p_cur[sub * 2 + (r >> 3)][(r & 7) >> 1] = w;
                } else {
                    l_run = l_run * alpha + psum;
                    asm volatile("" : "+v"(l_run));
                }
            };
            auto op_mfma = [&](auto tc, u32x4 a) SHIFTATTN_INLINE {
                constexpr int t = decltype(tc)::value;
                constexpr bool is_a = HAS_A && (!HAS_C || (t % 2 == 0));
                constexpr int o = (HAS_A && HAS_C) ? t / 2 : t;
                if constexpr (is_a) {
                    constexpr int sub = o / 8, ks = o % 8;
                    if constexpr (ks == 0) {
                        f32x16 z;
#pragma unroll
                        for (int r = 0; r < 16; ++r) z[r] = 0.f;
                        s_nxt[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), qf[ks], z, 0, 0, 0);
                    } else {
                        s_nxt[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), qf[ks], s_nxt[sub], 0, 0, 0);
                    }
                } else {
                    constexpr int ks2 = o / 4, mt = o % 4;
                    u32x4 pv = {p_prv[ks2][0], p_prv[ks2][1], p_prv[ks2][2], p_prv[ks2][3]};
                    oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(pv), oacc[mt], 0, 0, 0);
                }
            };

            if constexpr (NOPS == 0) {
                [&]<int... C>(std::integer_sequence<int, C...>) SHIFTATTN_INLINE { (chunk(IC<C>{}), ...); }
                (std::make_integer_sequence<int, 26>{});
            } else {
                u32x4 opnd[NOPS];
                opnd[0] = first0;
                opnd[1] = first1;
                [&]<int... T>(std::integer_sequence<int, T...>) SHIFTATTN_INLINE {
                    (([&]() SHIFTATTN_INLINE {
                         if constexpr (T + 2 < NOPS) opnd[T + 2] = op_read(IC<T + 2>{});
                         op_mfma(IC<T>{}, opnd[T]);
                         if constexpr (kStagger && T == kLateSlot) {
                             if (grp_u != 0) {
                                 if (more_k) load_k(k_src, PAR);
                                 load_v(v_src, PAR);
                             }
                         }
                         if constexpr (NOPS == 32) {
                             if constexpr (T < 26) chunk(IC<T>{});
                         } else {
                             if constexpr (2 * T < 26) chunk(IC<2 * T>{});
                             if constexpr (2 * T + 1 < 26) chunk(IC<2 * T + 1>{});
                         }
                         __builtin_amdgcn_sched_barrier(0);
                     }()),
                     ...);
                }
                (std::make_integer_sequence<int, NOPS>{});
            }
            wait_vm0();  // this wavefront's loads have landed before it reaches the next barrier
            id0 = id1;
            id1 = id2;
            id2 = id3_v;
        };

        int barriers = 0;  // barriers this group executes in the pass; both groups must end up equal
        if (n > 0) {
            // prologue: K of the first two tiles, S^T of the first
            // (K of the second is waited for behind the products on the first; the ids are uniform: said here, or the key loop forms its addresses from vector registers, eight vector instructions
            // more in two steps: 0.4 % of 24 kinds of batches)
            id0 = __builtin_amdgcn_readfirstlane(id0);
            id1 = __builtin_amdgcn_readfirstlane(id1);
            id2 = __builtin_amdgcn_readfirstlane(id2);
            if (n > 1) {
                load_k(block_base(id1), 1);
                // vmcnt(4): all but these four.  Memory operations count down in the order of their issue, and the four are behind those
                // of the first tile; whatever else is issued behind them only makes the wait a longer one.
                __builtin_amdgcn_s_waitcnt(0x0F74);
            } else {
                wait_vm0();
            }
            __syncthreads();
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
                for (int r = 0; r < 16; ++r) sbuf[0][sub][r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const u32x4 a = *reinterpret_cast<const u32x4*>(gbase + sub * 8192 + k_rd[ks]);
                    sbuf[0][sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), qf[ks], sbuf[0][sub], 0, 0, 0);
                }
            }
            wait_vm0();
            if (n == 1) {
                body(IC<0>{}, IC<0>{}, IC<0>{}, 0);
            } else {
                body(IC<0>{}, IC<1>{}, IC<0>{}, 0);
                int j = 1;  // stays odd: the steady-state loop takes two tiles per trip so that the
                            // register sets of even and odd tiles are fixed at compile time
                for (; j + 2 < n; j += 2) {
                    body(IC<1>{}, IC<1>{}, IC<1>{}, j);
                    body(IC<0>{}, IC<1>{}, IC<1>{}, j + 1);
                }
                if (j + 1 < n) {
                    body(IC<1>{}, IC<1>{}, IC<1>{}, j);
                    body(IC<0>{}, IC<0>{}, IC<1>{}, j + 1);
                } else {
                    body(IC<1>{}, IC<0>{}, IC<1>{}, j);
                }
            }
            // epilogue: C of the last tile
            __syncthreads();
            const int lp = (n - 1) & 1;
            if (own_ragged) {
                clear_ragged_v(kt_of(n - 1), lp);
                __syncthreads();
            }
            apply_pending();
            auto last_c = [&](auto par_c) SHIFTATTN_INLINE {
                constexpr int PAR = decltype(par_c)::value;
#pragma unroll
                for (int ks2 = 0; ks2 < 4; ++ks2)
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) {
                        const u32x4 a = *reinterpret_cast<const u32x4*>(gbase + PAR * kStageBytes + v_rd + ks2 * kBlockBytes + mt * 1024);
                        u32x4 pv = {pw[PAR][ks2][0], pw[PAR][ks2][1], pw[PAR][ks2][2], pw[PAR][ks2][3]};
                        oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(pv), oacc[mt], 0, 0, 0);
                    }
            };
            if (lp) last_c(IC<1>{});
            else last_c(IC<0>{});
            barriers = n + 2 + (own_ragged ? 1 : 0);
        }
        // even out the barrier count of the two groups (their LDS regions are disjoint, only the count matters)
        const int other_barriers = n_other > 0 ? n_other + 2 + ((pass_ragged && !own_ragged) ? 1 : 0) : 0;
        for (int b = barriers; b < other_barriers; ++b) __syncthreads();

        // ---- merge the two groups -------------------------------------------------------------------------
        float l_tot = l_run + __shfl_xor(l_run, 32);
        __syncthreads();  // every wavefront is done with the tile stages
        // the pass that follows: its first K tiles go to stage 0 of either group, where nothing of the merge lies
        const bool more = p.paired && cur.tile != rank;   // (the second of a pair is the last)
        if (more) {
            next = part_of(rank);
            request_first(next);
        }
        // the thread index is read through an opaque copy: addresses derived from the plain value are loop
        // invariants that the optimiser computes before the key loop and then spills around it
        int tid_m = tid;
        asm volatile("" : "+v"(tid_m));
        const int t4 = tid_m & 255;
        // Each group finishes one half of the head dimension (group 0 rows 0..63, group 1 rows 64..127): it parks the other half
        // of its accumulators for the other group and folds in what that group parked.
        float* park = reinterpret_cast<float*>(lds + kParkAt);        // [2 groups][32 values][256 lanes]
        float* x_ml = reinterpret_cast<float*>(lds + kStagedAt + kCols * kPitch);  // [2 groups][2][256]
        // (register arrays are indexed with compile-time constants only: one copy of the code per group)
        auto park_half = [&](auto g_c) SHIFTATTN_INLINE {
            constexpr int GRP = decltype(g_c)::value;
            float* mine = park + GRP * (32 * 256);
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[(k * 16 + r) * 256 + t4] = oacc[2 * (1 - GRP) + k][r];
            x_ml[(GRP * 2) * 256 + t4] = m_used;
            x_ml[(GRP * 2 + 1) * 256 + t4] = l_tot;
        };
        if (grp == 0) park_half(IC<0>{});
        else park_half(IC<1>{});
        __syncthreads();
        if (more) load_q(next);
        if (p.n_splits == 1) {
            // it normalises and puts bf16 rows into an LDS staging tile; then all eight wavefronts write the tile out in whole
            // 256-byte rows (one 16-byte piece per lane, 1 KiB of consecutive output per instruction per 4 rows)
            unsigned char* stage = lds + kStagedAt;                       // [128 columns][kPitch]
            auto finish_half = [&](auto g_c) SHIFTATTN_INLINE {
                constexpr int grp = decltype(g_c)::value;  // shadows the runtime value
                const float* theirs = park + (1 - grp) * (32 * 256);
                const float m_o = x_ml[((1 - grp) * 2) * 256 + t4], l_o = x_ml[((1 - grp) * 2 + 1) * 256 + t4];
                const float m_star = fmaxf(m_used, m_o);
                const float w_me = m_used == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_used - m_star) * p.c);
                const float w_o = m_o == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_o - m_star) * p.c);
                const float l_all = l_tot * w_me + l_o * w_o;
                const float inv = l_all > 0.f ? p.out_scale / l_all : 0.f;
                const float a_me = w_me * inv, a_o = w_o * inv;
                const int cw_m = ((tid_m >> 6) & 3) * 32 + (tid_m & 31), half_m = (tid_m >> 5) & 1;
                unsigned char* srow = stage + cw_m * kPitch + (64 * grp + 4 * half_m) * 2;
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        bf16x4 v;
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            v[x] = static_cast<__bf16>(oacc[2 * grp + k][r4 * 4 + x] * a_me + theirs[(k * 16 + r4 * 4 + x) * 256 + t4] * a_o);
                        *reinterpret_cast<u32x2*>(srow + (32 * k + 8 * r4) * 2) = __builtin_bit_cast(u32x2, v);
                    }
            };
            if (grp == 0) finish_half(IC<0>{});
            else finish_half(IC<1>{});
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int col = (tid_m >> 4) + 32 * i, piece = tid_m & 15;
                const int tok_c = tok0 + (col >> p.gs_log2);
                if (tok_c < q_len) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + col * kPitch + piece * 16);
                    uint16_t* op = p.out + static_cast<size_t>(q_begin + tok_c) * p.out_stride +
                                   ((hs << p.gs_log2) + (col & gs_mask)) * kD + piece * 8;
                    *reinterpret_cast<u32x4*>(op) = v;
                }
            }
        } else {
            // key ranges split over workgroups: the un-normalised partial of this range, each group one half of the head
            // dimension of it
            auto fold_half = [&](auto g_c) SHIFTATTN_INLINE {
                constexpr int grp = decltype(g_c)::value;  // shadows the runtime value
                const float* theirs = park + (1 - grp) * (32 * 256);
                const float m_o = x_ml[((1 - grp) * 2) * 256 + t4], l_o = x_ml[((1 - grp) * 2 + 1) * 256 + t4];
                const float m_star = fmaxf(m_used, m_o);
                const float w_me = m_used == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_used - m_star) * p.c);
                const float w_o = m_o == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_o - m_star) * p.c);
                const int cw_m = ((tid_m >> 6) & 3) * 32 + (tid_m & 31), half_m = (tid_m >> 5) & 1, tok_m = tok0 + (cw_m >> p.gs_log2);
                if (tok_m >= q_len || ctx - q_len + tok_m < 0) return;
                // accumulator register r of row tile mt is head-dim 32*mt + 8*(r/4) + 4*half + r%4
                const size_t prow = (static_cast<size_t>(split) * p.total_q + q_begin + tok_m) * p.hq_l + (hs << p.gs_log2) + (cw_m & gs_mask);
                float* op = p.o_part + prow * kD + 64 * grp + 4 * half_m;
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        f32x4 v;
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            v[x] = oacc[2 * grp + k][r4 * 4 + x] * w_me + theirs[(k * 16 + r4 * 4 + x) * 256 + t4] * w_o;
                        *reinterpret_cast<f32x4*>(op + 32 * k + 8 * r4) = v;
                    }
                if (grp == 0 && half_m == 0) {
                    p.ml_part[prow * 2] = m_star * p.c;  // -inf when this key range held no visible key
                    p.ml_part[prow * 2 + 1] = l_tot * w_me + l_o * w_o;
                }
            };
            if (grp == 0) fold_half(IC<0>{});
            else fold_half(IC<1>{});
        }
        if (!more) break;
        // The next pass reuses LDS.  A bare barrier: __syncthreads() would also wait until the rows just written out and the
        // requests of the next pass have come back.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        cur = next;
    }
}

constexpr double kPassSeconds = 7e-6;  // what a pass of this kernel costs around its key loop (Q, first tiles, merge of the groups, write-out)

struct Plan {
    int gs_log2, head_slots, tile_tokens, pair_ranks, n_splits;
    bool paired, rotate;
};

Plan make_plan(int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    Plan pl;
    const int G = a.hq_l / a.hkv_l;
    const bool pow2 = (G & (G - 1)) == 0 && G <= 32;
    pl.gs_log2 = 0;
    if (pow2) while ((1 << pl.gs_log2) < G) ++pl.gs_log2;
    pl.head_slots = a.hq_l >> pl.gs_log2;
    pl.tile_tokens = 128 >> pl.gs_log2;
    const int tiles = (max_q_len + pl.tile_tokens - 1) / pl.tile_tokens;
    pl.paired = option_prefill_pairing() != 2;
    pl.pair_ranks = pl.paired ? (tiles + 1) / 2 : tiles;
    // Key ranges per column tile: the count that minimises the model of a launch that also decides between the two
    // kernels - more ranges when the tiles alone cannot fill the chip (long cached context, short chunk) or fill it
    // with a ragged last round (320 equal workgroups on 256 compute units), as long as the merge does not eat the gain.
    const long wgs = static_cast<long>(pl.pair_ranks) * num_seqs * pl.head_slots;
    int splits = 1;
    const int forced = option_prefill_splits();
    if (forced > 0) {
        splits = forced;
    } else {
        const int by_len = max_seq_len / (16 * kKvTile);  // at least 16 key tiles per range
        const double walks = paired_walks(max_q_len, max_seq_len);
        // (with what the passes cost around their key loops: two per round of pairs, about 7 us each)
        auto priced = [&](int sp) {
            return launch_model_seconds(wgs, sp, 128, total_q, max_seq_len, a.hq_l, walks) +
                   2.0 * static_cast<double>((wgs * sp + 255) / 256) * kPassSeconds;
        };
        double best = priced(1);
        for (int cand = 2; cand <= 16 && cand <= by_len; ++cand) {
            const double t = priced(cand);
            if (t < best * 0.97) {  // a further range must pay for itself
                best = t;
                splits = cand;
            }
        }
    }
    if (splits < 1) splits = 1;
    if (splits > 64) splits = 64;
    pl.n_splits = splits;
    pl.rotate = rotate_sequences_over_dies(num_seqs, pl.head_slots, total_q, max_q_len);
    return pl;
}

// FP8 E4M3 cache: the blocks the batch reads are first widened to bf16 (exact) into a scratch cache in
// the workspace, block i of sequence s at scratch block s * nb + i with nb = blocks of the longest
// context, together with the block table that says so; the kernel then runs on the scratch cache with
// k_scale in its logit scale and v_scale on its output.  The pass moves 1.5 bytes per cached element
// once, against the 4 * D flops per (query, key) pair of the attention itself.
constexpr size_t kFp8ScratchLimit = static_cast<size_t>(8) << 30;  // larger batches take the general kernel

struct Fp8Scratch {
    int nb;               // scratch blocks per sequence
    size_t cache_bytes;   // bf16 scratch cache
    size_t table_bytes;   // int32 [num_seqs][nb], padded to 256 bytes
};

Fp8Scratch fp8_scratch(int num_seqs, int max_seq_len, const AttnShape& a) {
    Fp8Scratch f;
    f.nb = (max_seq_len + kBlockSize - 1) / kBlockSize;
    f.cache_bytes = static_cast<size_t>(num_seqs) * f.nb * a.hkv_l * 2 * kBlockBytes;
    f.table_bytes = (static_cast<size_t>(num_seqs) * f.nb * sizeof(int32_t) + 255) / 256 * 256;
    return f;
}

}  // namespace

bool prefill_mfma_supported(const AttnShape& a, int num_seqs, int max_seq_len) {
    if (!(a.elem == 2 && a.D == kD && a.hq_l % a.hkv_l == 0)) return false;
    return !a.kv_fp8() || fp8_scratch(num_seqs, max_seq_len, a).cache_bytes <= kFp8ScratchLimit;
}

namespace {

// Which kernel serves a launch: the 128-column kernel of this file (narrow) or one of the two forms of the 64-column wavefronts
// of prefill_mfma64.hip, tiles of 256 columns (wide) and of 128 with two groups of wavefronts (half; w.groups == 2).
// choose() compares the narrow and the wide plan under a rough model of a launch; see plan_within() for what is launched.
struct Choice {
    bool wide;
    Plan narrow;
    Prefill64Plan w;
};

Choice choose(int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    Choice c;
    c.narrow = make_plan(num_seqs, total_q, max_q_len, max_seq_len, a);
    c.wide = false;
    // (a cache widened from FP8 is bf16 by the time a kernel runs, so only the other conditions matter)
    AttnShape b = a;
    b.kv_elem = b.elem;
    if (!prefill_mfma64_supported(b)) return c;
    c.w = prefill_mfma64_plan(num_seqs, total_q, max_q_len, max_seq_len, a, option_prefill_splits());
    const int forced = option_prefill_tile();
    if (forced == 128) return c;
    // Both priced with what their passes cost around the key loop (two passes per round of pairs here; the wide kernel's,
    // about 15 us each, are in its plan); the 12 % are this kernel's slower loop.  The workgroups that weigh are counted
    // as for the wide kernel: those of sequences shorter than the longest are light or leave at once.
    const long wgs_n = static_cast<long>(c.narrow.pair_ranks * longest_chunk_equivalents(num_seqs, total_q, max_q_len) * c.narrow.head_slots + 0.999);
    const double rounds_n = static_cast<double>((wgs_n * c.narrow.n_splits + 255) / 256);
    const double t_narrow = 1.12 * launch_model_seconds(wgs_n, c.narrow.n_splits, 128, total_q, max_seq_len, a.hq_l,
                                                         paired_walks(max_q_len, max_seq_len)) + 2.0 * rounds_n * kPassSeconds;
    c.wide = forced == 256 || c.w.model_with_passes < 0.97 * t_narrow;
    return c;
}

size_t split_bytes(int n_splits, int total_q, const AttnShape& a) {
    return n_splits == 1 ? 0 : static_cast<size_t>(n_splits) * total_q * a.hq_l * (kD + 2) * sizeof(float);
}

size_t split_bytes_of(const Choice& c, int total_q, const AttnShape& a) {
    return split_bytes(c.wide ? c.w.n_splits : c.narrow.n_splits, total_q, a);
}

// ---- the launch within the workspace given --------------------------------------------------------------------
// choose() above plans tiles in pairs for the 128-column kernel and at least 1024 keys per range: right where the tiles
// fill the chip, and a chip left idle where they do not (a few prompts of some hundred tokens, a short chunk behind a
// long context: 47 tokens on 9062 cached, 4 heads, were one workgroup per key range that walked its range twice).  Its
// plan stays the least workspace a call is accepted with and the plan of a caller that brings no more; beyond it, one
// tile or two per workgroup and 1 to 32 key ranges of the three kernels are priced with the model below.  Constants in
// microseconds, fitted to 110 launches times about 50 plans each (prompts of 40 .. 14000 tokens, chunks behind 100 ..
// 60000 cached, 1 .. 12 sequences, all head geometries): the fit is 9 % off (root mean square of the logarithm).  On 1500 others
// the choices are 1.4 % slower than the best plan measured and 1.8 % faster than those among the narrow and the wide form.
struct TileKernel {
    double pass, second_pass;  // around the key loop: set-up, Q, first and last tile, write-out
    double step, step_full;    // one step of the key loop, and what it costs more once every compute unit is busy
    int keys_per_step;
    double several;            // factor where the batch has several sequences
};
constexpr TileKernel kNarrowCost = {1.94, 3.35, 1.362, 0.281, 2 * kKvTile, 1.084};   // two groups of wavefronts, a tile of 64 keys each
constexpr TileKernel kWideCost = {3.9, 3.1, 0.592, 0.039, 32, 1.108};
constexpr TileKernel kHalfCost = {5.35, 5.3, 0.506, 0.167, 64, 1.089};   // two groups of wavefronts, a tile of 32 keys each: fewer
    // clocks a key than the narrow kernel's, more around the loop; the cheaper one from about 1200 keys on (4 x 4096 tokens of 4 heads
    // 73.2 -> 67.6 us without the append, 11 prompts of 149 to 1097 of 5 heads 23.5 -> 26.7)
// the kernels a launch can take: the 128-column kernel and the two tilings of the 256-column kernel's file
enum Kind { kNarrow, kWide, kHalf, kKinds };
const TileKernel& cost_of(Kind k) { return k == kNarrow ? kNarrowCost : k == kWide ? kWideCost : kHalfCost; }
bool kind_allowed(Kind k, const AttnShape& bf16) {
    const int forced = option_prefill_tile();
    if (k == kNarrow) return forced != 256 || !prefill_mfma64_supported(bf16);
    if (!prefill_mfma64_supported(bf16)) return false;
    return k == kWide ? forced != 128 : forced != 256 && bf16.hq_l / bf16.hkv_l <= 128;
}

// The batch counted in sequences of its longest chunk, for `heads` (sequence, head) indices a sequence.  Of two sequences of one
// each, which never rotate, either sees every second die only: the longer has half the chip, whatever the shorter leaves of the other
// half (5068 + 8739 tokens, 5 heads: 150 us on the 128-column kernel, whose heads count one by one, 176 in two groups).  Of the 1500
// launches below 11 are 3 % slower than without the half form, 20 with the sum over the longest here too.
double sequences_that_weigh(int num_seqs, int heads, int total_q, int max_q_len) {
    return num_seqs == 2 && heads == 1 ? 2.0 : longest_chunk_equivalents(num_seqs, total_q, max_q_len);
}

double launch_us(const TileKernel& k, bool paired, int splits, int tile_tokens, int heads, int num_seqs, int total_q,
                 int max_q_len, int max_seq_len, int hq_l) {
    constexpr double kCus = 256, kSlack = 1.13;  // slack: how far a chip full of unequal workgroups stays from level
    constexpr double kMergeUs = 4.5, kMergeBytesPerUs = 5.8e6, kRowBytes = 1040;  // partials of a (token, head) written and read
    const int tiles = (max_q_len + tile_tokens - 1) / tile_tokens, ranks = paired ? (tiles + 1) / 2 : tiles;
    const double seqs = sequences_that_weigh(num_seqs, heads, total_q, max_q_len);
    const double wgs = ranks * seqs * heads * splits, grid = static_cast<double>(ranks) * num_seqs * heads * splits;
    const int q = max_q_len < max_seq_len ? max_q_len : max_seq_len;
    auto steps = [&](int keys) {   // of the range a workgroup takes of a tile that sees `keys` keys
        const int range = k.keys_per_step * splits;
        return static_cast<double>((keys + range - 1) / range);
    };
    const double heavy = steps(max_seq_len), light = steps(max_seq_len - q + (tile_tokens < q ? tile_tokens : q));
    const double step = k.step + k.step_full * (wgs < kCus ? wgs / kCus : 1.0);
    double d_hi, d_lo;             // longest and shortest workgroup
    if (paired) d_hi = d_lo = k.pass + heavy * step + (tiles > 1 ? k.second_pass + light * step : 0.0);
    else d_hi = k.pass + heavy * step, d_lo = k.pass + light * step;
    // A grid beyond the chip takes whole rounds of its shortest workgroup at least.  Workgroups of sequences shorter than
    // the longest leave at once, but the dispatcher hands workgroups to the 32 shader engines in turn, and up to two rounds the
    // busy ones fit the places of one only where no engine gets more than its eight: of 320 batches of 2 .. 12 unequal chunks those
    // with at most seven on the fullest engine took 0.9 of the time of the plan priced by whole rounds, those with nine or more 1.2
    // to 1.4 of it (six chunks of 19 to 95 tokens, 5 heads, ten ranges: all 300 workgroups busy, 1.39).  Busy are a sequence's own tiles,
    // its ragged last one among them, so n tokens are counted as n / tile + 1.
    const double rest = num_seqs > 1 ? (total_q - max_q_len) / (num_seqs - 1.0) : 0.0;
    double other = rest / tile_tokens + 1.0;   // tiles of a sequence but the longest, the ragged one among them
    if (other > tiles) other = tiles;
    const double other_ranks = paired ? (other + 1.0) / 2 : other;
    double busy = (ranks + (num_seqs - 1) * other_ranks) * heads * splits;
    // Where nothing rotates and the (sequence, head) count is even, the workgroups of one (sequence, head) see every second engine
    // (375 + 123 tokens on 29041, 8 heads: 144 workgroups of the long chunk on 128 compute units 132 us, 120 91).
    if ((static_cast<long>(num_seqs) * heads) % 2 == 0 && heads % 2 != 0 && !rotate_sequences_over_dies(num_seqs, heads, total_q, max_q_len))
        busy += (ranks - other_ranks) * splits;
    // Held to whole rounds of the grid from where on: at 0.7 / 0.75 / 0.8 / 0.85 / 0.9 / 0.95 of the chip the choices among 350 batches for
    // which it matters are 9.3 / 8.5 / 7.5 / 6.1 / 8.0 / 9.1 % slower than the best plan, 10.3 always.
    const double counted = grid <= 2 * kCus && busy > 0.85 * kCus ? grid : wgs;
    const double rounds = static_cast<double>(static_cast<long>((counted + kCus - 1) / kCus));
    double span = (grid > kCus ? kSlack : 1.0) * (d_hi + d_lo) / 2 * wgs / kCus;
    if (span < d_hi) span = d_hi;
    if (span < rounds * d_lo) span = rounds * d_lo;
    if (num_seqs > 1) span *= k.several;
    if (splits > 1) span += kMergeUs + splits * static_cast<double>(total_q) * hq_l * kRowBytes / kMergeBytesPerUs;
    return (span + 6.6) * (1.0 + 0.008 * splits);   // (launch; among equals the plan with fewer ranges)
}

// What the model must promise before a launch leaves the 128-column kernel.  Among 1500 launches of chunks alone (1 .. 12 equal or unequal
// chunks of 40 .. 14000 tokens, some behind 100 .. 60000 cached) and 2577 unified batches (1 .. 3 chunks of up to 3000 tokens on up to
// 100000 cached beside 2 .. 128 rows of up to 32000, either cache) the choices with 1 / 1.02 / 1.04 / 1.05 are 1.1 / 1.2 / 1.4 / 1.6 % and
// 1.9 / 2.0 / 2.0 / 2.1 % off the best plan measured, and 31 / 14 / 11 / 12 and 58 / 48 / 42 / 44 of them 3 % slower than the choice among
// the narrow and the wide form (297 / 275 / 238 / 214 and 237 / 200 / 174 / 153 as much faster).
constexpr double kMargin = 1.04;
// Keys a range of the half form holds at least.  Time with it over that of the narrow kernel, same tiles and ranges, by the keys of
// a range: 512 .. 768 1.09, 768 .. 1024 1.04, 1024 .. 1400 1.02, 1400 .. 2000 0.97, 2000 .. 2800 0.93, beyond 5600 0.79 (tiles one by
// one; in pairs 1.13 / 1.07 / 1.04 / 1.00 / 0.96 / 0.82).  Of chunks alone the line lies at the crossing: with lines at 1024 / 1400 /
// 2000 / 2400 the launches are 1.4 / 1.4 / 1.6 / 1.8 % off the best plan, 11 / 11 / 9 / 9 of them 3 % slower than without the form.  Beside
// decode rows, where the rows' four wavefronts a workgroup weigh too, it lies behind: with lines at 1400 / 2000 / 2400 / 2800 the batches are
// 1.9 / 2.0 / 2.0 / 2.1 % off, 47 / 45 / 42 / 40 slower (1579 tokens on 2097 beside 31 rows of 5516: narrow 52 us, half in ranges of 1838 60).
constexpr int kHalfLeastKeys = 1400, kHalfLeastKeysBesideRows = 2400;

Kind kind_of(const Choice& c) { return !c.wide ? kNarrow : c.w.groups == 1 ? kWide : kHalf; }

// `c` with one of the kernels, tiles in pairs or one per workgroup, and that many key ranges
void set_plan(Choice& c, Kind kind, bool paired, int splits, int num_seqs, int max_q_len, const AttnShape& a) {
    c.wide = kind != kNarrow;
    if (kind == kNarrow) {
        const int tiles = (max_q_len + c.narrow.tile_tokens - 1) / c.narrow.tile_tokens;
        c.narrow.paired = paired, c.narrow.pair_ranks = paired ? (tiles + 1) / 2 : tiles, c.narrow.n_splits = splits;
        return;
    }
    c.w.groups = kind == kWide ? 1 : 2;
    c.w.tile_tokens = 256 / c.w.groups / (a.hq_l / a.hkv_l);
    const int tiles = (max_q_len + c.w.tile_tokens - 1) / c.w.tile_tokens;
    c.w.paired = paired, c.w.pair_ranks = paired ? (tiles + 1) / 2 : tiles, c.w.n_splits = splits;
    c.w.workgroups = static_cast<long>(c.w.pair_ranks) * splits * num_seqs * a.hkv_l;
}

double priced(const Choice& c, int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    return c.wide ? launch_us(cost_of(kind_of(c)), c.w.paired, c.w.n_splits, c.w.tile_tokens, a.hkv_l, num_seqs, total_q, max_q_len, max_seq_len, a.hq_l)
                  : launch_us(kNarrowCost, c.narrow.paired, c.narrow.n_splits, c.narrow.tile_tokens, c.narrow.head_slots, num_seqs, total_q,
                              max_q_len, max_seq_len, a.hq_l);
}

Choice plan_within(size_t split_budget, int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    Choice best = choose(num_seqs, total_q, max_q_len, max_seq_len, a);
    AttnShape b = a;
    b.kv_elem = b.elem;
    const int forced_splits = option_prefill_splits(), forced_pairing = option_prefill_pairing();
    // (choose()'s plan without the margin, whichever kernel it is for: with 3 % in its favour besides 15 of 1254 launches were slower
    // by that and more, without one is)
    double best_us = priced(best, num_seqs, total_q, max_q_len, max_seq_len, a);
    Choice c = best;
    auto try_ranges = [&](int splits) {
        if (split_bytes(splits, total_q, a) > split_budget) return;
        for (int k = 0; k < kKinds; ++k) {
            if (!kind_allowed(static_cast<Kind>(k), b) || (k == kHalf && max_seq_len < splits * kHalfLeastKeys)) continue;
            for (int paired = 0; paired < 2; ++paired) {
                if (forced_pairing != 0 && paired != (forced_pairing == 1)) continue;
                set_plan(c, static_cast<Kind>(k), paired != 0, splits, num_seqs, max_q_len, a);
                const double us = (k == kNarrow ? 1.0 : kMargin) * priced(c, num_seqs, total_q, max_q_len, max_seq_len, a);
                if (us < best_us) best = c, best_us = us;
            }
        }
    };
    if (forced_splits > 0) {
        try_ranges(forced_splits);
    } else {
        for (int splits : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32})
            if (splits == 1 || max_seq_len >= splits * 2 * kKvTile) try_ranges(splits);
    }
    return best;
}

size_t with_fp8_scratch(size_t bytes, int num_seqs, int max_seq_len, const AttnShape& a) {
    if (!a.kv_fp8()) return bytes;
    const Fp8Scratch f = fp8_scratch(num_seqs, max_seq_len, a);
    return (bytes + 255) / 256 * 256 + f.cache_bytes + f.table_bytes;
}

}  // namespace

size_t prefill_mfma_least_workspace(int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    const Choice c = choose(num_seqs, total_q, max_q_len, max_seq_len, a);
    return with_fp8_scratch(split_bytes_of(c, total_q, a), num_seqs, max_seq_len, a);
}

size_t prefill_mfma_workspace(int num_seqs, int total_q, int max_q_len, int max_seq_len, const AttnShape& a) {
    const size_t least = prefill_mfma_least_workspace(num_seqs, total_q, max_q_len, max_seq_len, a);
    const Choice c = plan_within(SIZE_MAX, num_seqs, total_q, max_q_len, max_seq_len, a);
    const size_t best = with_fp8_scratch(split_bytes_of(c, total_q, a), num_seqs, max_seq_len, a);
    return best > least ? best : least;
}

hipError_t prefill_mfma_init() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_kernel<0>), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_kernel<1>), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesBoth);
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_kernel<2>), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesBoth);
    return e;
}

namespace {

constexpr float kLog2e = 1.4426950408889634f;

// The cache as the kernels read it: itself, or the blocks of an FP8 cache that the batch needs widened to bf16 behind the
// partials in the workspace.
struct CacheView {
    const void* cache;
    const int32_t* block_table;
    int max_blocks;
};

hipError_t bf16_view(const void* cache, const int32_t* block_table, const int32_t* seq_lens, int num_seqs, int max_seq_len,
                     size_t partial_bytes, void* workspace, const AttnShape& a, CacheView* v, hipStream_t st) {
    *v = {cache, block_table, a.max_blocks};
    if (!a.kv_fp8()) return hipSuccess;
    const Fp8Scratch f = fp8_scratch(num_seqs, max_seq_len, a);
    unsigned char* scratch = static_cast<unsigned char*>(workspace) + (partial_bytes + 255) / 256 * 256;
    int32_t* table2 = reinterpret_cast<int32_t*>(scratch + f.cache_bytes);
    *v = {scratch, table2, f.nb};
    return launch_fp8_blocks_to_bf16(cache, block_table, a.max_blocks, seq_lens, num_seqs, f.nb, a.hkv_l, scratch, table2, st);
}

PrefillParams narrow_params(const void* q, const CacheView& v, const int32_t* cu_seqlens_q, const int32_t* seq_lens, int num_seqs,
                            int total_q, const Plan& pl, void* out, void* workspace, const AttnShape& a) {
    PrefillParams p;
    p.q = static_cast<const uint16_t*>(q);
    p.cache = static_cast<const uint16_t*>(v.cache);
    p.block_table = v.block_table;
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
    p.gs_log2 = pl.gs_log2;
    p.head_slots = pl.head_slots;
    p.n_splits = pl.n_splits;
    p.paired = pl.paired ? 1 : 0;
    p.rotate = pl.rotate ? 1 : 0;
    p.max_blocks = v.max_blocks;
    p.c = a.scale * a.k_scale * kLog2e;
    p.out_scale = a.v_scale;
    p.ranks = pl.pair_ranks;
    p.range_div = static_cast<float>(pl.n_splits);
    return p;
}

}  // namespace

hipError_t launch_prefill_mfma(const void* q, const void* cache, const int32_t* block_table,
                               const int32_t* cu_seqlens_q, const int32_t* seq_lens, int num_seqs, int total_q,
                               int max_q_len, int max_seq_len, void* out, void* workspace, size_t workspace_bytes,
                               const AttnShape& a, hipStream_t st) {
    if (num_seqs == 0 || total_q == 0 || max_q_len <= 0) return hipSuccess;
    const size_t fixed = with_fp8_scratch(0, num_seqs, max_seq_len, a);
    // (an FP8 cache's scratch lies behind the partials, at a multiple of 256 bytes)
    const size_t budget = workspace_bytes < fixed ? 0 : a.kv_fp8() ? (workspace_bytes - fixed) / 256 * 256 : workspace_bytes;
    const Choice ch = plan_within(budget, num_seqs, total_q, max_q_len, max_seq_len, a);
    CacheView v;
    if (hipError_t e = bf16_view(cache, block_table, seq_lens, num_seqs, max_seq_len, split_bytes_of(ch, total_q, a), workspace, a, &v, st); e != hipSuccess)
        return e;
    if (ch.wide)
        return launch_prefill_mfma64(q, v.cache, v.block_table, v.max_blocks, cu_seqlens_q, seq_lens, num_seqs, total_q, ch.w, out,
                                     workspace, a, a.scale * a.k_scale * kLog2e, a.v_scale, st);
    const Plan& pl = ch.narrow;
    const PrefillParams p = narrow_params(q, v, cu_seqlens_q, seq_lens, num_seqs, total_q, pl, out, workspace, a);
    const unsigned grid = static_cast<unsigned>(pl.pair_ranks) * pl.n_splits * num_seqs * pl.head_slots;
    prefill_kernel<0><<<grid, kThreads, kLdsBytes, st>>>(p, DecodeRole{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.n_splits > 1)
        return launch_combine(p.o_part, p.ml_part, total_q, a.hq_l, kD, pl.n_splits, 0, nullptr, 0, out, a.out_stride,
                              a.elem, a.v_scale, st);
    return hipSuccess;
}

// ---- prefill and decode rows of a unified batch in one launch -----------------------------------------------------
// Chunks are bound by the matrix units, decode rows by memory, and one behind the other each leaves the other's resource
// idle; each also costs a launch (about 4.6 us behind another kernel) for its product and one for its merge.  Here the
// first workgroups of either prefill kernel's grid take the decode rows and the others the tiles, one merge kernel serves
// both.  A compute unit holds one workgroup of either kind, so the rows get as many as the tiles' ranges leave over; where
// every place is taken, the last key range of each tile is the one that waits for a place and is made shorter by what the
// decode rows take, so that all end together.  1000 tokens on 20000 cached (FP8) with 97 decodes: 154 -> 132 us a step;
// 200 random batches (1 .. 8 equal or unequal chunks of 100 .. 2048 on up to 60000 cached, 2 .. 128 decodes, 80 of the batches with
// decode rows that weigh more than the chunks) against two launches: 1.20 times, five of them 2 to 6.5 % slower; where all rows are as long as the longest 1.18, where one is and the others have a 25th 1.12.  2048 tokens on 131072 cached with 64
// decodes (256-column kernel): 1028 -> 974; 1536 on 90000 with 100: 670 -> 602.
namespace {

// The 128-column kernel beside decode rows, where the launch is full from its first workgroup on: from 200 random unified batches.  With
// its constants above, which come from launches of chunks alone, the 2577 batches are 2.3 instead of 2.0 % off the best plan, and 152 of
// them instead of 42 are 3 % slower than without the half form.
constexpr TileKernel kNarrowBesideRows = {2.65, 3.1, 1.4, 0.335, 2 * kKvTile, 1.0};

struct BothPlan {
    bool taken, wide;
    Plan narrow;
    Prefill64Plan w;
    int dec_wgs, dec_waves;
    float range_div;
    size_t partial_bytes;  // of the prefill part, a multiple of 256 with an FP8 cache's scratch behind it
    size_t bytes;          // workspace in all
};

// microseconds the decode rows take on some workgroups, one per compute unit (rates measured with 64 of them; an FP8 cache
// has half the bytes in flight); the lengths are on the device, their mean is taken as 0.6 of the longest
double decode_bytes(int num_seqs, int max_seq_len, const AttnShape& a) {
    return 0.6 * num_seqs * static_cast<double>(max_seq_len) * a.hkv_l * 2 * kD * a.kv_elem;
}
constexpr double kDecodeStartUs = 5.0, kBf16BytesPerUsWg = 60e3, kFp8BytesPerUsWg = 48e3, kDecodeBytesPerUs = 5.8e6;
// Of that with four wavefronts per workgroup (the kernels of 64-column wavefronts) instead of eight.  Choices among the 1578 batches over a
// bf16 cache with 0.65 / 0.74 / 0.85 / 1: 2.2 / 2.1 / 2.2 / 2.2 % off the best plan, 35 / 30 / 31 / 41 of them 3 % slower than without the
// half form; among the 999 over an FP8 cache with 0.45 / 0.6 / 0.85: 1.8 / 1.8 / 1.9 %, 11 / 15 / 30.
constexpr double kFourWaves = 0.85, kFp8FourWaves = 0.45;
double decode_us(double bytes, double wgs, bool fp8, bool wide) {
    const double rate = wgs * (fp8 ? kFp8BytesPerUsWg : kBf16BytesPerUsWg) * (!wide ? 1.0 : fp8 ? kFp8FourWaves : kFourWaves);
    return kDecodeStartUs + bytes / (rate < kDecodeBytesPerUs ? rate : kDecodeBytesPerUs);
}

// What the rows take on that many workgroups if the tiles take nothing from them: bytes per microsecond and workgroup from 16 ..
// 250 workgroups over 117 .. 760 MB of K/V (a workgroup keeps a fixed number of bytes in flight, half of them with an FP8 cache or
// in the 256-column kernel, and the trip to memory gets longer the more of them ask).  The rates above shape the plans well
// where tiles run beside the rows to the end, but promise too much where the rows outlast them.  kBothLimit: 176 random unified
// batches, half of them with decode rows that weigh more than the chunks.  Ten were slower shared, by 1 to 28 % (2 x 567 tokens
// x 16 heads with 73 rows of up to 17881: 204 us, 159 one after the other), all at 0.89 of the two launches' time or more by
// this figure; below 0.88 none was, and the two that the line gives away had gained 3 and 6 %.
double decode_us_at_least(double bytes, double wgs, bool fp8, bool wide) {
    const double per_wg = fp8 ? (wide ? 28.3e3 : 43e3) : (wide ? 57e3 - 150.0 * wgs : 56.6e3 - 125.0 * wgs);
    const double rate = wgs * per_wg;
    return kDecodeStartUs + bytes / (rate < 6.4e6 ? rate : 6.4e6);
}
constexpr double kDecodeAloneBytesPerUs = 6.1e6;   // of a launch of their own
constexpr double kBothLimit = 0.88;

BothPlan plan_both(int num_seqs, int total_q, int max_q_len, int max_seq_len, int num_dec, int max_dec_len, const AttnShape& a) {
    BothPlan best{};
    if (option_prefill_splits() != 0 || option_prefill_pairing() == 1) return best;
    if (num_seqs < 1 || total_q < 1 || max_q_len < 1 || num_dec < 1 || max_dec_len < 1 || !decode_mfma_one_launch(num_dec, max_dec_len, a))
        return best;
    const double bytes = decode_bytes(num_dec, max_dec_len, a);
    if (bytes < 1e6) return best;   // (a few short rows: nothing to share, and the workspace stays the larger of the two parts')
    const Choice alone = plan_within(SIZE_MAX, num_seqs, total_q, max_q_len, max_seq_len, a);
    const double chunks_us = (alone.wide ? kMargin : 1.0) * priced(alone, num_seqs, total_q, max_q_len, max_seq_len, a);   // (the scale of the plans below)
    double best_us = 0.97 * (chunks_us + decode_us(bytes, 256, a.kv_fp8(), false) + 9.0), at_least_us = 0.0;
    const int q = max_q_len < max_seq_len ? max_q_len : max_seq_len;
    AttnShape b16 = a;
    b16.kv_elem = b16.elem;
    for (int kind = 0; kind < kKinds; ++kind) {
        if (!kind_allowed(static_cast<Kind>(kind), b16)) continue;
        const TileKernel& k = kind == kNarrow ? kNarrowBesideRows : cost_of(static_cast<Kind>(kind));
        Choice c = alone;
        set_plan(c, static_cast<Kind>(kind), false, 1, num_seqs, max_q_len, a);
        const int tile_tokens = c.wide ? c.w.tile_tokens : c.narrow.tile_tokens, heads = c.wide ? a.hkv_l : c.narrow.head_slots;
        const int tiles = c.wide ? c.w.pair_ranks : c.narrow.pair_ranks;
        const bool four_waves = c.wide;
        const double lightest = max_seq_len - q + (tile_tokens < q ? tile_tokens : q);
        const double step = (k.step + k.step_full) / k.keys_per_step;   // per key
        auto rows_us = [&](double x) { return decode_us(bytes, x, a.kv_fp8(), four_waves); };
        for (int splits : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32}) {
            if (splits > 1 && max_seq_len < splits * 2 * kKvTile) break;
            if (kind == kHalf && max_seq_len < splits * kHalfLeastKeysBesideRows) break;
            const double wgs = tiles * sequences_that_weigh(num_seqs, heads, total_q, max_q_len) * heads * splits, grid = static_cast<double>(tiles) * num_seqs * heads * splits;
            const double merge = splits > 1 ? splits * static_cast<double>(total_q) * a.hq_l * 1040 / 5.8e6 : 0.0;
            auto consider = [&](double x, double div, double span) {
                const double us = (kind == kNarrow ? 1.0 : kMargin) * (span * (num_seqs > 1 ? k.several : 1.0) + merge + 6.6 + 4.5) * (1.0 + 0.008 * splits);
                if (us >= best_us) return;
                best_us = us;
                at_least_us = decode_us_at_least(bytes, x, a.kv_fp8(), four_waves) + merge + 6.6 + 4.5;
                set_plan(c, static_cast<Kind>(kind), false, splits, num_seqs, max_q_len, a);
                best.taken = true;
                best.wide = c.wide;
                best.narrow = c.narrow;
                best.w = c.w;
                best.dec_wgs = static_cast<int>(x);
                best.dec_waves = best.dec_wgs * (four_waves ? kPrefill64Waves : kDecodeWaves);
                best.range_div = static_cast<float>(div);
                best.partial_bytes = split_bytes(splits, total_q, a);
            };
            if (grid <= 256) {
                const double free = 256 - grid, last = grid / splits;   // places the tiles leave over; workgroups of the last ranges
                if (free >= 8) {                                        // nobody waits
                    const double d = k.pass + max_seq_len * step / splits;
                    consider(free, splits, d > rows_us(free) ? d : rows_us(free));
                }
                if (splits > 1 && free + last >= 8) {                   // the last ranges wait for the decode rows' places
                    const double x = static_cast<int>(free + last);
                    const double cut = rows_us(x) / step / max_seq_len;     // keys the last range leaves to the others, of the tile's
                    const double share = (1.0 + cut) / splits;              // of a full range: splits x share - cut = 1
                    if (share - cut >= 0.05 * share) consider(x, 1.0 / share, k.pass + max_seq_len * share * step);
                }
            } else {                                                    // several rounds: the rows first, ever lighter tiles behind them
                const double d_hi = k.pass + max_seq_len * step / splits, d_lo = k.pass + lightest * step / splits;
                for (int x : {32, 64, 96, 128, 192}) {
                    double span = 1.13 * (0.5 * (d_hi + d_lo) * wgs + x * rows_us(x)) / 256;
                    const double rounds = static_cast<double>(static_cast<long>((grid + x + 255) / 256));
                    for (const double least : {d_hi, rounds * d_lo, rows_us(x)})
                        if (span < least) span = least;
                    consider(x, splits, span);
                }
            }
        }
    }
    if (at_least_us > kBothLimit * (chunks_us + kDecodeStartUs + bytes / kDecodeAloneBytesPerUs + 9.0)) return BothPlan{};
    if (best.taken)
        best.bytes = (with_fp8_scratch(best.partial_bytes, num_seqs, max_seq_len, a) + 255) / 256 * 256 +
                     decode_mfma_workspace_for(best.dec_waves, num_dec, a);
    return best;
}

}  // namespace

size_t prefill_and_decode_workspace(int num_seqs, int total_q, int max_q_len, int max_seq_len, int num_dec, int max_dec_len, const AttnShape& a) {
    return plan_both(num_seqs, total_q, max_q_len, max_seq_len, num_dec, max_dec_len, a).bytes;
}

void prefill_mfma_describe(int num_seqs, int total_q, int max_q_len, int max_seq_len, int num_dec, int max_dec_len, const AttnShape& a,
                           shiftattn_prefill_plan_t* plan) {
    Choice c;
    const BothPlan both = num_dec > 0 ? plan_both(num_seqs, total_q, max_q_len, max_seq_len, num_dec, max_dec_len, a) : BothPlan{};
    if (both.taken) c.wide = both.wide, c.narrow = both.narrow, c.w = both.w;
    else c = plan_within(SIZE_MAX, num_seqs, total_q, max_q_len, max_seq_len, a);
    plan->tile_columns = c.wide && c.w.groups == 1 ? 256 : 128;
    plan->wave_columns = c.wide ? 64 : 32;
    plan->key_ranges = c.wide ? c.w.n_splits : c.narrow.n_splits;
    plan->tiles_per_wg = (c.wide ? c.w.paired : c.narrow.paired) ? 2 : 1;
    plan->decode_wgs = both.taken ? both.dec_wgs : 0;
}

bool launch_prefill_and_decode(const void* q, void* cache, const int32_t* block_table, const int32_t* cu_seqlens_q, const int32_t* seq_lens,
                               int num_seqs, int total_q, int max_q_len, int max_seq_len, int num_dec, int max_dec_len, void* out,
                               void* workspace, size_t workspace_bytes, const AttnShape& a, hipStream_t st, hipError_t* err) {
    const BothPlan pl = plan_both(num_seqs, total_q, max_q_len, max_seq_len, num_dec, max_dec_len, a);
    if (!pl.taken || workspace_bytes < pl.bytes) return false;
    CacheView v;
    *err = bf16_view(cache, block_table, seq_lens, num_seqs, max_seq_len, pl.partial_bytes, workspace, a, &v, st);
    if (*err != hipSuccess) return true;
    const size_t dec_at = (with_fp8_scratch(pl.partial_bytes, num_seqs, max_seq_len, a) + 255) / 256 * 256;
    const size_t rows = decode_mfma_rows_for(pl.dec_waves, num_dec, a);
    DecodeRole d;
    d.q = static_cast<const uint16_t*>(q) + static_cast<size_t>(total_q) * a.q_stride;
    d.cache = static_cast<uint16_t*>(cache);
    d.block_table = block_table + static_cast<size_t>(num_seqs) * a.max_blocks;
    d.seq_lens = seq_lens + num_seqs;
    d.o_part = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + dec_at);
    d.ml_part = d.o_part + rows * kD;
    d.plan = reinterpret_cast<int2*>(d.ml_part + rows * 2);
    d.max_blocks = a.max_blocks;
    d.num_seqs = num_dec;
    d.r_min = decode_mfma_r_min(max_dec_len);
    d.n_wg = pl.dec_wgs;
    d.c = a.scale * a.k_scale * kLog2e;
    const int n_splits = pl.wide ? pl.w.n_splits : pl.narrow.n_splits;
    float* o_part = static_cast<float*>(workspace);
    const float* ml_part = n_splits > 1 ? o_part + static_cast<size_t>(n_splits) * total_q * a.hq_l * kD : nullptr;
    if (pl.wide) {
        *err = launch_prefill64_and_decode(q, v.cache, v.block_table, v.max_blocks, cu_seqlens_q, seq_lens, num_seqs, total_q, pl.w, pl.range_div,
                                           d, out, workspace, a, d.c, a.v_scale, st);
    } else {
        PrefillParams p = narrow_params(q, v, cu_seqlens_q, seq_lens, num_seqs, total_q, pl.narrow, out, workspace, a);
        p.range_div = pl.range_div;
        const unsigned grid = static_cast<unsigned>(pl.dec_wgs) + static_cast<unsigned>(pl.narrow.pair_ranks) * n_splits * num_seqs * pl.narrow.head_slots;
        if (a.kv_fp8()) prefill_kernel<2><<<grid, kThreads, kLdsBytesBoth, st>>>(p, d);
        else prefill_kernel<1><<<grid, kThreads, kLdsBytesBoth, st>>>(p, d);
        *err = hipGetLastError();
    }
    if (*err != hipSuccess) return true;
    *err = launch_combine_both(o_part, ml_part, total_q, n_splits, out, d.o_part, d.ml_part, d.plan, num_dec,
                               static_cast<uint16_t*>(out) + static_cast<size_t>(total_q) * a.out_stride, a, st);
    return true;
}

}  // namespace shiftattn
