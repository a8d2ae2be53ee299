// The two projections that touch the exchange (Algorithm 1: qkv = embed * W_qkv in front of the first
// all-to-all, embed = attn_o * W_o behind the second), as one bf16 MFMA GEMM whose operand and result
// addressing carries the pack / unpack:
//   qkv_proj_pack : C[t][f] = sum_k x[t][k] W[f][k]; feature tile f lies in one head, and a head's
//                   columns go straight to the send buffer(s) of the rank(s) that own it (Sec. 3.2.1:
//                   fused q|k|v exchange, KV replication) - the pack kernel and its round trip
//                   through HBM disappear;
//   unpack_o_proj : C[t][c] = sum_k a[t][k] W_o[c][k] with a[t][(p hq_l + j) D + e] read in place from
//                   receive buffer p - the unpack kernel disappears.
// Weights are stored one row per output feature (K contiguous), as linear layers keep them.
//
// Kernel: an output tile per workgroup, four wavefronts (2 along the features x 2 along the tokens, one wavefront per SIMD
// with its accumulators in the AGPR half of the register file), the weight rows as A operand and the token rows as B
// operand, so a lane ends up with runs of four consecutive features of one token (8-byte stores).  Three tile shapes:
//   256 features x 256 token rows (128 x 128 per wavefront, 256 accumulator registers): the most flops per byte, for
//     batches of whole rounds of the chip; two k stages in LDS;
//   256 x 128: half the tile where 256 rows would leave compute units idle; three k stages;
//   128 x 128: few token rows, few features; four k stages - with two, a workgroup alone on its compute unit waits for
//     memory once per stage (65 rows x 10240 features x 8192 k unsplit: 0.80 us per stage with two, 0.33 with four).
// plan_gemm() chooses, with its figures.  k advances in stages of 128 bytes per row (64 bf16 or 128 FP8 elements: whole
// cache lines), the stage buffers filled by direct-to-LDS loads of 1 KiB (eight rows); a row keeps its eight
// 16-byte pieces at positions piece ^ ((row / 2) % 8), which makes the operand reads (16 or 32 consecutive rows, one
// piece column) conflict-free.  One barrier per stage.  bf16: v_mfma_f32_16x16x32_bf16; FP8: v_mfma_scale_f32_16x16x128_f8f6f4.
// What the main loop is built around (all measured on this kernel):
//   * the chip runs these kernels at its power limit: the clock settles where MFMA rate x energy per MFMA fits, so
//     the 16x16x32 form (less accumulator traffic per flop) sustains about 15 % more than 32x32x16;
//   * with one wavefront per SIMD and 16-clock MFMAs the matrix pipe stays fed only if at most one other instruction
//     sits between two MFMAs: every LDS read, every load (split in two: M0, then the load) and the scalar bookkeeping
//     has a slot of its own behind an MFMA;
//   * workgroups on different XCDs start their walk over k at different places (see rot0 below).
#include "internal.h"
#include "token_rows.h"

#include <math.h>

#include <type_traits>
#include <utility>

namespace shiftattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kTile = 256;                 // features (and for large batches token rows) per workgroup; N is a multiple of it
constexpr int kRowBytes = 128;             // bytes of a row per k stage: one cache line, 64 bf16 or 128 FP8 elements
constexpr int kWavesN = 2, kWavesM = 2;    // wavefronts along the features / along the tokens
constexpr int kGemmThreads = 64 * kWavesN * kWavesM;

// A workgroup's output tile: TN features x TM token rows, with ST k stages in LDS (one being multiplied, the others in
// flight), and what follows from it
template <int TN, int TM, int ST>
struct TileShape {
    static constexpr int kWaveN = TN / kWavesN, kWaveM = TM / kWavesM;   // rows of either operand that one wavefront multiplies
    static constexpr int kAT = kWaveN / 16, kBT = kWaveM / 16;           // ... in tiles of 16
    static constexpr int kMfmas = kAT * kBT;                             // MFMAs of one k step
    static constexpr int kReads = kAT + kBT;                             // operand tiles of one k step
    static constexpr int kRowsN = TN / 4, kRowsM = TM / 4;               // rows of either operand that one wavefront loads
    static constexpr int kLoadsN = kRowsN / 8, kLoadsM = kRowsM / 8;     // direct-to-LDS instructions: eight rows (1 KiB) each
    static constexpr int kLoads = kLoadsN + kLoadsM;                     // per wavefront and k stage
    static constexpr int kStage = (TN + TM) * kRowBytes;                 // weights, then tokens
    static constexpr int kStages = ST;
    static constexpr int kStagingPitch = 2 * kWaveN + 16;                // bytes between token rows of a wavefront's result staged in LDS
    static constexpr int kStagingWave = kWaveM * kStagingPitch;
    static constexpr int kLds = 4 * kStagingWave > kStages * kStage ? 4 * kStagingWave : kStages * kStage;
    static constexpr int kPerCu = kLds <= 80 * 1024 ? 2 : 1;             // workgroups per compute unit
};

// s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8
constexpr int wait_imm(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lgkm << 8); }
constexpr int kNoVm = 63, kNoLgkm = 15;
constexpr int kHeadDim = 128;

__device__ inline bf16x8 frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// The bf16 MFMA as assembly with its accumulator tied in place in an accumulation register: given the builtin, the
// register allocator rotated the 64 small accumulators of a wavefront through both register files (some 500 copies
// per k stage).  The compiler does not know this statement is an MFMA: its operands come straight from LDS reads
// (waited for by the compiler, which does track the registers), an accumulator is touched again 64 MFMAs later at the
// earliest, and compiler-generated reads of the results sit behind mfma_settle().
__device__ inline __attribute__((always_inline)) void mfma_16x16x32(f32x4& d, u32x4 a, u32x4 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
__device__ inline __attribute__((always_inline)) void mfma_settle() { asm volatile("s_nop 7\n\ts_nop 7" ::: "memory"); }

struct GemmParams {
    const unsigned char* __restrict__ w;   // [N][K], bf16 or FP8 E4M3 codes
    const unsigned char* __restrict__ x;   // token rows of the same type; see mode
    uint16_t* __restrict__ c;              // bf16
    const float* __restrict__ xs;          // FP8: one scale per token row
    const float* __restrict__ ws;          // FP8: one scale per output feature
    int M, M_out, N, K;               // M token rows exist, rows M..M_out-1 of the result are written as zeros
    // mode 0 (qkv_proj_pack): x dense [M][K]; result columns scattered to send buffers (XchgShape below)
    // mode 1 (unpack_o_proj): x gathered from recv [P][T_pad][hq_l][128] (k = (p hq_l + j) 128 + e); result dense [M][N]
    int mode;
    int k_splits;                     // workgroups that share an output tile, each with a range of k stages
    float* __restrict__ partial;      // k_splits > 1: fp32 partial results [k_splits][M_out - m_base][N] instead of c
    int items;                        // work items of the launch: output tiles x k ranges
    int m_base;                       // first token row of the launch's tiles (a multiple of the tile height)
    int m_tiles;                      // token tiles of the launch
    int group_rows;                   // order of the work items, see item_order()
    XchgShape s;
};

// kFp8: both operands are FP8 E4M3 codes (v_mfma_scale_f32_16x16x128_f8f6f4 with unit block scales, fp32
// accumulation); the result is multiplied by the token's and the feature's scale before it is rounded to bf16.
// kSplit: the workgroup covers one of p.k_splits ranges of k and leaves fp32 sums in p.partial (for FP8 operands: before
// the scales, which the finishing kernel applies).  One call is one output tile (and k range): work item `item` of the launch.
template <bool kFp8, bool kSplit, int TN, int TM, int ST>
__device__ __attribute__((always_inline)) void proj_gemm_tile(const GemmParams& p, const int item) {
    using S_ = TileShape<TN, TM, ST>;
    constexpr int kAT = S_::kAT, kBT = S_::kBT, kMfmas = S_::kMfmas, kReads = S_::kReads;
    constexpr int kLoadsN = S_::kLoadsN, kLoadsM = S_::kLoadsM, kLoads = S_::kLoads, kStage = S_::kStage, kStages = ST;
    constexpr int kTokenBytes = TN * kRowBytes;   // where a stage's token rows start
    constexpr int kElem = kFp8 ? 1 : 2;          // bytes per operand element
    constexpr int kBK = kRowBytes / kElem;       // k per stage
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // (an opaque copy of the thread index per work item, and another one for the epilogue below: as invariants of the
    // persistent loop, everything derived from it would be computed once and kept in registers through the main loop)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = tid >> 6, lane = tid & 63;
    const int wn = wave % kWavesN, wm = wave / kWavesN;
    // which output tile: see item_order()
    const int n_tiles = p.N / TN;
    const int n_splits = kSplit ? p.k_splits : 1;
    const int per_split = n_tiles * p.m_tiles;
    const int split = kSplit ? item / per_split : 0;
    const int tile_id = item - split * per_split;
    int n_idx, m_idx;
    if (!kSplit && p.group_rows == 0) {
        m_idx = tile_id / n_tiles;
        n_idx = tile_id - m_idx * n_tiles;
    } else {
        const int per_group = p.group_rows * n_tiles, group = tile_id / per_group, in_group = tile_id - group * per_group;
        const int rows = min(p.group_rows, p.m_tiles - group * p.group_rows);   // token tiles of this group
        n_idx = in_group / rows;
        m_idx = group * p.group_rows + in_group - n_idx * rows;
    }
    const int n0 = n_idx * TN, m0 = p.m_base + m_idx * TM;
    // this workgroup's k stages: [kt0, kt0 + k_steps) of all; with FP8 operands the very last stage may hold 64 k only
    const int kt_all = (p.K + kBK - 1) / kBK;
    const int kt0 = kSplit ? static_cast<int>(static_cast<int64_t>(kt_all) * split / n_splits) : 0;
    const int k_steps = kSplit ? static_cast<int>(static_cast<int64_t>(kt_all) * (split + 1) / n_splits) - kt0 : kt_all;
    const bool ragged = kFp8 && p.K % kBK != 0 && kt0 + k_steps == kt_all;

    // ---- direct-to-LDS loads: this wavefront fills a quarter of the rows of both operand tiles, eight rows of
    // 128 bytes (1 KiB, eight whole cache lines) per instruction; lane -> row 8 j + lane / 8, LDS piece position
    // lane % 8, logical piece = position ^ key.  (Half lines - 16 rows of 64 bytes per instruction - kept the address
    // path of the compute unit busy nine tenths of the time and every line was requested twice, one k tile apart.)
    // The address of a load is a wavefront-uniform base (tile origin + k, kept in scalar registers and advanced by
    // scalar adds) plus a 32-bit byte offset per lane that never changes, and the LDS destination is uniform too: no
    // vector ALU instruction is spent on a load.
    const int ld_row = lane >> 3, ld_pos = lane & 7;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const size_t k_bytes = static_cast<size_t>(p.K) * kElem;
    const size_t seg_bytes = p.mode == 0 ? k_bytes : static_cast<size_t>(p.s.hq_l) * kHeadDim * kElem;   // contiguous k of a token row
    uint32_t w_off[kLoadsN], x_off[kLoadsM];   // byte offsets of this lane's piece from the tile origin at k = 0
#pragma unroll
    for (int j = 0; j < kLoadsN; ++j) {
        const int row = S_::kRowsN * wave + 8 * j + ld_row;
        const int piece = ld_pos ^ ((row >> 1) & 7);
        w_off[j] = static_cast<uint32_t>(static_cast<size_t>(row) * k_bytes + piece * 16);
    }
#pragma unroll
    for (int j = 0; j < kLoadsM; ++j) {
        const int row = S_::kRowsM * wave + 8 * j + ld_row;
        const int piece = ld_pos ^ ((row >> 1) & 7);
        // (rows past the end re-read the last one; they are not stored)
        x_off[j] = static_cast<uint32_t>(static_cast<size_t>(tile_row(m0, row, p.M)) * seg_bytes + piece * 16);
    }
    // A half-filled last stage: the lanes of pieces 4..7 (past the end of the row) fetch pieces 0..3 once more.  The
    // key of row (32 or 64) wave + 8 j + lane / 8 has bit 2 equal to j % 2, so which lanes those are depends on j % 2 only.
    uint32_t tail_fix[2];
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) tail_fix[jp] = (((ld_pos >> 2) ^ jp) & 1) ? 64u : 0u;
    const unsigned char* w_tile = p.w + static_cast<size_t>(n0) * k_bytes;
    const unsigned char* x_tile = p.x + static_cast<size_t>(tile_origin(m0, p.M)) * seg_bytes;
    // A token row's k runs contiguously through the hq_l heads that one source rank returned, then jumps to the
    // next rank's buffer (mode 1); in mode 0 it is contiguous throughout.
    const int seg_tiles = max(static_cast<int>(seg_bytes / kRowBytes), 1);
    const size_t seg_jump = p.mode == 0 ? 0 : static_cast<size_t>(p.s.T_pad - 1) * seg_bytes;
    // The workgroups of a launch move through k in step, and rows lie a power of two apart: left alone, every compute
    // unit of the chip asks for the same few memory channels at the same time (measured: the address path stalled by the
    // cache twice as often, twice the bytes fetched into the L2s).  So the walk over k starts at a different place on
    // every XCD (workgroup i runs on XCD i % 8; the workgroups of one XCD stay together, they share operand panels
    // through its L2) and wraps around; a sum over k does not care where it starts.
    // With one token tile the workgroups of an XCD share no panels either, and start at places of their own.
    const int skew = p.m_tiles == 1 ? blockIdx.x / 8 % 32 : 0;
    const int rot0 = ragged ? 0 : static_cast<int>(((static_cast<int64_t>(blockIdx.x % 8) * k_steps) / 8 + skew) % k_steps);
    const unsigned char* const w_start = w_tile + static_cast<size_t>(kt0) * kRowBytes;
    const unsigned char* const x_start = x_tile + static_cast<size_t>(kt0) * kRowBytes + static_cast<size_t>(kt0 / seg_tiles) * seg_jump;
    const int left_start = seg_tiles - kt0 % seg_tiles;
    const int kt_first = kt0 + rot0;
    int ld_kt = 0, ld_left = seg_tiles - kt_first % seg_tiles;   // loads issued so far, and how many stages remain in the segment of the next one
    int wrap_left = k_steps - rot0;                              // stages until the walk is back at the start of its range
    w_tile += static_cast<size_t>(kt_first) * kRowBytes;
    x_tile += static_cast<size_t>(kt_first) * kRowBytes + static_cast<size_t>(kt_first / seg_tiles) * seg_jump;
    // 1 KiB from a wavefront-uniform base (scalar registers) + a 32-bit byte offset per lane into LDS at dst (uniform):
    // written as assembly so that the load forms the address itself instead of a 64-bit vector addition in front of it.
    // These loads are waited for with the explicit vmcnt waits below only.
    auto scalar_ptr = [](const unsigned char* ptr) -> const unsigned char* {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
        return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
    };
    auto dma_1k = [&](const unsigned char* base, uint32_t lane_off, unsigned char* dst) {
        const uint32_t m0v = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
        // (M0 is reserved by the compiler - it sets it right before each use of its own and keeps no value in it, and
        // rejects it on a clobber list - so writing it here needs no clobber.)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(m0v), "v"(lane_off), "s"(scalar_ptr(base)) : "memory");
    };
    auto load_one = [&](int j, bool tail) {          // first the token rows, then the weight rows
        unsigned char* dst = lds + (ld_kt % kStages) * kStage;
        const int jj = j < kLoadsM ? j : j - kLoadsM;
        const uint32_t fix = tail ? tail_fix[jj % 2] : 0u;
        if (j < kLoadsM) dma_1k(x_tile, x_off[jj] - fix, dst + kTokenBytes + (S_::kRowsM * wave_s) * kRowBytes + jj * 1024);
        else dma_1k(w_tile, w_off[jj] - fix, dst + (S_::kRowsN * wave_s) * kRowBytes + jj * 1024);
    };
    auto advance_x = [&]() {              // behind the last token-row load of a stage
        x_tile += kRowBytes;
        if (--ld_left == 0) {             // (a real branch, rarely taken: as selects this is a dozen scalar instructions)
            asm volatile("; next source buffer");
            ld_left = seg_tiles;
            x_tile += seg_jump;
        }
    };
    // LDS addresses of this wavefront's rows in the stage buffer that the next loads fill
    uint32_t ld_dst_w = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds + (S_::kRowsN * wave_s) * kRowBytes));
    uint32_t ld_dst_x = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds + kTokenBytes + (S_::kRowsM * wave_s) * kRowBytes));
    int ld_buf_left = kStages;            // buffers up to the last one, the next loads' included
    auto advance_w = [&]() {              // behind the last load of a stage
        ++ld_kt;
        w_tile += kRowBytes;
        if (--wrap_left == 0) {           // (rarely taken, a real branch)
            asm volatile("; back to the start of the k range");
            w_tile = w_start;
            x_tile = x_start;
            ld_left = left_start;
        }
        const bool last_buf = --ld_buf_left == 0;
        const uint32_t step = last_buf ? 0u - static_cast<uint32_t>((kStages - 1) * kStage) : static_cast<uint32_t>(kStage);
        ld_buf_left = last_buf ? kStages : ld_buf_left;
        ld_dst_w += step;
        ld_dst_x += step;
    };
    // The same load in two statements, for the loop of the 16-clock MFMAs, where the single wavefront of a SIMD keeps the
    // matrix pipe fed only if no more than one other instruction sits between two MFMAs: the LDS destination into M0
    // (one scalar addition; the MFMA behind it is the wait state the load needs), then, one MFMA later, the load.
    // Nothing else in this kernel writes M0 between the two (the compiler has no use of its own for it here).
    auto set_m0 = [&]<int j>() {
        constexpr int imm = (j < kLoadsM ? j : j - kLoadsM) * 1024;
        const uint32_t dst = j < kLoadsM ? ld_dst_x : ld_dst_w;
        asm volatile("s_add_u32 m0, %0, %1" :: "s"(dst), "n"(imm) : "scc");
    };
    auto issue_load = [&]<int j>(bool tail) {
        constexpr bool is_x = j < kLoadsM;
        constexpr int jj = is_x ? j : j - kLoadsM;
        const uint32_t* offs = is_x ? x_off : w_off;
        const uint32_t off = offs[jj] - (tail ? tail_fix[jj % 2] : 0u);
        const unsigned char* base = scalar_ptr(is_x ? x_tile : w_tile);
        asm volatile("global_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base) : "memory");
    };

    // ---- operand reads: tiles of 16 rows; this wavefront's weight rows and token rows in a stage buffer
    const int a_base = (wn * S_::kWaveN) * kRowBytes;
    const int b_base = kTokenBytes + (wm * S_::kWaveM) * kRowBytes;

    // accumulators: kAT x kBT tiles of 16 x 16 per wavefront (256 x 256 tile: 256 registers)
    f32x4 acc[kAT][kBT];
#pragma unroll
    for (int nt = 0; nt < kAT; ++nt)
#pragma unroll
        for (int mt = 0; mt < kBT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[nt][mt][r] = 0.f;

    // the first stages are requested (the last one of a short k with its half-row fix), stage 0 has landed everywhere
    auto prologue = [&]() {
        for (int t = 0; t < kStages && t < k_steps; ++t) {
            const bool tail = ragged && t == k_steps - 1;
#pragma unroll
            for (int j = 0; j < kLoads; ++j) load_one(j, tail);
            advance_x();
            advance_w();
        }
        if (k_steps >= kStages) __builtin_amdgcn_s_waitcnt(wait_imm((kStages - 1) * kLoads, kNoLgkm));
        else __builtin_amdgcn_s_waitcnt(wait_imm(0, kNoLgkm));
        asm volatile("s_barrier" ::: "memory");
    };
    // The stage loop.  kLoadMode 0: no loads (the last stages), 1: the loads of the stage that the buffer just left takes
    // next follow the meeting, 2: the same with the half-row fix (that stage is a half-filled last one).
    int rd_off = 0, rd_next = kStages > 1 ? kStage : 0;   // the buffers of stage st and of the next one
    auto next_buffer = [&]() {
        rd_off = rd_next;
        rd_next = rd_next == (kStages - 1) * kStage ? 0 : rd_next + kStage;
    };
    // this wavefront holds the rest of stage st in registers, and its loads of stage st + 1 have landed (younger ones stay
    // in flight; without kLoadMode fewer than the usual number are left behind it)
    auto meet = [&]<int kLoadMode>(int st) {
        if constexpr (kLoadMode > 0 || kStages == 2) {
            __builtin_amdgcn_s_waitcnt(wait_imm((kStages - 2) * kLoads, 0));
        } else {
            const int younger = k_steps - 2 - st;
            if (younger >= 2 && kStages >= 4) __builtin_amdgcn_s_waitcnt(wait_imm(2 * kLoads, 0));
            else if (younger == 1) __builtin_amdgcn_s_waitcnt(wait_imm(kLoads, 0));
            else __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
        }
        asm volatile("s_barrier" ::: "memory");
    };
    auto run_stages = [&](auto&& stage) {
        int st = 0;
        const int n_plain = k_steps - kStages - (ragged ? 1 : 0);
        for (; st < n_plain; ++st) stage.template operator()<1>(st);
        if constexpr (kFp8) {
            if (ragged && st + kStages < k_steps) {
                stage.template operator()<2>(st);
                ++st;
            }
        }
        for (; st < k_steps; ++st) stage.template operator()<0>(st);
    };

    // Operands are read from LDS one MFMA k step (a "slice": 32 bytes of every row for bf16, 64 for FP8) ahead of the
    // MFMAs that use them, into the other of two register sets, one read behind an MFMA, in the order in which the
    // MFMAs of the coming slice need them: the matrix pipe never waits behind a burst of reads (with one wavefront per
    // SIMD nothing else would feed it meanwhile).  The workgroup meets once per stage, in front of the stage's last
    // slice: by then a wavefront holds that slice in registers (it is done with the stage's buffer) and its loads of
    // the next stage have landed.  Behind the meeting the first slice of the next stage is read and the stage after
    // next is requested into the buffer just left, one load behind every MFMA.
    if constexpr (!kFp8) {
        // v_mfma_f32_16x16x32_bf16 (at the chip's power limit it sustains about 15 % more than the 32x32x16 form: it
        // reads and writes a quarter of the accumulator registers per MFMA for half the work).  A slice is 32 k, half
        // a stage: lane -> row lane % 16 of a 16-row tile, piece 4 slice + lane / 16 of its 128-byte row; kAT x kBT
        // MFMAs per slice.
        const int r16 = lane & 15, kg = lane >> 4;
        int rd[2];
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) rd[sl] = r16 * kRowBytes + (((4 * sl + kg) ^ ((r16 >> 1) & 7)) << 4);
        u32x4 a[2][kAT], b[2][kBT];   // [set]
        // read r of a slice into set S, in the order of first use by MFMA (i, j) = (I / kBT, I % kBT): a[0], b[0 ..], a[1 ..]
        auto read_one = [&]<int r, int S>(const unsigned char* base, int sl) {
            if constexpr (r == 0) a[S][0] = *reinterpret_cast<const u32x4*>(base + a_base + rd[sl]);
            else if constexpr (r <= kBT) b[S][r - 1] = *reinterpret_cast<const u32x4*>(base + b_base + (r - 1) * 16 * kRowBytes + rd[sl]);
            else a[S][r - kBT] = *reinterpret_cast<const u32x4*>(base + a_base + (r - kBT) * 16 * kRowBytes + rd[sl]);
        };
        // the MFMAs of one slice on set S; the reads of (rd_base, rd_sl) into the other set spread behind them (kDense:
        // over the first three quarters, so that they are back before the slice ends); kLoadMode > 0: the loads of the
        // stage after next, M0 and the load behind MFMAs of their own
        auto slice = [&]<int S, bool kDense, int kLoadMode>(const unsigned char* rd_base, int rd_sl) {
            [&]<int... I>(std::integer_sequence<int, I...>) {
                (([&]() {
                     constexpr int i = I / kBT, j = I % kBT;
                     mfma_16x16x32(acc[i][j], a[S][i], b[S][j]);
                     // read r goes behind MFMA r * span / kReads, load l behind l * kMfmas / kLoads + kLoadSkew (M0) and the next
                     constexpr int kSpan = kDense ? 3 * kMfmas / 4 : kMfmas;
                     constexpr int r = (I * kReads + kSpan - 1) / kSpan;
                     if constexpr (r < kReads && r * kSpan / kReads == I) read_one.template operator()<r, 1 - S>(rd_base, rd_sl);
                     if constexpr (kLoadMode > 0) {
                         constexpr int kLoadSkew = kMfmas / kLoads >= 4 ? 1 : 0;
                         constexpr auto m0_at = [](int l) { return l * kMfmas / kLoads + kLoadSkew; };
                         constexpr int l = I < kLoadSkew ? kLoads : ((I - kLoadSkew) * kLoads + kMfmas - 1) / kMfmas;   // the load whose M0 may be here
                         constexpr int l1 = I < kLoadSkew + 1 ? kLoads : ((I - 1 - kLoadSkew) * kLoads + kMfmas - 1) / kMfmas;
                         if constexpr (l1 < kLoads && m0_at(l1) + 1 == I) issue_load.template operator()<l1>(kLoadMode == 2);
                         if constexpr (l < kLoads && m0_at(l) == I) set_m0.template operator()<l>();
                         if constexpr (I == m0_at(kLoadsM - 1) + 2) advance_x();   // (scalar work)
                         if constexpr (I == kMfmas - 1) advance_w();
                     }
                     __builtin_amdgcn_sched_barrier(0);
                 }()),
                 ...);
            }(std::make_integer_sequence<int, kMfmas>{});
        };
        prologue();
        [&]<int... R>(std::integer_sequence<int, R...>) {
            (read_one.template operator()<R, 0>(lds, 0), ...);
        }(std::make_integer_sequence<int, kReads>{});
        auto stage = [&]<int kLoadMode>(int st) {
            // (where two copies of this body meet, the compiler moves accumulators between registers; the wait states
            // an MFMA needs behind such a move are put here, since it cannot know that one follows)
            asm volatile("s_nop 4" ::: "memory");
            slice.template operator()<0, true, 0>(lds + rd_off, 1);
            meet.template operator()<kLoadMode>(st);
            // (behind the last stage: stale data, not used)
            slice.template operator()<1, false, kLoadMode>(lds + rd_next, 0);
            next_buffer();
        };
        run_stages(stage);
        mfma_settle();
    } else {
        // v_mfma_scale_f32_16x16x128_f8f6f4 with unit block scales: a stage (128 bytes of a row) is one MFMA k step,
        // 64 MFMAs of 32 clocks; lane -> row lane % 16 of a 16-row tile, pieces lane / 16 and 4 + lane / 16 of its row (which
        // k a lane holds does not matter as long as both operands agree; with pieces 2 (lane / 16) and the next one, every read met
        // two lanes of the sixteen that LDS serves at a time on the same banks).  Registers hold the eight token
        // tiles of the stage (b, 64 registers) and eight weight tiles (a, 64): rows i = 0..3 of the MFMA grid fetch
        // weight tiles 4..7 of the stage, the workgroup meets in front of row 4 (all of the stage's operands are in
        // registers or on their way, the next stage has landed), rows 4..7 fetch weight tiles 0..3 of the next stage and
        // request the stage after next, and token tile j of the next stage is fetched right behind MFMA (7, j), the
        // last one that uses its registers, eight MFMAs ahead of the first one that needs it.
        const int r16 = lane & 15, kg = lane >> 4;
        int rd[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) rd[h] = r16 * kRowBytes + (((4 * h + kg) ^ ((r16 >> 1) & 7)) << 4);
        i32x8 a[kAT], b[kBT];
        int unit_scale;   // E8M0 code of 1.0, in a vector register as the instruction wants it
        asm volatile("v_mov_b32 %0, 127" : "=v"(unit_scale));
        auto join = [](u32x4 lo, u32x4 hi) -> i32x8 {
            return i32x8{static_cast<int>(lo[0]), static_cast<int>(lo[1]), static_cast<int>(lo[2]), static_cast<int>(lo[3]),
                         static_cast<int>(hi[0]), static_cast<int>(hi[1]), static_cast<int>(hi[2]), static_cast<int>(hi[3])};
        };
        auto read_a = [&]<int i>(const unsigned char* base) {
            const unsigned char* row = base + a_base + i * 16 * kRowBytes;
            a[i] = join(*reinterpret_cast<const u32x4*>(row + rd[0]), *reinterpret_cast<const u32x4*>(row + rd[1]));
        };
        auto read_b = [&]<int j>(const unsigned char* base) {
            const unsigned char* row = base + b_base + j * 16 * kRowBytes;
            b[j] = join(*reinterpret_cast<const u32x4*>(row + rd[0]), *reinterpret_cast<const u32x4*>(row + rd[1]));
        };
        // (assembly with the accumulator tied in place, as for bf16 above)
        auto mfma = [&](f32x4& d, const i32x8& av, const i32x8& bv) {
            asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %3 op_sel_hi:[0,0,0]"
                         : "+a"(d) : "v"(av), "v"(bv), "v"(unit_scale));
        };
        prologue();
        [&]<int... R>(std::integer_sequence<int, R...>) {
            (read_b.template operator()<R>(lds), ...);
        }(std::make_integer_sequence<int, kBT>{});
        [&]<int... R>(std::integer_sequence<int, R...>) {
            (read_a.template operator()<R>(lds), ...);
        }(std::make_integer_sequence<int, kAT / 2>{});
        auto stage = [&]<int kLoadMode>(int st) {
            const unsigned char* cur = lds + rd_off;
            const unsigned char* nxt = lds + rd_next;
            next_buffer();
            asm volatile("s_nop 4" ::: "memory");   // (accumulator moves between two copies of this body, see above)
            if (kLoadMode == 0 && ragged && st == k_steps - 1) {
                // a half-filled last stage: the upper 64 bytes of its rows repeat the lower ones (see the loads); the
                // second pieces, which lie there, are multiplied by zero
#pragma unroll
                for (int j = 0; j < kBT; ++j)
#pragma unroll
                    for (int e = 4; e < 8; ++e) b[j][e] = 0;
                asm volatile("s_nop 4" ::: "memory");
            }
            [&]<int... I>(std::integer_sequence<int, I...>) {
                (([&]() {
                     constexpr int i = I / kBT, j = I % kBT;
                     if constexpr (I == kMfmas / 2) meet.template operator()<kLoadMode>(st);
                     mfma(acc[i][j], a[i], b[j]);
                     if constexpr (i < kAT / 2 && j == 0) read_a.template operator()<i + kAT / 2>(cur);
                     if constexpr (i >= kAT / 2 && j == 1) read_a.template operator()<i - kAT / 2>(nxt);   // (behind the last stage: stale, unused)
                     if constexpr (i == kAT - 1) read_b.template operator()<j>(nxt);
                     if constexpr (kLoadMode > 0 && i >= kAT / 2) {   // the loads, behind the meeting: M0, then the load
                         // step q (M0 of load q / 2, or the load) goes into slot q * slots / steps of the kMfmas / 2 slots
                         constexpr int slot = I - kMfmas / 2, kSlots = kMfmas / 2, kSteps = 2 * kLoads;
                         constexpr int q0 = (slot * kSteps + kSlots - 1) / kSlots, q1 = ((slot + 1) * kSteps + kSlots - 1) / kSlots;
                         [&]<int... Q>(std::integer_sequence<int, Q...>) {
                             (([&]() {
                                  constexpr int q = q0 + Q;
                                  if constexpr (q % 2 == 0) {
                                      set_m0.template operator()<q / 2>();
                                  } else {
                                      if constexpr (Q > 0) asm volatile("s_nop 0");   // no MFMA between M0 and its load
                                      issue_load.template operator()<q / 2>(kLoadMode == 2);
                                      if constexpr (q / 2 == kLoadsM - 1) advance_x();
                                      if constexpr (q / 2 == kLoads - 1) advance_w();
                                  }
                              }()),
                              ...);
                         }(std::make_integer_sequence<int, q1 - q0>{});
                     }
                     __builtin_amdgcn_sched_barrier(0);
                 }()),
                 ...);
            }(std::make_integer_sequence<int, kMfmas>{});
        };
        run_stages(stage);
        mfma_settle();
    }

    // ---- result.  A lane holds runs of four consecutive features of one token: acc[i][j] is features
    // 16 i + 4 (lane / 16) .. + 3 of token 16 j + lane % 16.
    int tid_e = threadIdx.x;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63;
    constexpr int kTokStep = 16;
    constexpr int kQuads = kAT;
    const int tok_lane = lane_e & 15;
    auto quad_feature = [&](int q) { return 16 * q + 4 * (lane_e >> 4); };
    auto quad_value = [&](int q, int t, int e) -> float { return acc[q][t][e]; };
    const int f_wave = n0 + wn * S_::kWaveN;     // first feature of this wavefront; its features lie in one head
    // The bf16 result goes through LDS (the stage buffers are free by now): a wavefront lays its 128 tokens x 128
    // features down as rows of 256 bytes (pitch 272: the 8-byte writes of 16 token rows then spread over all banks),
    // reads them back 16 bytes per lane and stores whole rows - 256 contiguous bytes per token instead of the 8-byte
    // pieces the accumulator layout would give (those cost 4 % of the kernel).  A wavefront reads only what it wrote
    // itself, so the workgroup does not meet; what other wavefronts may still be reading there is discarded anyway
    // (the last stage's look-ahead reads).
    unsigned char* stg = lds + wave * S_::kStagingWave;
    auto stage_result = [&]() {
#pragma unroll
        for (int t = 0; t < kBT; ++t) {
            const int tok = t * kTokStep + tok_lane;
            const int m = m0 + wm * S_::kWaveM + tok;
            float row_scale = 1.f;
            if constexpr (kFp8) row_scale = m < p.M ? p.xs[m] : 0.f;
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const int f = quad_feature(q);
                f32x4 col_scale = {1.f, 1.f, 1.f, 1.f};
                if constexpr (kFp8) col_scale = *reinterpret_cast<const f32x4*>(p.ws + f_wave + f);
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y = m < p.M ? quad_value(q, t, e) : 0.f;   // rows M .. M_out - 1 of the result are zeros
                    if constexpr (kFp8) y = y * row_scale * col_scale[e];
                    v[e] = static_cast<__bf16>(y);
                }
                *reinterpret_cast<u32x2*>(stg + tok * S_::kStagingPitch + f * 2) = __builtin_bit_cast(u32x2, v);
            }
        }
    };
    auto store_rows = [&](uint16_t* dst_row0, size_t row_stride) {   // dst_row0: feature f_wave of token row 0
        constexpr int kLanes = S_::kWaveN / 8, kRowsAtOnce = 64 / kLanes;   // lanes per row of the wavefront's features
#pragma unroll 8
        for (int r = 0; r < S_::kWaveM / kRowsAtOnce; ++r) {
            const int tok = kRowsAtOnce * r + lane_e / kLanes;
            const int m = m0 + wm * S_::kWaveM + tok;
            if (m >= p.M_out) continue;
            const u32x4 v = *reinterpret_cast<const u32x4*>(stg + tok * S_::kStagingPitch + (lane_e % kLanes) * 16);
            *reinterpret_cast<u32x4*>(dst_row0 + static_cast<size_t>(m) * row_stride + (lane_e % kLanes) * 8) = v;
        }
    };
    if constexpr (kSplit) {   // this k range's fp32 sums, [split][token][feature]; proj_finish adds the ranges and does the layout
        float* base = p.partial + static_cast<size_t>(split) * (p.M_out - p.m_base) * p.N + f_wave;   // [split][row - m_base][feature]
#pragma unroll
        for (int t = 0; t < kBT; ++t) {
            const int m = m0 + wm * S_::kWaveM + t * kTokStep + tok_lane;
            if (m >= p.M) continue;   // rows past the last token are zeros in the result and are not read
            float* row = base + static_cast<size_t>(m - p.m_base) * p.N;
#pragma unroll
            for (int q = 0; q < kQuads; ++q)
                *reinterpret_cast<f32x4*>(row + quad_feature(q)) =
                    f32x4{quad_value(q, t, 0), quad_value(q, t, 1), quad_value(q, t, 2), quad_value(q, t, 3)};
        }
        return;
    }
    stage_result();
    if (p.mode == 1) {
        store_rows(p.c + f_wave, static_cast<size_t>(p.N));
        return;
    }
    // send buffers [P][T_pad][hq_l + 2 hkv_l][128]: which buffer(s) own this head (wavefront-uniform)
    const XchgShape& s = p.s;
    const int head = f_wave / kHeadDim, col = f_wave % kHeadDim;
    const int w_out = s.hq_l + 2 * s.hkv_l;
    const size_t row_stride = static_cast<size_t>(w_out) * kHeadDim;
    const size_t buf_stride = static_cast<size_t>(s.T_pad) * row_stride;
    if (head < s.h) {
        const int dest = head / s.hq_l, local = head - dest * s.hq_l;
        store_rows(p.c + dest * buf_stride + local * kHeadDim + col, row_stride);
    } else {
        const bool is_v = head >= s.h + s.h_kv;
        const int g = head - s.h - (is_v ? s.h_kv : 0);   // K or V head on the source side
        const int slot0 = s.hq_l + (is_v ? s.hkv_l : 0);
        if (s.h_kv >= s.P) {   // each destination owns hkv_l consecutive heads
            const int dest = g / s.hkv_l, local = slot0 + (g - dest * s.hkv_l);
            store_rows(p.c + dest * buf_stride + local * kHeadDim + col, row_stride);
        } else {               // replication: head g goes to the P / h_kv destinations whose first KV head it is
            for (int dest = 0; dest < s.P; ++dest)
                if (static_cast<int>((static_cast<int64_t>(dest) * s.h_kv) / s.P) == g)
                    store_rows(p.c + dest * buf_stride + slot0 * kHeadDim + col, row_stride);
        }
    }
}

// The grid is persistent: as many workgroups as the chip holds walk the launch's work items (output tile, k range) in
// rounds, so a compute unit goes from one tile to the next without waiting to be scheduled (ten rounds of tiles at the
// 70B shape).  Workgroup b runs on XCD b % 8, see item_order() for which item of a round it takes.
template <bool kFp8, bool kSplit, int TN, int TM, int ST>
__global__ __launch_bounds__(kGemmThreads, (TileShape<TN, TM, ST>::kPerCu)) void proj_gemm_kernel(GemmParams p) {
    const int xcd = blockIdx.x % 8, in_xcd = blockIdx.x / 8;
    for (int base = 0; base + static_cast<int>(blockIdx.x) < p.items; base += gridDim.x) {
        const int count = min(static_cast<int>(gridDim.x), p.items - base);   // items of this round
        const int item = !kSplit && p.group_rows == 0 ? static_cast<int>(blockIdx.x) : xcd * (count / 8) + min(xcd, count % 8) + in_xcd;
        proj_gemm_tile<kFp8, kSplit, TN, TM, ST>(p, base + item);
        // the next item's loads go where other wavefronts may still be reading their staged result rows
        __builtin_amdgcn_s_waitcnt(wait_imm(kNoVm, 0));
        asm volatile("s_barrier" ::: "memory");
    }
}

// In which order a launch's work items are dealt to the XCDs, so that the 32 compute units of one share operand panels
// through its L2.  0: item i of a round goes to XCD i % 8 with the feature tiles fastest, so that an XCD keeps the same
// n_tiles / 8 feature panels from the first round to the last: launches of several rounds (16384 rows of the 70B shape:
// both projections 3255 us against 3277 in groups).  Otherwise token tiles in groups of up to `most`, and an XCD takes a
// stretch of consecutive items of one k range: the panels of a group's token rows x a few feature panels (1280 features x
// 8192 k, 512 rows in five k ranges: 31.8 us dealt out singly, 25 in stretches; groups of 2 or 16 tiles at 16384 rows: 5 %
// slower than 6).  Where the line lies, both projections of 64 + 16 heads x 8192 / x 5120 in bf16, order 0 against groups: 16384
// rows 3261 / 2117 us against 3324 / 2118, 8192 rows 1651 / 1125 against 1685 / 1143.  Below 1024 tiles the gain is not certain:
// 2048 to 6000 rows of three models, order 0 is 0.8 % slower to 1.6 % faster.
inline int item_order(int n_tiles, int m_tiles, int k_splits, int most) {
    if (k_splits == 1 && n_tiles % 8 == 0 && n_tiles >= 24 && n_tiles * m_tiles >= 1024) return 0;
    const int groups = (m_tiles + most - 1) / most;
    return (m_tiles + groups - 1) / groups;
}

template <bool kFp8, int TN, int TM, int ST>
hipError_t launch(const GemmParams& p, hipStream_t st) {
    using S = TileShape<TN, TM, ST>;
    const int64_t items = static_cast<int64_t>(p.N / TN) * p.m_tiles * p.k_splits;
    if (items == 0) return hipSuccess;
    if (items > 0x7FFFFFFF) return hipErrorInvalidValue;
    GemmParams q = p;
    q.items = static_cast<int>(items);
    q.group_rows = item_order(p.N / TN, p.m_tiles, p.k_splits, TM == TN ? 6 : 8);
    int cus = 0, device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    const int slots = cus * S::kPerCu;
    const unsigned grid = static_cast<unsigned>(items < slots ? items : slots);
    if (p.k_splits > 1) proj_gemm_kernel<kFp8, true, TN, TM, ST><<<grid, kGemmThreads, S::kLds, st>>>(q);
    else proj_gemm_kernel<kFp8, false, TN, TM, ST><<<grid, kGemmThreads, S::kLds, st>>>(q);
    return hipGetLastError();
}

enum TileKind { kTile256x256, kTile256x128, kTile128x128, kTileKinds };   // features x token rows
constexpr int kTileFeatures[kTileKinds] = {256, 256, 128}, kTileTokens[kTileKinds] = {256, 128, 128};

// How a product is laid over the 256 compute units: `lead_tiles` token tiles of `lead` shape are done whole (as many as
// fill rounds of the chip), the token rows behind them in tiles of `tail` shape, with k in `splits` ranges whose fp32 sums
// go to the caller's workspace and are added by the finishing kernel (splits == 1: whole as well, no workspace).
struct GemmPlan {
    TileKind lead, tail;
    int lead_tiles, splits;
    double us;   // the model's time
};

// The model that chooses: microseconds of one launch, fitted to 2000 timed launches (65 .. 4096 token rows, the nine
// feature / k sizes of the served models' projections, all tile shapes and k ranges; a workgroup's walk over k at a given
// share of the chip in use is what differs between the shapes).  The choice it makes is 0.7 % slower on average than the
// best of them, 19 % at worst; against the 256 x 256 tile alone it is 1.0x at 2048 and more rows of the 70B shape, 1.35x
// at 701 rows over FP8 operands and up to 2x where features or k are few.
struct TileCost {
    double launch, tile, stage, stage_full;      // launch; per tile; per k stage on an idle chip and what a full chip adds
    double finish, partial_tbs, weight_tbs;      // finishing kernel; partial results (TB/s); weights at most at this rate
};
constexpr TileCost kTileCost[2][kTileKinds] = {
    {{1.0, 8.5, 1.05, 0.22, 0.5, 6.1, 5.1}, {2.0, 4.7, 0.566, 0.20, 2.7, 5.8, 6.0}, {2.9, 2.9, 0.317, 0.124, 2.1, 3.9, 6.2}},
    {{1.0, 9.6, 1.17, 0.09, 0.5, 6.2, 8.0}, {3.5, 5.0, 0.560, 0.18, 1.5, 5.6, 8.0}, {3.1, 3.6, 0.374, 0.082, 1.3, 3.8, 8.0}}};

double launch_us(TileKind kind, int64_t m_tiles, int rows, int N, int K, int splits, bool fp8) {
    const TileCost& c = kTileCost[fp8][kind];
    const int elem = fp8 ? 1 : 2;
    const int64_t items = m_tiles * (N / kTileFeatures[kind]) * splits;
    const double rounds = static_cast<double>((items + 255) / 256), full = items / (256.0 * rounds);
    const int stages = ((static_cast<int64_t>(K) * elem + kRowBytes - 1) / kRowBytes + splits - 1) / splits;
    const double walk = rounds * (c.tile + stages * (c.stage + c.stage_full * full));
    const double weights = static_cast<double>(N) * K * elem / (c.weight_tbs * 1e6);
    const double w2 = walk * walk, b2 = weights * weights;
    const double loop = sqrt(sqrt(w2 * w2 + b2 * b2));   // the longer of the two, rounded off where they are alike
    return c.launch + loop + (splits > 1 ? c.finish + splits * (8.0 * rows * N) / (c.partial_tbs * 1e6) : 0.0);
}

size_t split_bytes(int splits, int64_t rows, int N) { return splits > 1 ? static_cast<size_t>(splits) * rows * N * sizeof(float) : 0; }

GemmPlan plan_gemm(int M_out, int N, int K, bool fp8, size_t workspace_bytes) {
    GemmPlan best = {kTile256x256, kTile256x256, 0, 1, 1e30};
    if (M_out < 1 || N < kTile) return best;
    const int stages = (K * (fp8 ? 1 : 2) + kRowBytes - 1) / kRowBytes;
    // the tail: `rows` token rows, in tiles and k ranges that keep to one round of the chip (more rounds: whole)
    auto with_tail = [&](TileKind lead, int lead_tiles, double lead_us) {
        const int rows = M_out - lead_tiles * kTileTokens[lead];
        for (int kind = 0; kind < kTileKinds; ++kind) {
            const TileKind tail = static_cast<TileKind>(kind);
            const int64_t m_tiles = (rows + kTileTokens[tail] - 1) / kTileTokens[tail], tiles = m_tiles * (N / kTileFeatures[tail]);
            for (int sp = 1; sp <= 16 && (sp == 1 || (tiles * sp <= 256 && stages / sp >= 4)); ++sp) {
                if (split_bytes(sp, rows, N) > workspace_bytes) break;
                const double us = lead_us + launch_us(tail, m_tiles, rows, N, K, sp, fp8);
                if (us < best.us) best = {lead, tail, lead_tiles, sp, us};
            }
        }
    };
    with_tail(kTile256x256, 0, 0.0);
    for (int kind = 0; kind < kTileKinds; ++kind) {   // whole rounds of the chip first (the last full one may go to the tail too)
        const TileKind lead = static_cast<TileKind>(kind);
        const int n_tiles = N / kTileFeatures[lead];
        const int full_rounds = static_cast<int>(static_cast<int64_t>(M_out / kTileTokens[lead]) * n_tiles / 256);
        for (int r = full_rounds; r > 0 && r >= full_rounds - 1; --r) {
            const int lead_tiles = r * 256 / n_tiles;
            if (lead_tiles == 0 || lead_tiles * kTileTokens[lead] >= M_out) continue;
            with_tail(lead, lead_tiles, launch_us(lead, lead_tiles, lead_tiles * kTileTokens[lead], N, K, 1, fp8));
        }
    }
    return best;
}

template <bool kFp8>
hipError_t launch_kind(TileKind kind, const GemmParams& p, hipStream_t st) {
    switch (kind) {
        case kTile256x256: return launch<kFp8, 256, 256, 2>(p, st);
        case kTile256x128: return launch<kFp8, 256, 128, 3>(p, st);
        default: return launch<kFp8, 128, 128, 4>(p, st);
    }
}

template <bool kFp8, int TN, int TM, int ST>
hipError_t init_tile() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&proj_gemm_kernel<kFp8, false, TN, TM, ST>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, TileShape<TN, TM, ST>::kLds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&proj_gemm_kernel<kFp8, true, TN, TM, ST>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, TileShape<TN, TM, ST>::kLds);
}

}  // namespace

// bf16, head_dim 128; the feature dimension of either product must be a multiple of the 256-wide tile
template <int TN, int TM, int ST>
hipError_t init_shape() {
    const hipError_t e = init_tile<false, TN, TM, ST>();
    return e == hipSuccess ? init_tile<true, TN, TM, ST>() : e;
}

hipError_t proj_gemm_init() {
    hipError_t e = init_shape<256, 256, 2>();
    if (e == hipSuccess) e = init_shape<256, 128, 3>();
    if (e == hipSuccess) e = init_shape<128, 128, 4>();
    return e;
}

bool qkv_proj_pack_supported(const XchgShape& s, int d_model, int elem) {
    return elem == 2 && s.vec_per_head * 8 == kHeadDim && d_model > 0 && d_model % 64 == 0 && (s.h + 2 * s.h_kv) % 2 == 0;
}
bool unpack_o_proj_supported(const XchgShape& s, int d_model, int elem) {
    return elem == 2 && s.vec_per_head * 8 == kHeadDim && d_model > 0 && d_model % kTile == 0 && s.h > 0;
}

// The workspace that the size query names for a product of this size: the partial results of 256 x 256 tiles with k in as many
// ranges as a rougher model of the launch takes.  Callers allocate by these sizes once and tests pin them, so they are part of
// the interface; plan_gemm() uses what fits.  What that costs against a workspace without limit, by plan_gemm()'s model over
// 529 products that this kernel takes (9 .. 8192 rows, twelve feature / k sizes, both types): 0.2 % on average, more than
// 2 % in 16 of them, 15 % at worst (64 rows x 8192 features x 8192 k over FP8 operands).
size_t proj_gemm_workspace(int M_out, int N, int K, bool fp8) {
    const int n_tiles = N / kTile, m_tiles = (M_out + kTile - 1) / kTile;
    if (n_tiles == 0 || m_tiles == 0) return 0;
    const double walk = 2.0 * kTile * kTile * static_cast<double>(K) / (fp8 ? 12.5e12 : 6.5e12);   // one workgroup over all of k
    auto rounds = [](int64_t items) { return static_cast<double>((items + 255) / 256); };
    const int by_length = K / (fp8 ? 64 : 32) / 16;
    const double t_whole = rounds(static_cast<int64_t>(n_tiles) * m_tiles) * walk;
    double t_best = t_whole;
    size_t bytes = 0;
    for (int ma = 0; ma < m_tiles; ++ma) {
        const int64_t tiles_b = static_cast<int64_t>(n_tiles) * (m_tiles - ma);
        const double rows_b = static_cast<double>(M_out - ma * kTile);
        const double partial = 2.0 * rows_b * N * sizeof(float) / 3.2e12;   // written once, read once
        const double t_a = ma > 0 ? rounds(static_cast<int64_t>(n_tiles) * ma) * walk + 3.0e-6 : 0.0;
        for (int sp = 2; sp <= 16 && sp <= by_length; ++sp) {
            const double t = t_a + rounds(tiles_b * sp) / sp * walk + sp * partial + 5.0e-6;
            if (t < t_best && t < 0.97 * t_whole) {
                t_best = t;
                bytes = split_bytes(sp, M_out - ma * kTile, N);
            }
        }
    }
    return bytes;
}

void proj_gemm_describe(int M_out, int N, int K, bool fp8, size_t workspace_bytes, shiftattn_proj_plan_t* plan) {
    const GemmPlan pl = plan_gemm(M_out, N, K, fp8, workspace_bytes);
    *plan = shiftattn_proj_plan_t{0, pl.splits, 0, 0, pl.lead_tiles, kTileFeatures[pl.lead], kTileTokens[pl.lead],
                                  kTileFeatures[pl.tail], kTileTokens[pl.tail]};
}

double proj_gemm_us(int M_out, int N, int K, bool fp8, size_t workspace_bytes) { return plan_gemm(M_out, N, K, fp8, workspace_bytes).us; }

// runs the product in the best way for which the workspace has room
static hipError_t run_gemm(GemmParams& p, void* workspace, size_t workspace_bytes, hipStream_t st) {
    const bool fp8 = p.xs != nullptr;
    const GemmPlan pl = plan_gemm(p.M_out, p.N, p.K, fp8, workspace ? workspace_bytes : 0);
    p.partial = nullptr;
    p.k_splits = 1;
    if (pl.lead_tiles > 0) {
        p.m_base = 0;
        p.m_tiles = pl.lead_tiles;
        const hipError_t e = fp8 ? launch_kind<true>(pl.lead, p, st) : launch_kind<false>(pl.lead, p, st);
        if (e != hipSuccess) return e;
    }
    p.m_base = pl.lead_tiles * kTileTokens[pl.lead];
    p.m_tiles = (p.M_out - p.m_base + kTileTokens[pl.tail] - 1) / kTileTokens[pl.tail];
    p.k_splits = pl.splits;
    if (pl.splits > 1) p.partial = static_cast<float*>(workspace);
    const hipError_t e = fp8 ? launch_kind<true>(pl.tail, p, st) : launch_kind<false>(pl.tail, p, st);
    if (e != hipSuccess || pl.splits == 1) return e;
    return launch_proj_finish(p.partial, p.k_splits, p.M_out - p.m_base, p.c, p.M, p.M_out, p.N, p.mode, p.s, p.xs, p.ws, st,
                              p.m_base);
}

hipError_t launch_qkv_proj_pack(const void* x, const void* w_qkv, void* send, int d_model, const XchgShape& s,
                                const float* x_scales, const float* w_scales, void* workspace, size_t workspace_bytes,
                                hipStream_t st) {
    GemmParams p;
    p.w = static_cast<const unsigned char*>(w_qkv);
    p.x = static_cast<const unsigned char*>(x);
    p.c = static_cast<uint16_t*>(send);
    p.xs = x_scales;
    p.ws = w_scales;
    p.M = s.T;
    p.M_out = s.T_pad;
    p.N = (s.h + 2 * s.h_kv) * kHeadDim;
    p.K = d_model;
    p.mode = 0;
    p.s = s;
    if (s.T == 0) return launch_pack(nullptr, send, s, st);  // only padding rows: the pack kernel writes the zeros
    return run_gemm(p, workspace, workspace_bytes, st);
}

hipError_t launch_unpack_o_proj(const void* recv, const void* w_o, void* out, int d_model, const XchgShape& s,
                                const float* a_scales, const float* w_scales, void* workspace, size_t workspace_bytes,
                                hipStream_t st) {
    GemmParams p;
    p.w = static_cast<const unsigned char*>(w_o);
    p.x = static_cast<const unsigned char*>(recv);
    p.c = static_cast<uint16_t*>(out);
    p.xs = a_scales;
    p.ws = w_scales;
    p.M = s.T;
    p.M_out = s.T;
    p.N = d_model;
    p.K = s.h * kHeadDim;
    p.mode = 1;
    p.s = s;
    if (s.T == 0) return hipSuccess;
    return run_gemm(p, workspace, workspace_bytes, st);
}

}  // namespace shiftattn
