// The two projections next to the exchange (Algorithm 1: qkv = embed * W_qkv, embed = attn_o * W_o) for the few
// tokens of a decode step (Algorithm 2, the small-batch side of the threshold).  With few token rows the product
// is bound by reading the weight matrix once from HBM, not by the matrix cores, so the kernel is organised around
// that stream:
//
//   * 256 workgroups, one per compute unit, each owning a contiguous block of output features (N / 256 rows, so every
//     compute unit reads the same number of weight bytes; more than 40 features each: several rounds);
//   * the eight wavefronts of a workgroup (four where a step is large) split k.  A wavefront multiplies all features of the
//     block in one walk over its slice: per step of 128 bytes of k (64 bf16 or 128 FP8 elements) it fetches UX pieces of
//     eight token rows and UW pieces of eight weight rows, and holds the sums of all (token, feature) pairs in registers (at
//     most 24 up to 32 rows, 48 up to 64, 72 up to 96, 64 up to 128).  The token rows arrive with the weights they meet, so there is no limit on k;
//   * few features with long rows leave compute units idle or one long walk to each: there k is cut into 2, 4 or 8 ranges, each a
//     workgroup of its own, if the caller's workspace has room for their fp32 sums, and a small second kernel (4 to 5 us with its
//     launch, or 2 where the sums are few) adds them in range order;
//   * both arrive by direct-to-LDS loads (1 KiB per instruction: eight rows x 128 bytes, whole cache lines; weights
//     marked non-temporal: they are used once, the token rows by every workgroup) into a ring private to the wavefront -
//     no workgroup barrier in the stream, a wavefront waits for its own loads by count - and are read back as MFMA
//     operands (two v_mfma_f32_16x16x32_bf16 per step and pair of tiles, or one v_mfma_scale_f32_16x16x128_f8f6f4 over
//     FP8 codes); the 128 bytes of a row keep their eight 16-byte pieces at positions piece ^ (row / 2) % 8, which makes
//     those reads conflict-free;
//   * at the end the wavefronts' partial results meet in LDS and are summed in wavefront order (bitwise
//     reproducible), multiplied by the token's and the feature's scale when the operands are FP8 codes, rounded once
//     to bf16 and stored where the pack / unpack would have put them.
//
// Measured (us a call in a replayed graph, weights in rotation; the kernel before - tiles of 16 features one after the
// other against token rows held in registers, k split over workgroups and a finishing launch where they did not fit - ->
// this one): 10240 x 8192 bf16, 1 / 16 / 19 / 32 rows 27.2 / 32.4 / 33.8 / 36.9 -> 27.0 / 26.7 / 27.0 / 29.0 (168 MB: 6.3
// TB/s at 16 rows); 5120 x 2048 9.1 / 10.2 / 10.8 / 12.3 -> 6.7 / 7.3 / 7.6 / 8.0; FP8 codes, 10240 x 8192 16.1 / 18.3 / 19.8 / 22.4 ->
// 15.0 / 15.1 / 15.4 / 16.4, 64 rows 26.1 -> 20.8.  Few features, bf16, whole -> in ranges (the kernel before in brackets): 256 x
// 65536, 1 row 41.9 -> 11.6 (16.4); 2304 x 16384, 32 rows 27.6 -> 17.8 (23.2); 1024 x 8192, 64 rows 18.1 -> 11.0 (16.1, the tiled
// kernel).
// What is left over the weights' pass at the read probe's 6.9 TB/s: launch, first round trip and the meeting (about 3 us), and
// with many rows the token rows, which every workgroup reads whole (about 0.1 us per row at k = 8192).  Tried and not kept: as
// many wavefronts as hold two steps each (16 at most; small products 2 to 20 % slower), weights requested further ahead than
// the token rows in what is left of the LDS (within 2 %), at least 16 features a workgroup (up to 17 % slower).
#include "internal.h"

#include <math.h>

namespace shiftattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kSWaves = 8;                         // wavefronts that the size query counts with
constexpr int kSGrid = 256;                        // workgroups: one per compute unit
constexpr int kStepRowBytes = 128;                 // bytes of a weight row per step of a wavefront: 64 bf16 or 128 FP8 k
constexpr int kMaxRows = 40;                       // features per workgroup at most
constexpr int kRotSteps = 3;                       // steps of k between the starts of neighbouring blocks
constexpr int kHeadDim = 128;
#define SHIFTATTN_STREAM_HINT " nt"   // weights are read once: non-temporal

struct StreamParams {
    const unsigned char* __restrict__ w;   // [N][K] bf16 or FP8 E4M3 codes
    const unsigned char* __restrict__ x;   // token rows, see mode
    uint16_t* __restrict__ c;              // bf16 result
    float* __restrict__ partial;           // kg > 1: [kg][rows][N] fp32
    const float* __restrict__ xs;          // FP8 products: one scale per token row ...
    const float* __restrict__ ws;          // ... and one per output feature (nullptr: none)
    int M, M_out, N, K;                    // M token rows exist, rows M .. M_out - 1 of the result are zeros
    int mode;                              // 0: x dense [M][K], result into the send buffers; 1: x gathered from the
                                           // receive buffers (k = (p hq_l + j) 128 + e), result dense [M][N]
    int kg, kg_log2;                       // k ranges, each a workgroup of its own; the streaming kernel's are a power of two
    int rows_per_block;                    // features per block, a multiple of 4
    XchgShape s;
};

__device__ inline bf16x8 frag(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Four bf16 results of token t, features f .. f + 3 (one head, col = f % 128), to their place(s):
// mode 1: out[t][f]; mode 0: the send buffer(s) of the rank(s) owning the head (Sec. 3.2.1: fused q|k|v exchange,
// KV replication when there are fewer KV heads than ranks).
__device__ inline void store4(const StreamParams& p, int t, int f, u32x2 v) {
    if (p.mode == 1) {
        *reinterpret_cast<u32x2*>(p.c + static_cast<size_t>(t) * p.N + f) = v;
        return;
    }
    const XchgShape& s = p.s;
    const int head = f / kHeadDim, col = f % kHeadDim;
    const size_t row_stride = static_cast<size_t>(s.hq_l + 2 * s.hkv_l) * kHeadDim;
    const size_t buf_stride = static_cast<size_t>(s.T_pad) * row_stride;
    uint16_t* row = p.c + static_cast<size_t>(t) * row_stride + col;
    if (head < s.h) {
        const int dest = head / s.hq_l, local = head - dest * s.hq_l;
        *reinterpret_cast<u32x2*>(row + dest * buf_stride + local * kHeadDim) = v;
        return;
    }
    const bool is_v = head >= s.h + s.h_kv;
    const int g = head - s.h - (is_v ? s.h_kv : 0);
    const int slot0 = s.hq_l + (is_v ? s.hkv_l : 0);
    if (s.h_kv >= s.P) {
        const int dest = g / s.hkv_l, local = slot0 + (g - dest * s.hkv_l);
        *reinterpret_cast<u32x2*>(row + dest * buf_stride + local * kHeadDim) = v;
    } else {
        for (int dest = 0; dest < s.P; ++dest)
            if (static_cast<int>((static_cast<int64_t>(dest) * s.h_kv) / s.P) == g)
                *reinterpret_cast<u32x2*>(row + dest * buf_stride + slot0 * kHeadDim) = v;
    }
}

__device__ inline u32x2 round4(f32x4 v) {
    bf16x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = static_cast<__bf16>(v[e]);
    return __builtin_bit_cast(u32x2, r);
}

// Wavefronts of a workgroup and steps in a wavefront's ring: all of the LDS.  Eight wavefronts where their rings hold two steps,
// four with rings twice as long beyond (four everywhere from six pieces a step on: 8192 x 8192, 16 rows 21.7 -> 24.0 us).
template <int UX, int UW>
constexpr int stream_waves() { return UX + UW <= 10 ? 8 : 4; }
template <int UX, int UW>
constexpr int stream_steps() { return 160 / stream_waves<UX, UW>() / (UX + UW); }

// UX: pieces of eight token rows, UW: pieces of eight weight rows per step; kFp8: both operands are FP8 E4M3 codes
template <int UX, int UW, bool kFp8>
__global__ __launch_bounds__((64 * stream_waves<UX, UW>())) void proj_stream_kernel(StreamParams p) {
    constexpr int kElem = kFp8 ? 1 : 2;
    constexpr int kStepK = kStepRowBytes / kElem;
    constexpr int kWaves = stream_waves<UX, UW>(), kUnits = UX + UW, kRing = stream_steps<UX, UW>(), kSlot = kUnits * 1024;
    constexpr int TB = (UX + 1) / 2, TW = (UW + 1) / 2;
    static_assert(kRing >= 2 && kRing * kUnits <= 62, "outstanding loads fit the counter");
    static_assert(TB * TW <= kRing * kUnits, "a wavefront's sums fit its ring");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, grp = lane >> 4;
    // k range and block of features (workgroup i runs on XCD i % 8: a range's token rows enter few L2s)
    const int kr = blockIdx.x & (p.kg - 1), rb = blockIdx.x >> p.kg_log2;
    const int row_begin = rb * p.rows_per_block;
    const int row_end = min(p.N, row_begin + p.rows_per_block);   // row_begin < N: the grid has no empty workgroup
    const size_t k_bytes = static_cast<size_t>(p.K) * kElem;
    const int all_steps = p.K / kStepK;
    const int my_slice = kr * kWaves + wave, slices_log2 = p.kg_log2 + (kWaves == 8 ? 3 : 2);
    const int slice = all_steps * my_slice >> slices_log2, n = (all_steps * (my_slice + 1) >> slices_log2) - slice;   // this wavefront's steps (none, if k is that short)
    // Neighbouring blocks start their walk kRotSteps apart and wrap around: rows lie k apart, often a power of two, and with
    // the same start everywhere all workgroups ask the same memory channels at the same time (in the kernel before: 8192
    // features x 8192 k, 1 / 16 rows 27.2 / 29.4 us in bf16, 16.6 / 16.8 with FP8 codes; three steps further per block 23.7 /
    // 26.5 and 13.1 / 14.8; other sizes within 1 % or faster, any odd step alike).
    const int first = static_cast<int>((static_cast<uint32_t>(slice) + static_cast<uint32_t>(rb) * kRotSteps) % all_steps);
    unsigned char* const ring_ptr = lds + wave * (kRing * kSlot);
    const uint32_t ring = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds)) + wave * (kRing * kSlot);

    // piece u holds rows 8 u .. 8 u + 7; lane: row 8 u + lane / 8, position lane % 8 holds piece position ^ (row / 2) % 8.
    // Rows past the last one re-read it; they are not stored.
    const uint32_t seg_bytes = p.mode == 0 ? static_cast<uint32_t>(k_bytes) : p.s.hq_l * kHeadDim * kElem;   // consecutive k of a token
    uint32_t xoff[UX], woff[UW];
#pragma unroll
    for (int u = 0; u < UX; ++u) {
        const int r = 8 * u + (lane >> 3);
        xoff[u] = min(r, p.M - 1) * seg_bytes + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int u = 0; u < UW; ++u) {
        const int r = 8 * u + (lane >> 3);
        woff[u] = static_cast<uint32_t>(min(r, row_end - row_begin - 1) * k_bytes + (((lane & 7) ^ ((r >> 1) & 7)) << 4));
    }
    auto scalar_ptr = [](const unsigned char* ptr) -> const unsigned char* {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
        return reinterpret_cast<const unsigned char*>((static_cast<uint64_t>(hi) << 32) | lo);
    };
    // (M0: the compiler sets it right before each use of its own and keeps no value in it)
    auto load_token = [&](const unsigned char* base, uint32_t off, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst), "v"(off), "s"(scalar_ptr(base)) : "memory");
    };
    auto load_weight = [&](const unsigned char* base, uint32_t off, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" SHIFTATTN_STREAM_HINT
                     :: "s"(dst), "v"(off), "s"(scalar_ptr(base)) : "memory");
    };
    int rq_step = first, rq_slot = 0;   // the next step to request and its place
    const uint32_t seg_steps = seg_bytes / kStepRowBytes;   // token rows: consecutive steps before the next receive buffer
    const uint32_t seg = first / seg_steps;
    uint32_t seg_left = (seg + 1) * seg_steps - first;
    const unsigned char* w_base = p.w + row_begin * k_bytes + static_cast<size_t>(first) * kStepRowBytes;
    const unsigned char* x_base = p.x + (p.mode == 0 ? 0 : static_cast<size_t>(seg) * p.s.T_pad * seg_bytes) +
                                  static_cast<size_t>(first - seg * seg_steps) * kStepRowBytes;
    auto request = [&]() {
        const uint32_t dst = ring + rq_slot * kSlot;
#pragma unroll
        for (int u = 0; u < UX; ++u) load_token(x_base, xoff[u], dst + 1024 * u);
#pragma unroll
        for (int u = 0; u < UW; ++u) load_weight(w_base, woff[u], dst + 1024 * (UX + u));
        rq_slot = rq_slot + 1 == kRing ? 0 : rq_slot + 1;
        w_base += kStepRowBytes;
        x_base += kStepRowBytes;
        if (--seg_left == 0) {
            seg_left = seg_steps;
            x_base += static_cast<size_t>(p.s.T_pad - 1) * seg_bytes;   // mode 0 has one segment: the wrap below
        }
        if (++rq_step == all_steps) {
            rq_step = 0;
            w_base -= k_bytes;
            x_base = p.x;
        }
    };
#pragma unroll
    for (int g = 0; g < kRing; ++g)
        if (g < n) request();

    // operand reads: row l16 of a tile of 16, piece 4 kb + grp (FP8: two of a lane's k halves, in the same order for both
    // operands) at position piece ^ key(row); a tile of one piece reads its eight rows twice
    int rd[2], rd_half[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int piece = 4 * kb + grp;
        rd[kb] = l16 * kStepRowBytes + ((piece ^ (l16 >> 1)) << 4);
        rd_half[kb] = (l16 & 7) * kStepRowBytes + ((piece ^ ((l16 & 7) >> 1)) << 4);
    }
    f32x4 acc[TW][TB];
#pragma unroll
    for (int tw = 0; tw < TW; ++tw)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[tw][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
    int slot = 0;
    for (int j = 0; j < n; ++j) {
        // loads return in order: step j has landed when only those of the steps behind it are outstanding
        const int younger = min(kRing - 1, n - 1 - j);
#pragma unroll
        for (int y = 0; y < kRing; ++y)
            if (younger == y) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kUnits * y) : "memory");
        const unsigned char* stage = ring_ptr + slot * kSlot;
        u32x4 a[TW][2], b[TB][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int tb = 0; tb < TB; ++tb)
                b[tb][kb] = *reinterpret_cast<const u32x4*>(stage + 2048 * tb + (2 * tb + 1 == UX ? rd_half[kb] : rd[kb]));
#pragma unroll
            for (int tw = 0; tw < TW; ++tw)
                a[tw][kb] = *reinterpret_cast<const u32x4*>(stage + 1024 * UX + 2048 * tw + (2 * tw + 1 == UW ? rd_half[kb] : rd[kb]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot is in registers: the step kRing ahead goes there
        if (j + kRing < n) request();
        slot = slot + 1 == kRing ? 0 : slot + 1;
        if constexpr (kFp8) {
            auto both = [](const u32x4 (&v)[2]) {
                return i32x8{static_cast<int>(v[0][0]), static_cast<int>(v[0][1]), static_cast<int>(v[0][2]), static_cast<int>(v[0][3]),
                             static_cast<int>(v[1][0]), static_cast<int>(v[1][1]), static_cast<int>(v[1][2]), static_cast<int>(v[1][3])};
            };
#pragma unroll
            for (int tw = 0; tw < TW; ++tw)
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
                    acc[tw][tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(both(a[tw]), both(b[tb]), acc[tw][tb], 0, 0, 0, 127, 0, 127);
        } else {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int tw = 0; tw < TW; ++tw)
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb)
                        acc[tw][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(a[tw][kb]), frag(b[tb][kb]), acc[tw][tb], 0, 0, 0);
        }
    }
    // ---- the wavefronts' k slices meet, each in its wavefront's ring, which has been read and into which nothing is on its way
#pragma unroll
    for (int tw = 0; tw < TW; ++tw)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) reinterpret_cast<f32x4*>(ring_ptr)[(tw * TB + tb) * 64 + lane] = acc[tw][tb];
    __syncthreads();
    for (int i = tid; i < TW * TB * 64; i += 64 * kWaves) {
        const int tile = i >> 6, tw = tile / TB, tb = tile - tw * TB;
        // register r of a lane is feature 4 grp + r of token l16
        const int t = 16 * tb + l16, f = row_begin + 16 * tw + 4 * grp;
        if (f >= row_end || t >= p.M_out) continue;
        f32x4 sum = reinterpret_cast<const f32x4*>(lds)[i];
#pragma unroll
        for (int w2 = 1; w2 < kWaves; ++w2) {
            const f32x4 v = reinterpret_cast<const f32x4*>(lds + w2 * (kRing * kSlot))[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += v[e];
        }
        if (p.kg > 1) {   // rows past the last token are not read
            if (t < p.M) *reinterpret_cast<f32x4*>(p.partial + (static_cast<size_t>(kr) * p.M_out + t) * p.N + f) = sum;
            continue;
        }
        if constexpr (kFp8) {
            if (t < p.M) {
                const float row_scale = p.xs[t];
                const f32x4 col_scale = *reinterpret_cast<const f32x4*>(p.ws + f);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = sum[e] * row_scale * col_scale[e];
            }
        }
        store4(p, t, f, t < p.M ? round4(sum) : u32x2{0u, 0u});
    }
}

template <int UX, int UW>
constexpr int stream_lds() { return stream_waves<UX, UW>() * stream_steps<UX, UW>() * (UX + UW) * 1024; }

#define SHIFTATTN_STREAM_SHAPES(X) \
    X(1, 1) X(1, 2) X(1, 3) X(1, 4) X(1, 5) X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(2, 5) \
    X(3, 1) X(3, 2) X(3, 3) X(3, 4) X(3, 5) X(4, 1) X(4, 2) X(4, 3) X(4, 4) X(4, 5) \
    X(6, 1) X(6, 2) X(6, 3) X(6, 4) X(6, 5) X(8, 1) X(8, 2) X(8, 3) X(8, 4) X(8, 5) \
    X(12, 1) X(12, 2) X(12, 3) X(12, 4) X(12, 5) X(16, 1) X(16, 2) X(16, 3) X(16, 4)

// features per workgroup: the chip's compute units read equally many bytes, in as many rounds of at most kMaxRows features as it takes
int stream_rows(int N, int kg) {
    const int blocks = kSGrid / kg, rounds = (N + blocks * kMaxRows - 1) / (blocks * kMaxRows);
    return ((N + blocks * rounds - 1) / (blocks * rounds) + 3) / 4 * 4;
}

struct StreamShape {
    int ux, uw;   // pieces of eight token rows and of eight weight rows
};

StreamShape stream_shape(int M_out, int rows_per_block) {
    const int octets = (M_out + 7) / 8;
    return {octets <= 4 ? octets : octets <= 8 ? (octets + 1) / 2 * 2 : (octets + 3) / 4 * 4, (rows_per_block + 7) / 8};
}

bool stream_built(StreamShape shape) {
#define SHIFTATTN_STREAM_IS(ux_, uw_) if (shape.ux == ux_ && shape.uw == uw_) return true;
    SHIFTATTN_STREAM_SHAPES(SHIFTATTN_STREAM_IS)
#undef SHIFTATTN_STREAM_IS
    return false;
}

hipError_t launch_stream(const StreamParams& p, hipStream_t st) {
    const auto [ux, uw] = stream_shape(p.M_out, p.rows_per_block);
    const unsigned grid = (p.N + p.rows_per_block - 1) / p.rows_per_block * p.kg;
#define SHIFTATTN_STREAM_LAUNCH(ux_, uw_)                                                                   \
    if (ux == ux_ && uw == uw_) {                                                                         \
        if (p.xs) proj_stream_kernel<ux_, uw_, true><<<grid, 64 * stream_waves<ux_, uw_>(), stream_lds<ux_, uw_>(), st>>>(p);     \
        else proj_stream_kernel<ux_, uw_, false><<<grid, 64 * stream_waves<ux_, uw_>(), stream_lds<ux_, uw_>(), st>>>(p);         \
        return hipGetLastError();                                                                         \
    }
    SHIFTATTN_STREAM_SHAPES(SHIFTATTN_STREAM_LAUNCH)
#undef SHIFTATTN_STREAM_LAUNCH
    return hipErrorInvalidValue;
}

// Behind either kernel with k ranges: result[t][f .. f + 3] = sum over the ranges in their order, rounded once
// (row_base: partial row r is row row_base + r of the result)
constexpr int kFinishAhead = 4;
__global__ __launch_bounds__(256) void proj_stream_finish_kernel(StreamParams p, int t_rows, int row_base) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int quads = p.N / 4;
    if (i >= static_cast<int64_t>(p.M_out - row_base) * quads) return;
    const int r = static_cast<int>(i / quads), f = static_cast<int>(i % quads) * 4;
    const int t = row_base + r;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    if (t < p.M) {
        sum = *reinterpret_cast<const f32x4*>(p.partial + static_cast<size_t>(r) * p.N + f);
        // four ranges are requested at a time: added one by one, each would be a round trip to memory of its own
        const float* src = p.partial + static_cast<size_t>(r) * p.N + f;
        const size_t range = static_cast<size_t>(t_rows) * p.N;
        for (int c = 1; c < p.kg; c += kFinishAhead) {
            f32x4 v[kFinishAhead];
#pragma unroll
            for (int x = 0; x < kFinishAhead; ++x)
                if (c + x < p.kg) v[x] = *reinterpret_cast<const f32x4*>(src + (c + x) * range);
#pragma unroll
            for (int x = 0; x < kFinishAhead; ++x) {
                if (c + x < p.kg) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += v[x][e];
                }
            }
        }
        if (p.xs) {   // the scales of FP8 operands, applied as the unsplit kernel applies them
            const float row_scale = p.xs[t];
            const f32x4 col_scale = *reinterpret_cast<const f32x4*>(p.ws + f);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = sum[e] * row_scale * col_scale[e];
        }
    }
    store4(p, t, f, round4(sum));
}

}  // namespace

// result = sum over kg partial results [kg][t_rows][N] (fp32) in group order, rounded once, stored with the layout of `mode`
hipError_t launch_proj_finish(const float* partial, int kg, int t_rows, void* c, int M, int M_out, int N, int mode,
                              const XchgShape& s, const float* x_scales, const float* w_scales, hipStream_t st, int row_base) {
    StreamParams p = {};
    p.xs = x_scales;
    p.ws = w_scales;
    p.partial = const_cast<float*>(partial);
    p.c = static_cast<uint16_t*>(c);
    p.M = M;
    p.M_out = M_out;
    p.N = N;
    p.mode = mode;
    p.kg = kg;
    p.s = s;
    const int64_t items = static_cast<int64_t>(M_out - row_base) * (N / 4);
    if (items <= 0) return hipSuccess;
    proj_stream_finish_kernel<<<static_cast<unsigned>((items + 255) / 256), 256, 0, st>>>(p, t_rows, row_base);
    return hipGetLastError();
}

hipError_t proj_stream_init() {
    hipError_t e = hipSuccess;
#define SHIFTATTN_STREAM_INIT(ux_, uw_)                                                                                 \
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&proj_stream_kernel<ux_, uw_, false>),  \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, stream_lds<ux_, uw_>());  \
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&proj_stream_kernel<ux_, uw_, true>),   \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, stream_lds<ux_, uw_>());
    SHIFTATTN_STREAM_SHAPES(SHIFTATTN_STREAM_INIT)
#undef SHIFTATTN_STREAM_INIT
    return e;
}

// Microseconds of a call with k in kg ranges (one round of workgroups), for the choice of kg: launch and meeting, the walk of one
// wavefront or the weights' pass, whichever is longer (rounded off where they are alike), the finishing launch with the sums written and
// read.  Fitted to 3666 timed launches of 1 .. 64 rows, 256 .. 8192 features and 1024 .. 65536 k of both types, kg = 1, 2, 4, 8: 6 % off in one
// of ten, 12 to 15 % in one of a hundred.
static double stream_us(int M_out, int N, int64_t k_bytes, int kg) {
    const auto [ux, uw] = stream_shape(M_out, stream_rows(N, kg));
    const bool eight = ux + uw <= 10;   // wavefronts, see stream_waves()
    const double step = eight ? 0.034 + 0.096 * ux + 0.178 * uw : 0.096 * (ux + uw) - 0.30;
    const double walk = static_cast<double>(k_bytes) / kStepRowBytes / (kg * (eight ? 8 : 4)) * step;
    const double weights = static_cast<double>(N) * k_bytes / 7.7e6;
    const double w2 = walk * walk, b2 = weights * weights;
    return 3.2 + 0.03 * (ux + uw) + sqrt(sqrt(w2 * w2 + b2 * b2)) + (kg > 1 ? 1.9 + kg * (8.0 * M_out * N) / 2.4e6 : 0.0);
}

// Served: up to 128 token rows, and expected to be no slower than the large-batch kernel with its small tiles and k ranges.
// That kernel shares the weights among all of a tile's token rows, so it can win from 33 rows on; every block of features
// reads all token rows here.  Measured, us, this kernel / that one:
//   * up to 16 rows, up to 32 but for the sizes of the third point, or up to 64 with rows of at most 8 KiB (4096 bf16 or 8192 FP8 elements), this one throughout: bf16, 64
//     rows, 6144 x 4096 16.7 / 21.4, 5120 x 2048 11.3 / 17.3, 8192 x 1024 7.2 / 10.6; FP8 8192 x 8192 18.0 / 23.1;
//   * 33 to 64 longer rows: 10240 x 8192, 64 rows 35.9 / 37.7, 10240 x 5120 27.6 / 27.7; 8192 x 8192, 40 / 48 rows
//     26.2 / 26.3, 27.5 / 26.6; 5120 x 5120, 40 rows 16.3 / 15.5; 1280 x 5120, 40 rows 12.0 / 11.5: the line in N is drawn
//     through these.  Without the workspace that its k ranges want that kernel is several times slower, with a short one slower:
//     1280 x 8192, 48 rows, where the query names a quarter of what it wants, 16.4 / 17.9;
//   * more features than one round takes, or rows of more than 16 KiB: by a model of both (this one: launch, the weights' pass at
//     6.4 TB/s, and per round the token rows past the tenth at 66 GB/s a compute unit).  bf16 14336 x 12288, 24 / 32 rows
//     64.1 / 65.3, 71.1 / 66.1; 18432 x 8192, 32 / 64 rows 54.1 / 63.2, 71.9 / 63.2; 4096 x 15360, 24 rows 29.9 / 27.6; FP8
//     8192 x 16384, 32 rows 24.5 / 37.6.  The model prices this one too high near the line, so some calls stay with the tiled kernel
//     that this one would serve sooner: bf16 8192 x 16384, 32 rows 45.6 / 51.5; 24576 x 8192, 24 rows 67.2 / 71.5; 17408 x 4096, 48
//     rows 33.0 / 36.0; FP8 14336 x 12288, 17 rows 33.8 / 37.6; 24576 x 8192, 24 rows 37.2 / 40.5;
//   * 65 to 128 rows: FP8 6144 x 4096, 96 / 128 rows 12.6 / 17.0, 14.7 / 18.6; 10240 x 5120 19.8 / 23.3, 25.4 / 25.5;
//     1280 x 5120 11.9 / 12.5, 13.8 / 13.6; 8192 x 8192 21.7 / 21.5; bf16 8192 x 1024 8.2 / 11.0, 9.4 / 11.2; 5120 x 2048
//     14.4 / 15.3, 16.9 / 16.6; 2048 x 4096 15.1 / 13.9.  (More than 32 features a workgroup and 96 rows: a ring of one step.)
//     The figures of the tiled kernel are those with its workspace; a call without one is not told apart here and takes that kernel
//     unsplit for longer rows, as it always has (2304 x 5120 in bf16: 65 rows 45 us, 64 rows here 17).
static bool proj_stream_takes(int M_out, int N, int K, bool fp8, size_t workspace_bytes) {
    const int elem = fp8 ? 1 : 2;
    if (M_out < 1 || M_out > 128 || N % 4 != 0 || K % (kStepRowBytes / elem) != 0) return false;
    const int64_t k_bytes = static_cast<int64_t>(K) * elem;
    if (M_out > 16 && (N > kSGrid * kMaxRows || k_bytes > 16384)) {
        const int rounds = (N + kSGrid * kMaxRows - 1) / (kSGrid * kMaxRows);
        const double us = 3.0 + static_cast<double>(N) * k_bytes / 6.4e6 + static_cast<double>(rounds) * (M_out - 10) * k_bytes / 66e3;
        return M_out <= 64 && us <= proj_gemm_us(M_out, N, K, fp8, workspace_bytes);
    }
    if (M_out > 64) return M_out <= 96 ? k_bytes <= (fp8 ? 5120 : 4096) : k_bytes <= (fp8 ? 4096 : 2048) && stream_rows(N, 1) <= 32;
    if (M_out <= 32 || k_bytes <= 8192 || M_out <= (N - 4096) / 96) return true;
    return proj_gemm_us(M_out, N, K, fp8, workspace_bytes) > 1.1 * proj_gemm_us(M_out, N, K, fp8, SIZE_MAX);
}

int proj_stream_ranges(int M_out, int N, int K, bool fp8, size_t workspace_bytes) {
    const int elem = fp8 ? 1 : 2;
    if (M_out < 1 || N % 4 != 0 || K % (kStepRowBytes / elem) != 0) return 0;
    // k ranges only where the model has them 5 % ahead of the walk in one piece, or 10 % of the tiled kernel where that takes the call
    // (with 5 %: 3072 x 12288, 48 rows 23.1 us in two ranges, 21.8 there).  The
    // choice over 1424 measured products of up to 64 rows with the workspace of the size query: within 3 % of the best kernel and kg
    // in nine of ten, 15 % off in one of a hundred; none slower than the kernel before (2512 products).  Above 64 rows
    // the size query's workspace is the tiled kernel's, which uses it.
    const bool whole = proj_stream_takes(M_out, N, K, fp8, workspace_bytes);
    if (M_out > 64) return whole ? 1 : 0;
    const int64_t k_bytes = static_cast<int64_t>(K) * elem;
    int best = whole ? 1 : 0;
    double best_us = whole ? stream_us(M_out, N, k_bytes, 1) : proj_gemm_us(M_out, N, K, fp8, workspace_bytes);
    for (int kg = 2; kg <= 8; kg *= 2) {
        if (N > kSGrid / kg * kMaxRows || k_bytes < static_cast<int64_t>(kg) * 8 * kStepRowBytes ||
            static_cast<size_t>(kg) * M_out * N * sizeof(float) > workspace_bytes) break;
        const double us = (whole ? 1.05 : 1.1) * stream_us(M_out, N, k_bytes, kg);
        if (us < best_us && stream_built(stream_shape(M_out, stream_rows(N, kg)))) {
            best = kg;
            best_us = us;
        }
    }
    return best;
}

// Host query: the instance that a call which this kernel takes launches; false if it is not built
bool proj_stream_describe(int M_out, int N, int kg, shiftattn_proj_plan_t* plan) {
    const StreamShape shape = stream_shape(M_out, stream_rows(N, kg));
    *plan = shiftattn_proj_plan_t{1, kg, shape.ux, shape.uw, 0, 0, 0, 0, 0};
    return stream_built(shape);
}

// What the size query names: for up to 64 rows whose k divides by that of eight wavefronts' steps, room for k ranges of token rows
// (rounded up to 16, 32 or 64) x features in fp32, else what the large-batch kernel's plan wants.  Callers allocate by these sizes and
// tests pin them, so they are part of the interface and no longer follow either kernel: which kernel runs, in how many ranges, is
// decided per call by what fits.  They are more than a call uses where it streams whole (17 to 32 rows x 10240 x 8192: 2.6 MB, none
// used), and less than the tiled kernel would take for 33 to 64 rows of 8192 x 8192 and the like (within 2 % there; where features
// are few the ranges of this kernel make up for it: 48 rows x 1280 x 8192).
size_t proj_workspace(int M_out, int N, int K, bool fp8) {
    const int per_step = kSWaves * kStepRowBytes / (fp8 ? 1 : 2);
    if (M_out <= 64 && N % 4 == 0 && K % per_step == 0) {
        const int tb = M_out <= 16 ? 1 : M_out <= 32 ? 2 : 4;
        for (int kwb = 16 / tb; kwb >= 1; kwb /= 2) {
            const int kg = K / per_step / kwb;
            if (K / per_step % kwb == 0 && kg <= 8 && kSGrid % kg == 0) return kg == 1 ? 0 : static_cast<size_t>(kg) * 16 * tb * N * sizeof(float);
        }
    }
    return proj_gemm_workspace(M_out, N, K, fp8);
}

static hipError_t run_stream(StreamParams& p, int kg, void* workspace, hipStream_t st) {
    p.kg = kg;
    p.kg_log2 = __builtin_ctz(kg);
    p.partial = static_cast<float*>(workspace);
    p.rows_per_block = stream_rows(p.N, kg);
    const hipError_t e = launch_stream(p, st);
    if (e != hipSuccess || kg == 1) return e;
    return launch_proj_finish(p.partial, kg, p.M_out, p.c, p.M, p.M_out, p.N, p.mode, p.s, p.xs, p.ws, st, 0);
}

// kg: k ranges, see proj_stream_ranges(); x_scales / w_scales: nullptr for bf16 operands, the row scales of FP8 E4M3 codes otherwise
hipError_t launch_qkv_proj_stream(const void* x, const void* w_qkv, void* send, int d_model, const XchgShape& s,
                                  const float* x_scales, const float* w_scales, int kg, void* workspace, hipStream_t st) {
    StreamParams p = {};
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
    return run_stream(p, kg, workspace, st);
}

hipError_t launch_o_proj_stream(const void* recv, const void* w_o, void* out, int d_model, const XchgShape& s,
                                const float* a_scales, const float* w_scales, int kg, void* workspace, hipStream_t st) {
    StreamParams p = {};
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
    return run_stream(p, kg, workspace, st);
}

}  // namespace shiftattn
