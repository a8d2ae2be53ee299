// Causal prefill attention of fp32 shards over the paged KV cache (Algorithm 1, boxed attention line, prefill rows):
// fp32 throughout, head_dim 64 or 128, up to 16 query heads per KV head.  The general kernel takes everything else.
//
// A workgroup owns 16 "columns" - (new token, query head) pairs, the heads that share a KV head next to each other - and
// its eight wavefronts split the keys: wavefront w takes cache blocks 16 w .. of 32 keys, and every eighth such pair of
// blocks behind it.  Partial results meet in LDS at the end.
//   S^T[key][col]  = K[key][:] . Q^T[:][col]       16x16x4 fp32 MFMA, A = K rows, B = Q^T
//   O^T[d][col]   += V^T[d][key] . P^T[key][col]   A = V^T rows, B = P^T
// Operands come straight from the cache in 16-byte pieces: the four elements of a lane's piece serve four MFMAs, and the
// same four of Q (or P) go with them, so the order in which head-dim elements and keys enter the sums is the pieces' own.
// With V stored dimension-major, the four S^T values a lane holds are the P^T operands of its own V pieces.
//
// What bounds it: fp32 batches are small (hundreds of tokens), so time is the chain sequence -> block id -> K/V -> two
// products -> merge; eight wavefronts per 16 columns put a 256-key row at one trip round that chain, and a workgroup per 16
// columns fills the chip from about a thousand tokens of four heads on.  256 tokens,
// 4 heads, D = 64: 8.2 us, against 19.5 of the general kernel (a wavefront per row, keys over lanes, no matrix unit); 990
// tokens in two sequences, D = 128: 21. Error against fp64 5 to 15 % below the general kernel's (2.1e-7 .. 3.1e-7).
#include "internal.h"

namespace shiftattn {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kCols = 16;
constexpr int kStep = 2 * kBlockSize;  // keys per wavefront step

template <int D>
__global__ __launch_bounds__(kWaves * 64, 2) void prefill_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ cache, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ cu_seqlens_q, const int32_t* __restrict__ seq_lens, int num_seqs, float* __restrict__ out,
    AttnShape a, int G, int tile_tokens) {
    constexpr int kJ = D / 16, kPitch = D + 4;
    __shared__ __attribute__((aligned(16))) float o_s[kWaves][kCols][kPitch];
    __shared__ float m_s[kWaves][kCols], l_s[kWaves][kCols];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 15, grp = lane >> 4;

    // ---- which (sequence, tile, KV head): sequence s owns workgroups cu[s] / tile_tokens + s and following, at least as
    // many as it has tiles (the lengths are on the device); later tokens see more keys and start first
    const int item = static_cast<int>(gridDim.x - 1 - blockIdx.x);
    const int hk = item % a.hkv_l, x = item / a.hkv_l;
    int s = 0;
    for (int base = 0; base < num_seqs; base += 64) {
        const int i = base + lane;
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(i < num_seqs && cu_seqlens_q[i] / tile_tokens + i <= x));
        if (n > 0) s = base + n - 1;
        if (n < 64) break;
    }
    const int q_begin = cu_seqlens_q[s], q_len = cu_seqlens_q[s + 1] - q_begin;
    const int tok0 = (x - (q_begin / tile_tokens + s)) * tile_tokens;
    if (tok0 >= q_len) return;  // uniform
    const int ctx = seq_lens[s];
    const int pos0 = ctx - q_len + tok0;                                                    // first token's position
    const int pos_max = pos0 + min(tile_tokens, q_len - tok0) - 1;
    const int n_blocks = pos_max < 0 ? 0 : pos_max / kBlockSize + 1;
    const int cols_used = tile_tokens * G;
    const bool valid = col < cols_used && tok0 + col / G < q_len;
    const int pos = valid ? pos0 + col / G : -1;
    const int32_t* table = block_table + static_cast<size_t>(s) * a.max_blocks;

    f32x4 qf[kJ];
    {   // a column beyond the tile or the sequence reads the nearest real one's row: its logits are masked, its result dropped
        const int cr = min(col, cols_used - 1), tr = min(tok0 + cr / G, q_len - 1);
        const float* qp = q + static_cast<size_t>(q_begin + tr) * a.q_stride + static_cast<size_t>(hk * G + cr % G) * D + 4 * grp;
#pragma unroll
        for (int j = 0; j < kJ; ++j) qf[j] = *reinterpret_cast<const f32x4*>(qp + 16 * j);
    }
    const float scale = a.scale * a.k_scale;

    f32x4 kf[2][kJ], vf[2][kJ], o[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    auto block_ptr = [&](int b, int part) {
        return cache + cache_part_offset(table[min(b, n_blocks - 1)], hk, part, a.hkv_l, D);
    };
    auto load_k = [&](int st) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const float* p = block_ptr(2 * st + b, 0) + col * D + 4 * grp;
#pragma unroll
            for (int j = 0; j < kJ; ++j) kf[b][j] = *reinterpret_cast<const f32x4*>(p + 16 * j);
        }
    };
    if (2 * wave < n_blocks) load_k(wave);
    for (int st = wave; 2 * st < n_blocks; st += kWaves) {   // uniform per wavefront
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const float* p = block_ptr(2 * st + b, 1) + col * kBlockSize + 4 * grp;
#pragma unroll
            for (int mt = 0; mt < kJ; ++mt) vf[b][mt] = *reinterpret_cast<const f32x4*>(p + 16 * mt * kBlockSize);
        }
        f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[0][j][e], qf[j][e], sc[0], 0, 0, 0);
                sc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[1][j][e], qf[j][e], sc[1], 0, 0, 0);
            }
        // the next step's K: under the softmax where the registers hold it beside V (at D = 128 they spilled)
        if constexpr (D == 64)
            if (2 * (st + kWaves) < n_blocks) load_k(st + kWaves);
        // keys of this lane's values: key0 + 16 b + r
        const int key0 = kStep * st + 4 * grp;
        float m_loc = -INFINITY;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sc[b][r] = key0 + 16 * b + r <= pos ? sc[b][r] * scale : -INFINITY;
                m_loc = fmaxf(m_loc, sc[b][r]);
            }
        m_loc = fmaxf(m_loc, __shfl_xor(m_loc, 16));
        m_loc = fmaxf(m_loc, __shfl_xor(m_loc, 32));
        const float m_new = fmaxf(m_run, m_loc);
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;   // (no visible key yet)
        const float alpha = expf(m_run - m_ref);
        float p[2][4], l_add = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[b][r] = expf(sc[b][r] - m_ref);
                l_add += p[b][r];
            }
        l_run = l_run * alpha + l_add;
        m_run = m_new;
#pragma unroll
        for (int mt = 0; mt < kJ; ++mt) o[mt] *= alpha;
        // A key that a column does not see has P = 0 there, which must not meet a V that is no number: slots past the
        // context may hold anything and are cleared; infinities and NaNs of tokens that only later columns see send the
        // step down the element-wise path.
        bool odd = false;
        if (kStep * st + kStep - 1 > pos0) {   // uniform: the step reaches past some column's position
            float t = 0.f;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int mt = 0; mt < kJ; ++mt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (key0 + 16 * b + e >= ctx) vf[b][mt][e] = 0.f;
                        t = fmaf(vf[b][mt][e], 0.f, t);
                    }
            odd = __builtin_amdgcn_ballot_w64(t != 0.f) != 0;
        }
        if (__builtin_expect(!odd, 1)) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int mt = 0; mt < kJ; ++mt) o[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[b][mt][e], p[b][e], o[mt], 0, 0, 0);
        } else {
            // (the sums go through this lane's places in LDS: a loop over them there costs the usual path no registers)
#pragma unroll
            for (int mt = 0; mt < kJ; ++mt) *reinterpret_cast<f32x4*>(&o_s[wave][col][16 * mt + 4 * grp]) = o[mt];
#pragma unroll 1
            for (int k = 0; k < kStep; ++k) {
                const int e = k & 3;
                const float lo = e == 0 ? p[0][0] : e == 1 ? p[0][1] : e == 2 ? p[0][2] : p[0][3];
                const float hi = e == 0 ? p[1][0] : e == 1 ? p[1][1] : e == 2 ? p[1][2] : p[1][3];
                const float pk = __shfl(k < 16 ? lo : hi, ((k & 15) >> 2) * 16 + col);
                const float* vp = block_ptr(2 * st + (k >> 4), 1) + (k & 15);
                if (kStep * st + k <= pos)
#pragma unroll 1
                    for (int i = 0; i < D / 4; ++i) {
                        const int d = 16 * (i >> 2) + 4 * grp + (i & 3);
                        o_s[wave][col][d] = fmaf(vp[d * kBlockSize], pk, o_s[wave][col][d]);
                    }
            }
#pragma unroll
            for (int mt = 0; mt < kJ; ++mt) o[mt] = *reinterpret_cast<const f32x4*>(&o_s[wave][col][16 * mt + 4 * grp]);
        }
        if constexpr (D != 64)
            if (2 * (st + kWaves) < n_blocks) load_k(st + kWaves);
    }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int mt = 0; mt < kJ; ++mt) *reinterpret_cast<f32x4*>(&o_s[wave][col][16 * mt + 4 * grp]) = o[mt];
    if (grp == 0) {
        m_s[wave][col] = m_run;
        l_s[wave][col] = l_run;
    }
    __syncthreads();
    // 32 threads per column, D / 32 elements each; wavefronts' parts in their order
    constexpr int kE = D / 32;
    typedef float vec __attribute__((ext_vector_type(kE)));
    const int c = threadIdx.x >> 5, d = (threadIdx.x & 31) * kE;
    if (c >= cols_used || tok0 + c / G >= q_len) return;
    float m_star = m_s[0][c];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m_star = fmaxf(m_star, m_s[w][c]);
    float l = 0.f;
    vec acc = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const float f = m_s[w][c] == -INFINITY ? 0.f : expf(m_s[w][c] - m_star);
        l = fmaf(l_s[w][c], f, l);
        acc += *reinterpret_cast<const vec*>(&o_s[w][c][d]) * f;
    }
    const float inv = l > 0.f ? a.v_scale / l : 0.f;   // a row without visible keys is zero
    *reinterpret_cast<vec*>(out + static_cast<size_t>(q_begin + tok0 + c / G) * a.out_stride + static_cast<size_t>(hk * G + c % G) * D + d) = acc * inv;
}

}  // namespace

bool prefill_f32_supported(const AttnShape& a) {
    return a.elem == 4 && !a.kv_fp8() && (a.D == 64 || a.D == 128) && a.hq_l % a.hkv_l == 0 && a.hq_l / a.hkv_l <= kCols;
}

hipError_t launch_prefill_f32(const void* q, const void* cache, const int32_t* block_table, const int32_t* cu_seqlens_q,
                              const int32_t* seq_lens, int num_seqs, int total_q, void* out, const AttnShape& a, hipStream_t st) {
    if (total_q == 0) return hipSuccess;
    const int G = a.hq_l / a.hkv_l, tile_tokens = kCols / G;
    const unsigned grid = static_cast<unsigned>(total_q / tile_tokens + num_seqs) * a.hkv_l;
    auto run = [&](auto kernel) {
        kernel<<<grid, kWaves * 64, 0, st>>>(static_cast<const float*>(q), static_cast<const float*>(cache), block_table, cu_seqlens_q,
                                             seq_lens, num_seqs, static_cast<float*>(out), a, G, tile_tokens);
        return hipGetLastError();
    };
    return a.D == 64 ? run(prefill_f32_kernel<64>) : run(prefill_f32_kernel<128>);
}

}  // namespace shiftattn
