// Decode attention: the kernel around decode_flat_body (decode_body.h, which says how it works) and its launches.
#include "decode_body.h"

#include <stdlib.h>

namespace shiftattn {

namespace {

using namespace decode_flat;

constexpr int kWaves = 4;
constexpr int kFlatWorkgroups = 512;                      // two resident per compute unit
constexpr int kFlatWorkers = kFlatWorkgroups * kWaves;    // wavefronts, each with its own token range

template <bool kFp8, bool kAppend>
__global__ __launch_bounds__(kWaves * 64, 2) void decode_flat_kernel(
    const uint16_t* __restrict__ q, int64_t q_stride, uint16_t* __restrict__ cache,
    const int32_t* __restrict__ block_table, int max_blocks, const int32_t* __restrict__ seq_lens,
    float* __restrict__ o_part, float* __restrict__ ml_part, int2* __restrict__ plan, int num_seqs, int hq_l, int hkv_l,
    float c, int r_min, AppendArgs ap) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kWaves * kStageBytes];
    __shared__ int index[kIndexInts];
    decode_flat_body<kFp8, kAppend, kWaves, false>(q, q_stride, cache, block_table, max_blocks, seq_lens, o_part, ml_part, plan, num_seqs, hq_l,
                                            hkv_l, c, r_min, ap, smem, index, blockIdx.x, kFlatWorkgroups);
}

}  // namespace

namespace {

inline int padded_len(int max_seq_len) { return max_seq_len / kGroup * kGroup + kGroup; }  // >= the padded longest context
// sequences per launch: as many as give the kernel's pair index its fill, and few enough that the padded token line of a
// launch (pairs x padded longest context) stays below 2^31, the range of the kernel's 32-bit prefix sums
inline int seqs_per_launch(int max_seq_len, const AttnShape& a) {
    const int64_t by_line = (static_cast<int64_t>(0x7FFFFFFF) - kGroup) / padded_len(max_seq_len > 0 ? max_seq_len : 1) / a.hkv_l;
    const int64_t by_index = kFlatMaxPairs / a.hkv_l;
    return static_cast<int>(by_line < by_index ? by_line : by_index);
}
inline size_t flat_rows(int n, const AttnShape& a) { return decode_mfma_rows_for(kFlatWorkers, n, a); }

}  // namespace

size_t decode_mfma_rows_for(int workers, int n, const AttnShape& a) {
    return (static_cast<size_t>(workers) + static_cast<size_t>(n) * a.hkv_l) * (a.hq_l / a.hkv_l);
}

size_t decode_mfma_workspace_for(int workers, int n, const AttnShape& a) {
    return decode_mfma_rows_for(workers, n, a) * (kD + 2) * sizeof(float) + static_cast<size_t>(n) * a.hkv_l * sizeof(int2);
}

bool decode_mfma_one_launch(int num_seqs, int max_seq_len, const AttnShape& a) {
    return decode_mfma_supported(a, num_seqs, max_seq_len) && num_seqs <= seqs_per_launch(max_seq_len, a);
}

// tokens per wavefront never fall below this, so that no output row has more parts than the
// merge kernel holds (and tiny batches are not shredded into one-group partials)
int decode_mfma_r_min(int max_seq_len) {
    const int padded_max = (max_seq_len + kGroup - 1) / kGroup * kGroup;
    const int r_min = (padded_max / (kMaxParts - 24) + kGroup) / kGroup * kGroup;
    return r_min < 2 * kGroup ? 2 * kGroup : r_min;
}

bool decode_mfma_supported(const AttnShape& a, int /*num_seqs*/, int max_seq_len) {
    return a.elem == 2 && a.D == kD && a.hq_l % a.hkv_l == 0 && a.hq_l / a.hkv_l <= 16 && a.hkv_l <= kFlatMaxPairs &&
           max_seq_len <= 0x7FFFFFFF - 2 * kGroup && seqs_per_launch(max_seq_len, a) >= 1;
}

size_t decode_mfma_workspace(int num_seqs, int max_seq_len, const AttnShape& a) {
    const int per = seqs_per_launch(max_seq_len, a);
    const int n = num_seqs < per ? num_seqs : per;
    return decode_mfma_workspace_for(kFlatWorkers, n, a);
}

bool decode_mfma_appends(int /*num_seqs*/, const AttnShape& /*a*/) { return true; }

hipError_t launch_decode_mfma(const void* q, const void* k_new, const void* v_new, const int64_t* slots, void* cache,
                              const int32_t* block_table, const int32_t* seq_lens, int num_seqs, int max_seq_len,
                              void* out, void* workspace, const AttnShape& a, hipStream_t st) {
    if (num_seqs == 0) return hipSuccess;  // max_seq_len 0: every row is padding, the kernels write their zeros
    const float c = a.scale * a.k_scale * 1.4426950408889634f;  // logits of an FP8 cache carry k_scale
    const int r_min = decode_mfma_r_min(max_seq_len);
    const bool append = k_new != nullptr;
    const int per = seqs_per_launch(max_seq_len, a);
    for (int s0 = 0; s0 < num_seqs; s0 += per) {  // runs share the workspace: same stream, one after the other
        const int n = num_seqs - s0 < per ? num_seqs - s0 : per;
        const size_t rows = flat_rows(n, a);
        float* o_part = static_cast<float*>(workspace);
        float* ml_part = o_part + rows * kD;
        int2* plan = reinterpret_cast<int2*>(ml_part + rows * 2);
        const uint16_t* q_run = static_cast<const uint16_t*>(q) + static_cast<size_t>(s0) * a.q_stride;
        uint16_t* out_run = static_cast<uint16_t*>(out) + static_cast<size_t>(s0) * a.out_stride;
        const AppendArgs ap = {append ? static_cast<const uint16_t*>(k_new) + static_cast<size_t>(s0) * a.kv_stride : nullptr,
                               append ? static_cast<const uint16_t*>(v_new) + static_cast<size_t>(s0) * a.kv_stride : nullptr,
                               append ? slots + s0 : nullptr, a.kv_stride, a.k_scale, a.v_scale};
        auto launch = [&](auto kernel) {
            kernel<<<kFlatWorkgroups, kWaves * 64, 0, st>>>(q_run, a.q_stride, static_cast<uint16_t*>(cache),
                                                            block_table + static_cast<size_t>(s0) * a.max_blocks, a.max_blocks,
                                                            seq_lens + s0, o_part, ml_part, plan, n, a.hq_l, a.hkv_l, c, r_min, ap);
        };
        if (a.kv_fp8()) {
            if (append) launch(decode_flat_kernel<true, true>);
            else launch(decode_flat_kernel<true, false>);
        } else {
            if (append) launch(decode_flat_kernel<false, true>);
            else launch(decode_flat_kernel<false, false>);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = launch_combine_flat(o_part, ml_part, plan, n, a.hq_l, a.hq_l / a.hkv_l, out_run, a.out_stride, a.v_scale, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace shiftattn
