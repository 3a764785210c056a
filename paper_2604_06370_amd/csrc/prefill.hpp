// What the two prefill kernels and their entry point share.
#pragma once

#include <hip/hip_runtime.h>

#include "mfma.hpp"

namespace fkvp {

struct PrefillArgs {
    const uint16_t *q, *base_kv, *res_kv, *lora_b;
    const int32_t *adapter_idx, *base_bt, *res_bt, *seq_lens, *q_indptr;
    const float *rope_cos, *rope_sin;
    uint16_t *out;
    int32_t n_agents, hq, hkv, max_pages, blocks_per_agent_head;
    float scale_log2;
    int32_t rope_rows;  // positions the RoPE tables hold
};

constexpr int kXcds = 8;
constexpr int kCus = 256;  // compute units of the GPU

// Rows of an agent's chunk that its query blocks do not reach (a max_q_per_agent below the
// agent's row count) are written as NaN by the agent's last block, so the shortfall shows in
// the output instead of leaving stale memory there.
__device__ __forceinline__ void poison_unreached_rows(const PrefillArgs &p, int q0, int nq, int h, int g, int reach) {
    using namespace fkvk;
    const uint32_t nan2 = 0x7fc07fc0u;  // two bf16 quiet NaNs
    for (int64_t i = threadIdx.x; i < (int64_t)(nq - reach) * g * 32; i += blockDim.x) {
        const int64_t row = i / 32, c = i % 32;
        const int tok = reach + (int)(row / g), j = (int)(row % g);
        uint16_t *orow = p.out + ((int64_t)(q0 + tok) * p.hq + h * g + j) * 128;
        *reinterpret_cast<u32x2 *>(orow + 4 * c) = u32x2{nan2, nan2};
    }
}

// Launch of the pipelined kernel (prefill_stream.hip) with 128 or 256 query rows per workgroup.
hipError_t launch_stream(int r, int g, bool rope, bool rows128, const PrefillArgs &pa, hipStream_t st, void *const *ev);

}  // namespace fkvp
