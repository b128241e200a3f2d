// tppo_plan_build: the work plan of a batch layout (plan.h), built once and
// handed to tppo_egae*, tppo_ppo_losses and tppo_ppo_losses_backward so that
// none of them has to cut the batch into tiles again.  tppo_select builds the
// same plan as a by-product of the token filter (Sec. 3.2).
#include <atomic>

#include "plan_build.h"

namespace tppo {

uint32_t next_call_tag() {
    static std::atomic<uint32_t> counter{0};
    uint32_t t = counter.fetch_add(1, std::memory_order_relaxed) + 1;
    if (t == 0) t = counter.fetch_add(1, std::memory_order_relaxed) + 1;   // 0 means "never written"
    return t;
}

int device_compute_units() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> known[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
    if (dev < kMaxDevices) {
        const int v = known[dev].load(std::memory_order_relaxed);
        if (v > 0) return v;
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (dev < kMaxDevices && cus > 0) known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// Workgroups 0 .. parts-1 build the list, workgroup `parts` counts the two token sets meanwhile, the remaining
// workgroups zero the tagged words.
__global__ __launch_bounds__(kBuildThreads) void plan_build_kernel(const int32_t* __restrict__ resp_off,
                                                                   const int32_t* __restrict__ keep_len,
                                                                   const int32_t* __restrict__ done, int B,
                                                                   int n_resp, int cap, int parts, void* plan_raw,
                                                                   int32_t* status) {
    __shared__ union {
        BuildLds build;
        SetLds sets;
    } s;
    const Plan pl = plan_view(plan_raw, cap);
    const int block = blockIdx.x;
    if (block > parts) {
        clear_words(pl, block - parts - 1, (int)gridDim.x - parts - 1);
    } else if (block == parts) {
        count_sets(pl, s.sets, resp_off, keep_len, done, B);
    } else {
        if (block == 0 && threadIdx.x == 0 && (resp_off[0] != 0 || resp_off[B] != n_resp))
            set_status(status, TPPO_STATUS_BAD_LAYOUT);
        build_list(pl, s.build, resp_off, keep_len, done, keep_len != nullptr, B, n_resp, block, parts, status);
    }
}

int launch_plan_build(const int32_t* resp_off, const int32_t* keep_len, const int32_t* done, int64_t B,
                      int64_t n_resp, int64_t cap, void* plan_raw, int32_t* status, hipStream_t s) {
    const int parts = build_parts(B);
    int64_t zero_groups = (plan_words(cap) + kBuildThreads * 8 - 1) / (kBuildThreads * 8);
    zero_groups = zero_groups < 1 ? 1 : zero_groups > 4096 ? 4096 : zero_groups;
    hipLaunchKernelGGL(plan_build_kernel, dim3(parts + 1 + (int)zero_groups), dim3(kBuildThreads), 0, s, resp_off,
                       keep_len, done, (int)B, (int)n_resp, (int)cap, parts, plan_raw, status);
    return launch_result();
}

}  // namespace tppo

extern "C" size_t tppo_plan_bytes(int64_t n_resp, int64_t B) {
    if (n_resp < 0 || B < 0) return 256;
    return tppo::plan_bytes_for(tppo::plan_max_tiles(n_resp, B));
}

extern "C" int tppo_plan_build(const int32_t* resp_off, const int32_t* keep_len, const int32_t* done, int64_t B,
                               int64_t n_resp, void* plan, size_t plan_bytes, int32_t* status, void* stream) {
    using namespace tppo;
    if (B < 0 || n_resp < 0 || n_resp > INT32_MAX - kTileTokens || B > INT32_MAX / 4) return TPPO_ERR_SIZE;
    if (n_resp > 0 && B == 0) return TPPO_ERR_SIZE;
    if (!resp_off || (B > 0 && !done)) return TPPO_ERR_NULL;
    if (plan_max_tiles(n_resp, B) > INT32_MAX / 8) return TPPO_ERR_SIZE;
    if (!plan || !is_aligned(plan, 256) || plan_bytes < tppo_plan_bytes(n_resp, B)) return TPPO_ERR_WORKSPACE;
    return launch_plan_build(resp_off, keep_len, done, B, n_resp, plan_max_tiles(n_resp, B), plan, status,
                             static_cast<hipStream_t>(stream));
}
