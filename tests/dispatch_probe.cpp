// The library's host layer (pam_api.cpp) with its kernel launches and the HIP
// calls around them replaced by records of what would be launched, so that the
// choice of kernel and plan can be tested through the C ABI without a GPU.
// Built by dispatch_probe.py.

#include "pam_api.cpp"

namespace {
// kernel: 1 tiled product, 2 few rows, 3 small product, 4 exact derivative,
// 5 reduction of K slices, 6 zero fill.
struct Launch {
    int64_t kernel, tile_m, tile_n, kgroups, splits, k_per_split, whole, split_tiles, few_rows_of_a, batch;
};
constexpr int kMost = 8;
Launch g_launches[kMost];
int g_count = 0;

hipError_t record(const Launch &l) {
    if (g_count < kMost)
        g_launches[g_count] = l;
    ++g_count;
    return hipSuccess;
}
Launch of(int64_t kernel, int64_t tm, int64_t tn, int64_t kg, const pamk::GemmParams &p) {
    return {kernel, tm, tn, kg, p.splits, p.k_per_split, p.whole, p.split_tiles, 0, 0};
}
}  // namespace

namespace pamk {
hipError_t launch_pam_mul(const float *, const float *, float *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_pad(const float *, const float *, float *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_palog2(const float *, float *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_paexp2(const float *, float *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_round_mantissa(const float *, float *, int64_t, int, hipStream_t) { return hipSuccess; }
hipError_t launch_pam_gemm(int tm, int tn, int kg, bool, bool, bool, const GemmParams &p, hipStream_t) {
    return record(of(1, tm, tn, kg, p));
}
hipError_t launch_pam_skinny(bool rows, bool, const GemmParams &, int64_t batch, hipStream_t) {
    return record({2, 0, 0, 0, 0, 0, 0, 0, rows, batch});
}
hipError_t launch_pam_small(bool, bool, bool, GemmParams, int64_t batch, hipStream_t) {
    return record({3, 0, 0, 0, 0, 0, 0, 0, 0, batch});
}
hipError_t launch_pam_exact_grad(bool, const GemmParams &p, hipStream_t) {
    return record(of(4, kExactTileM, kExactTileN, 1, p));
}
hipError_t launch_split_tile_reduce(int tm, int tn, const GemmParams &p, hipStream_t) {
    return record(of(5, tm, tn, 0, p));
}
hipError_t launch_fill_zero(float *, int32_t, int32_t, int64_t, int64_t, int64_t, hipStream_t) {
    return record({6, 0, 0, 0, 0, 0, 0, 0, 0, 0});
}
hipError_t scratch_address(void **out) {
    *out = reinterpret_cast<void *>(uintptr_t{4096});
    return hipSuccess;
}
}  // namespace pamk

extern "C" {
// The launches since the last call (at most kMost of them), and their count.
int probe_take(Launch *out) {
    const int n = g_count;
    std::memcpy(out, g_launches, sizeof g_launches);
    g_count = 0;
    return n;
}
hipError_t hipGetDevice(int *dev) {
    *dev = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *prop, int) {
    std::memset(prop, 0, sizeof *prop);
    std::strcpy(prop->gcnArchName, "gfx950");
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "no GPU here"; }
hipError_t hipDeviceGetAttribute(int *, hipDeviceAttribute_t, int) { return hipErrorNoDevice; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipErrorNoDevice; }
hsa_status_t hsa_init() { return HSA_STATUS_ERROR; }
hsa_status_t hsa_shut_down() { return HSA_STATUS_ERROR; }
hsa_status_t hsa_iterate_agents(hsa_status_t (*)(hsa_agent_t, void *), void *) { return HSA_STATUS_ERROR; }
hsa_status_t hsa_agent_get_info(hsa_agent_t, hsa_agent_info_t, void *) { return HSA_STATUS_ERROR; }
}
