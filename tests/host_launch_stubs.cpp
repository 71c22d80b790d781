// Stand-ins for the kernel launchers, for a host-only build of the library's host code (argument
// checks, shape bookkeeping, the Eq. 3 schedule) under AddressSanitizer and UBSan on the CPU.
// Nothing here touches a GPU: a launch that the host code lets through is recorded as done.  For the tests of the rule by
// which stage 3 hands out its rows, stem_test_attention_grid gives what it says for a device of so many compute units.
#include "stem_common.h"

namespace stem {

int launch_pool(const Problem&, int, const void*, const void*, const void*, float*, float*, float*, hipStream_t) {
    return STEM_OK;
}
int launch_block_scores(const Problem&, int, const float*, const float*, const float*, float, float, bool, float*,
                        hipStream_t) {
    return STEM_OK;
}
int launch_group_scores(const Problem&, const float*, int, float*, hipStream_t) { return STEM_OK; }
int launch_select(const Problem&, int, const float*, const int32_t*, int32_t, int32_t, int32_t*, int32_t*, int32_t,
                  hipStream_t) {
    return STEM_OK;
}
int launch_score_select(const Problem&, int, const float*, const float*, const float*, float, float, const int32_t*,
                        int32_t, int32_t, int32_t*, int32_t*, int32_t, float*, hipStream_t) {
    return STEM_OK;
}
int launch_sparse_attn(const Problem&, const void*, const void*, const void*, const int32_t*, const int32_t*, int32_t,
                       bool, float, void*, float*, int32_t*, hipStream_t) {
    return STEM_OK;
}

}  // namespace stem

// lives in a file of its own with the device array it uses; the host-only build has no device
extern "C" int stem_estimate_static(const stem_shape*, const void*, const void*, const void*, float, float, int32_t,
                                    float*, void*) {
    return STEM_ERR_HIP;
}

extern "C" hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
extern "C" hipError_t hipDeviceGetAttribute(int*, hipDeviceAttribute_t, int) { return hipErrorNoDevice; }

// grid: claims, xcds_per_kv_head, items_per_xcd, claim_from, slots, then the rows of each of the eight XCDs
static int units_of_device, units_asked;
static int give_units() { ++units_asked; return units_of_device; }
extern "C" int stem_test_attention_grid(const stem_shape* shape, int32_t kmax, int32_t units, int32_t queue, int64_t* grid,
                                        int32_t* asked) {
    stem::Problem p;
    const int st = stem::make_problem(shape, &p);
    if (st != STEM_OK) return st;
    units_of_device = units;
    units_asked = 0;
    grid[0] = stem::attention_claims_rows(p, kmax, give_units);
    *asked = units_asked;
    const stem::AttentionGrid ag = stem::attention_grid(p, kmax, queue != 0, give_units);
    grid[1] = ag.xcds_per_kv_head;
    grid[2] = ag.items_per_xcd;
    grid[3] = ag.claim_from;
    grid[4] = ag.slots;
    for (int x = 0; x < 8; ++x)
        grid[5 + x] = stem::rows_of_xcd(x, p.Hq, p.R, p.G, ag.items_per_xcd, ag.xcds_per_kv_head);
    return STEM_OK;
}
