// C ABI of the linear layer (declared and documented in include/sarathi.h): argument checks, the
// split-K decision, the launch.  Stateless: no handle, nothing allocated.
#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "internal.h"
#include "sarathi.h"

using namespace sarathi;

namespace {

bool shape_ok(int32_t T, int32_t N, int32_t K) {
    if (T < 0 || N <= 0 || K <= 0) return false;
    if (N % 128 != 0 || K % 64 != 0 || K > (1 << 20)) return false;
    return (int64_t)T * N < ((int64_t)1 << 40);
}

}  // namespace

extern "C" size_t sarathi_linear_workspace_bytes(int32_t num_tokens, int32_t out_features, int32_t in_features) {
    if (!shape_ok(num_tokens, out_features, in_features) || num_tokens == 0) return 0;
    return plan_linear_parts(num_tokens, out_features, in_features, SIZE_MAX).workspace_bytes(num_tokens, out_features);
}

static sarathi_status plan_part(int part, int32_t num_tokens, int32_t out_features, int32_t in_features, size_t workspace_bytes,
                                sarathi_linear_plan *out) {
    if (!out || num_tokens == 0) return SARATHI_EINVAL;
    if (!shape_ok(num_tokens, out_features, in_features)) return SARATHI_ESHAPE;
    const LinearPlan pl = plan_linear_parts(num_tokens, out_features, in_features, workspace_bytes).part[part];
    *out = sarathi_linear_plan{pl.feature_tile, pl.token_tile, pl.n_tiles, pl.t_tiles, pl.splits, pl.k_per_split};
    return SARATHI_OK;
}

extern "C" sarathi_status sarathi_plan_linear(int32_t num_tokens, int32_t out_features, int32_t in_features,
                                              size_t workspace_bytes, sarathi_linear_plan *out) {
    return plan_part(0, num_tokens, out_features, in_features, workspace_bytes, out);
}

extern "C" sarathi_status sarathi_plan_linear_rest(int32_t num_tokens, int32_t out_features, int32_t in_features,
                                                   size_t workspace_bytes, sarathi_linear_plan *out) {
    return plan_part(1, num_tokens, out_features, in_features, workspace_bytes, out);
}

extern "C" sarathi_status sarathi_linear(const void *x, const void *w, void *y, int32_t num_tokens,
                                         int32_t out_features, int32_t in_features, void *workspace,
                                         size_t workspace_bytes, void *stream) {
    if (!shape_ok(num_tokens, out_features, in_features)) return SARATHI_ESHAPE;
    if (num_tokens == 0) return SARATHI_OK;
    if (!x || !w || !y) return SARATHI_EINVAL;
    const LinearParts parts = plan_linear_parts(num_tokens, out_features, in_features, workspace ? workspace_bytes : 0);
    const hipError_t e = (hipError_t)launch_linear_parts(parts, x, w, y, num_tokens, out_features, in_features, workspace, stream);
    return e == hipSuccess ? SARATHI_OK : SARATHI_EHIP;
}
