// Prints the decode plans of the built library, for tests that run without a GPU: one problem per
// input line, "batch n_q_heads n_kv_heads n_kept bits group outliers decode_splits workspace_bytes"
// (workspace_bytes 0: as many as the library states), one answer per line, "accepted n_splits n_waves
// part_bytes part_off counter_bytes stated_bytes".
// Test infrastructure only.
#include <cstdio>

#include "kvqp_internal.h"

int main() {
    int batch, hq, hkv, n, bits, group, outliers, splits;
    size_t bytes;
    while (std::scanf("%d %d %d %d %d %d %d %d %zu", &batch, &hq, &hkv, &n, &bits, &group, &outliers, &splits, &bytes) == 9) {
        kvqp_cfg c{};
        c.batch = batch; c.n_q_heads = hq; c.n_kv_heads = hkv; c.head_dim = 128; c.bits = bits; c.group_size = group;
        c.outlier_threshold = outliers ? 6.0f : 0.0f; c.decode_splits = splits; c.sm_scale = 0.088f;
        const size_t stated = kvqp::decode_ws_bound(c);
        kvqp::DecodePlan p = kvqp::plan_decode(c, n);
        const bool ok = p.fit(bytes ? bytes : stated);
        std::printf("%d %d %d %zu %zu %zu %zu\n", (int)ok, p.n_splits, p.n_waves, p.part_bytes, p.part_off,
                    kvqp::decode_ws_header_bytes(c), stated);
    }
    return 0;
}
