// C entry points over csrc/psd_rules.h for tests/test_rules.py.
#include "psd_rules.h"

extern "C" {
int64_t max_items() { return psd::kMaxItems; }
int32_t dense_threads(int64_t keys, int64_t shards) { return psd::dense_threads_for(keys, shards); }
int32_t dense_chunks(int64_t n, int32_t S, int32_t threads) { return psd::dense_chunks_for(n, S, threads); }
int64_t pack_rows(int64_t cu, int64_t cv) { return psd::pack_rows_per_launch(cu, cv); }
int32_t f32_reach(int64_t K, int64_t ldu, int64_t ldv) { return psd::factors_in_reach(K, ldu, ldv, 4, psd::kF32Reserve); }
int32_t bf16_reach(int64_t K, int64_t ldu, int64_t ldv, int64_t rows) { return psd::factors_in_reach(K, ldu, ldv, 2, psd::bf16_reserve(rows)); }
}
