// Structure-aware chunking of a token stream (Section 4.3, Appendix B separator table).
// Host code only: the boundaries feed lc_build_index and the close bits of lc_append.
#include "lc_chunker.h"

extern "C" int lc_chunk_tokens(const char* text, const int64_t* offsets, int n, int min_len, int max_len,
                               int32_t* bounds, int capacity, int* n_chunks) {
    if (!offsets || !bounds || !n_chunks || n < 0 || min_len < 1 || max_len < min_len || (!text && n > 0))
        return LC_ERR_INVALID_ARG;
    for (int i = 0; i < n; ++i)
        if (offsets[i + 1] < offsets[i]) return LC_ERR_INVALID_ARG;
    if (capacity < 1) return LC_ERR_CAPACITY;
    int m = 0;
    bounds[0] = 0;
    const bool done = lc_chunk_cuts(
        n, min_len, max_len,
        [&](int64_t i) { return lc_separator_level({text + offsets[i], offsets[i + 1] - offsets[i]}); },
        [&](int64_t end) {
            if (m + 2 > capacity) return false;
            bounds[++m] = (int32_t)end;
            return true;
        });
    if (!done) return LC_ERR_CAPACITY;
    *n_chunks = m;
    return LC_OK;
}
