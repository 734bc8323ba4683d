// Which batches take the kernels for few rows (k_few.hip).  Host code only, no HIP.
#pragma once

#include <stdint.h>

namespace bz {

constexpr int kFewThreads = 512;             // of a workgroup
constexpr int kFewRows = 4;                  // most rows of a batch

inline int few_vectors(int H) { return (H / 8 + kFewThreads - 1) / kFewThreads; }       // 8-element vectors per thread and row

// M rows on a model of hidden size H, qd = query heads * d, nqkv rows of the QKV projection, feed-forward width F.  The norm keeps
// up to two vectors per thread and row (H <= 8192, by which the products with a residual, of H weight rows, are also one tile per
// workgroup), and the weights are addressed with 32-bit byte offsets: every one of the four
// matrices has to end below 2^32 bytes, as in the kernels for more rows.
inline bool few_rows([[maybe_unused]] int M, [[maybe_unused]] int H, [[maybe_unused]] int qd, [[maybe_unused]] int nqkv,
                     [[maybe_unused]] int F) {
#ifdef BZ_FP32_DEBUG
    return false;
#else
    auto addressable = [](int64_t rows, int64_t cols) { return rows * cols < 0x7fffffff; };
    return M >= 1 && M <= kFewRows && few_vectors(H) <= 2 && H % 8 == 0 && F % 8 == 0 && qd % 8 == 0 && addressable(nqkv, H) &&
           addressable(H, qd) && addressable(2 * (int64_t)F, H);
#endif
}

}  // namespace bz
