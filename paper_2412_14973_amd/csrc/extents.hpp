// Sizes that the FP32 product kernel's 32-bit byte offsets reach (host code).
#pragma once
#include <cstdint>

namespace tlr {

constexpr int64_t OFFSETS_END = (int64_t)1 << 32;

// The buffers of a product's operands, A as M x K (ta: K x M) with pitch lda and B as K x N with pitch ldb (GM_LINE: B2
// b2_off entries after B). Their lengths come from the true sizes: what lies past the last row reads zero. The offsets
// run over the padded ones, and one past 2^32 would come round to the operand's first rows, so those have to fit too.
struct Extents {
    bool fit;
    uint32_t bytesA, bytesB;
};
inline Extents gemm_extents(int64_t M, int64_t N, int64_t K, int64_t Mt, int64_t Kt, bool ta, int64_t lda, int64_t ldb,
                            int64_t b2_off) {
    auto over = [](int64_t cols, int64_t ld) { return cols > ld ? cols - ld : 0; };   // columns past a last row
    const int64_t endA = (ta ? K * lda + over(M, lda) : M * lda) * 8, endB = (K * ldb + over(N, ldb) + b2_off) * 8;
    return Extents{endA < OFFSETS_END && endB < OFFSETS_END, (uint32_t)((ta ? Kt : Mt) * lda * 8),
                   (uint32_t)((Kt * ldb + b2_off) * 8)};
}

// A field (ns x nr, padded to lds x ldk) of an FP32 call: the same limit whether D is read in place or from a padded copy
inline bool field_fits(int64_t lds, int64_t ldk) { return lds * ldk * 8 < OFFSETS_END; }

}  // namespace tlr
