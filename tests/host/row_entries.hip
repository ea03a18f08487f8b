// Every entry of a derivative row that a thread of a compiled tile shape reads
// lies inside the row.
#include <cstdio>

#include "pass_kernel.hpp"
#include "pass_variants.hpp"

int main() {
    int shapes = 0, bad = 0;
#define CHECK_SHAPE(N_, A_, B_, M_, P_, S_, PART_)                                                   \
    {                                                                                                \
        ++shapes;                                                                                    \
        int out = 0;                                                                                 \
        for (int t = 0; t < P_ * (A_ > B_ ? A_ : B_); ++t)                                           \
            for (int rows = 0; rows < 2; ++rows)                                                     \
                for (int n1 = 0; n1 < A_; ++n1) {                                                    \
                    const int e = pstd::row_entry<N_, A_, B_>(rows ? t % B_ : t / P_, n1);           \
                    out += e < 0 || e >= N_;                                                         \
                }                                                                                    \
        if (out) std::printf("%d = %d x %d, %d pencils: %d entries out of range\n", N_, A_, B_, P_, out); \
        bad += out;                                                                                  \
    }
    PSTD_VARIANTS(CHECK_SHAPE)
    std::printf("%d shapes\n", shapes);
    return bad || !shapes;
}
