// CPU test of the folded grids: every workgroup has one place, and each dimension
// stays within what a launch holds.
#include <cstdio>

#include "../paper_2303_14495_amd/csrc/gl_fold.hpp"

static int fails = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
            ++fails;                                                \
        }                                                           \
    } while (0)

int main() {
    const int64_t rows = (int64_t)1 << 31;
    const int64_t sizes[] = {1, 2, 255, gl::kFoldRow - 1, gl::kFoldRow, gl::kFoldRow + 1, 3 * gl::kFoldRow,
                             ((int64_t)1 << 28) * 16 / 256,  // 2^28 rows of 16 lanes: 2^32 threads
                             rows * 16 / 256,                // the most rows, 16 lanes each
                             rows / 4,                       // a wavefront per point, the most points
                             rows * 2 * 13 / 256 + 1};       // 26 vectors per point
    for (const int64_t blocks : sizes) {
        const gl::Fold f = gl::fold_blocks(blocks);
        CHECK((int64_t)f.x * 1024 < ((int64_t)1 << 32));
        CHECK(f.y >= 1 && f.y <= 65535);
        CHECK((int64_t)f.x * f.y >= blocks);
        CHECK((int64_t)f.x * (f.y - 1) < blocks);
        CHECK(gl::folded(0, 0, f.x) == 0);
        CHECK(gl::folded(f.x - 1, f.y - 1, f.x) == (int64_t)f.x * f.y - 1);
        if (f.y > 1) CHECK(gl::folded(0, 1, f.x) == gl::folded(f.x - 1, 0, f.x) + 1);
    }
    std::printf(fails ? "%d failures\n" : "ok\n", fails);
    return fails ? 1 : 0;
}
