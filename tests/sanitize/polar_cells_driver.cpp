// The polar encoder's phase cells and shares on the CPU, for a build with -fsanitize=undefined,float-cast-overflow.  The exit status
// is what the test reads.
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <initializer_list>

#include "qamw_polar_cells.hpp"

using namespace qamw;

static int fails = 0;
constexpr double PI = 3.14159265358979323846;
#define EXPECT(c) do { if (!(c)) { std::printf("FAILED: %s (line %d)\n", #c, __LINE__); ++fails; } } while (0)

static uint32_t cell(float x0, float x1) {
    const bool upper = x1 < 0.0f || (x1 == 0.0f && x0 < 0.0f);
    return polar_phase_cell(x0, x1, upper, [](float s) { return s < FLT_MIN ? INFINITY : 1.0f / s; });   // as the hardware's, subnormals flushed
}

int main() {
    // every conversion is of a number in range: zeros of either sign, subnormal pairs, pairs on the axes, the largest
    const float tiny[] = {0.0f, -0.0f, FLT_TRUE_MIN, -FLT_TRUE_MIN, 0x1p-130f, FLT_MIN, -FLT_MIN, 1e-30f, 1.0f, -1.0f, 0.99e15f, -0.99e15f};
    for (float x0 : tiny)
        for (float x1 : tiny) EXPECT(cell(x0, x1) < (uint32_t)PF_PHASE_CELLS);
    // and the cell is that of the angle, within the margin of 1e-5 that the table's entries leave
    for (int i = 0; i < 100000; ++i) {
        const double a = PI * i / 100000, place = std::cos(a) / (std::fabs(std::cos(a)) + std::fabs(std::sin(a)));
        for (double r : {1e-25, 1.0, 1e14})
            for (int sign : {1, -1}) {
                const int at = (int)cell((float)(sign * r * std::cos(a)), (float)(sign * r * std::sin(a)));
                const double lo = 2.0 * at / PF_PHASE_CELLS - 1.0, hi = 2.0 * (at + 1) / PF_PHASE_CELLS - 1.0;
                if (i) EXPECT((at == 0 || place > lo - 1e-5) && (at + 1 == PF_PHASE_CELLS || place < hi + 1e-5));
            }
    }
    // the parts of a row's items are all of them, once; tables by what a workgroup encodes
    for (int n = 1; n <= 64; ++n)
        for (int parts = 1; parts <= (n + 7) / 8; ++parts) {
            int at = 0;
            for (int p = 0; p < parts; ++p) {
                const PolarPart s = polar_part(n, p, parts, 64);
                EXPECT(s.from == at && s.to >= s.from);
                EXPECT(s.tables == (s.to - s.from >= PF_LUT_ITEMS));
                EXPECT(!polar_part(n, p, parts, 4).tables && !polar_part(n, p, parts, 512).tables);
                at = s.to;
            }
            EXPECT(at == n);
        }
    if (fails == 0) std::printf("polar cells driver ok\n");
    return fails != 0;
}
