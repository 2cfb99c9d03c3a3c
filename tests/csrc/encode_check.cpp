// The threaded bfloat16 encoding of a grid's arrays against one value after the
// other: biases and every encoded value, bit for bit.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <limits>
#include <random>
#include <vector>

#include "cpu_nests.hpp"

using namespace ofl;

namespace {

float reference_bias(const std::vector<float> &x) {
    float lo = std::numeric_limits<float>::infinity(), hi = -lo;
    bool exact = true;
    for (float v : x) {
        uint32_t u;
        std::memcpy(&u, &v, sizeof u);
        lo = std::min(lo, v);
        hi = std::max(hi, v);
        exact = exact && (u & 0xffffu) == 0;
    }
    return exact ? 0.f : static_cast<float>(0.5 * (static_cast<double>(lo) + static_cast<double>(hi)));
}

}  // namespace

int main() {
    const float inf = std::numeric_limits<float>::infinity(), nan = std::numeric_limits<float>::quiet_NaN();
    std::mt19937 rng(5);
    // below, at and past the lanes of the scan and the slices of the work
    for (size_t n : {1u, 15u, 16u, 17u, 27u, 65535u, 65536u, 65537u, 300001u, 600000u}) {
        constexpr int kArrays = 7;
        std::vector<std::vector<float>> x(kArrays, std::vector<float>(n));
        std::uniform_real_distribution<float> u(-2.f, 3.f);
        for (int a = 0; a < kArrays; ++a)
            for (size_t t = 0; t < n; ++t)
                x[a][t] = a == 1 ? 1.f : (a == 2 ? -0.f : u(rng));  // 1, 2: exact in bfloat16
        x[3][n / 2] = nan;
        x[4][n - 1] = inf;
        x[5].assign(n, nan);
        x[6][0] = -5.f;
        x[6][n - 1] = 9.f;
        for (bool offset : {false, true}) {
            std::vector<std::vector<uint16_t>> q(kArrays, std::vector<uint16_t>(n, 0xdead));
            const float *src[kArrays];
            uint16_t *dst[kArrays];
            float bias[kArrays];
            for (int a = 0; a < kArrays; ++a) {
                src[a] = x[a].data();
                dst[a] = q[a].data();
            }
            cpu_encode_bf16(src, kArrays, n, offset, bias, dst);
            for (int a = 0; a < kArrays; ++a) {
                const float want = offset ? reference_bias(x[a]) : 0.f;
                if (std::memcmp(&want, &bias[a], sizeof want) != 0 && !(want != want && bias[a] != bias[a])) {
                    std::printf("n %zu array %d offset %d: bias %g, want %g\n", n, a, offset, bias[a], want);
                    return 1;
                }
                for (size_t t = 0; t < n; ++t)
                    if (q[a][t] != f32_to_bf16_rne(x[a][t] - want) && want == want) {
                        std::printf("n %zu array %d offset %d: value %zu differs\n", n, a, offset, t);
                        return 1;
                    }
            }
        }
    }
    std::puts("encoding ok");
    return 0;
}
