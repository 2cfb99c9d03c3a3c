// CPU loop nests (gene bit 0) and the host-side bfloat16 encoder.
#pragma once

#include <cstddef>
#include <cstdint>

namespace ofl {

float bf16_bits_to_f32(uint16_t q);
uint16_t f32_to_bf16_rne(float x);

void cpu_sweep_f32(int I, int J, int K, const float *const coef[12], const float *p, float *wrk2, float omega);
void cpu_sweep_bf16(int I, int J, int K, const uint16_t *const coef[12], const float bias[12], const float *p,
                    float *wrk2, float omega);
double cpu_residual(int I, int J, int K, const float *p, const float *wrk2, float omega);
void cpu_copyback(int I, int J, int K, const float *wrk2, float *p);
// q[a][t] = bfloat16(fl32(x[a][t] - bias[a])), round to nearest even, for arrays of
// n values; bias: 0, or with `offset` the middle of the array's range where
// bfloat16 does not hold the array exactly.
void cpu_encode_bf16(const float *const *x, int arrays, size_t n, bool offset, float *bias, uint16_t *const *q);
int cpu_threads();

}  // namespace ofl
