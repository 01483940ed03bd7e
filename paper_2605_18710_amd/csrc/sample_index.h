// The sample that a position belongs to, without an integer division: kernels and host tests compile the same function.
#pragma once

// floor(e / N) for positions e >= 0 of N to a sample, inv = 1 / N in fp32: e + 1/2 is exact, the two roundings (of inv and of the product)
// move the quotient by about 2^-23 of itself, and it lies 1 / 2N or more from a whole number, so the result is exact below 2^22 - 1.
constexpr int kSampleMax = 1 << 21;
constexpr int sample_of(int e, float inv) { return (int)(((float)e + 0.5f) * inv); }
