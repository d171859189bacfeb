// tail.h -- the normal upper tail Q(z) = erfc(z / sqrt 2) / 2 as a table of
// linear cells, shared by the screening kernels of libqlm.
//
// 1024 cells cover z in [-6, 6] (beyond, Q is within 1e-9 of 0 or 1).  A kernel
// forms t = 1536 - (1024 / 12) z in single precision and clamps it to
// [1024, 2048): there every float has exponent 10, so the ten leading mantissa
// bits are the cell.  Cell k holds the line that best fits Q over its width
// (the chord, moved by half its largest deviation), as (a, b) with
// Q ~ a + b t; the two end cells are the constants 0 and 1.  The largest
// error of the lines is below 2.2e-6.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qlm_tail {

constexpr int kCells = 1024;
constexpr double kZ = 6.0;
constexpr double kScale = kCells / (2.0 * kZ);                  // cells per unit z
constexpr float kMid = 1536.0f;
constexpr float kLo = 1024.0f;
constexpr float kHi = 2047.9998779296875f;                      // 2048 - 2^-13
constexpr uint32_t kCellBits = 0x7FE000u;                       // mantissa bits 22..13
// Variances multiplied by this make the reciprocal square root of their sum
// come out in cells per unit of margin.
constexpr double kVarScale = 1.0 / (kScale * kScale);

// The table itself, formed by the compiler in double precision and kept in
// device memory: a kernel copies its 8 KiB into LDS.  (Formed by the kernels,
// three double-precision erfc per thread: k_score took 10.8 us on 8 groups and
// 256 plans, 6.8 with the copy, and the search and the per-request calls spent a
// launch of 4.6 us on it.)
struct alignas(16) Table {
    float c[2 * kCells];                                        // (a, b) of each cell
};

// e^-y for 0 <= y <= 18: e^(y / 4) by its series, to the fourth power.
constexpr double exp_neg(double y)
{
    const double w = y / 4.0;
    double term = 1.0, sum = 1.0;
    for (int n = 1; term > 1e-18 * sum; ++n) {
        term *= w / n;
        sum += term;
    }
    for (int k = 0; k < 2; ++k) sum *= sum;
    return 1.0 / sum;
}

// Q(z) = 1/2 - erf(z / sqrt 2) / 2, 0 <= z <= 6, from the series of positive terms
// erf x = (2 / sqrt pi) e^(-x^2) sum_n 2^n x^(2n+1) / (1 3 5 ... (2n+1))
// (Abramowitz and Stegun 7.1.6; no cancellation, so Q is good to about 1e-15).
constexpr double upper_tail(double z)
{
    const double x = z * 0.70710678118654752440;
    double term = x, sum = x;
    for (int n = 1; term > 1e-18 * sum; ++n) {
        term *= 2.0 * x * x / (2 * n + 1);
        sum += term;
    }
    return 0.5 - 0.56418958354775628695 * exp_neg(x * x) * sum;   // 1 / sqrt pi
}

constexpr Table make_table()
{
    // Q at the cells' edges and middles, half a cell apart, from z = 6 down to
    // -6 (where Q(-z) = 1 - Q(z))
    double q[2 * kCells + 1] = {};
    for (int j = 0; j <= kCells; ++j) {
        q[j] = upper_tail((512.0 - 0.5 * j) / kScale);
        q[2 * kCells - j] = 1.0 - q[j];
    }
    Table t{};
    for (int k = 0; k < kCells; ++k) {
        const double p0 = q[2 * k], pm = q[2 * k + 1], p1 = q[2 * k + 2];
        double c1 = p1 - p0;
        double c0 = p0 + 0.5 * (pm - 0.5 * (p0 + p1));
        // the end cells are flat at exactly 0 and 1 (their Q is within 2e-9 of it),
        // so that clamped margins give exact zero and one terms
        if (k == 0 || k == kCells - 1) {
            c0 = k == 0 ? 0.0 : 1.0;
            c1 = 0.0;
        }
        // the line in t itself (c0 - c1 (1024 + k) + c1 t): no fraction to form
        // in the kernel; the constant is at most 9.6 in size, so its rounding adds
        // below 6e-7
        t.c[2 * k] = (float)(c0 - c1 * (kLo + k));
        t.c[2 * k + 1] = (float)c1;
    }
    return t;
}

static __device__ const Table kTable = make_table();

// Copies the table into LDS (16-byte aligned); every thread tid of a workgroup
// of nthreads calls it.
__device__ inline void stage(float2 *tab, int tid, int nthreads)
{
    const float4 *src = reinterpret_cast<const float4 *>(kTable.c);
    float4 *dst = reinterpret_cast<float4 *>(tab);
    for (int k = tid; k < kCells / 2; k += nthreads) dst[k] = src[k];
}

// Q at the margin num (seconds, slo - E[W]) for the scaled variance vz
// (variance in s^2 times kVarScale): rsq(vz) is in cells per second of margin.
// vz = 0 gives 0 or 1 by the sign of num (0 for num = 0).
__device__ inline float q_of(const float2 *tab, float num, float vz)
{
    const float rs = __builtin_amdgcn_rsqf(vz);
    float t = fmaf(-num, rs, kMid);
    t = __builtin_amdgcn_fmed3f(t, kLo, kHi);         // NaN (0 * inf) -> low end
    const float2 c = tab[(__float_as_uint(t) & kCellBits) >> 13];
    return fmaf(c.y, t, c.x);
}

}  // namespace qlm_tail
