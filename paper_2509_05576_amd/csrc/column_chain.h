// The sequential steps inside one column block (Section 4.2 steps 4-5), device code shared by quant.hip and flow.hip.
#pragma once
#include "fobq_internal.h"

namespace fobq {

constexpr int CB = 64;

__device__ __forceinline__ double chain_readlane(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// The 64 sequential steps of NR rows by one wavefront (lane = block column; the rows do not interact, their steps
// interleave).  Us: the block's pivot rows Un[j][lane] in LDS, row stride LDU, 0 for lanes <= j, so that a lane keeps the value
// it was quantized at to the end.  The loop therefore holds nothing but the dependent chain -- multiply, rint, max, min, fma,
// readlane, fma; a wavefront is bound by its instruction count (about 4.5 cycles each with two wavefronts on the SIMD) --
// and every lane takes its code and its difference w - q from its final value afterwards, by the same operations.
// EXACT = false forms the quotient w / s as w * (1 / s) (the product is within 2 ulp of the true quotient, so rint of it can
// differ from rint(w / s) only when it lies within 2 ulp of a half-integer) and reports through `suspect` whether any
// column came that close when it was quantized, or ended with a difference that is not finite: such a difference times the
// 0 of a column quantized before it is NaN, and that column's final value is no longer what it was quantized at.
// EXACT = true uses the true division and takes code and difference at the column's own step.
template <bool EXACT, int NR, int LDU>
__device__ __forceinline__ void chain_steps(double (&w)[NR], const double* Us, const double (&s)[NR], const double (&z)[NR],
                                            double maxq, int nb, int lane, double (&mycode)[NR], double (&mydiff)[NR],
                                            bool& suspect)
{
    double rcp_s[NR], lo[NR], hi[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        rcp_s[r] = 1.0 / s[r];
        lo[r] = -z[r];
        hi[r] = maxq - z[r];                      // clamp(c + z, 0, maxq) - z = clamp(c, -z, maxq - z)
    }
    // This lane's pivot-row entries u_j = Us[j][lane] come from LDS 16 steps ahead of their use, so that no memory
    // access sits on the sequential chain and only 32 of the 64 are in registers at a time.
    double ub[2][16];
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) ub[0][jj] = Us[jj * LDU + lane];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g < 3) {
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) ub[(g + 1) & 1][jj] = Us[(16 * (g + 1) + jj) * LDU + lane];
        }
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            const int j = 16 * g + jj;
            if (j < nb) {                             // uniform
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const double tq = EXACT ? w[r] / s[r] : w[r] * rcp_s[r];
                    const double cz = fmin(fmax(rint(tq), lo[r]), hi[r]);        // code - zero
                    const double df = w[r] - s[r] * cz;
                    if (EXACT && lane == j) { mycode[r] = cz + z[r]; mydiff[r] = df; }
                    w[r] -= chain_readlane(df, j) * ub[g & 1][jj];
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);            // keeps the loads of the group after the next from moving up here
    }
    if (EXACT) return;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const double tq = w[r] * rcp_s[r];
        const double c0 = rint(tq);
        const double cz = fmin(fmax(c0, lo[r]), hi[r]);
        mycode[r] = cz + z[r];
        mydiff[r] = w[r] - s[r] * cz;
        suspect |= (fabs(fabs(tq - c0) - 0.5) < 1.0e-9 * fmax(1.0, fabs(tq))) | __builtin_amdgcn_class(mydiff[r], 0x207);      // NaN, -inf, inf
    }
}

}  // namespace fobq
