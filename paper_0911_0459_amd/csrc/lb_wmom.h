// The binary model's post-collision state stored as seven moment planes ("moment
// storage", schedule 6; the step over it is lb_block_bin).
//
// With the rates of Appendix A the moments e, eps, qx and qy relax fully to
// their equilibria, so the nine post-collision populations of a node follow
// from seven numbers (PostState: rho - rho_ref, j*, the axis and diagonal
// common parts b and d, pxx*, pxy*).  Schedule 6 stores those seven (j* as
// j*/3), FP32, and phi: 32 bytes per node instead of 40 of the population
// storage.  phi is in fixed point, as in every binary step (phi_of_fixed).
// Streaming needs the populations of the neighbours, so a step rebuilds them
// (FP32, from j/3) into LDS, where the pulls read them.
#pragma once
#include "lb_strip.h"

namespace lbk {

constexpr int NMOM = 7;   // planes of the stored post-collision state

// The stored planes: rho - rho_ref, jx*/3, jy*/3, b, d, pxx*, pxy*.  The
// momentum is stored divided by 3 because the populations take j/3 and
// j/12 = (j/3)/4: rebuilt from j itself in FP32, the rounded constants 1/3 and
// 1/12 (both 3e-8 too large) would amplify the streamed momentum by that much
// every step, a bias that moves an interface measurably over 10^4 steps.  From
// j/3 the rebuild uses exact scalings by powers of two and rounded sums only.
__device__ __forceinline__ void pops_of_stored(const float (&m)[NMOM], float (&f)[9]) {
    const float a7 = 0.25f * m[5], a8 = 0.25f * m[6];
    const float jx3 = m[1], jy3 = m[2];
    const float jpp = 0.25f * (jx3 + jy3), jpm = 0.25f * (jx3 - jy3);
    const float cx = m[3] + a7, cy = m[3] - a7, cp = m[4] + a8, cm = m[4] - a8;
    f[1] = cx + jx3;
    f[2] = cx - jx3;
    f[3] = cy + jy3;
    f[4] = cy - jy3;
    f[5] = cp + jpp;
    f[6] = cp - jpp;
    f[7] = cm - jpm;
    f[8] = cm + jpm;
    f[0] = m[0] - 4.f * (m[3] + m[4]);
}

// In-place conversion of one arena's f regions (every capillary: blockIdx.y
// strides over them)
// between the nine populations and the seven-plane post-collision state: the
// library switches the storage when a launch configuration of the other
// storage is set.  From populations (which a step leaves in the seven-
// dimensional post-collision space): drho = sum f, j/3 with j = sum e f, b and
// d the means of the axis and of the diagonal populations,
// pxx* = (f1+f2)-(f3+f4), pxy* = (f5+f6)-(f7+f8); back by the inverse map.
// FP64 arithmetic, one rounding per stored value.  (phi is in fixed point in
// either storage.)
template <bool TO_STATE>
__global__ void __launch_bounds__(256) lb_convert_kernel(const CapDev* caps, int ncaps, float* arena) {
    for (int cap = blockIdx.y; cap < ncaps; cap += gridDim.y) {
        const CapDev c = caps[cap];
        float* base = arena + c.off_f;
        for (long long k = blockIdx.x * 256LL + threadIdx.x; k < c.plane; k += 256LL * gridDim.x) {
            float* p = base + k;
            if (TO_STATE) {
                double f[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) f[i] = p[i * c.plane];
                const double ax = (f[1] + f[2]), ay = (f[3] + f[4]), dp = (f[5] + f[6]), dm = (f[7] + f[8]);
                const float m[NMOM] = {(float)(f[0] + ((ax + ay) + (dp + dm))),
                                       (float)((((f[1] - f[2]) + (f[5] - f[6])) + (f[8] - f[7])) / 3.0),
                                       (float)((((f[3] - f[4]) + (f[5] - f[6])) + (f[7] - f[8])) / 3.0),
                                       (float)(0.25 * (ax + ay)),
                                       (float)(0.25 * (dp + dm)),
                                       (float)(ax - ay),
                                       (float)(dp - dm)};
#pragma unroll
                for (int i = 0; i < NMOM; ++i) p[i * c.plane] = m[i];
            } else {
                double m[NMOM], o[9];
#pragma unroll
                for (int i = 0; i < NMOM; ++i) m[i] = p[i * c.plane];
                pops_of_state(PostState<double>{m[0], 3.0 * m[1], 3.0 * m[2], m[3], m[4], m[5], m[6]}, o);
#pragma unroll
                for (int i = 0; i < 9; ++i) p[i * c.plane] = (float)o[i];
            }
        }
    }
}

}  // namespace lbk
