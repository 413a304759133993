// One time step of the curvilinear wave LBM (BGK, tau = 1/2), fused
// collide-and-push-stream with walls, plus probe recording.
//
// Per node x (Sec. III; c_s = c, w_0 = 1 - D c^2, w_l = c^2/2):
//   S   = sqrt(g) P = sum_l f_l
//   A^{de} = c^2 S Mhat^{de}            (metric part of the stress)
//   K_d = sqrt(g) J'^d = f_{+d} - f_{-d} - (c^2/2) S Gamh^d
//         - (1/4) sum_e [A^{de}(x + e_e) - A^{de}(x - e_e)]
//   f*_0 = 2 w_0 S - f_0,  f*_{+-d} = c^2 S +- K_d - f_{+-d}   (2 f^eq - f)
//   push: f_l(x + xi_l, t + 1) = f*_l(x); a link that crosses a wall feeds
//   the opposite population at x: bounce-back D f*_l, free f*_{lbar},
//   fixed -f*_l.
// Beyond a wall A is mirrored: even for bounce-back and free walls, odd for
// fixed walls.  The gradient uses S of the same (pre-collision) time level.
#include "march_common.h"

namespace lbw {
namespace {

constexpr int kBlock = 256;

__device__ inline float node_sum(const float* __restrict__ f, int64_t N, int64_t m) {
    float s = f[m];
#pragma unroll
    for (int l = 1; l < 5; ++l) s += f[l * N + m];
    return s;
}

// One thread per node, the neighbours' sums read through the caches; the
// last workgroup records the probes.
__global__ __launch_bounds__(kBlock) void step_simple_kernel(GeomDev g, ProbeArgs pr, const float* __restrict__ fin,
                                                            float* __restrict__ fout) {
    constexpr int Q = 5;
    if (blockIdx.x == gridDim.x - 1) {
        march::record_probes<Q>(g, pr, 1, fin);
        return;
    }
    const int64_t n = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.N) return;
    const int64_t N = g.N;
    const int n0 = g.n0, n1 = g.n1;
    const int i0 = (int)((uint32_t)n % (uint32_t)n0);
    const int i1 = (int)((uint32_t)n / (uint32_t)n0);

    float f[Q];
#pragma unroll
    for (int l = 0; l < Q; ++l) f[l] = fin[l * N + n];
    float S = f[0];
#pragma unroll
    for (int l = 1; l < Q; ++l) S += f[l];

    const float* te = g.tab + (size_t)i0 * kTabF32;
    const float cM00 = te[0], cM11 = te[3], hG0 = te[4];

    float A00[2], A11[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int s = side == 0 ? 1 : -1;
        int wall = 0;
        int j = link_coord(i0, s, n0, g.bc_lo[0], g.bc_hi[0], &wall);
        A00[side] = j >= 0 ? g.tab[(size_t)j * kTabF32] * node_sum(fin, N, n + (j - i0))
                           : march::ghost(wall, cM00 * S);
        // (the axis-1 coefficients do not depend on i1)
        j = link_coord(i1, s, n1, g.bc_lo[1], g.bc_hi[1], &wall);
        A11[side] = j >= 0 ? cM11 * node_sum(fin, N, n + (int64_t)(j - i1) * n0) : march::ghost(wall, cM11 * S);
    }
    float fs[Q];
    march::collide_2d(f, S, A00[0], A00[1], A11[0], A11[1], hG0, g.c2, g.two_w0, fs);

    fout[n] = fs[0];
    const int idx[2] = {i0, i1};
    const int nn[2] = {n0, n1};
    const int64_t stride[2] = {1, n0};
#pragma unroll
    for (int l = 1; l < Q; ++l) {
        const int a = (l - 1) >> 1;
        const int s = (l & 1) ? 1 : -1;
        const int lb = (l & 1) ? l + 1 : l - 1;
        int wall = 0;
        const int j = link_coord(idx[a], s, nn[a], g.bc_lo[a], g.bc_hi[a], &wall);
        if (j >= 0)
            fout[l * N + n + (int64_t)(j - idx[a]) * stride[a]] = fs[l];
        else
            fout[lb * N + n] = march::bounce(wall, g.damp, fs[l], fs[lb]);
    }
}

}  // namespace

hipError_t launch_step(const GeomDev& g, const ProbeArgs& pr, const float* fin, float* fout, hipStream_t st) {
    const unsigned blocks = (unsigned)((g.N + kBlock - 1) / kBlock) + 1;  // + probe block
    hipLaunchKernelGGL(step_simple_kernel, dim3(blocks), dim3(kBlock), 0, st, g, pr, fin, fout);
    return hipGetLastError();
}

}  // namespace lbw
