// kern_mfma_cb.hip -- the MFMA path's pipelined kernels (kern_mfma_unit.h) with
// the B tiles built in registers from the compact crossbar (column words,
// per-type plane bytes, axon types) instead of read as int8 weight planes:
// used when one workgroup covers all samples of a core, so that the core's
// B source is read once per tick; and the kernel that builds the planes at load.
// Kept in a translation unit of its own, apart from the plane form
// (kern_mfma.hip).
#include <algorithm>

#include "kern_mfma_unit.h"

namespace ranc {

hipError_t launch_integrate_mfma_cb(const DevNet &n, const TickArgs &a, int two_planes, int samples_per_wg,
                                    hipStream_t st)
{
    return launch_mfma_shape<true>(n, a, two_planes, samples_per_wg, st);
}

hipError_t launch_integrate_mfma_group_cb(const MfmaGroupArgs &g, int total, int k, int code, int ext,
                                          hipStream_t st)
{
    return launch_group_code<true>(g, total, k, code, ext, st);
}

// The int8 planes from the compact source, once at load: [C][N/32][A/32][planes]
// [64 lanes][16 bytes]; lane l, byte b of k-step k covers axon 32k + 16(l/32) + b
// and neuron 32nb + l%32. Two planes: w >> 7 first, then w & 127. One thread per
// lane's bytes of every plane. Packed on the host and uploaded, the planes were
// most of the load: 512 cores of 256 x 256 102 ms, now 11; 256 cores of 512 x 512
// 186, 24.
template <int PL>
__global__ __launch_bounds__(256) void k_build_planes(DevNet n, v4i *planes)
{
    const int KS = n.A / 32;
    const long long total = (long long)n.C * n.NW * KS * 64;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
        const int lane = (int)(i & 63), h = lane >> 5;
        const long long u = i >> 6;   // (c, nb, k)
        const int k = (int)(u % KS), nb = (int)(u / KS % n.NW);
        const size_t c = (size_t)(u / KS / n.NW);
        const int j = 32 * nb + (lane & 31);
        const uint32_t *wsel = mfma_bsrc_wsel(n) + c * PL * 2 * n.N + j;
        uint32_t wl[PL], wh[PL];
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            wl[p] = wsel[(size_t)(2 * p) * n.N];
            wh[p] = wsel[(size_t)(2 * p + 1) * n.N];
        }
        const uint32_t bits = n.colbits[(c * n.W + k) * n.N + j] >> (16 * h);
        const uint4 t4 = reinterpret_cast<const uint4 *>(mfma_bsrc_types(n, PL) + c * n.A)[2 * k + h];
        v4i b[PL];
        compact_b_tile(bits, t4, wl, wh, b);
#pragma unroll
        for (int p = 0; p < PL; ++p)
            planes[(u * PL + p) * 64 + lane] = b[p];
    }
}

hipError_t launch_build_planes(const DevNet &n, int two_planes, uint4 *planes, hipStream_t st)
{
    if (n.vlayout != VLAYOUT_BRICK || !n.colbits || !planes || n.A % 32 || n.W != n.A / 32 || n.NW != n.N / 32)
        return hipErrorInvalidValue;
    const long long total = (long long)n.C * n.NW * n.W * 64;
    const unsigned blocks = (unsigned)std::min<long long>((total + 255) / 256, 16384);
    if (two_planes)
        hipLaunchKernelGGL((k_build_planes<2>), dim3(blocks), dim3(256), 0, st, n, reinterpret_cast<v4i *>(planes));
    else
        hipLaunchKernelGGL((k_build_planes<1>), dim3(blocks), dim3(256), 0, st, n, reinterpret_cast<v4i *>(planes));
    return hipGetLastError();
}

}  // namespace ranc
