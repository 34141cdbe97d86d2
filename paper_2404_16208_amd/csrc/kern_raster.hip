// kern_raster.hip -- the output file of Sec. IV in bulk: the output-bus spikes
// of every sample over a range of retained ticks, packed into one bit array
// the caller owns, so that a run can be drained chunk by chunk while the next
// chunk runs (streaming, Sec. V) and the host decodes off the critical path.
//
// Output neurons are numbered in ascending (core, neuron) order among the
// neurons whose destination is the output bus. Two layouts:
//   by neuron: u64 [T][Nout][HG], HG = ceil(S / 64); bit i of word (t, o, w)
//              = sample 64 w + i spiked from output neuron o at tick t0 + t;
//   by sample: u32 [T][S][ceil(Nout / 32)]; bit o % 32 of word (t, s, o / 32)
//              = the same event (the compact form for few samples).
// Bits of samples >= S and of output neurons >= Nout are zero; every word of
// the range is written.
//
// Sources: the MFMA and event-driven paths keep the raster neuron-major
// already (history words; on the MFMA path the bits of each 32-sample half
// follow the MFMA result row order sigma32 and are permuted back); the plain
// path keeps, per sample, the cores' neuron words that hold output neurons
// (raster columns).
#include <algorithm>

#include "kern_bits.h"
#include "ranc_internal.h"

namespace ranc {

// Sample-ordered 32-bit word from an MFMA-ordered one: bit i of the result is
// bit sigma32_inv(i) of x. The order permutes nibbles: nibble (b4 b3 b2) goes
// to place (b3 b2 b4), by an exchange of the middle bytes (b4 with b3) and
// of the middle nibbles of each half (b4 with b2).
__device__ inline uint32_t unsigma32(uint32_t x)
{
    uint32_t t = (x ^ (x >> 8)) & 0x0000FF00u;
    x ^= t ^ (t << 8);
    t = (x ^ (x >> 4)) & 0x00F000F0u;
    return x ^ t ^ (t << 4);
}

// ---- by neuron

__global__ __launch_bounds__(256) void k_raster_hist_by_neuron(DevNet n, long long t0, int T, uint64_t *dst)
{
    const long long HG = n.S64 / 64;
    const long long total = (long long)T * n.Nout * HG;
    const bool mfma = n.vlayout == VLAYOUT_BRICK;
    const uint64_t *src = reinterpret_cast<const uint64_t *>(n.raster);
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long t = i / ((long long)n.Nout * HG);
        const long long rest = i - t * n.Nout * HG;   // o * HG + w
        const int row = (int)((t0 + t) % n.RT);
        uint64_t w = src[(size_t)row * n.Nout * HG + rest];
        if (mfma)
            w = (uint64_t)unsigma32((uint32_t)w) | (uint64_t)unsigma32((uint32_t)(w >> 32)) << 32;
        dst[i] = w;
    }
}

// outcol[ow] = (index c * NW + w of raster column ow's neuron word, output
// index of the column's first output neuron). One wavefront per (tick, raster
// column, 64 samples), lane = sample.
__global__ __launch_bounds__(256) void k_raster_plain_by_neuron(DevNet n, const int2 *outcol, long long t0, int T,
                                                                uint64_t *dst)
{
    const int HG = n.S64 / 64;
    const long long wv = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (wv >= (long long)T * n.Wout * HG)
        return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    const int w = (int)(wv % HG);
    const long long r = wv / HG;
    const int ow = (int)(r % n.Wout);
    const int t = (int)(r / n.Wout);
    const int row = (int)((t0 + t) % n.RT);
    const int s = 64 * w + lane;
    const uint32_t word = s < n.S ? n.raster[((size_t)row * n.S + s) * n.Wout + ow] : 0u;
    const int2 oc = outcol[ow];
    uint32_t mask = n.outmask[oc.x];   // uniform
    int o = oc.y;
    uint64_t *drow = dst + ((size_t)t * n.Nout) * HG + w;
    while (mask) {
        const int b = __builtin_ctz(mask);
        mask &= mask - 1u;
        const uint64_t bits = __ballot((word >> b) & 1u);
        if (lane == 0)
            drow[(size_t)o * HG] = bits;
        ++o;
    }
}

// ---- by sample

// A bit transpose, bound by memory (it reads and writes every bit once).
// Workgroup (tick, block of 128 WAVES_ output neurons, TILES_ tiles of 64
// samples): a lane loads its output neuron's words (TILES_ * 8 bytes in a run),
// each 32 neurons x 32 samples is transposed across the lanes of a half-wave,
// and the words go through LDS, so that each sample's 4 WAVES_ words are
// written as one run, 128 bytes with 8 waves. Blocks of samples that read the
// same lines are neighbours in the unit order, which gives each die (blockIdx
// mod 8) a contiguous range, so that the lines are fetched into one L2.
// 32 ticks of 32768 output neurons: 1024 samples (134 MB read and written) 617
// us with 32-byte runs and one broadcast load per neuron, 94 now (2.9 TB/s); 100
// samples 46, 8.4. Few units: 16 ticks, 64 samples, 7 us, 4.7. Streaming stores
// (ordinary ones 73 us when repeated on one raster, 69; 8.3, 7.3).
template <int WAVES_, int TILES_>
__global__ __launch_bounds__(64 * WAVES_) void k_raster_hist_by_sample(DevNet n, long long t0, int total, uint32_t *dst)
{
    constexpr int OWS = 4 * WAVES_;   // output words of a sample
    __shared__ uint32_t sw[64 * TILES_][OWS + 1];
    const int per = gridDim.x >> 3;   // (gridDim.x is a multiple of 8)
    const int u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (u >= total)
        return;   // whole workgroups, before the barrier
    const int HG = n.S64 / 64;
    const int NOW = (n.Nout + 31) / 32;
    const int OB = (NOW + OWS - 1) / OWS, SB = (HG + TILES_ - 1) / TILES_;
    const int tile0 = u % SB * TILES_;
    const int ob = u / SB % OB;
    const int t = u / SB / OB;
    const int row = (int)((t0 + t) % n.RT);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const uint64_t *src = reinterpret_cast<const uint64_t *>(n.raster) + (size_t)row * n.Nout * HG;
    const int sl = n.vlayout == VLAYOUT_BRICK ? sigma32(lane & 31) : lane & 31;   // sample of the lane's bit
    uint64_t w[2][TILES_];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int o = 32 * OWS * ob + 128 * wave + 64 * h + lane;
#pragma unroll
        for (int i = 0; i < TILES_; ++i)
            w[h][i] = o < n.Nout && tile0 + i < HG ? src[(size_t)o * HG + tile0 + i] : 0ull;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TILES_; ++i) {
            const int g = 4 * wave + 2 * h + (lane >> 5);
            sw[64 * i + sl][g] = transpose32((uint32_t)w[h][i], lane);
            sw[64 * i + 32 + sl][g] = transpose32((uint32_t)(w[h][i] >> 32), lane);
        }
    __syncthreads();
    const int words = min(OWS, NOW - OWS * ob);
    const int g = threadIdx.x % OWS;
    for (int k = threadIdx.x / OWS; k < 64 * TILES_; k += 64 * WAVES_ / OWS) {
        const int s = 64 * tile0 + k;
        if (s < n.S && g < words)
            __builtin_nontemporal_store(sw[k][g], dst + (((size_t)t * n.S + s) * NOW + OWS * ob + g));
    }
}

template <int WAVES_, int TILES_>
static void launch_hist_by_sample(const DevNet &n, long long t0, int T, uint32_t *dst, hipStream_t st)
{
    const int NOW = (n.Nout + 31) / 32;
    const long long total = (long long)T * ((NOW + 4 * WAVES_ - 1) / (4 * WAVES_)) * ((n.S64 / 64 + TILES_ - 1) / TILES_);
    hipLaunchKernelGGL((k_raster_hist_by_sample<WAVES_, TILES_>), dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * WAVES_),
                       0, st, n, t0, (int)total, dst);
}

// opos[o] = raster column of output neuron o << 5 | its bit in the column.
// One wavefront per (tick, sample) and 1024 output neurons: lane = output neuron
// of 16 blocks of 64, each two loads deep (position, word) and a ballot; lane i
// keeps word i, so that the words leave as one 128-byte run (the destination
// may be host memory).
// 128 ticks of one sample with 32768 output neurons: 8.5 us with 32 loads in a
// row per word, 5.3 now.
constexpr int RASTER_BLOCKS = 16;
__global__ __launch_bounds__(256) void k_raster_plain_by_sample(DevNet n, const int32_t *opos, long long t0, int T,
                                                                uint32_t *dst)
{
    const int NOW = (n.Nout + 31) / 32;
    const int OB = (NOW + 2 * RASTER_BLOCKS - 1) / (2 * RASTER_BLOCKS);
    const long long wv = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ob = (int)(wv % OB);
    const long long r = wv / OB;   // t * S + s
    if (r >= (long long)T * n.S)
        return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    const long long t = r / n.S;
    const uint32_t *rrow = n.raster + ((size_t)((t0 + t) % n.RT) * n.S + (r - t * n.S)) * n.Wout;
    const int o0 = 64 * RASTER_BLOCKS * ob + lane;
    int p[RASTER_BLOCKS];
    uint32_t x[RASTER_BLOCKS];
#pragma unroll
    for (int i = 0; i < RASTER_BLOCKS; ++i)
        p[i] = opos[min(o0 + 64 * i, n.Nout - 1)];
#pragma unroll
    for (int i = 0; i < RASTER_BLOCKS; ++i)
        x[i] = rrow[p[i] >> 5];
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < RASTER_BLOCKS; ++i) {
        const uint64_t b = __ballot(o0 + 64 * i < n.Nout && ((x[i] >> (p[i] & 31)) & 1u));
        if ((lane >> 1) == i)
            word = (uint32_t)(b >> (32 * (lane & 1)));
    }
    if (lane < 2 * RASTER_BLOCKS && 2 * RASTER_BLOCKS * ob + lane < NOW)
        dst[r * NOW + 2 * RASTER_BLOCKS * ob + lane] = word;
}

hipError_t launch_pack_raster(const DevNet &n, const int2 *outcol, const int32_t *opos, int by_sample, long long t0,
                              int T, void *dst, hipStream_t st)
{
    if (T < 1 || !dst)
        return hipErrorInvalidValue;
    if (n.Nout == 0)
        return hipSuccess;
    const bool plain = n.vlayout == VLAYOUT_CSN;
    if (plain && !(by_sample ? (const void *)opos : (const void *)outcol))
        return hipErrorInvalidValue;
    const int HG = n.S64 / 64;
    if (by_sample) {
        uint32_t *d = static_cast<uint32_t *>(dst);
        if (plain) {
            const long long waves = (long long)T * n.S * ((n.Nout + 64 * RASTER_BLOCKS - 1) / (64 * RASTER_BLOCKS));
            if ((waves + 3) / 4 > INT32_MAX)
                return hipErrorInvalidValue;
            hipLaunchKernelGGL(k_raster_plain_by_sample, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, n, opos, t0,
                               T, d);
        } else {
            // large workgroups (long runs to write) where there are two for
            // every CU, else four times as many small ones
            const long long large = (long long)T * ((n.Nout + 1023) / 1024) * ((HG + 3) / 4);
            if (large >= 512)
                HG == 1   ? launch_hist_by_sample<8, 1>(n, t0, T, d, st)
                : HG == 2 ? launch_hist_by_sample<8, 2>(n, t0, T, d, st)
                          : launch_hist_by_sample<8, 4>(n, t0, T, d, st);
            else
                HG == 1 ? launch_hist_by_sample<2, 1>(n, t0, T, d, st) : launch_hist_by_sample<2, 2>(n, t0, T, d, st);
        }
    } else {
        uint64_t *d = static_cast<uint64_t *>(dst);
        if (plain) {
            const long long waves = (long long)T * n.Wout * HG;
            hipLaunchKernelGGL(k_raster_plain_by_neuron, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, n,
                               outcol, t0, T, d);
        } else {
            const long long total = (long long)T * n.Nout * HG;
            const long long blocks = std::min<long long>((total + 255) / 256, 8192);
            hipLaunchKernelGGL(k_raster_hist_by_neuron, dim3((unsigned)blocks), dim3(256), 0, st, n, t0, T, d);
        }
    }
    return hipGetLastError();
}

}  // namespace ranc
