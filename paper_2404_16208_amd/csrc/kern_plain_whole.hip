// kern_plain_whole.hip -- all ticks of a call (2^16 per launch at most) for a
// small network, one workgroup per sample.
//
// A network of up to PLAIN_WHOLE_NEURONS neurons fits one CU: its crossbar
// columns, weights, parameters and potentials stay in registers (up to 4
// neurons per thread) and its scheduler (a byte per axon and slot) in LDS for
// the whole call, so a tick needs no launch and no memory but the output
// raster, which nothing waits for. Samples are independent, so the workgroups
// never talk to each other.
// Per tick: (1) a wavefront takes 64 axons of a core at a time, sorted by type
// (see k_plain_ticks), reads their scheduler bytes and input bits and ballots
// them into two axon words in LDS; barrier; (2) per 64-neuron block: one AND
// and population count per word, leak/threshold/reset, spikes stored as bytes
// into the slots of their delays; the slot just read is cleared; barrier.
// Bound: issue. 12 cores of 256 x 256 are 48 blocks of about 60 vector
// instructions on 4 SIMDs, plus two barriers and four LDS round trips.
// Measured, one sample, calls of 128 ticks, us per tick: 12 cores of 256 x 256
// with 4 types 8.4 with a router launch per tick, 3.4 with one launch per tick
// (k_plain_ticks), 1.9 here; 5 cores, 10 samples 9.3 -> 1.3. All 64-axon tasks
// of a wavefront read together instead of one after another spill and lose
// (2.0 and, with 16 cores of 2 types, 4.0 instead of 2.5).
#include "kern_bits.h"
#include "kern_common.h"
#include "ranc_internal.h"

namespace ranc {

static constexpr int WH_THREADS = 1024, WH_WAVES = WH_THREADS / 64;
static constexpr int WH_TASKS = 8;          // 64-axon tasks per wavefront, at most
static_assert(64ull * 512 * PLAIN_WHOLE_TICKS_MAX < 1ull << 32 &&
                  64ull * WH_TASKS * WH_WAVES * PLAIN_WHOLE_TICKS_MAX < 1ull << 32, "a launch's counts overflow");

// LDS (dynamic), in bytes: D + 1 scheduler slots, each the bytes of all axons,
// 64 bytes that stay zero (read for padding positions) and 64 that are never
// read (written for neurons without a destination core); axon words; input
// words of WH_EXT_TICKS ticks.
static constexpr int WH_EXT_TICKS = 32;
struct WholeLds {
    int stride, words, ext, total;   // bytes per slot; offsets
};
__host__ __device__ inline WholeLds whole_lds(int C, int A, int D, int nb, int cin_words)
{
    WholeLds l;
    l.stride = C * A + 128;
    l.words = (D + 1) * l.stride;
    l.ext = l.words + C * nb * 8;
    l.total = l.ext + WH_EXT_TICKS * cin_words * 4;
    return l;
}

// EXT: the extended potential update (lif_update).
template <int G_, int PW, int NPT, bool EXT>
__global__ __launch_bounds__(WH_THREADS) void k_plain_whole(DevNet n, BlockArgs a)
{
    constexpr int SW = G_ * PW;            // axon words
    constexpr int NB = (SW + 1) / 2;       // 64-axon tasks per core
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ unsigned s_de;   // delivered spikes
    const int A = n.A, CA = n.C * A, D1 = n.D + 1;
    const int CinW = a.ext_base ? n.Cin * n.W : 0;
    const WholeLds l = whole_lds(n.C, A, n.D, NB, CinW);
    uint8_t *ring = lds;
    const int stride = l.stride, ring_bytes = D1 * stride;
    uint32_t *words = reinterpret_cast<uint32_t *>(lds + l.words);   // [core][2 NB]
    uint32_t *ext = reinterpret_cast<uint32_t *>(lds + l.ext);       // [tick][Cin W]
    const int s = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = a.ticks;
    const int q0 = (n.tick[0] + a.k0) % n.Q;
    int row = (n.tick[1] + a.k0) % n.RT;

    // the wave's neuron blocks: wave * NPT + i
    const int nbn = n.N >> 6, blocks = n.C * nbn;
    uint32_t col[NPT][SW], dst[NPT];
    int32_t wt[NPT][G_], v[NPT], leak[NPT], thr[NPT], rst[NPT], fl[NPT];
    bool lin[NPT];
    uint32_t om[NPT];   // lanes 0, 1: output-bus neurons of the block's two words, ...
    int ow[NPT];        // ... and their raster columns (-1: none)
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int blk = min(wave * NPT + i, blocks - 1);
        const int c = blk / nbn, j = (blk % nbn) * 64 + lane;
        const size_t cj = (size_t)c * n.N + j;
#pragma unroll
        for (int w = 0; w < SW; ++w)
            col[i][w] = a.cols[((size_t)c * SW + w) * n.N + j];
#pragma unroll
        for (int g = 0; g < G_; ++g)
            wt[i][g] = n.wts[((size_t)c * G_ + g) * n.N + j];
        leak[i] = n.leak[cj];
        thr[i] = n.thr[cj];
        rst[i] = n.rst[cj];
        // LDS offset of the destination's byte, from the slot of the tick
        const uint32_t d = a.dst[cj];
        dst[i] = d != PLAIN_NO_DEST ? (d & 15u) * stride + (d >> 4) : (uint32_t)(stride + CA + 64 + (lane & 63));
        v[i] = n.V[((size_t)c * n.S + s) * n.N + j];
        const size_t m0 = (size_t)c * n.NW + 2 * (blk % nbn);
        om[i] = n.outmask[m0 + (lane & 1)];
        ow[i] = lane < 2 ? n.outword[m0 + lane] : -1;
        fl[i] = n.vmin;
        lin[i] = false;
        if constexpr (EXT) {
            fl[i] = n.floor[cj];
            lin[i] = (n.linmask[cj >> 5] >> (j & 31)) & 1u;
        }
    }
    // the wave's axon tasks (core, 64 positions): LDS byte of the lane's axon
    // within a slot and its bit among a tick's input words
    const int tasks = n.C * NB;
    int ax_byte[WH_TASKS];   // (CA: padding)
    int in_bit[WH_TASKS];    // uniform: what to add for the input bit; NO_INPUT: the core takes none
    constexpr int NO_INPUT = INT32_MIN;
#pragma unroll
    for (int i = 0; i < WH_TASKS; ++i) {
        const int t = wave + WH_WAVES * i;
        ax_byte[i] = CA;
        in_bit[i] = NO_INPUT;
        if (t < tasks) {
            const int c = t / NB, p = a.pos[(size_t)c * (64 * NB) + 64 * (t % NB) + lane];
            const int ci = CinW ? n.in_index[c] : -1;
            if (p < 0x8000)
                ax_byte[i] = c * A + p;
            if (ci >= 0)
                in_bit[i] = (ci - c) * A;
        }
    }

    // scheduled spikes of the next D ticks from the byte ring, which is left
    // empty (the slot before the next tick's still holds what that tick read)
    for (int i = tid; i < ring_bytes / 4; i += WH_THREADS)
        reinterpret_cast<uint32_t *>(ring)[i] = 0u;
    if (tid == 0)
        s_de = 0u;
    lds_barrier();
    for (int d = -1; d < n.D; ++d) {
        const int q = q0 + d < 0 ? n.Q - 1 : (q0 + d) % n.Q;
        uint32_t *g = reinterpret_cast<uint32_t *>(a.ring8 + ((size_t)q * n.S + s) * CA);
        for (int i = tid; i < CA / 4; i += WH_THREADS) {
            if (d >= 0)
                reinterpret_cast<uint32_t *>(ring + d * stride)[i] = g[i];
            g[i] = 0u;
        }
    }
    __syncthreads();

    unsigned de = 0, fired[NPT], ev[NPT];   // per lane: delivered spikes, spikes of its neurons, synaptic events
#pragma unroll
    for (int i = 0; i < NPT; ++i)
        fired[i] = ev[i] = 0;
    int base = 0;   // LDS slot of tick k (k % (D + 1)), in bytes
#pragma unroll 1
    for (int k = 0; k < T; ++k) {
        if (CinW && k % WH_EXT_TICKS == 0) {
            // the input words of the next ticks (every wavefront is past those before)
            const int nk = min(WH_EXT_TICKS, T - k);
            const uint32_t *g = a.ext_base + (size_t)s * a.ext_sstride + (size_t)(a.k0 + k) * a.tick_words;
            for (int i = tid; i < nk * CinW; i += WH_THREADS)
                ext[i] = g[i];
            __syncthreads();
        }
        // 1. axon words: lane i collects task i's pair
        const uint32_t *es = ext + (k % WH_EXT_TICKS) * CinW;
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int i = 0; i < WH_TASKS; ++i) {
            if (wave + WH_WAVES * i >= tasks)
                break;   // wave-uniform
            const bool r = ring[base + ax_byte[i]] != 0;
            de += r;
            uint64_t x = __ballot(r);
            if (in_bit[i] != NO_INPUT) {   // wave-uniform
                const int bit = max(ax_byte[i] + in_bit[i], 0);
                x |= __ballot(ax_byte[i] < CA && ((es[bit >> 5] >> (bit & 31)) & 1u));
            }
            lo = lane == i ? (uint32_t)x : lo;
            hi = lane == i ? (uint32_t)(x >> 32) : hi;
        }
        if (lane < WH_TASKS && wave + WH_WAVES * lane < tasks)
            reinterpret_cast<uint2 *>(words)[wave + WH_WAVES * lane] = uint2{lo, hi};
        lds_barrier();
        // 2. neurons
        for (int i = tid; i < CA / 4; i += WH_THREADS)
            reinterpret_cast<uint32_t *>(ring + base)[i] = 0u;
        uint32_t *rr = n.raster + ((size_t)row * n.S + s) * n.Wout;
        const uint32_t wrap = ring_bytes - base;   // offsets from here on lie in slot 0 and up
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int blk = wave * NPT + i;
            if (blk >= blocks)
                break;   // wave-uniform
            const uint32_t *xw = words + (blk / nbn) * (2 * NB);
            int in = leak[i];
            unsigned evs = 0;
#pragma unroll
            for (int g = 0; g < G_; ++g) {
                unsigned cnt = 0;
#pragma unroll
                for (int w = 0; w < PW; ++w)
                    cnt += __popc(col[i][g * PW + w] & xw[g * PW + w]);
                in += __mul24((int)cnt, wt[i][g]);
                evs += cnt;
            }
            ev[i] += evs;
            bool fire;
            if constexpr (EXT) {
                int32_t vnew;
                fire = lif_update(v[i], in, 0, thr[i], rst[i], n.vmin, n.vmax, fl[i], lin[i], vnew);
                v[i] = vnew;
            } else {
                // 32-bit potentials, absolute reset, no floor: the saturating
                // add is the whole clamp
                const int32_t u = __builtin_elementwise_add_sat(v[i], in);
                fire = u >= thr[i];
                v[i] = fire ? rst[i] : u;
            }
            if (fire)
                ring[base + dst[i] - (dst[i] >= wrap ? ring_bytes : 0)] = 1;
            fired[i] += fire;
            const uint64_t b = __ballot(fire);
            if (ow[i] >= 0)
                rr[ow[i]] = (lane ? (uint32_t)(b >> 32) : (uint32_t)b) & om[i];
        }
        lds_barrier();
        base = base + stride == ring_bytes ? 0 : base + stride;
        row = row + 1 == n.RT ? 0 : row + 1;
    }

    de = wave_sum_dpp(de);
    if (lane == 0)
        atomicAdd(&s_de, de);
    lds_barrier();
    // potentials, counts, and the spikes still scheduled back into the byte ring
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int blk = wave * NPT + i;
        if (blk >= blocks)
            break;
        const int c = blk / nbn, j = (blk % nbn) * 64 + lane;
        n.V[((size_t)c * n.S + s) * n.N + j] = v[i];
        const size_t m = (size_t)c * n.NW + j / 32;
        const unsigned em = wave_sum_dpp(fired[i]), e = wave_sum_dpp(ev[i]);
        const unsigned ro = wave_sum_dpp((n.coremask[m] >> (j & 31)) & 1u ? fired[i] : 0u);
        const unsigned ou = wave_sum_dpp((n.outmask[m] >> (j & 31)) & 1u ? fired[i] : 0u);
        // (delivered spikes of all cores go to the first row: the rows are summed when read)
        const unsigned add = lane == CNT_EMITTED ? em : lane == CNT_ROUTED ? ro : lane == CNT_DELIVERED ? (blk == 0 ? s_de : 0u)
                             : lane == CNT_OUT ? ou : e;
        if (lane < CNT_N)
            n.cnt[((size_t)blk * n.S + s) * CNT_N + lane] += add;
    }
    for (int d = 0; d < n.D; ++d) {
        const int q = (q0 + T + d) % n.Q;
        int ls = base + d * stride;
        ls = ls >= ring_bytes ? ls - ring_bytes : ls;
        uint32_t *g = reinterpret_cast<uint32_t *>(a.ring8 + ((size_t)q * n.S + s) * CA);
        for (int i = tid; i < CA / 4; i += WH_THREADS)
            g[i] = reinterpret_cast<uint32_t *>(ring + ls)[i];
    }
}

bool plain_whole_supported(int C, int A, int N, int G, int D, int Cin, int sorted_words)
{
    const int per = (C * (N / 64) + WH_WAVES - 1) / WH_WAVES;   // neurons per thread
    // more columns per thread spill (16 cores of 256 x 256 with 4 types, 48: 5.0 us per tick, one launch per tick 3.4)
    if (!sorted_words || G * sorted_words > 12 || C * N > PLAIN_WHOLE_NEURONS || per * G * sorted_words > 40)
        return false;
    const int nb = (G * sorted_words + 1) / 2;
    return C * nb <= WH_TASKS * WH_WAVES && whole_lds(C, A, D, nb, Cin * A / 32).total <= 64 * 1024;
}

template <int G_, int PW, int NPT> static void launch_whole_n(const DevNet &n, const BlockArgs &a, int lds, hipStream_t st)
{
    if (n.model_ext)
        hipLaunchKernelGGL((k_plain_whole<G_, PW, NPT, true>), dim3(n.S), dim3(WH_THREADS), lds, st, n, a);
    else
        hipLaunchKernelGGL((k_plain_whole<G_, PW, NPT, false>), dim3(n.S), dim3(WH_THREADS), lds, st, n, a);
}

template <int G_, int PW>
static hipError_t launch_whole_k(const DevNet &n, const BlockArgs &a, hipStream_t st)
{
    const int lds = whole_lds(n.C, n.A, n.D, (G_ * PW + 1) / 2, a.ext_base ? n.Cin * n.W : 0).total;
    switch ((n.C * (n.N / 64) + WH_WAVES - 1) / WH_WAVES) {
    case 1: launch_whole_n<G_, PW, 1>(n, a, lds, st); break;
    case 2: launch_whole_n<G_, PW, 2>(n, a, lds, st); break;
    case 3: launch_whole_n<G_, PW, 3>(n, a, lds, st); break;
    case 4: launch_whole_n<G_, PW, 4>(n, a, lds, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_plain_whole(const DevNet &n, const BlockArgs &a, hipStream_t st)
{
    if (n.vlayout != VLAYOUT_CSN || n.cnt_rows != n.N / 64 || n.S > 65535 || n.Q < n.D + 2 || !a.ring8 || !a.dst ||
        !a.cols || !a.pos || !plain_whole_supported(n.C, n.A, n.N, n.G, n.D, n.Cin, a.sorted_words) || a.ticks < 1 || a.ticks > PLAIN_WHOLE_TICKS_MAX || a.k0 < 0 ||
        a.k0 + a.ticks > n.RT)
        return hipErrorInvalidValue;
    switch (n.G * 32 + a.sorted_words) {
#define RANC_WHOLE(G, PW) case G * 32 + PW: return launch_whole_k<G, PW>(n, a, st);
        RANC_WHOLE(1, 2) RANC_WHOLE(1, 4) RANC_WHOLE(1, 8) RANC_WHOLE(2, 1) RANC_WHOLE(2, 2) RANC_WHOLE(2, 3)
        RANC_WHOLE(2, 4) RANC_WHOLE(2, 5) RANC_WHOLE(2, 6) RANC_WHOLE(4, 1) RANC_WHOLE(4, 2) RANC_WHOLE(4, 3)
        RANC_WHOLE(8, 1)
#undef RANC_WHOLE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ranc
