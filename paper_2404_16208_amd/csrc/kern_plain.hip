// kern_plain.hip -- one tick of integrate + leak/threshold/reset, plain path.
//
// One workgroup per (core, sample), one lane per neuron (N = 64..512 lanes).
// The tick's axon spikes of the core (scheduler slot OR external input) are
// A/32 words that every lane needs, so they are loaded with uniform (scalar)
// loads and pre-masked per axon type. Each lane then reads its neuron's
// crossbar column as A/32 words (coalesced across lanes: colbits is
// [C][W][N]) and counts, per axon type, the spiking connected axons with
// popcount; the input is sum_g count_g * weight[g] (GPU-RANC Sec. II: the
// axon type selects the neuron's weight). Spikes are gathered with a
// wavefront ballot into 32-bit words; output-bus spikes go to the raster.
//
// Two forms. On handles with the byte ring one kernel does the whole tick
// (k_plain_ticks, and k_plain_ticks_batch): every firing lane stores its spike
// in the destination's scheduler itself. On the others, and where a router is asked
// for (k_integrate_plain, k_integrate_plain_batch), the spikes go out as words and
// the router kernels (kern_route.hip) deliver them.
#include <algorithm>

#include "kern_bits.h"
#include "kern_common.h"
#include "ranc_internal.h"

namespace ranc {

static constexpr int PLAIN_BLOCK_TICKS = MFMA_BLOCK_TICKS_MAX;   // ticks per launch, at most

// One (core, sample) on a workgroup of at least N threads (threads past N
// take part in the ballots and the barrier only).
template <int W_, int G_>
__device__ __forceinline__ void integrate_plain_unit(const DevNet &n, const TickArgs &ta, int c, int s)
{
    const int N = n.N;
    const int jt = threadIdx.x;
    const bool live = jt < N;
    const int j = live ? jt : N - 1;   // idle threads mirror the last neuron's loads
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    // Axon spikes of this tick: scheduler slot t%Q OR the external input.
    const uint32_t *slot = n.ring + (((size_t)tick_slot(n, ta.k) * n.S + s) * n.C + c) * W_;
    const int ci = n.in_index[c];
    const uint32_t *ext = (ta.ext_t != nullptr && ci >= 0)
                              ? ta.ext_t + (size_t)s * ta.ext_sstride + (size_t)ci * W_
                              : nullptr;
    uint32_t xt[G_][W_];
    unsigned delivered = 0;
#pragma unroll
    for (int w = 0; w < W_; ++w) {
        const uint32_t r = slot[w];
        delivered += __popc(r);
        const uint32_t x = r | (ext ? ext[w] : 0u);
#pragma unroll
        for (int g = 0; g < G_; ++g)
            xt[g][w] = x & n.typemask[((size_t)c * G_ + g) * W_ + w];
    }

    // Integration: per-type counts of spiking connected axons.
    unsigned cnt[G_];
#pragma unroll
    for (int g = 0; g < G_; ++g)
        cnt[g] = 0;
    const uint32_t *col = n.colbits + (size_t)c * W_ * N + j;
#pragma unroll
    for (int w = 0; w < W_; ++w) {
        const uint32_t cw = col[(size_t)w * N];
#pragma unroll
        for (int g = 0; g < G_; ++g)
            cnt[g] += __popc(cw & xt[g][w]);
    }
    const int32_t *wt = n.wts + (size_t)c * G_ * N + j;
    int in = 0;
    unsigned ev = 0;
#pragma unroll
    for (int g = 0; g < G_; ++g) {
        in += __mul24((int)cnt[g], wt[(size_t)g * N]);
        ev += cnt[g];
    }

    // Leak, threshold, reset.
    const size_t cj = (size_t)c * N + j;
    const size_t vi = ((size_t)c * n.S + s) * N + j;
    int32_t vnew;
    int32_t fl = n.vmin;
    bool lin = false;
    if (n.model_ext) {   // uniform
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (j & 31)) & 1u;
    }
    const bool fire = lif_update(n.V[vi], in, n.leak[cj], n.thr[cj], n.rst[cj], n.vmin, n.vmax, fl, lin, vnew) && live;
    if (live)
        n.V[vi] = vnew;
    if (!live)
        ev = 0;

    // Spike words (ballot), counters, output raster. Each wavefront adds its
    // 64 neurons' counts to its own counter row (no reduction across waves);
    // wave 0 also counts the core's delivered spikes.
    const unsigned long long b = __ballot(fire);
    ev = wave_sum(ev);
    if (lane == 0 && wave < (N >> 6)) {
        unsigned em = 0, ro = 0, ou = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int nw = wave * 2 + h;
            const uint32_t wd = (uint32_t)(b >> (32 * h));
            const size_t m = (size_t)c * n.NW + nw;
            n.spk[((size_t)s * n.C + c) * n.NW + nw] = wd;
            const uint32_t om = wd & n.outmask[m];
            em += __popc(wd);
            ro += __popc(wd & n.coremask[m]);
            ou += __popc(om);
            const int ow = n.outword[m];
            if (ow >= 0)
                n.raster[((size_t)tick_row(n, ta.k) * n.S + s) * n.Wout + ow] = om;
        }
        // the core's delivered spikes are counted once, in row 0
        store_counts(n, ta.k, (size_t)c * (N >> 6) + wave, s, pack_counts(em, ro, ou, wave == 0 ? delivered : 0u, ev));
    }
}

template <int W_, int G_>
__global__ __launch_bounds__(512) void k_integrate_plain(DevNet n, TickArgs ta)
{
    integrate_plain_unit<W_, G_>(n, ta, blockIdx.x, blockIdx.y);
}

// Whole ticks of one core per workgroup (N threads, lane = neuron), delivery
// included. The scheduler is the byte ring: one byte per axon and slot, so that
// a firing neuron delivers its spike with one plain byte store of 1 (several
// spikes to one axon and tick store the same byte, in any order) and no
// router, table or atomic is needed (atomic ORs into the bit ring ran at 18 G
// per second on this GPU, three times the time of the rest of the tick at
// 128 cores x 23 samples). A wavefront's load of 64 axons' bytes and a ballot
// give two axon words.
// SORTED: the axons are taken in order of their type (pos: axon of each
// position, PW words per type), so one AND and one population count per word
// replace one of each per word and type: 24 instead of 64 for four types of
// 256 axons. The columns are 12 instead of 8 words then, so networks whose
// parameters come from memory every tick keep the natural order.
// One tick per launch (several samples per workgroup, the next one's state
// loaded ahead): the slot of the tick before is cleared, which no other
// workgroup reads or writes (the ring has D + 2 slots or more), so no wavefront
// waits for another. BLOCK: a block of ticks of a feed-forward network, whose
// slots are complete before the launch: their words are collected in LDS
// first, so the loop over ticks loads nothing and has no barrier.
// Bound: with one tick, a launch's latency (about 3 us: tick counter -> ring
// bytes -> potential store through memory shared by the XCDs); parameters,
// potentials and the counters' old values are loaded beside it. Measured, us
// per tick, integration and router launch before -> this: 512 cores of 256 x
// 256, one sample 10.9 -> 4.7 (4.4 natural, 4.2 sorted order); 4096 cores 30.6
// -> 19.5 (77 MB of parameters and state, 4 TB/s); 128 cores x 23 samples 18.3
// -> 10.5 (10.3 sorted, 10.7 natural). 512 cores in four layers, 32 ticks, eight
// per launch: 10.9 -> 2.0. Adding the counts in the per-tick ring instead of
// the totals was slower (11.9 at 128 x 23).
enum PlainForm { ONE_SAMPLE, SAMPLES, BLOCK_OF_TICKS };
template <int G_, int SW, bool SORTED, PlainForm FORM>
__global__ __launch_bounds__(512) void k_plain_ticks(DevNet n, BlockArgs a)
{
    constexpr bool BLOCK = FORM == BLOCK_OF_TICKS;
    constexpr int NB = (SW + 1) / 2;             // 64-axon ballots per tick
    constexpr int PW = SORTED ? SW / G_ : SW;    // words per type
    __shared__ uint32_t x_lds[BLOCK ? PLAIN_BLOCK_TICKS : 1][2 * NB];
    const int N = n.N;
    const int c = a.order ? a.order[a.first + blockIdx.x] : (int)blockIdx.x;
    const int s0 = FORM == SAMPLES ? blockIdx.y * a.spw : blockIdx.y, ns = FORM == SAMPLES ? min(a.spw, n.S - s0) : 1;
    const int kb = a.level ? a.k0 + (a.step - a.level[c]) * a.block : a.k0;
    const int nt = BLOCK ? min(kb + a.block, a.k0 + a.ticks) - kb : 1;
    if (kb < a.k0 || nt < 1)
        return;   // whole workgroups, before any barrier
    const int j = threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = N >> 6;

    // axon of the lane in each ballot (past the axons: a valid one, masked)
    int ax[NB];
    uint64_t has[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if constexpr (SORTED) {
            const int p = a.pos[(size_t)c * (64 * NB) + 64 * b + lane];
            ax[b] = p & 0x7FFF;
            has[b] = __ballot(p < 0x8000);
        } else {
            ax[b] = 64 * b + lane;
            has[b] = ~0ull;
        }
    }
    const size_t CA = (size_t)n.C * n.A;
    const uint32_t *cols = (SORTED ? a.cols : n.colbits) + (size_t)c * SW * N + j;
    uint32_t col[SW];
#pragma unroll
    for (int w = 0; w < SW; ++w)
        col[w] = cols[(size_t)w * N];
    int32_t wt[G_];
#pragma unroll
    for (int g = 0; g < G_; ++g)
        wt[g] = n.wts[((size_t)c * G_ + g) * N + j];
    const size_t cj = (size_t)c * N + j;
    const int32_t leak = n.leak[cj], thr = n.thr[cj], rst = n.rst[cj];
    const uint32_t dst = a.dst[cj];
    int32_t fl = n.vmin;
    bool lin = false;
    if (n.model_ext) {   // uniform
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (j & 31)) & 1u;
    }
    int32_t *vp = n.V + ((size_t)c * n.S + s0) * N + j;
    int32_t v_next = *vp;
    // this wave's counter row, lane i < CNT_N its i-th total
    unsigned long long *cp = n.cnt + (((size_t)c * nw + wave) * n.S + s0) * CNT_N + (lane < CNT_N ? lane : 0);
    unsigned long long c_next = *cp;
    const uint32_t *tmask = n.typemask + (size_t)c * G_ * SW;   // (natural order only)
    const size_t m0 = (size_t)c * n.NW + 2 * wave;   // the wave's two neuron words
    const uint64_t cmask = n.coremask[m0] | (uint64_t)n.coremask[m0 + 1] << 32;
    const uint64_t omask = n.outmask[m0] | (uint64_t)n.outmask[m0 + 1] << 32;
    const int ow = lane < 2 ? n.outword[m0 + lane] : -1;
    const uint32_t om = (uint32_t)(omask >> (32 * (lane & 1)));
    const int ci = n.in_index[c];
    const bool has_ext = a.ext_base != nullptr && ci >= 0;   // uniform

    const int q0 = (n.tick[0] + kb) % n.Q, row0 = (n.tick[1] + kb) % n.RT;
    auto slot_of = [&](int q, int s) -> uint8_t * { return a.ring8 + ((size_t)q * n.S + s) * CA; };
    // ring bytes and input words of the lane's axons at tick kb + k
    struct Axons {
        uint32_t ring[NB], ext[NB];
    };
    auto load_axons = [&](int k, int q, int s) -> Axons {
        Axons x;
        const uint8_t *rp = slot_of(q, s) + (size_t)c * n.A;
        const uint32_t *ep = has_ext ? a.ext_base + (size_t)s * a.ext_sstride + (size_t)(kb + k) * a.tick_words + (size_t)ci * n.W : nullptr;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            x.ring[b] = rp[ax[b]];
            x.ext[b] = has_ext ? ep[ax[b] >> 5] : 0u;
        }
        return x;
    };
    // their two words per ballot, and the number of delivered spikes
    auto words_of = [&](const Axons &x, uint64_t (&m)[NB]) -> unsigned {
        unsigned de = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint64_t r = __ballot(x.ring[b] != 0u) & has[b];
            de += (unsigned)__popcll(r);
            m[b] = r | (has_ext ? __ballot((x.ext[b] >> (ax[b] & 31)) & 1u) & has[b] : 0ull);
        }
        return de;
    };
    // clear this core's bytes of slot q: 4 axons per thread
    auto clear_slot = [&](int q, int s) {
        uint32_t *p = reinterpret_cast<uint32_t *>(slot_of(q, s) + (size_t)c * n.A);
        for (int i = j; i < n.A / 4; i += N)
            p[i] = 0u;
    };
    unsigned de = 0;   // uniform: delivered spikes this wavefront counts
    Axons x_next;
    if constexpr (BLOCK) {
        for (int k = wave; k < nt; k += nw) {
            const int q = q0 + k >= n.Q ? q0 + k - n.Q : q0 + k;
            uint64_t m[NB];
            de += words_of(load_axons(k, q, s0), m);
            if (lane == 0) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    x_lds[k][2 * b] = (uint32_t)m[b];
                    x_lds[k][2 * b + 1] = (uint32_t)(m[b] >> 32);
                }
            }
        }
        __syncthreads();   // the slots are read: they can be cleared
        for (int k = -1; k < nt; ++k) {
            const int q = q0 + k < 0 ? n.Q - 1 : q0 + k >= n.Q ? q0 + k - n.Q : q0 + k;
            clear_slot(q, s0);
        }
    } else {
        x_next = load_axons(0, q0, s0);
    }

    for (int si = 0; si < ns; ++si) {
        const int s = s0 + si;
        int32_t v = v_next;
        const unsigned long long c_old = c_next;
        uint32_t xw[2 * NB];
        if constexpr (!BLOCK) {
            uint64_t m[NB];
            de = words_of(x_next, m);
            if (wave != 0)
                de = 0;   // every wavefront reads them all: counted in row 0
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                xw[2 * b] = (uint32_t)m[b];
                xw[2 * b + 1] = (uint32_t)(m[b] >> 32);
            }
            if (FORM == SAMPLES && si + 1 < ns) {
                v_next = vp[N];
                c_next = cp[CNT_N];
                x_next = load_axons(0, q0, s + 1);
            }
            clear_slot(q0 ? q0 - 1 : n.Q - 1, s);
        }
        unsigned em = 0, ro = 0, ou = 0, ev = 0;   // em, ro, ou uniform
        int q = q0, row = row0;
#pragma unroll 1
        for (int k = 0; k < nt; ++k) {
            if constexpr (BLOCK) {
#pragma unroll
                for (int w = 0; w < SW; ++w)
                    xw[w] = x_lds[k][w];
            }
            unsigned cnt[G_];
#pragma unroll
            for (int g = 0; g < G_; ++g) {
                cnt[g] = 0;
#pragma unroll
                for (int w = 0; w < PW; ++w) {
                    const int i = SORTED ? g * PW + w : w;
                    cnt[g] += __popc(col[i] & (SORTED ? xw[i] : xw[i] & tmask[g * SW + w]));
                }
            }
            int in = 0;
#pragma unroll
            for (int g = 0; g < G_; ++g) {
                in += __mul24((int)cnt[g], wt[g]);
                ev += cnt[g];
            }
            int32_t vnew;
            const bool fire = lif_update(v, in, leak, thr, rst, n.vmin, n.vmax, fl, lin, vnew);
            v = vnew;
            if (fire && dst != PLAIN_NO_DEST) {
                const int qd = q + (int)(dst & 15u);
                slot_of(qd >= n.Q ? qd - n.Q : qd, s)[dst >> 4] = 1;
            }
            const uint64_t b = __ballot(fire);
            em += (unsigned)__popcll(b);
            ro += (unsigned)__popcll(b & cmask);
            ou += (unsigned)__popcll(b & omask);
            if (lane < 2) {   // the wave's two neuron words
                const uint32_t word = (uint32_t)(b >> (32 * lane));
                if (a.want_spk)
                    n.spk[((size_t)s * n.C + c) * n.NW + 2 * wave + lane] = word;
                if (ow >= 0)
                    n.raster[((size_t)row * n.S + s) * n.Wout + ow] = word & om;
            }
            q = q + 1 == n.Q ? 0 : q + 1;
            row = row + 1 == n.RT ? 0 : row + 1;
        }
        *vp = v;
        ev = wave_sum_dpp(ev);
        // (delivered spikes: each wavefront adds those it counted; the rows are summed when read)
        const unsigned add = lane == CNT_EMITTED ? em : lane == CNT_ROUTED ? ro : lane == CNT_DELIVERED ? de : lane == CNT_OUT ? ou : ev;
        if (lane < CNT_N)
            *cp = c_old + add;
        vp += N;
        cp += CNT_N;
    }
}

template <int G_, int SW, bool SORTED>
static hipError_t launch_plain_ticks_k(const DevNet &n, const BlockArgs &a, hipStream_t st)
{
    const dim3 grid(a.count, (n.S + a.spw - 1) / a.spw), block(n.N);
    if (a.level)
        hipLaunchKernelGGL((k_plain_ticks<G_, SW, SORTED, BLOCK_OF_TICKS>), grid, block, 0, st, n, a);
    else if (a.spw > 1)
        hipLaunchKernelGGL((k_plain_ticks<G_, SW, SORTED, SAMPLES>), grid, block, 0, st, n, a);
    else
        hipLaunchKernelGGL((k_plain_ticks<G_, SW, SORTED, ONE_SAMPLE>), grid, block, 0, st, n, a);
    return hipGetLastError();
}

// Words per type of the sorted form that is built for G types; 0: none fits
// (24 words are the most; with one type, the natural order).
int plain_sorted_words(int G, int longest)
{
    const int pw = std::max(1, (longest + 31) / 32);
    return G == 1 && pw <= 16 ? pw : G == 2 && pw <= 8 ? pw : G == 4 && pw <= 6 ? pw : G == 8 && pw <= 3 ? pw : 0;
}

hipError_t launch_plain_ticks(const DevNet &n, const BlockArgs &a, hipStream_t st)
{
    if (n.vlayout != VLAYOUT_CSN || n.N < 64 || n.N > 512 || n.N % 64 != 0 || n.cnt_rows != n.N / 64 || n.S > 65535 ||
        !a.dst || !a.ring8 || n.Q < n.D + 2 || a.spw < 1 || a.first < 0 || a.count < 1 || a.first + a.count > n.C ||
        a.block < 1 || a.ticks < 1 || a.k0 < 0 || a.k0 + a.ticks > n.RT || (!a.order) != (!a.level) ||
        (a.level ? a.spw != 1 || a.block > PLAIN_BLOCK_TICKS || a.ticks + n.D + 1 > n.Q : a.ticks != 1))
        return hipErrorInvalidValue;
    if (a.sorted_words) {
        if (!a.cols || !a.pos)
            return hipErrorInvalidValue;
        switch (n.G * 32 + a.sorted_words) {
#define RANC_SORTED(G, PW) case G * 32 + PW: return launch_plain_ticks_k<G, G * PW, true>(n, a, st);
            RANC_SORTED(1, 2) RANC_SORTED(1, 4) RANC_SORTED(1, 8) RANC_SORTED(1, 16) RANC_SORTED(2, 1) RANC_SORTED(2, 2) RANC_SORTED(2, 3) RANC_SORTED(2, 4) RANC_SORTED(2, 5) RANC_SORTED(2, 6)
            RANC_SORTED(2, 7) RANC_SORTED(2, 8) RANC_SORTED(4, 1) RANC_SORTED(4, 2) RANC_SORTED(4, 3) RANC_SORTED(4, 4)
            RANC_SORTED(4, 5) RANC_SORTED(4, 6) RANC_SORTED(8, 1) RANC_SORTED(8, 2) RANC_SORTED(8, 3)
#undef RANC_SORTED
        default: return hipErrorInvalidValue;
        }
    }
    switch (n.W * 16 + n.G) {
#define RANC_NATURAL(W, G) case W * 16 + G: return launch_plain_ticks_k<G, W, false>(n, a, st);
        RANC_NATURAL(2, 1) RANC_NATURAL(2, 2) RANC_NATURAL(2, 4) RANC_NATURAL(2, 8) RANC_NATURAL(4, 1) RANC_NATURAL(4, 2)
        RANC_NATURAL(4, 4) RANC_NATURAL(4, 8) RANC_NATURAL(8, 1) RANC_NATURAL(8, 2) RANC_NATURAL(8, 4) RANC_NATURAL(8, 8)
        RANC_NATURAL(16, 1) RANC_NATURAL(16, 2) RANC_NATURAL(16, 4) RANC_NATURAL(16, 8)
#undef RANC_NATURAL
    default: return hipErrorInvalidValue;
    }
}

// The deliveries still scheduled, from the bit ring to the byte ring or back:
// each is moved (the other ring is left empty), so a second run moves nothing.
// A thread takes the 32 axons of one scheduler word; the slots hold the ticks
// from the next one on, and, one before it in the byte ring, the slot that the
// next tick would have cleared.
__global__ __launch_bounds__(256) void k_move_ring(DevNet n, uint8_t *ring8, int to_bytes)
{
    const size_t words = (size_t)n.S * n.C * n.W;
    const int last = n.tick[0] ? n.tick[0] - 1 : n.Q - 1;   // slot of the last tick run
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words * n.Q; i += (size_t)gridDim.x * blockDim.x) {
        const int q = (int)(i / words);
        uint32_t *w = n.ring + i;
        uint4 *b = reinterpret_cast<uint4 *>(ring8 + i * 32);   // (a word's 32 axons: [q][s][c][A] and [q][s][c][A / 32])
        uint32_t by[8] = {b[0].x, b[0].y, b[0].z, b[0].w, b[1].x, b[1].y, b[1].z, b[1].w};
        uint32_t bits = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            bits |= ((((by[k] & 0x01010101u) * 0x10204080u) >> 28) & 15u) << (4 * k);
        if (q == last)
            bits = 0;   // read already
        bits |= *w;
        if (to_bytes) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                by[k] = (((bits >> (4 * k)) & 15u) * 0x00204081u) & 0x01010101u;
            *w = 0u;
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                by[k] = 0u;
            *w = bits;
        }
        b[0] = uint4{by[0], by[1], by[2], by[3]};
        b[1] = uint4{by[4], by[5], by[6], by[7]};
    }
}

hipError_t launch_move_ring(const DevNet &n, uint8_t *ring8, int to_bytes, hipStream_t st)
{
    if (n.vlayout != VLAYOUT_CSN || !ring8 || n.Q < n.D + 2)
        return hipErrorInvalidValue;
    const size_t words = (size_t)n.Q * n.S * n.C * n.W;
    hipLaunchKernelGGL(k_move_ring, dim3((unsigned)std::min<size_t>((words + 255) / 256, 4096)), dim3(256), 0, st, n, ring8, to_bytes);
    return hipGetLastError();
}

// The same tick for one 64-neuron block of one (core, sample) on a single
// wavefront (the batched launch, where networks of every N share one launch
// shape); the block's counts go to its own counter row.
template <int W_, int G_>
__device__ __forceinline__ void integrate_plain_wave(const DevNet &n, const TickArgs &ta, int c, int s, int nb)
{
    const int N = n.N;
    const int lane = threadIdx.x & 63;
    const uint32_t *slot = n.ring + (((size_t)tick_slot(n, ta.k) * n.S + s) * n.C + c) * W_;
    const int ci = n.in_index[c];
    const uint32_t *ext = (ta.ext_t != nullptr && ci >= 0)
                              ? ta.ext_t + (size_t)s * ta.ext_sstride + (size_t)ci * W_
                              : nullptr;
    const uint32_t *tmask = n.typemask + (size_t)c * G_ * W_;
    const int j = nb * 64 + lane;
    unsigned cnt[G_];
#pragma unroll
    for (int g = 0; g < G_; ++g)
        cnt[g] = 0;
    unsigned delivered = 0;
    const uint32_t *col = n.colbits + (size_t)c * W_ * N + j;
    // axon words and type masks are wave-uniform (scalar loads)
#pragma unroll 2
    for (int w = 0; w < W_; ++w) {
        const uint32_t r = slot[w];
        delivered += __popc(r);
        const uint32_t cw = col[(size_t)w * N] & (r | (ext ? ext[w] : 0u));
#pragma unroll
        for (int g = 0; g < G_; ++g)
            cnt[g] += __popc(cw & tmask[g * W_ + w]);
    }
    const int32_t *wt = n.wts + (size_t)c * G_ * N + j;
    int in = 0;
    unsigned e = 0;
#pragma unroll
    for (int g = 0; g < G_; ++g) {
        in += __mul24((int)cnt[g], wt[(size_t)g * N]);
        e += cnt[g];
    }
    const size_t cj = (size_t)c * N + j;
    const size_t vi = ((size_t)c * n.S + s) * N + j;
    int32_t vnew;
    int32_t fl = n.vmin;
    bool lin = false;
    if (n.model_ext) {   // uniform
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (j & 31)) & 1u;
    }
    const bool fire = lif_update(n.V[vi], in, n.leak[cj], n.thr[cj], n.rst[cj], n.vmin, n.vmax, fl, lin, vnew);
    n.V[vi] = vnew;
    const unsigned long long b = __ballot(fire);
    const unsigned ev = wave_sum(e);
    if (lane == 0) {
        unsigned em = 0, ro = 0, ou = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int nw = nb * 2 + h;
            const uint32_t wd = (uint32_t)(b >> (32 * h));
            const size_t m = (size_t)c * n.NW + nw;
            const uint32_t om = wd & n.outmask[m];
            em += __popc(wd);
            ro += __popc(wd & n.coremask[m]);
            ou += __popc(om);
            n.spk[((size_t)s * n.C + c) * n.NW + nw] = wd;
            const int ow = n.outword[m];
            if (ow >= 0)
                n.raster[((size_t)tick_row(n, ta.k) * n.S + s) * n.Wout + ow] = om;
        }
        store_counts(n, ta.k, (size_t)c * (N >> 6) + nb, s, pack_counts(em, ro, ou, nb == 0 ? delivered : 0u, ev));
    }
}

// One tick of one 64-neuron block of one (core, sample) on a single wavefront,
// delivery included (the batched form of k_plain_ticks, natural order): words
// and type masks are wave-uniform, the columns are read as they are used.
template <int W_, int G_>
__device__ __forceinline__ void plain_tick_wave(const BatchEntry &e, int k, int c, int s, int nb)
{
    constexpr int NB = W_ / 2;
    const DevNet &n = e.n;
    const int N = n.N;
    const int lane = threadIdx.x & 63;
    const int q = tick_slot(n, k);
    const size_t CA = (size_t)n.C * n.A;
    auto slot_of = [&](int q) -> uint8_t * { return e.ring8 + ((size_t)q * n.S + s) * CA; };
    const uint8_t *rp = slot_of(q) + (size_t)c * n.A + lane;
    const int ci = n.in_index[c];
    const bool has_ext = e.ext_base != nullptr && ci >= 0;   // uniform
    const uint32_t *ep = has_ext ? e.ext_base + (size_t)s * e.ext_sstride + (size_t)k * e.tick_words + (size_t)ci * W_ : nullptr;
    uint32_t rb[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        rb[b] = rp[64 * b];
    const int j = nb * 64 + lane;
    const size_t cj = (size_t)c * N + j;
    const size_t vi = ((size_t)c * n.S + s) * N + j;
    const int32_t v = n.V[vi], leak = n.leak[cj], thr = n.thr[cj], rst = n.rst[cj];
    const uint32_t dst = e.dst[cj];
    const size_t row = (size_t)c * (N >> 6) + nb;
    unsigned long long *cp = n.cnt + (row * n.S + s) * CNT_N + (lane < CNT_N ? lane : 0);
    const unsigned long long c_old = *cp;
    uint32_t xw[W_];
    unsigned de = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint64_t r = __ballot(rb[b] != 0u);
        de += (unsigned)__popcll(r);
        xw[2 * b] = (uint32_t)r | (has_ext ? ep[2 * b] : 0u);
        xw[2 * b + 1] = (uint32_t)(r >> 32) | (has_ext ? ep[2 * b + 1] : 0u);
    }
    const uint32_t *tmask = n.typemask + (size_t)c * G_ * W_;
    const uint32_t *col = n.colbits + (size_t)c * W_ * N + j;
    unsigned cnt[G_];
#pragma unroll
    for (int g = 0; g < G_; ++g)
        cnt[g] = 0;
#pragma unroll
    for (int w = 0; w < W_; ++w) {
        const uint32_t cw = col[(size_t)w * N] & xw[w];
#pragma unroll
        for (int g = 0; g < G_; ++g)
            cnt[g] += __popc(cw & tmask[g * W_ + w]);
    }
    const int32_t *wt = n.wts + (size_t)c * G_ * N + j;
    int in = 0;
    unsigned ev = 0;
#pragma unroll
    for (int g = 0; g < G_; ++g) {
        in += __mul24((int)cnt[g], wt[(size_t)g * N]);
        ev += cnt[g];
    }
    int32_t vnew;
    int32_t fl = n.vmin;
    bool lin = false;
    if (n.model_ext) {   // uniform
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (j & 31)) & 1u;
    }
    const bool fire = lif_update(v, in, leak, thr, rst, n.vmin, n.vmax, fl, lin, vnew);
    n.V[vi] = vnew;
    if (fire && dst != PLAIN_NO_DEST) {
        const int qd = q + (int)(dst & 15u);
        slot_of(qd >= n.Q ? qd - n.Q : qd)[dst >> 4] = 1;
    }
    // this wavefront's share of the core's bytes of the slot before
    {
        const int share = n.A / (N >> 6);   // bytes, a multiple of 8
        uint32_t *p = reinterpret_cast<uint32_t *>(slot_of(q ? q - 1 : n.Q - 1) + (size_t)c * n.A + nb * share);
        if (lane < share / 4)
            p[lane] = 0u;
        if (share > 256 && lane < share / 4 - 64)   // (512 axons, 64 neurons)
            p[64 + lane] = 0u;
    }
    const uint64_t b = __ballot(fire);
    ev = wave_sum_dpp(ev);
    const size_t m0 = (size_t)c * n.NW + 2 * nb;
    const unsigned em = (unsigned)__popcll(b);
    const unsigned ro = (unsigned)__popcll(b & (n.coremask[m0] | (uint64_t)n.coremask[m0 + 1] << 32));
    const unsigned ou = (unsigned)__popcll(b & (n.outmask[m0] | (uint64_t)n.outmask[m0 + 1] << 32));
    if (lane < 2) {
        const uint32_t word = (uint32_t)(b >> (32 * lane));
        if (e.form & BATCH_WANT_SPK)
            n.spk[((size_t)s * n.C + c) * n.NW + 2 * nb + lane] = word;
        const int ow = n.outword[m0 + lane];
        if (ow >= 0)
            n.raster[((size_t)tick_row(n, k) * n.S + s) * n.Wout + ow] = word & n.outmask[m0 + lane];
    }
    const unsigned add = lane == CNT_EMITTED ? em : lane == CNT_ROUTED ? ro : lane == CNT_DELIVERED ? (nb == 0 ? de : 0u)
                         : lane == CNT_OUT ? ou : ev;
    if (lane < CNT_N)
        *cp = c_old + add;
}

int plain_shape_code(int W, int G)
{
    const int wi = W == 2 ? 0 : W == 4 ? 1 : W == 8 ? 2 : 3;
    const int gi = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : 3;
    return wi * 4 + gi;
}

// Several networks on the plain path, one tick, one launch: unit u is
// (64-neuron block, core, sample) of the network whose unit range holds u,
// on one wavefront.
__global__ __launch_bounds__(64) void k_integrate_plain_batch(const BatchEntry *__restrict__ tab, int num, int k)
{
    const int u = blockIdx.x;
    const BatchEntry &e = tab[batch_entry_of(tab, num, u, false)];
    const int local = u - e.unit_begin;
    const int nbs = e.n.N >> 6;
    const int nb = local % nbs, c = (local / nbs) % e.n.C, s = local / nbs / e.n.C;
    TickArgs ta;
    ta.k = k;
    ta.ext_t = e.ext_base ? e.ext_base + (size_t)k * e.tick_words : nullptr;
    ta.ext_sstride = e.ext_sstride;
    switch (e.code) {
#define RANC_PLAIN_CASE(WI, W, GI, G) \
    case WI * 4 + GI: integrate_plain_wave<W, G>(e.n, ta, c, s, nb); break;
        RANC_PLAIN_CASE(0, 2, 0, 1) RANC_PLAIN_CASE(0, 2, 1, 2) RANC_PLAIN_CASE(0, 2, 2, 4) RANC_PLAIN_CASE(0, 2, 3, 8)
        RANC_PLAIN_CASE(1, 4, 0, 1) RANC_PLAIN_CASE(1, 4, 1, 2) RANC_PLAIN_CASE(1, 4, 2, 4) RANC_PLAIN_CASE(1, 4, 3, 8)
        RANC_PLAIN_CASE(2, 8, 0, 1) RANC_PLAIN_CASE(2, 8, 1, 2) RANC_PLAIN_CASE(2, 8, 2, 4) RANC_PLAIN_CASE(2, 8, 3, 8)
        RANC_PLAIN_CASE(3, 16, 0, 1) RANC_PLAIN_CASE(3, 16, 1, 2) RANC_PLAIN_CASE(3, 16, 2, 4)
        RANC_PLAIN_CASE(3, 16, 3, 8)
#undef RANC_PLAIN_CASE
    default: break;
    }
}

// The same units, one per wavefront, for networks with the byte ring.
__global__ __launch_bounds__(256) void k_plain_ticks_batch(const BatchEntry *__restrict__ tab, int num, int total, int k)
{
    const int u = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (u >= total)
        return;   // whole wavefronts
    const BatchEntry &e = tab[batch_entry_of(tab, num, u, false)];
    const int local = u - e.unit_begin;
    const int nbs = e.n.N >> 6;
    const int nb = local % nbs, c = (local / nbs) % e.n.C, s = local / nbs / e.n.C;
    switch (e.code) {
#define RANC_PLAIN_CASE(WI, W, GI, G) \
    case WI * 4 + GI: plain_tick_wave<W, G>(e, k, c, s, nb); break;
        RANC_PLAIN_CASE(0, 2, 0, 1) RANC_PLAIN_CASE(0, 2, 1, 2) RANC_PLAIN_CASE(0, 2, 2, 4) RANC_PLAIN_CASE(0, 2, 3, 8)
        RANC_PLAIN_CASE(1, 4, 0, 1) RANC_PLAIN_CASE(1, 4, 1, 2) RANC_PLAIN_CASE(1, 4, 2, 4) RANC_PLAIN_CASE(1, 4, 3, 8)
        RANC_PLAIN_CASE(2, 8, 0, 1) RANC_PLAIN_CASE(2, 8, 1, 2) RANC_PLAIN_CASE(2, 8, 2, 4) RANC_PLAIN_CASE(2, 8, 3, 8)
        RANC_PLAIN_CASE(3, 16, 0, 1) RANC_PLAIN_CASE(3, 16, 1, 2) RANC_PLAIN_CASE(3, 16, 2, 4)
        RANC_PLAIN_CASE(3, 16, 3, 8)
#undef RANC_PLAIN_CASE
    default: break;
    }
}

hipError_t launch_plain_ticks_batch(const BatchEntry *tab, int num, int total, int k, hipStream_t st)
{
    if (num < 1 || total < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_plain_ticks_batch, dim3((total + 3) / 4), dim3(256), 0, st, tab, num, total, k);
    return hipGetLastError();
}

hipError_t launch_integrate_plain_batch(const BatchEntry *tab, int num, int total, int k, hipStream_t st)
{
    if (num < 1 || total < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_integrate_plain_batch, dim3(total), dim3(64), 0, st, tab, num, k);
    return hipGetLastError();
}

template <int W_>
static hipError_t launch_plain_w(const DevNet &n, const TickArgs &a, hipStream_t st)
{
    const dim3 grid(n.C, n.S), block(n.N);
    switch (n.G) {
    case 1: hipLaunchKernelGGL((k_integrate_plain<W_, 1>), grid, block, 0, st, n, a); break;
    case 2: hipLaunchKernelGGL((k_integrate_plain<W_, 2>), grid, block, 0, st, n, a); break;
    case 4: hipLaunchKernelGGL((k_integrate_plain<W_, 4>), grid, block, 0, st, n, a); break;
    case 8: hipLaunchKernelGGL((k_integrate_plain<W_, 8>), grid, block, 0, st, n, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_integrate_plain(const DevNet &n, const TickArgs &a, hipStream_t st)
{
    if (n.N < 64 || n.N > 512 || n.N % 64 != 0 || n.S > 65535)
        return hipErrorInvalidValue;
    switch (n.W) {
    case 2: return launch_plain_w<2>(n, a, st);
    case 4: return launch_plain_w<4>(n, a, st);
    case 8: return launch_plain_w<8>(n, a, st);
    case 16: return launch_plain_w<16>(n, a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ranc
