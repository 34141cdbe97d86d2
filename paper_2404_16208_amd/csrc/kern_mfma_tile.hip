// kern_mfma_tile.hip -- the MFMA path's tick where a workgroup covers one tile
// of 64 samples (all of a network with up to 64 samples, or samples_per_wg =
// 64): the same work as kern_mfma_unit.h, without a pipeline over tiles.
//
// One tile per workgroup is a chain of dependent loads (source list, history
// word), two barriers, products and update, and nothing in the workgroup
// hides it: the bytes (potentials read and written, 512 per neuron) would
// take a fifth of the time. So the form is built to keep many workgroups on a
// CU: potentials come straight into registers, B tiles are used as they are
// read (or built) and not held, single LDS buffers (20 KB with 256 axons where the
// pipelined form has 92 to 140), and cores of 64 neurons have workgroups of
// four wavefronts instead of eight with four idle. Loads are issued in the
// order of their use, the potentials last, so that the wait for history words
// does not wait for them.
// us per tick at 64 samples, pipelined form and this: 1024 cores of 256 x 64 27.7,
// 13.0 (at 5.2 TB/s the potentials take 6.5); of 128 x 128 (9 bits) 44.7, 20.5
// (13.0); of 256 x 256 (8 bits) 47.6, 35.0 (26.0); of 512 x 512 (9 bits) 188, 97
// (52.0); 16 cores of 256 x 256 10.5, 9.0. Potentials by ordinary loads and stores
// instead of streaming ones: 133 to 166 us for 4096 cores of 256 x 256.
#include "kern_common.h"
#include "kern_bits.h"
#include "kern_mfma_unit.h"
#include "ranc_internal.h"

namespace ranc {

// NB_: 32-neuron blocks of the workgroup (2, 4 or 8). A wavefront has one
// block and 32 samples, or with 8 blocks and one plane 64 samples; with two
// planes its sums and potentials would not fit 128 registers (1024 cores of 256 x
// 256, 9 bits: 56 us with spills, 45 with 16 wavefronts; 8 bits: 36 and 43).
template <int A_, int NB_, bool TWO> struct TileShape {
    static constexpr int WAVES = NB_ == 8 && !TWO ? 8 : 2 * NB_;
    static constexpr int STW = 2 * NB_ / WAVES;   // 32-sample groups per wavefront
    static constexpr int APW = A_ / 64;           // 64-axon blocks of the gather
    static constexpr int GPW = 2 * APW > WAVES ? 2 : 1;   // 32-sample groups per gather task
    static constexpr int TASKS = GPW == 2 ? APW : 2 * APW;
    static constexpr int TPW = (TASKS + WAVES - 1) / WAVES;
    static constexpr int WPW = (A_ / 32 + WAVES - 1) / WAVES;   // axon words expanded per wavefront
    static constexpr int ROWB = A_ + 16;          // padded LDS row of the int8 tile (bytes)
};

template <int A_> struct TileLds {
    __attribute__((aligned(16))) int8_t a[MFMA_TS * (A_ + 16)];   // int8 axon spikes
    uint32_t x[MFMA_TS][A_ / 32 + 1];             // delivered axon words
    unsigned cnt[2][MFMA_TS];                     // as s_cnt of integrate_mfma_unit
};

template <int A_, int NB_, bool TWO, bool CB>
__device__ __forceinline__ void integrate_tile(const DevNet &n, const TickArgs &ta, int bid, TileLds<A_> &lds)
{
    typedef TileShape<A_, NB_, TWO> T;
    constexpr int KS = A_ / 32, W_ = A_ / 32, PL = TWO ? 2 : 1, STW = T::STW, TPW = T::TPW, WPW = T::WPW;
    constexpr int DP = WPW < 2 ? WPW : 2;   // axon words whose connection counts are loaded ahead
    typedef typename RawWord<T::GPW == 2>::type RawT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int c, v;
    const int HG = n.S64 / 64;   // tiles
    core_unit_of(bid, n.C, n.slices * HG, c, v);
    const int slice = v % n.slices, tile = v / n.slices;
    const int s0 = tile * MFMA_TS, s_end = min(n.S, s0 + MFMA_TS);
    const int h = lane >> 5, jj = lane & 31;
    const int sig = sigma32(jj);
    const int nb = wave % NB_, stg = wave / NB_;
    const int nbc = slice * NB_ + nb;   // 32-neuron block within the core
    const int jc = nbc * 32 + jj;       // neuron within the core
    const size_t cj = (size_t)c * n.N + jc;

    for (int i = threadIdx.x; i < 2 * MFMA_TS; i += 64 * T::WAVES)
        (&lds.cnt[0][0])[i] = 0u;

    // source lists of the wave's gather tasks (64 axons x one or both groups)
    int axb[TPW], grp[TPW];
    uint32_t e_beg[TPW], e_end[TPW];
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        const int task = min(wave + T::WAVES * k, T::TASKS - 1);
        axb[k] = T::GPW == 2 ? task : task % T::APW;
        grp[k] = T::GPW == 2 ? 0 : task / T::APW;
        const uint32_t *p = n.rtx_ptr + (size_t)c * A_ + axb[k] * 64 + lane;
        e_beg[k] = p[0];
        e_end[k] = p[1];
    }
    const int ci = n.in_index[c];
    const uint32_t *ext_c = (ta.ext_t != nullptr && ci >= 0) ? ta.ext_t + (size_t)ci * W_ : nullptr;
    uint32_t xe[WPW];
#pragma unroll
    for (int k = 0; k < WPW; ++k) {
        const int wi = wave + T::WAVES * k;
        xe[k] = ext_c && wi < W_ && s0 + lane < s_end ? ext_c[(size_t)(s0 + lane) * ta.ext_sstride + wi] : 0u;
    }
    const int32_t lk = n.leak[cj], th = n.thr[cj], rs = n.rst[cj];
    const int oi = n.outidx[cj];
    int32_t fl = n.vmin;
    bool lin = false;
    if (n.model_ext) {   // uniform
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (cj & 31)) & 1u;
    }
    const int q_now = tick_slot(n, ta.k), r_row = tick_row(n, ta.k);
    const size_t CN = (size_t)n.C * n.N;
    auto word_of = [&](uint32_t ent, int g) -> RawT {
        int slot = q_now - (int)(ent & 15u) - 1;
        if (slot < 0)
            slot += n.Q;
        const uint64_t *row = n.hist + ((size_t)slot * CN + (ent >> 4)) * HG + tile;
        if constexpr (T::GPW == 2)
            return *row;
        else
            return reinterpret_cast<const uint32_t *>(row)[g];
    };
    uint32_t ent[TPW];
#pragma unroll
    for (int k = 0; k < TPW; ++k)
        ent[k] = e_beg[k] < e_end[k] ? n.rtx_ent[e_beg[k]] : 0u;
    RawT raw[TPW];
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        raw[k] = 0;
        if (e_beg[k] < e_end[k])
            raw[k] = word_of(ent[k], grp[k]);
    }
    // What the products need first, ahead of the barriers: the B tiles of two
    // k-steps, or all column words, the plane values and the types of two k-steps
    // (with four, no faster); and the connection counts. 1024 cores of 512 x 512
    // (9 bits) 110.6 us per tick without, 97.4 with; the sweep of eight networks
    // 1037 and 993 us.
    constexpr int KP = STW == 2 ? (CB ? 1 : 2) : KS < 2 ? KS : 2;
    const uint32_t *colw = n.colbits + (size_t)c * W_ * n.N + jc;
    const uint4 *ts = reinterpret_cast<const uint4 *>(mfma_bsrc_types(n, PL) + (size_t)c * A_) + h;
    const v4i *planes = reinterpret_cast<const v4i *>(n.planes) + ((size_t)c * n.NW + nbc) * KS * PL * 64 + lane;
    v4i bpre[KP][PL];
    uint32_t bits[KS], wl[PL], wh[PL];
    uint4 types[KP];
    if constexpr (CB) {
        const uint32_t *wsel = mfma_bsrc_wsel(n) + (size_t)c * PL * 2 * n.N + jc;
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            wl[p] = wsel[(size_t)(2 * p) * n.N];
            wh[p] = wsel[(size_t)(2 * p + 1) * n.N];
        }
#pragma unroll
        for (int k = 0; k < KS; ++k)
            bits[k] = colw[(size_t)k * n.N];
#pragma unroll
        for (int k = 0; k < KP; ++k)
            types[k] = ts[2 * k];
    } else {
#pragma unroll
        for (int k = 0; k < KP; ++k)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                bpre[k][p] = planes[(k * PL + p) * 64];
    }
    const size_t dg = (size_t)c * n.slices + slice;
    uint32_t degl[DP][8], degh[DP][8];
#pragma unroll
    for (int k = 0; k < DP; ++k) {
        const int wi = min(wave + T::WAVES * k, W_ - 1);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            degl[k][q] = n.degb[(dg * 2 + 0) * (A_ / 4) + wi * 8 + q];
            degh[k][q] = n.degb[(dg * 2 + 1) * (A_ / 4) + wi * 8 + q];
        }
    }
    const uint32_t cm32 = n.coremask[(size_t)c * n.NW + nbc];
    const uint32_t om32 = n.outmask[(size_t)c * n.NW + nbc];
    compiler_fence();
    v4i *vb = reinterpret_cast<v4i *>(n.V) + (((size_t)c * n.NW + nbc) * (n.S64 / 32) + 2 * tile + stg * STW) * 256 + lane;
    // (a group past the last sample has nothing to read or keep: it loads the tile's first)
    auto group_of = [&](int t) { return s0 + 32 * (stg * STW + t) < s_end ? t : -stg * STW; };
    v4i vr[STW][4];
#pragma unroll
    for (int t = 0; t < STW; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            vr[t][q] = __builtin_nontemporal_load(vb + (group_of(t) * 4 + q) * 64);
    compiler_fence();
    // Lane (h, j) holds, for axon 64 axb + 32 h + j, the bits of a 32-sample
    // group; after the transpose lane (h, i) holds the axon word 2 axb + h of
    // the sample of bit i.
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        if (__ballot(e_end[k] > e_beg[k] + 1) != 0)   // wave-uniform: axons with several sources
            for (uint32_t e = e_beg[k] + 1; e < e_end[k]; ++e)
                raw[k] |= word_of(n.rtx_ent[e], grp[k]);
        if (TPW * T::WAVES == T::TASKS || wave + T::WAVES * k < T::TASKS) {
#pragma unroll
            for (int g = 0; g < T::GPW; ++g)
                lds.x[32 * (T::GPW == 2 ? g : grp[k]) + sig][2 * axb[k] + h] =
                    transpose32((uint32_t)((uint64_t)raw[k] >> (32 * g)), lane);
        }
    }
    lds_barrier();

    // expansion, one lane per sample: delivered | external spikes of this
    // wave's axon words to int8, delivered and event counts
    {
        unsigned pdl = 0u, pev = 0u, pevh = 0u;
#pragma unroll
        for (int k = 0; k < WPW; ++k) {
            const int wi = wave + T::WAVES * k;
            if (wi < W_) {
                const uint32_t xd = lds.x[lane][wi];
                const uint32_t x = xd | xe[k];
                pdl += (unsigned)__popc(xd);
                uint32_t dl[8], dh[8], d[8], any_hi = 0;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    dl[q] = k < DP ? degl[k < DP ? k : 0][q] : n.degb[(dg * 2 + 0) * (A_ / 4) + wi * 8 + q];
                    dh[q] = k < DP ? degh[k < DP ? k : 0][q] : n.degb[(dg * 2 + 1) * (A_ / 4) + wi * 8 + q];
                    any_hi |= dh[q];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    d[q] = (((x >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
                    pev = __builtin_amdgcn_udot4(d[q], dl[q], pev, false);
                }
                if (any_hi) {   // uniform: a core of 256 connected neurons on an axon
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        pevh = __builtin_amdgcn_udot4(d[q], dh[q], pevh, false);
                }
                v4i *dst = reinterpret_cast<v4i *>(&lds.a[lane * T::ROWB + 32 * wi]);
                dst[0] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
                dst[1] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
            }
        }
        const unsigned dlev = (pev + (pevh << 8)) | (pdl << 18);
        if (s0 + lane < s_end && dlev)
            atomicAdd(&lds.cnt[1][lane], dlev);
    }
    lds_barrier();

    v16i lo[STW], hi[STW];
#pragma unroll
    for (int t = 0; t < STW; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            lo[t][r] = lk;
            hi[t][r] = 0;
        }
    const int8_t *arow = &lds.a[(stg * STW * 32 + jj) * T::ROWB + 16 * h];
    auto multiply = [&](int k, const v4i (&b)[PL]) {
#pragma unroll
        for (int t = 0; t < STW; ++t) {
            const v4i a = *reinterpret_cast<const v4i *>(arow + t * 32 * T::ROWB + 32 * k);
            if constexpr (TWO)
                hi[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[0], hi[t], 0, 0, 0);
            lo[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[PL - 1], lo[t], 0, 0, 0);
        }
    };
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        v4i b[PL];
        if constexpr (CB) {
            compact_b_tile(bits[k] >> (16 * h), k < KP ? types[k < KP ? k : 0] : ts[2 * k], wl, wh, b);
        } else {
#pragma unroll
            for (int p = 0; p < PL; ++p)
                b[p] = k < KP ? bpre[k < KP ? k : 0][p] : planes[(k * PL + p) * 64];
        }
        multiply(k, b);
    }

    const NeuronParams np{th, rs, fl, n.vmin, n.vmax, lin};
    uint32_t hword[STW];
#pragma unroll
    for (int t = 0; t < STW; ++t) {
        const int first = s0 + 32 * (stg * STW + t);   // the group's first sample
        uint32_t f = 0;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            int32_t in[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                in[e] = TWO ? lo[t][4 * q + e] + hi[t][4 * q + e] * 128 : lo[t][4 * q + e];
            if (n.model_ext)   // uniform
                update_rows<true>(vr[t][q], in, np, f);
            else
                update_rows<false>(vr[t][q], in, np, f);
            if (first < s_end)
                __builtin_nontemporal_store(vr[t][q], vb + (t * 4 + q) * 64);
        }
        // samples past the end never fire (their potentials are never read)
        if (first + 32 > s_end) {   // wave-uniform
            uint32_t vm = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                vm |= (uint32_t)(first + 8 * (r >> 2) + 4 * h + (r & 3) < s_end) << r;
            f &= vm;
        }
        // the neuron's spike word: bits r from lane jj, bits 16 + r from lane jj + 32
        hword[t] = f | ((uint32_t)__shfl_xor((int)f, 32, 64) << 16);
        // per-sample spike words of the wave's 32 neurons, and their counts
        const uint32_t sw = transpose32(hword[t], lane);
        const unsigned pc = (unsigned)__popc(sw) | ((unsigned)__popc(sw & cm32) << 10) | ((unsigned)__popc(sw & om32) << 20);
        if (h == 0 && first + sig < s_end && pc)
            atomicAdd(&lds.cnt[0][first - s0 + sig], pc);
    }
    if (h == 0) {
        uint64_t *ho = n.hist + ((size_t)q_now * CN + cj) * HG + tile;
        uint64_t *ro = reinterpret_cast<uint64_t *>(n.raster) + ((size_t)r_row * n.Nout + max(oi, 0)) * HG + tile;
        if constexpr (STW == 2) {
            const uint64_t w = (uint64_t)hword[0] | (uint64_t)hword[STW - 1] << 32;
            *ho = w;
            if (oi >= 0)
                *ro = w;
        } else {
            reinterpret_cast<uint32_t *>(ho)[stg] = hword[0];
            if (oi >= 0)
                reinterpret_cast<uint32_t *>(ro)[stg] = hword[0];
        }
    }
    lds_barrier();
    const int i = threadIdx.x;
    if (s0 + i < s_end && i < MFMA_TS) {
        const unsigned sp = lds.cnt[0][i], ev = lds.cnt[1][i];
        n.cring[((size_t)r_row * n.C * n.cnt_rows + (size_t)c * n.cnt_rows + slice) * n.S + s0 + i] =
            pack_counts(sp & 1023u, (sp >> 10) & 1023u, sp >> 20, slice == 0 ? ev >> 18 : 0u, ev & ((1u << 18) - 1u));
    }
}

template <int A_, int NB_, bool TWO, bool CB>
__global__ __launch_bounds__((64 * TileShape<A_, NB_, TWO>::WAVES)) __attribute__((amdgpu_waves_per_eu(4))) void k_integrate_tile(
    DevNet n, TickArgs ta)
{
    __shared__ TileLds<A_> lds;
    integrate_tile<A_, NB_, TWO, CB>(n, ta, blockIdx.x, lds);
}

// Several networks of one shape, as k_integrate_mfma_group.
template <int A_, int NB_, bool TWO, bool CB>
__global__ __launch_bounds__((64 * TileShape<A_, NB_, TWO>::WAVES)) __attribute__((amdgpu_waves_per_eu(4))) void k_integrate_tile_group(
    MfmaGroupArgs g, int k)
{
    __shared__ TileLds<A_> lds;
    const int u = blockIdx.x;
    int idx = 0;   // the last entry whose first unit is <= u (independent scalar loads)
    for (int i = 1; i < MFMA_GROUP_MAX; ++i)
        if (i < g.num && g.e[i].unit_begin <= u)
            idx = i;
    const MfmaGroupEntry &e = g.e[idx];
    TickArgs ta;
    ta.k = k;
    ta.ext_t = e.ext_base ? e.ext_base + (size_t)k * e.tick_words : nullptr;
    ta.ext_sstride = e.ext_sstride;
    integrate_tile<A_, NB_, TWO, CB>(e.n, ta, u - e.unit_begin, lds);
}

template <int A_, int NB_, bool TWO, bool CB>
static void launch_tile_k(const DevNet *n, const TickArgs &a, const MfmaGroupArgs *g, int total, int k, hipStream_t st)
{
    constexpr int threads = 64 * TileShape<A_, NB_, TWO>::WAVES;
    if (g)
        hipLaunchKernelGGL((k_integrate_tile_group<A_, NB_, TWO, CB>), dim3(total), dim3(threads), 0, st, *g, k);
    else
        hipLaunchKernelGGL((k_integrate_tile<A_, NB_, TWO, CB>), dim3(total), dim3(threads), 0, st, *n, a);
}

template <int A_, int NB_>
static void launch_tile_an(const DevNet *n, const TickArgs &a, const MfmaGroupArgs *g, int total, int k, int two, int cb,
                           hipStream_t st)
{
    if (two)
        cb ? launch_tile_k<A_, NB_, true, true>(n, a, g, total, k, st) : launch_tile_k<A_, NB_, true, false>(n, a, g, total, k, st);
    else
        cb ? launch_tile_k<A_, NB_, false, true>(n, a, g, total, k, st) : launch_tile_k<A_, NB_, false, false>(n, a, g, total, k, st);
}

// code: mfma_shape_code, plus MFMA_TILE_N64 for cores of 64 neurons
static hipError_t launch_tile(const DevNet *n, const TickArgs &a, const MfmaGroupArgs *g, int total, int k, int code, int cb,
                              hipStream_t st)
{
    const int two = code & 1;
    const int nb = (code & MFMA_TILE_N64) ? 2 : (code & 2) ? 8 : 4;
    switch ((code & (MFMA_TILE_N64 - 1)) / 4 * 16 + nb) {
#define RANC_TILE(AI, A) \
    case AI * 16 + 2: launch_tile_an<A, 2>(n, a, g, total, k, two, cb, st); break; \
    case AI * 16 + 4: launch_tile_an<A, 4>(n, a, g, total, k, two, cb, st); break; \
    case AI * 16 + 8: launch_tile_an<A, 8>(n, a, g, total, k, two, cb, st); break;
        RANC_TILE(0, 64) RANC_TILE(1, 128) RANC_TILE(2, 256) RANC_TILE(3, 512)
#undef RANC_TILE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_integrate_tile(const DevNet &n, const TickArgs &a, int two, int compact, hipStream_t st)
{
    if (n.C < 1 || n.slices < 1 || (long long)n.C * n.slices * (n.S64 / 64) > INT32_MAX)
        return hipErrorInvalidValue;
    const int code = mfma_shape_code(n.A, mfma_width(n.A, n.N, two), two) | (n.N == 64 ? MFMA_TILE_N64 : 0);
    return launch_tile(&n, a, nullptr, n.C * n.slices * (n.S64 / 64), 0, code, compact, st);
}

hipError_t launch_integrate_tile_group(const MfmaGroupArgs &g, int total, int k, int code, int compact, hipStream_t st)
{
    return launch_tile(nullptr, TickArgs(), &g, total, k, code, compact, st);
}

}  // namespace ranc
