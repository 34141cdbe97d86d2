// kern_mfma_ticks.hip -- several ticks of the batched MFMA path in one launch,
// for feed-forward networks.
//
// When the core graph has no cycle (a layered classifier), a core's spikes of
// any number of ticks depend only on its external input and on the spikes of
// cores in earlier levels (level = longest path from a core without sources).
// The cores of a level can therefore run a whole block of ticks at once, with
// their potentials in registers for the block, as soon as the levels before
// have run it. The history ring holds Q >= D + (ticks of the block's
// segment) slots for that (the runtime's Plan). One launch is one `step` of
// the skewed schedule: a core of level l runs block step - l.
//
// What bounds it: with one tick per launch every tick moves each potential
// from and to HBM (8 bytes per neuron, sample and tick; 1.07 GB per tick on
// the 512-core net at 1024 samples, 5.4 TB/s, the HBM read-modify-write
// limit). Here potentials move once per block, and a tick is bound by issue:
// per wavefront about 300 vector instructions and 32 MFMA of 32 cycles.
// Measured on that net, 32 ticks per call: 220 -> 84 us per tick at 1024
// samples (whole pass 7.77 -> 3.15 ms, of it 0.62 ms raster packing), 35 ->
// 11 us at 100 samples (1.17 -> 0.38 ms).
//
// Mapping: one workgroup of 8 wavefronts per (core, neuron slice, 64-sample
// tile); wave w owns the 32 neurons of block w % (slice / 32). Its B tiles
// (int8 planes), its potentials (32 registers per lane at 256-neuron slices)
// and its source-row addresses stay in registers for the block. Per tick:
//   A. the tick's axon words (LDS) OR external input, expanded to the int8
//      tile; the next tick's history bits, loaded a tick ahead, transposed to
//      axon words in LDS; the loads for the tick after are issued;
//   B. one LDS barrier (both LDS buffers are doubled);
//   C. products and potential update as in kern_mfma.hip, in place;
//   D. the loads of A are waited for, then the spike words are stored, so
//      that no wait ever covers a store of the same tick.
// The two 32-sample halves of a neuron's 16-bit fire masks are joined by one
// v_permlane32_swap: lane (h, j) then holds the word of sub-tile h.
// Spike counts are kept as vertical counters (bit plane i of a lane holds bit
// i of the count of each of its 32 samples; ten bitwise operations per tick
// and lane) and turned into per-sample totals once per block, where the
// per-tick kernel transposes every tick's words.
#include "kern_mfma_unit.h"

namespace ranc {

// Bit planes of the vertical counters: a block runs at most 2^6 - 1 ticks.
static constexpr int TICK_PLANES = 6;
static_assert(MFMA_BLOCK_TICKS_MAX < (1 << TICK_PLANES), "vertical counters overflow");

template <int A_, int N_, bool TWO, bool EXT>
__global__ __launch_bounds__(512) void k_integrate_mfma_ticks(DevNet n, BlockArgs ba)
{
    typedef MfmaLds<A_, N_> L;
    constexpr int NB = N_ / 32;          // 32-neuron blocks (4 or 8)
    constexpr int KS = A_ / 32;          // 32-axon k-steps
    constexpr int PL = TWO ? 2 : 1;      // B planes
    constexpr int STW = NB / 4;          // 32-sample sub-tiles per wave
    constexpr int W_ = A_ / 32;          // axon words
    constexpr int ROWB = L::ROWB;
    constexpr int WPW = (W_ + 7) / 8;    // axon words expanded per wave
    constexpr int APW = A_ / 64;         // 64-axon blocks of the gather
    constexpr int GPW = APW == 8 ? 2 : 1;  // 32-sample groups gathered per wave
    constexpr int FMAX = 4;              // sources per axon kept in registers
    typedef typename RawWord<GPW == 2>::type RawT;
    static_assert(NB == 4 || NB == 8, "N must be 128 or 256");
    static_assert(!(TWO && A_ == 512), "the plane split has no block form");

    __shared__ __attribute__((aligned(16))) typename L::ATile a_lds[2];
    __shared__ typename L::XTile x_lds[2];
    __shared__ unsigned s_cnt[CNT_N][MFMA_TS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int tiles = n.S64 / MFMA_TS;
    int ci_, v;
    core_unit_of(blockIdx.x, ba.count, n.slices * tiles, ci_, v);
    const int c = ba.order[ba.first + ci_];
    const int slice = v % n.slices;
    const int tile = v / n.slices;
    const int s0 = tile * MFMA_TS;
    const int kb = ba.k0 + (ba.step - ba.level[c]) * ba.block;   // first tick (position in the call)
    const int ke = min(kb + ba.block, ba.k0 + ba.ticks);
    if (kb < ba.k0 || kb >= ke)
        return;   // whole workgroups, before any barrier
    const int h = lane >> 5, jj = lane & 31;
    const int sig = sigma32(jj);
    const int nb = wave % NB;
    const int stg = wave / NB;
    const bool live = N_ == 256 || slice * NB + nb < n.NW;   // see integrate_mfma_unit
    const int nbu = live ? nb : 0;
    const int nbc = slice * NB + nbu;

    for (int i = threadIdx.x; i < CNT_N * MFMA_TS; i += blockDim.x)
        (&s_cnt[0][0])[i] = 0u;

    // ---- sources of the gather's axon (lane = axon)
    const bool gatherer = wave < 2 * APW;   // wave-uniform
    const int axb = wave % APW;
    const int grp = GPW == 2 ? 0 : wave / APW;
    uint32_t e_beg = 0, e_end = 0;
    if (gatherer) {
        const int ga = axb * 64 + lane;
        e_beg = n.rtx_ptr[(size_t)c * A_ + ga];
        e_end = n.rtx_ptr[(size_t)c * A_ + ga + 1];
    }
    const size_t HG = (size_t)n.S64 / 64;
    const size_t CN = (size_t)n.C * n.N;
    const size_t slot_words = CN * HG;       // history words per slot
    int q_now = (n.tick[0] + kb) % n.Q, r_row = (n.tick[1] + kb) % n.RT;
    const uint64_t *src_base[FMAX];          // slot 0 row of the source (neuron 0 where unused)
    int src_slot[FMAX];                      // slot read for the next load
    RawT src_mask[FMAX];                     // all ones where the source exists
#pragma unroll
    for (int k = 0; k < FMAX; ++k) {
        const bool used = e_beg + k < e_end;
        const uint32_t ent = used ? n.rtx_ent[e_beg + k] : 0u;
        int slot = q_now - (int)(ent & 15u) - 1;
        src_slot[k] = slot < 0 ? slot + n.Q : slot;
        src_base[k] = n.hist + (size_t)(ent >> 4) * HG + tile;
        src_mask[k] = used ? ~(RawT)0 : (RawT)0;
    }
    const bool multi = __ballot(e_end - e_beg > 1) != 0;          // wave-uniform
    const bool long_lists = __ballot(e_end - e_beg > FMAX) != 0;  // wave-uniform
    auto raw_word = [&](const uint64_t *w) -> RawT {
        if constexpr (GPW == 2)
            return *w;
        else
            return reinterpret_cast<const uint32_t *>(w)[grp];
    };
    auto next_word = [&](int k) -> RawT {
        const RawT w = raw_word(src_base[k] + (size_t)(unsigned)src_slot[k] * slot_words);
        src_slot[k] = src_slot[k] + 1 == n.Q ? 0 : src_slot[k] + 1;
        return w;
    };
    // history words of the next tick in order (called for kb, kb + 1, ...;
    // q: that tick's slot). Loads past the block read a slot of the ring that
    // is never used.
    auto load_mask = [&](int q, RawT (&raw)[FMAX]) {
        raw[0] = next_word(0);
        if (multi) {
#pragma unroll
            for (int k = 1; k < FMAX; ++k)
                raw[k] = next_word(k);
            for (uint32_t e = e_beg + FMAX; long_lists && e < e_end; ++e) {
                const uint32_t ent = n.rtx_ent[e];
                int slot = q - (int)(ent & 15u) - 1;
                if (slot < 0)
                    slot += n.Q;
                // (a lane with this source has all FMAX register sources)
                raw[1] |= raw_word(n.hist + ((size_t)slot * CN + (ent >> 4)) * HG + tile);
            }
        }
    };
    auto mask_of = [&](const RawT (&raw)[FMAX]) -> RawT {
        RawT m = raw[0] & src_mask[0];
        if (multi) {
#pragma unroll
            for (int k = 1; k < FMAX; ++k)
                m |= raw[k] & src_mask[k];
        }
        return m;
    };
    auto transpose_store = [&](RawT m, int buf) {
#pragma unroll
        for (int g = 0; g < GPW; ++g) {
            const uint32_t t = transpose32((uint32_t)(m >> (32 * g)), lane);
            x_lds[buf][32 * (GPW == 2 ? g : grp) + sig][2 * axb + h] = t;
        }
    };
    const int ci = n.in_index[c];
    const bool svalid = s0 + lane < n.S;
    const uint32_t *ext_s =
        (ba.ext_base != nullptr && ci >= 0)
            ? ba.ext_base + (size_t)min(s0 + lane, n.S - 1) * ba.ext_sstride + (size_t)kb * ba.tick_words + (size_t)ci * W_
            : nullptr;
    uint32_t xe[WPW];
#pragma unroll
    for (int k = 0; k < WPW; ++k)
        xe[k] = 0u;
    auto load_ext = [&]() {   // external input words of the next tick in order
        if (!ext_s)
            return;
#pragma unroll
        for (int k = 0; k < WPW; ++k) {
            const int wi = wave + 8 * k;
            if (wi < W_)
                xe[k] = ext_s[wi];
        }
        ext_s += ba.tick_words;
    };
    RawT raw[FMAX] = {};
    if (gatherer)
        load_mask(q_now, raw);
    load_ext();

    // ---- what stays in registers for the block
    v4i breg[KS][PL];
    {
        const v4i *planes = reinterpret_cast<const v4i *>(n.planes);
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                breg[k][p] = planes[((((size_t)c * n.NW + nbc) * KS + k) * PL + p) * 64 + lane];
    }
    const size_t cj = (size_t)c * n.N + slice * N_ + nbu * 32 + jj;
    const int32_t lk = n.leak[cj], th = n.thr[cj], rs = n.rst[cj];
    const int32_t vmin = n.vmin, vmax = n.vmax;
    int32_t fl = vmin;
    bool lin = false;
    if constexpr (EXT) {
        fl = n.floor[cj];
        lin = (n.linmask[cj >> 5] >> (cj & 31)) & 1u;
    }
    const int oi = n.outidx[cj];
    const uint32_t cm32 = n.coremask[(size_t)c * n.NW + nbc];
    const uint32_t om32 = n.outmask[(size_t)c * n.NW + nbc];
    const size_t dg = (size_t)c * n.slices + slice;
    uint32_t degl[WPW][8], degh[WPW][8];
    bool any_hi = false;
#pragma unroll
    for (int k = 0; k < WPW; ++k) {
        const int wi = wave + 8 * k;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            degl[k][q] = wi < W_ ? n.degb[(dg * 2 + 0) * (A_ / 4) + wi * 8 + q] : 0u;
            degh[k][q] = wi < W_ ? n.degb[(dg * 2 + 1) * (A_ / 4) + wi * 8 + q] : 0u;
            any_hi |= degh[k][q] != 0u;
        }
    }
    v4i *vb = reinterpret_cast<v4i *>(n.V) + ((size_t)c * n.NW + nbc) * (2 * HG) * 256 + lane;
    v4i vr[STW][4];   // potentials: element (t, q, e) = row 8q + 4h + e of sub-tile stg * STW + t
#pragma unroll
    for (int t = 0; t < STW; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            vr[t][q] = __builtin_nontemporal_load(vb + ((size_t)(2 * tile + stg * STW + t) * 4 + q) * 64);

    // sub-tiles whose samples end before their 32 rows: rows that exist
    uint32_t vm[STW];
#pragma unroll
    for (int t = 0; t < STW; ++t) {
        vm[t] = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            vm[t] |= (uint32_t)(s0 + 32 * (stg * STW + t) + 8 * (r >> 2) + 4 * h + (r & 3) < n.S) << r;
    }
    // the lane's 32-sample half-word of its neuron's history and raster words
    // (two sub-tiles per wave: lane half h stores sub-tile h)
    const int half = STW == 2 ? h : stg;
    const bool writer = live && (STW == 2 || h == 0);
    uint32_t *hist_w = reinterpret_cast<uint32_t *>(n.hist + cj * HG + tile) + half;
    uint32_t *rast_w = oi >= 0 ? reinterpret_cast<uint32_t *>(reinterpret_cast<uint64_t *>(n.raster) + (size_t)oi * HG + tile) + half
                               : nullptr;
    const size_t rast_row = 2 * (size_t)n.Nout * HG;   // u32 words per raster row

    uint32_t plane[TICK_PLANES];
#pragma unroll
    for (int i = 0; i < TICK_PLANES; ++i)
        plane[i] = 0u;
    unsigned pev = 0, pevh = 0, pdl = 0;   // events (by low and high degree bytes), delivered, of sample s0 + lane

    RawT m = 0;
    if (gatherer) {
        transpose_store(mask_of(raw), 0);
        load_mask(q_now + 1 == n.Q ? 0 : q_now + 1, raw);
        m = mask_of(raw);
    }
    lds_barrier();

#pragma unroll 1
    for (int k = kb; k < ke; ++k) {
        const int buf = (k - kb) & 1;
        int8_t *A = a_lds[buf];
        // A. expansion of tick k, then the words of tick k + 1 into LDS and
        //    the loads for tick k + 2 (history) and k + 1 (input)
#pragma unroll
        for (int i = 0; i < WPW; ++i) {
            const int wi = wave + 8 * i;
            if (wi < W_) {
                const uint32_t xd = x_lds[buf][lane][wi];
                const uint32_t x = xd | (svalid ? xe[i] : 0u);
                pdl += (unsigned)__popc(xd);
                uint32_t d[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    d[q] = (((x >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
                    pev = __builtin_amdgcn_udot4(d[q], degl[i][q], pev, false);
                    if (any_hi)
                        pevh = __builtin_amdgcn_udot4(d[q], degh[i][q], pevh, false);
                }
                v4i *dst = reinterpret_cast<v4i *>(&A[lane * ROWB + 32 * wi]);
                dst[0] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
                dst[1] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
            }
        }
        const bool more = k + 1 < ke;
        if (more) {
            if (gatherer) {
                transpose_store(m, buf ^ 1);
                int q2 = q_now + 2;
                load_mask(q2 >= n.Q ? q2 - n.Q : q2, raw);
            }
            load_ext();
        }
        lds_barrier();

        // C. products and potential update
        uint32_t hb[STW];
        if (live) {
#pragma unroll
            for (int t = 0; t < STW; ++t) {
                v16i acc_lo, acc_hi;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc_lo[r] = lk;
                    acc_hi[r] = 0;
                }
                const int8_t *arow = &A[((stg * STW + t) * 32 + jj) * ROWB + 16 * h];
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const v4i a = *reinterpret_cast<const v4i *>(arow + 32 * s);
                    if constexpr (TWO) {
                        acc_hi = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, breg[s][0], acc_hi, 0, 0, 0);
                        acc_lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, breg[s][1], acc_lo, 0, 0, 0);
                    } else {
                        acc_lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, breg[s][0], acc_lo, 0, 0, 0);
                    }
                }
                uint32_t f = 0;
#pragma unroll
                for (int r = 15; r >= 0; --r) {
                    const int32_t in_leak = TWO ? acc_lo[r] + acc_hi[r] * 128 : acc_lo[r];
                    int32_t u = __builtin_elementwise_add_sat(vr[t][r >> 2][r & 3], in_leak);
                    if constexpr (EXT)
                        u = min(max(u, vmin), vmax);
                    const bool fire = u >= th;
                    if constexpr (EXT)
                        vr[t][r >> 2][r & 3] = fire ? lif_reset(u, th, rs, vmax, lin) : max(u, fl);
                    else
                        vr[t][r >> 2][r & 3] = fire ? rs : u;
                    f = f + f + (uint32_t)fire;
                }
                hb[t] = f & vm[t];
            }
        }
        // D. wait for the loads of A, then store the spike words
        if (gatherer && more)
            m = mask_of(raw);
        asm volatile("" : "+v"(m));
#pragma unroll
        for (int i = 0; i < WPW; ++i)
            asm volatile("" : "+v"(xe[i]));
        if (live) {
            // lane (h, j), two sub-tiles: fire bits of rows 4h' of sub-tile h,
            // h' = 0 in lo, 1 in hi; one sub-tile: both halves the same
            const auto sw = __builtin_amdgcn_permlane32_swap(hb[0], hb[STW - 1], false, false);
            const uint32_t word = (uint32_t)sw[0] | ((uint32_t)sw[1] << 16);
            if (writer) {
                hist_w[(size_t)(unsigned)q_now * (2 * slot_words)] = word;
                if (rast_w)
                    rast_w[(size_t)(unsigned)r_row * rast_row] = word;
            }
            uint32_t carry = word;
#pragma unroll
            for (int i = 0; i < TICK_PLANES; ++i) {
                const uint32_t up = plane[i] & carry;
                plane[i] ^= carry;
                carry = up;
            }
        }
        q_now = q_now + 1 == n.Q ? 0 : q_now + 1;
        r_row = r_row + 1 == n.RT ? 0 : r_row + 1;
    }

    // ---- end of the block: potentials back, counts into the totals
    if (live) {
#pragma unroll
        for (int t = 0; t < STW; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_nontemporal_store(vr[t][q], vb + ((size_t)(2 * tile + stg * STW + t) * 4 + q) * 64);
        unsigned em = 0, ro = 0, ou = 0;
#pragma unroll
        for (int i = 0; i < TICK_PLANES; ++i) {
            const uint32_t sw = transpose32(plane[i], lane);
            em += (unsigned)__popc(sw) << i;
            ro += (unsigned)__popc(sw & cm32) << i;
            ou += (unsigned)__popc(sw & om32) << i;
        }
        if (STW == 2 || h == 0) {
            const int sl = 32 * half + sig;
            atomicAdd(&s_cnt[CNT_EMITTED][sl], em);
            atomicAdd(&s_cnt[CNT_ROUTED][sl], ro);
            atomicAdd(&s_cnt[CNT_OUT][sl], ou);
        }
    }
    atomicAdd(&s_cnt[CNT_EVENTS][lane], pev + (pevh << 8));
    atomicAdd(&s_cnt[CNT_DELIVERED][lane], pdl);
    lds_barrier();
    if (threadIdx.x < MFMA_TS && s0 + (int)threadIdx.x < n.S) {
        unsigned long long *cp = n.cnt + (((size_t)c * n.cnt_rows + slice) * n.S + s0 + threadIdx.x) * CNT_N;
#pragma unroll
        for (int i = 0; i < CNT_N; ++i)
            if (i != CNT_DELIVERED || slice == 0)   // the core's delivered spikes are counted once
                cp[i] += s_cnt[i][threadIdx.x];
    }
}

template <int A_, int N_, bool TWO>
static void launch_ticks_k(const DevNet &n, const BlockArgs &a, unsigned grid, hipStream_t st)
{
    if (n.model_ext)
        hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, true>), dim3(grid), dim3(512), 0, st, n, a);
    else
        hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, false>), dim3(grid), dim3(512), 0, st, n, a);
}

template <int A_, int N_>
static hipError_t launch_ticks_an(const DevNet &n, const BlockArgs &a, int two, unsigned grid, hipStream_t st)
{
    if (!two)
        launch_ticks_k<A_, N_, false>(n, a, grid, st);
    else if constexpr (A_ <= 256)
        launch_ticks_k<A_, N_, true>(n, a, grid, st);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

bool mfma_ticks_supported(int A, int N, int two_planes)
{
    // the plane split (512 axons, two planes) runs tick by tick
    return mfma_shape_supported(A, N, two_planes) && A * (two_planes ? 2 : 1) <= 512;
}

hipError_t launch_integrate_mfma_ticks(const DevNet &n, const BlockArgs &a, int two, hipStream_t st)
{
    const long long grid = (long long)a.count * n.slices * (n.S64 / MFMA_TS);
    if (!mfma_ticks_supported(n.A, n.N, two) || n.slices != mfma_slices(n.A, n.N, two) || n.cnt_rows != n.slices ||
        n.vlayout != VLAYOUT_BRICK || n.S64 % MFMA_TS || n.S > n.S64 || !n.planes || !a.order || !a.level ||
        a.first < 0 || a.count < 1 || a.first + a.count > n.C || a.block < 1 || a.block > MFMA_BLOCK_TICKS_MAX ||
        a.ticks < 1 || a.ticks + n.D > n.Q || a.k0 < 0 || a.k0 + a.ticks > n.RT || grid > INT32_MAX)
        return hipErrorInvalidValue;
    const int w = mfma_width(n.A, n.N, two);
    switch (n.A * 2 + (w == 256 ? 1 : 0)) {
    case 128: return launch_ticks_an<64, 128>(n, a, two, (unsigned)grid, st);
    case 129: return launch_ticks_an<64, 256>(n, a, two, (unsigned)grid, st);
    case 256: return launch_ticks_an<128, 128>(n, a, two, (unsigned)grid, st);
    case 257: return launch_ticks_an<128, 256>(n, a, two, (unsigned)grid, st);
    case 512: return launch_ticks_an<256, 128>(n, a, two, (unsigned)grid, st);
    case 513: return launch_ticks_an<256, 256>(n, a, two, (unsigned)grid, st);
    case 1024: return launch_ticks_an<512, 128>(n, a, two, (unsigned)grid, st);
    case 1025: return launch_ticks_an<512, 256>(n, a, two, (unsigned)grid, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ranc
