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
// per wavefront about 230 vector instructions and 32 MFMA of 32 cycles.
// Measured on that net, 32 ticks per call: 220 -> 64 us per tick at 1024
// samples, of it 53 per further tick and 10 for moving the potentials and
// setting up (509 us per level); 35 -> 9 us at 100 samples. With the packed
// output raster 7.77 -> 2.13 ms and 1.17 -> 0.29 ms per call, of it 0.62 and 0.05
// -> 0.09 and 0.01 for packing.
//
// Mapping: one workgroup per (core, neuron slice, 32-sample group), of 4
// wavefronts that own 64 neurons each (two 32-neuron blocks; 32 neurons each
// in 128-neuron slices and, on 8 wavefronts, with 512 axons). A wavefront's B
// tiles (int8 planes) and potentials stay in registers for the block of ticks:
// 128 + 32 of the 256 registers that two workgroups per CU leave a lane, so
// the axon operands come from LDS in two halves, and what is only summed over
// the block (spike words, axon spike counts) lives in LDS: a register spilled
// to memory in the loop makes its reload wait for the history loads in flight
// (794 us per level of 128 cores, 1024 samples and 32 ticks, where the form
// without spills took 566). One workgroup of 8 wavefronts per 64 samples, whose
// barrier stops the whole CU, took 587 then.
// The MFMA chain of one neuron block (16 of 32 cycles each) and the vector
// work of the other are independent, so the loop pairs them and the two pipes
// of a SIMD run side by side; with one barrier per tick:
//   first half   products of block 1, tick k; update of block 0, tick k;
//                expansion of tick k + 1 to the int8 tile; axon words of tick
//                k + 2 into LDS;
//   barrier      (LDS only; the int8 tile and the axon words are doubled)
//   second half  products of block 0, tick k + 1; update of block 1 and spike
//                words of tick k; history bits of tick k + 3 transposed, those
//                of tick k + 4 and the input of tick k + 3 loaded.
// (One block per wavefront: products of tick k + 1 beside the update of tick
// k.) Stores are issued after the loads of the same half, so no wait for a
// load covers a store of its tick.
// The two halves of a neuron's 16-bit fire masks are joined by one
// v_permlane32_swap: lane (h, j) then holds the word of neuron j of block h.
// Spike counts come from the lane's spike words at the end of the block, by
// vertical counters (bit plane p of a lane holds bit p of the count of each of
// its 32 samples), synaptic events from the axons' spike counts; the per-tick
// kernel transposes and multiplies every tick's words for them.
#include <type_traits>

#include "kern_mfma_unit.h"

namespace ranc {

// Bit planes of the vertical counters: a block runs at most 2^6 - 1 ticks.
static constexpr int TICK_PLANES = 6;
// scheduling fence that scalar and memory instructions may cross
static constexpr int SCHED_MEMORY_MAY_CROSS = 0x4 | 0x10 | 0x80;
static constexpr uint32_t NO_SOURCE = 0xFFFFFFFFu;   // (a source entry is below 2^27)
static_assert(MFMA_BLOCK_TICKS_MAX < (1 << TICK_PLANES), "vertical counters overflow");

// Wavefronts per workgroup and 32-neuron blocks per wavefront.
template <int A_, int N_> struct TicksShape {
    static constexpr int NPB = N_ == 256 && A_ <= 256 ? 2 : 1;
    static constexpr int WAVES = N_ / 32 / NPB;
};

// MULTI: some axon has several sources (FMAX in registers, the rest read from
// the table every tick).
template <int A_, int N_, bool TWO, bool EXT, bool MULTI>
__global__ __launch_bounds__((64 * TicksShape<A_, N_>::WAVES), (A_ == 512 && N_ == 128 ? 1 : 2)) void k_integrate_mfma_ticks(DevNet n, BlockArgs ba)
{
    constexpr int NPB = TicksShape<A_, N_>::NPB;
    constexpr int WAVES = TicksShape<A_, N_>::WAVES;
    constexpr int KS = A_ / 32;                // 32-axon k-steps
    constexpr int KC = KS > 8 ? 8 : (TWO && NPB == 2 && KS > 4) ? 4 : KS;        // k-steps whose operands are held at a time
    constexpr int PL = TWO ? 2 : 1;            // B planes
    constexpr int W_ = A_ / 32;                // axon words
    constexpr int ROWB = A_ + 16;              // padded LDS row of the int8 tile (bytes)
    constexpr int WPW = (W_ + 2 * WAVES - 1) / (2 * WAVES);   // axon words expanded per lane
    constexpr int APW = A_ / 64;               // 64-axon blocks of the gather
    constexpr int GB = (APW + WAVES - 1) / WAVES;   // of them per wavefront
    constexpr int FMAX = MULTI ? 4 : 1;        // sources per axon kept in registers
    constexpr int THREADS = 64 * WAVES;
    constexpr int TS = 32;                     // samples per workgroup

    __shared__ __attribute__((aligned(16))) int8_t a_lds[2][TS * ROWB];
    __shared__ uint32_t x_lds[2][TS][W_ + 1];
    __shared__ unsigned s_cnt[CNT_N][TS];
    // per lane: the spike word of every tick, and the spikes of each axon of
    // the lane's words so far, one byte per axon
    __shared__ uint32_t word_lds[MFMA_BLOCK_TICKS_MAX][THREADS];
    __shared__ uint32_t spike_lds[WPW * 8][THREADS];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int groups = (n.S + TS - 1) / TS;
    int ci_, v;
    core_unit_of(blockIdx.x, ba.count, n.slices * groups, ci_, v);
    const int c = ba.order[ba.first + ci_];
    const int slice = v % n.slices;
    const int grp = v / n.slices;
    const int s0 = grp * TS;
    const int kb = ba.k0 + (ba.step - ba.level[c]) * ba.block;   // first tick (position in the call)
    const int ke = min(kb + ba.block, ba.k0 + ba.ticks);
    if (kb < ba.k0 || kb >= ke)
        return;   // whole workgroups, before any barrier
    const int h = lane >> 5, jj = lane & 31;
    const int sig = sigma32(jj);
    // 32-neuron blocks of the core that this wavefront owns; 64-neuron cores
    // run as a 128-neuron slice whose upper two blocks are dead (wave-uniform)
    const int nb0 = slice * (N_ / 32) + wave * NPB;
    const bool live = N_ == 256 || nb0 < n.NW;
    const int nbu = live ? nb0 : 0;

    for (int i = threadIdx.x; i < CNT_N * TS; i += THREADS)
        (&s_cnt[0][0])[i] = 0u;
#pragma unroll
    for (int q = 0; q < WPW * 8; ++q)
        spike_lds[q][threadIdx.x] = 0u;

    // ---- sources of the gather's axons (lane = axon of block wave + WAVES g)
    const bool gatherer = APW >= WAVES || wave < APW;   // wave-uniform
    const size_t HG = (size_t)n.S64 / 64;
    const size_t CN = (size_t)n.C * n.N;
    const int Q = n.Q;
    // (the ring is below 4 GiB: offsets into it fit 32 bits)
    const uint32_t slot_bytes = (uint32_t)(CN * HG * 8), ring_bytes = (uint32_t)Q * slot_bytes;
    const int q0 = (n.tick[0] + kb) % Q, r0 = (n.tick[1] + kb) % n.RT;
    const char *hist_g = reinterpret_cast<const char *>(n.hist) + 4 * grp;   // the group's half words
    // the first source as the offset of its word of the next tick to load
    // (neuron 0 where the axon has none), the others as table entries
    uint32_t src0[GB], mask0[GB], ents[GB][FMAX], e_beg[GB] = {}, e_end[GB] = {};
    int delay0[GB];
    bool long_lists = false;   // wave-uniform
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        if (gatherer) {
            const int ga = (wave + WAVES * g) * 64 + lane;
            e_beg[g] = n.rtx_ptr[(size_t)c * A_ + ga];
            e_end[g] = n.rtx_ptr[(size_t)c * A_ + ga + 1];
        }
        const bool any = e_beg[g] < e_end[g];
        const uint32_t ent0 = any ? n.rtx_ent[e_beg[g]] : 0u;
        delay0[g] = (int)(ent0 & 15u) + 1;
        src0[g] = (ent0 >> 4) * (uint32_t)(HG * 8) + (uint32_t)(q0 - delay0[g] + (q0 < delay0[g] ? Q : 0)) * slot_bytes;
        mask0[g] = any ? ~0u : 0u;
#pragma unroll
        for (int k = 1; k < FMAX; ++k)
            ents[g][k] = e_beg[g] + k < e_end[g] ? n.rtx_ent[e_beg[g] + k] : NO_SOURCE;
        long_lists |= __ballot(e_end[g] - e_beg[g] > FMAX) != 0;
    }
    // History words of the next tick in order (q_load: its slot). Loads past
    // the block read a slot of the ring that is never used.
    int q_load = q0;
    auto word_of = [&](uint32_t ent) -> uint32_t {
        const int slot = q_load - (int)(ent & 15u) - 1;
        return *reinterpret_cast<const uint32_t *>(hist_g + ((ent >> 4) * (uint32_t)(HG * 8) +
                                                             (uint32_t)(slot < 0 ? slot + Q : slot) * slot_bytes));
    };
    auto load_mask = [&](uint32_t (&raw)[GB][FMAX]) {
#pragma unroll
        for (int g = 0; g < GB; ++g)
            raw[g][0] = *reinterpret_cast<const uint32_t *>(hist_g + src0[g]);
        if constexpr (MULTI) {
#pragma unroll
            for (int g = 0; g < GB; ++g) {
#pragma unroll
                for (int k = 1; k < FMAX; ++k) {
                    raw[g][k] = 0;
                    if (ents[g][k] != NO_SOURCE)
                        raw[g][k] = word_of(ents[g][k]);
                }
                for (uint32_t e = e_beg[g] + FMAX; long_lists && e < e_end[g]; ++e)
                    raw[g][1] |= word_of(n.rtx_ent[e]);
            }
        }
        q_load = q_load + 1 == Q ? 0 : q_load + 1;
        // (sources of delay q_load go on from slot Q - 1 to slot 0)
#pragma unroll
        for (int g = 0; g < GB; ++g)
            src0[g] += slot_bytes - (delay0[g] == q_load ? ring_bytes : 0);
    };
    // lane (h, j): bits of axon 32 h + j of the 64-axon block; after the
    // transpose lane (h, i) holds the block's axon word h of the sample of bit i
    auto words_of = [&](const uint32_t (&raw)[GB][FMAX], uint32_t (&t)[GB]) {
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            uint32_t m = raw[g][0] & mask0[g];
#pragma unroll
            for (int k = 1; k < FMAX; ++k)
                m |= raw[g][k];
            t[g] = transpose32(m, lane);
        }
    };
    auto store_words = [&](const uint32_t (&t)[GB], int buf) {
#pragma unroll
        for (int g = 0; g < GB; ++g)
            x_lds[buf][sig][2 * (wave + WAVES * g) + h] = t[g];
    };
    // external input words of the next tick in order: lane (h, j) takes words
    // 2 (wave + WAVES w) + h of sample s0 + j (a row of zeros where the core
    // takes none); the last tick of the block is loaded again past its end
    const int ci = n.in_index[c];
    const bool has_ext = ba.ext_base != nullptr && ci >= 0;
    const uint32_t svalid = s0 + jj < n.S ? ~0u : 0u;
    const uint32_t *ext_t = has_ext ? ba.ext_base + (size_t)s0 * ba.ext_sstride + (size_t)kb * ba.tick_words + (size_t)ci * W_
                                    : reinterpret_cast<const uint32_t *>(n.hist_zero);   // uniform
    const uint32_t ext_s = has_ext ? (uint32_t)(min(jj, n.S - 1 - s0) * ba.ext_sstride) : 0u;
    const long long ext_step = has_ext ? ba.tick_words : 0;
    int k_ext = kb;
    uint32_t xe[WPW], xn[WPW];
    auto load_ext = [&]() {
#pragma unroll
        for (int w = 0; w < WPW; ++w)
            xe[w] = ext_t[ext_s + min(2 * (wave + WAVES * w) + h, W_ - 1)];
        ++k_ext;
        ext_t += k_ext < ke ? ext_step : 0;
    };
    auto take_ext = [&]() {   // the loaded words are waited for here
#pragma unroll
        for (int w = 0; w < WPW; ++w) {
            xn[w] = xe[w];
            asm volatile("" : "+v"(xn[w]));
        }
    };
    uint32_t raw0[GB][FMAX] = {}, raw1[GB][FMAX] = {}, raw2[GB][FMAX] = {};
    if (gatherer) {
        load_mask(raw0);
        load_mask(raw1);
        load_mask(raw2);
    }
    load_ext();

    // ---- what stays in registers for the block of ticks
    v4i breg[NPB][KS][PL];
    const v4i *planes = reinterpret_cast<const v4i *>(n.planes);
#pragma unroll
    for (int t = 0; t < NPB; ++t)
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                breg[t][k][p] = planes[((((size_t)c * n.NW + nbu + t) * KS + k) * PL + p) * 64 + lane];
    const size_t cj = (size_t)c * n.N + nbu * 32 + jj;   // neuron of block 0
    const int32_t vmin = n.vmin, vmax = n.vmax;
    int32_t lk[NPB], th[NPB], rs[NPB], fl[NPB];
    bool lin[NPB];
#pragma unroll
    for (int t = 0; t < NPB; ++t) {
        lk[t] = n.leak[cj + 32 * t];
        th[t] = n.thr[cj + 32 * t];
        rs[t] = n.rst[cj + 32 * t];
        fl[t] = vmin;
        lin[t] = false;
        if constexpr (EXT) {
            fl[t] = n.floor[cj + 32 * t];
            lin[t] = (n.linmask[(cj >> 5) + t] >> jj) & 1u;
        }
    }
    v4i *vb = reinterpret_cast<v4i *>(n.V) + (((size_t)c * n.NW + nbu) * (2 * HG) + grp) * 256 + lane;
    const size_t vb_step = 2 * HG * 256;   // to the next neuron block
    v4i vr[NPB][4];   // potentials: element (t, q, e) = neuron j of block t, sample 8q + 4h + e
#pragma unroll
    for (int t = 0; t < NPB; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            vr[t][q] = __builtin_nontemporal_load(vb + t * vb_step + q * 64);

    // spike-word bits whose samples exist
    uint32_t vmask = 0;
    for (int b = 0; b < 32; ++b)
        vmask |= (uint32_t)(s0 + sigma32(b) < n.S) << b;
    // the lane's neuron when spike words are written (two blocks: lane half h
    // writes block h) and its history and raster words of the group
    const int tw_ = NPB == 2 ? h : 0;
    const size_t cw = cj + 32 * tw_;
    const bool writer = live && (NPB == 2 || h == 0);
    const uint32_t hist_o = (uint32_t)(cw * (HG * 8)) + 4 * grp;
    const int oi = n.outidx[cw];
    const uint32_t rast_o = (uint32_t)(oi >= 0 ? oi : 0) * (uint32_t)(HG * 8) + 4 * grp;   // (a row is below 4 GiB)
    const size_t row_bytes = (size_t)n.Nout * HG * 8;
    int q_now = q0, r_row = r0;
    unsigned pdl = 0;          // delivered spikes in the lane's words

    // axon words of tick i of the block (i < ticks: on = ~0, else 0) to int8
    auto expand = [&](int i, uint32_t on) {
#pragma unroll
        for (int w = 0; w < WPW; ++w) {
            const int wi = 2 * (wave + WAVES * w) + h;
            if (2 * WAVES * (w + 1) <= W_ || wave + WAVES * w < W_ / 2) {   // wave-uniform
                const uint32_t xd = x_lds[i & 1][jj][wi] & on;
                const uint32_t x = xd | (xn[w] & svalid & on);
                pdl += (unsigned)__popc(xd);
                uint32_t d[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    // nibble b3b2b1b0 -> bytes: bit i moves to bit 8i, no carries
                    d[q] = (((x >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
                    atomicAdd(&spike_lds[8 * w + q][threadIdx.x], d[q]);
                }
                v4i *dst = reinterpret_cast<v4i *>(&a_lds[i & 1][jj * ROWB + 32 * wi]);
                dst[0] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
                dst[1] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
            }
        }
    };
    // axon operands of k-steps [k, k + KC) of tick i of the block
    v4i ax[KC];
    auto load_axons = [&](int i, int k) {
        const int8_t *arow = &a_lds[i & 1][jj * ROWB + 16 * h];
#pragma unroll
        for (int s = 0; s < KC; ++s)
            ax[s] = *reinterpret_cast<const v4i *>(arow + 32 * (k + s));
    };
    // leak, threshold and reset of samples 8q + 4h + [0, 4) of block t from
    // their input plus leak; f = fire bits so far, doubled per row
    auto update_rows = [&](const v16i &a, int t, int q, uint32_t &f) {
        int32_t u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            u[e] = __builtin_elementwise_add_sat(vr[t][q][e], a[4 * q + e]);
            if constexpr (EXT)
                u[e] = min(max(u[e], vmin), vmax);
        }
        if constexpr (EXT) {
            int32_t v[4], r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = max(u[e], fl[t]);
                r[e] = lif_reset(u[e], th[t], rs[t], vmax, lin[t]);
            }
            fire_rows(f, v[0], v[1], v[2], v[3], u[0], u[1], u[2], u[3], r[0], r[1], r[2], r[3], th[t]);
            vr[t][q] = v4i{v[0], v[1], v[2], v[3]};
        } else {
            fire_rows(f, u[0], u[1], u[2], u[3], rs[t], th[t]);
            vr[t][q] = v4i{u[0], u[1], u[2], u[3]};
        }
    };
    // Products of block tp on the loaded operands (tick i of the block of
    // ticks), plus leak, into `out`, beside the update of block tu from `in`
    // (tu < 0: none); returns the update's fire bits. Two planes go through
    // one accumulator: the high plane's sums are shifted up in place and the
    // low plane's added on (16 registers fewer than two sums). The scheduling
    // fences keep the update spread over the first plane's products; the
    // second plane's run beside what follows.
    auto products = [&](auto tp_, auto tu_, int i, v16i &out, const v16i &in) -> uint32_t {
        constexpr int tp = decltype(tp_)::value, tu = decltype(tu_)::value;
        uint32_t f = 0;
        v16i a;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            a[r] = TWO ? 0 : lk[tp];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int s = q * KS / 4; s < (q + 1) * KS / 4; ++s) {
                if (KS > KC && s > 0 && s % KC == 0)
                    load_axons(i, s);
                a = __builtin_amdgcn_mfma_i32_32x32x32_i8(ax[s % KC], breg[tp][s][0], a, 0, 0, 0);
            }
            if constexpr (tu >= 0) {
                update_rows(in, tu, 3 - q, f);
                __builtin_amdgcn_sched_barrier(SCHED_MEMORY_MAY_CROSS);
            }
        }
        if constexpr (TWO) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                a[r] = a[r] * 128 + lk[tp];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (KS > KC && s % KC == 0)
                    load_axons(i, s);
                a = __builtin_amdgcn_mfma_i32_32x32x32_i8(ax[s % KC], breg[tp][s][1], a, 0, 0, 0);
            }
            if (KS > KC && NPB == 2 && tp == 0)
                load_axons(i, 0);   // for block 1
        }
        out = a;
        return f;
    };
    constexpr std::integral_constant<int, 0> blk0{};
    constexpr std::integral_constant<int, NPB - 1> blk1{};
    constexpr std::integral_constant<int, -1> no_update{};

    uint32_t tw[GB] = {};   // axon words of the tick two ahead
    if (gatherer) {
        words_of(raw0, tw);
        store_words(tw, 0);
        words_of(raw1, tw);
        store_words(tw, 1);
        words_of(raw2, tw);
        load_mask(raw0);
    }
    lds_barrier();
    const int ticks = ke - kb;
    take_ext();
    load_ext();
    expand(0, ~0u);
    take_ext();
    load_ext();
    lds_barrier();
    v16i acc0, acc1;
    load_axons(0, 0);
    products(blk0, no_update, 0, acc0, acc0);

#pragma unroll 1
    for (int i = 0; i < ticks; ++i) {
        // first half
        uint32_t hb[NPB];
        if constexpr (NPB == 2)
            hb[0] = products(blk1, blk0, i, acc1, acc0);
        expand(i + 1, i + 1 < ticks ? ~0u : 0u);
        if (gatherer)
            store_words(tw, i & 1);
        lds_barrier();

        // second half
        load_axons(i + 1, 0);
        if (gatherer) {
            words_of(raw0, tw);
            load_mask(raw0);
        }
        take_ext();
        load_ext();
        if constexpr (NPB == 2) {
            hb[1] = products(blk0, blk1, i + 1, acc0, acc1);
        } else {
            hb[0] = products(blk0, blk0, i + 1, acc1, acc0);
            acc0 = acc1;
        }
        // lane (h, j), two blocks: fire bits of samples 4h' of neuron j of
        // block h, h' = 0 in the low half, 1 in the high; one block: its word
        // in both lane halves
        rows_settled(hb[NPB - 1]);
        const auto sw = __builtin_amdgcn_permlane32_swap(hb[0], hb[NPB - 1], false, false);
        const uint32_t word = ((uint32_t)sw[0] | ((uint32_t)sw[1] << 16)) & vmask;
        word_lds[i][threadIdx.x] = word;
        if (writer) {
            *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(n.hist) + (size_t)(unsigned)q_now * slot_bytes + hist_o) = word;
            if (oi >= 0)
                *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(n.raster) + (unsigned)r_row * row_bytes + rast_o) = word;
        }
        q_now = q_now + 1 == Q ? 0 : q_now + 1;
        r_row = r_row + 1 == n.RT ? 0 : r_row + 1;
    }

    // ---- end of the block: potentials back, counts into the totals
    if (live) {
#pragma unroll
        for (int t = 0; t < NPB; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_nontemporal_store(vr[t][q], vb + t * vb_step + q * 64);
        const uint32_t cm32 = n.coremask[(size_t)c * n.NW + nbu + tw_], om32 = n.outmask[(size_t)c * n.NW + nbu + tw_];
        // vertical counters over the block's spike words: bit plane p of a lane
        // holds bit p of the count of each of its 32 samples
        uint32_t plane[TICK_PLANES] = {};
        for (int i = 0; i < ticks; ++i) {
            uint32_t carry = word_lds[i][threadIdx.x];
#pragma unroll
            for (int p = 0; p < TICK_PLANES; ++p) {
                const uint32_t up = plane[p] & carry;
                plane[p] ^= carry;
                carry = up;
            }
        }
        unsigned em = 0, ro = 0, ou = 0;
#pragma unroll
        for (int p = 0; p < TICK_PLANES; ++p) {
            const uint32_t sw = transpose32(plane[p], lane);
            em += (unsigned)__popc(sw) << p;
            ro += (unsigned)__popc(sw & cm32) << p;
            ou += (unsigned)__popc(sw & om32) << p;
        }
        if (NPB == 2 || h == 0) {
            atomicAdd(&s_cnt[CNT_EMITTED][sig], em);
            atomicAdd(&s_cnt[CNT_ROUTED][sig], ro);
            atomicAdd(&s_cnt[CNT_OUT][sig], ou);
        }
    }
    // synaptic events: each axon's spikes times its connected neurons
    unsigned pev = 0, pevh = 0;
    const size_t dg = (size_t)c * n.slices + slice;
#pragma unroll
    for (int w = 0; w < WPW; ++w) {
        const int wi = min(2 * (wave + WAVES * w) + h, W_ - 1);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            pev = __builtin_amdgcn_udot4(spike_lds[8 * w + q][threadIdx.x], n.degb[(dg * 2 + 0) * (A_ / 4) + wi * 8 + q], pev, false);
            pevh = __builtin_amdgcn_udot4(spike_lds[8 * w + q][threadIdx.x], n.degb[(dg * 2 + 1) * (A_ / 4) + wi * 8 + q], pevh, false);
        }
    }
    atomicAdd(&s_cnt[CNT_EVENTS][jj], pev + (pevh << 8));
    atomicAdd(&s_cnt[CNT_DELIVERED][jj], pdl);
    lds_barrier();
    if (threadIdx.x < TS && s0 + (int)threadIdx.x < n.S) {
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
    const dim3 block(64 * TicksShape<A_, N_>::WAVES);
    switch ((n.model_ext ? 2 : 0) + (a.multi ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, false, false>), dim3(grid), block, 0, st, n, a); break;
    case 1: hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, false, true>), dim3(grid), block, 0, st, n, a); break;
    case 2: hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, true, false>), dim3(grid), block, 0, st, n, a); break;
    default: hipLaunchKernelGGL((k_integrate_mfma_ticks<A_, N_, TWO, true, true>), dim3(grid), block, 0, st, n, a); break;
    }
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

// Offsets into the history ring, a raster row and a group's inputs fit 32 bits.
bool mfma_ticks_offsets_fit(int C, int N, int S64, int Q, int Nout, long long ext_sstride)
{
    const unsigned long long word = (unsigned long long)S64 / 64 * 8, lim = 1ull << 32;
    return (unsigned long long)C * N * word * Q < lim && (unsigned long long)Nout * word < lim &&
           (unsigned long long)ext_sstride * 32 < lim / 4;
}

hipError_t launch_integrate_mfma_ticks(const DevNet &n, const BlockArgs &a, int two, hipStream_t st)
{
    const long long grid = (long long)a.count * n.slices * ((n.S + 31) / 32);   // 32 samples per workgroup
    if (!mfma_ticks_supported(n.A, n.N, two) || n.slices != mfma_slices(n.A, n.N, two) || n.cnt_rows != n.slices ||
        n.vlayout != VLAYOUT_BRICK || n.S64 % MFMA_TS || n.S > n.S64 || !n.planes || !a.order || !a.level ||
        a.first < 0 || a.count < 1 || a.first + a.count > n.C || a.block < 1 || a.block > MFMA_BLOCK_TICKS_MAX ||
        a.ticks < 1 || a.ticks + n.D > n.Q || !mfma_ticks_offsets_fit(n.C, n.N, n.S64, n.Q, n.Nout, a.ext_sstride) || a.k0 < 0 || a.k0 + a.ticks > n.RT || grid > INT32_MAX)
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
