// runtime.cpp -- host side of the C ABI declared in include/ranc.h.
//
// Validation of the network description, the workspace layout, host-side
// packing of the description into the device layouts of ranc_internal.h
// (crossbar columns, per-type masks, MFMA weight planes, the inverted routing
// table), the tick loop that queues the per-tick kernels (per launch or as a
// captured HIP graph), batches of several networks, the launch-shape
// autotuner, and readback.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/ranc.h"
#include "ranc_internal.h"

using namespace ranc;

namespace {

thread_local std::string g_err;

ranc_status fail(ranc_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

ranc_status hip_fail(hipError_t e, const char *what)
{
    return fail(RANC_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

enum Region {
    R_COLBITS, R_TYPEMASK, R_WTS, R_LEAK, R_THR, R_RST, R_VINIT, R_COREMASK, R_OUTMASK, R_OUTWORD,
    R_ININDEX, R_RTDCNT, R_RTGOFF, R_RTENT, R_DEGB, R_OUTIDX, R_RTXPTR, R_RTXENT, R_HZERO,
    R_FLOOR, R_LINMASK, R_ECSRPTR, R_ECSRENT, R_LINKREC, R_OUTCOL, R_OUTPOS, R_LINKPTR, R_LINKENT, R_PLAINDST, R_SCOLS, R_SPOS,
    R_PARAMS_END,  // everything before this is uploaded once at load
    R_V = R_PARAMS_END, R_RING, R_SPK, R_HIST, R_RASTER, R_CNT, R_CRING, R_TICK, R_BATCH, R_EXT, R_LINKD,
    R_RSYNC,
    // MFMA path: the compact B source, uploaded at load as well; kept past
    // the state regions so that their placement does not depend on it; and the
    // int8 planes, built from it on the GPU
    R_BSRC, R_PLANES,
    // feed-forward networks (MFMA and plain paths): cores by level, then each
    // core's level; uploaded at load
    R_ORDER,
    // plain path, small networks: the byte ring
    R_RING8, R_NREG
};

struct Plan {
    int C, A, N, G, W, NW, D, Q, S, S64, RT, Wout, Nout, Cin, path, two, spw, spw_pipelined;
    int bsrc;            // MFMA path B source: -1 by mfma_compact_b, 0 the planes, 1 the compact crossbar
    int grid_w, grid_h;  // mesh size
    int slices;          // MFMA and sparse: neuron slices per core (one workgroup each)
    int cnt_rows;        // counter rows per core
    long long E;         // routed (CORE) neurons
    long long ell_words; // u32 words of the wave-interleaved routing table
    long long ecsr_entries; // sparse path: row entries, each slice's rows padded to sparse_row_align()
    size_t off[R_NREG], size[R_NREG], params_bytes, total;
    // MFMA path, feed-forward networks (kern_mfma_ticks.hip): cores by
    // ascending level, each core's level, the levels' first positions in
    // `order` (levels + 1 entries), and the ticks a segment of a call may run
    // at most (the history ring holds D more). No levels: tick by tick.
    int levels = 0, seg_ticks = 1;
    bool auto_mid = false;       // the MFMA path chosen for fewer than 64 samples
    bool multi_source = false;   // some axon has several sources
    int sorted_words = 0;        // plain path: words per axon type of the sorted columns, 0: none
    std::vector<int32_t> order, level, level_first;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Batch tables (several networks advanced by one launch per tick) live in the
// workspace of the batch's first network: up to BATCH_MAX entries for the
// MFMA path, then up to BATCH_MAX for the plain path, then two queue counters.
constexpr int BATCH_MAX = 128;
constexpr size_t BATCH_TABLE_BYTES = 2 * BATCH_MAX * sizeof(BatchEntry) + 256;

bool pow2_in(int v, int lo, int hi) { return v >= lo && v <= hi && (v & (v - 1)) == 0; }

ranc_status validate(const ranc_net_desc *d, int32_t S, int32_t RT, int32_t path)
{
    if (!d)
        return fail(RANC_EINVAL, "desc is NULL");
    if (d->abi_version != RANC_ABI_VERSION)
        return fail(RANC_EINVAL, "abi_version %u != %u", d->abi_version, RANC_ABI_VERSION);
    if (S < 1)
        return fail(RANC_EINVAL, "num_samples must be >= 1 (got %d)", S);
    if (S > 65535)
        return fail(RANC_EUNSUPPORTED, "num_samples must be <= 65535 (got %d)", S);
    if (RT < 1)
        return fail(RANC_EINVAL, "max_ticks_per_call must be >= 1 (got %d)", RT);
    if (path < RANC_PATH_AUTO || path > RANC_PATH_SPARSE)
        return fail(RANC_EINVAL, "unknown path %d", path);
    if (d->num_cores < 1)
        return fail(RANC_EINVAL, "num_cores must be >= 1");
    if (d->grid_w < 1 || d->grid_h < 1 || (long long)d->grid_w * d->grid_h != d->num_cores)
        return fail(RANC_EINVAL, "grid %dx%d does not hold %d cores", d->grid_w, d->grid_h, d->num_cores);
    if (!pow2_in(d->num_axons, 64, 512))
        return fail(RANC_EUNSUPPORTED, "num_axons must be 64, 128, 256 or 512 (got %d)", d->num_axons);
    if (!pow2_in(d->num_neurons, 64, 512))
        return fail(RANC_EUNSUPPORTED, "num_neurons must be 64, 128, 256 or 512 (got %d)", d->num_neurons);
    if (!pow2_in(d->num_types, 1, 8))
        return fail(RANC_EUNSUPPORTED, "num_types must be 1, 2, 4 or 8 (got %d)", d->num_types);
    if (d->weight_bits < 2 || d->weight_bits > 9)
        return fail(RANC_ERANGE, "weight_bits must be in [2, 9] (got %d)", d->weight_bits);
    if (d->potential_bits < 2 || d->potential_bits > 32)
        return fail(RANC_ERANGE, "potential_bits must be in [2, 32] (got %d)", d->potential_bits);
    if (d->max_delay < 1 || d->max_delay > 15)
        return fail(RANC_ERANGE, "max_delay must be in [1, 15] (got %d)", d->max_delay);
    if ((long long)d->num_cores * d->num_neurons > RT_MAX_NEURONS)
        return fail(RANC_EUNSUPPORTED, "num_cores * num_neurons must be <= 2^23");
    if (!d->crossbar || !d->axon_type || !d->weight || !d->leak || !d->threshold || !d->reset ||
        !d->v_init || !d->dest_kind || !d->dest_dx || !d->dest_dy || !d->dest_axon || !d->dest_delay)
        return fail(RANC_EINVAL, "a parameter array pointer is NULL");
    if (d->num_input_cores < 0 || d->num_input_cores > d->num_cores)
        return fail(RANC_EINVAL, "num_input_cores out of range (%d)", d->num_input_cores);
    if (d->num_input_cores > 0 && !d->input_cores)
        return fail(RANC_EINVAL, "input_cores is NULL");
    const int C = d->num_cores, A = d->num_axons, N = d->num_neurons, G = d->num_types;
    for (size_t i = 0; i < (size_t)C * A; ++i)
        if (d->axon_type[i] >= G)
            return fail(RANC_ERANGE, "axon_type[%zu] = %u is not < num_types", i, d->axon_type[i]);
    const int wlo = -(1 << (d->weight_bits - 1)), whi = (1 << (d->weight_bits - 1)) - 1;
    for (size_t i = 0; i < (size_t)C * N * G; ++i)
        if (d->weight[i] < wlo || d->weight[i] > whi)
            return fail(RANC_ERANGE, "weight[%zu] = %d outside %d-bit range", i, d->weight[i], d->weight_bits);
    const int leak_bits = d->leak_bits ? d->leak_bits : 32, reset_bits = d->reset_bits ? d->reset_bits : 32;
    if (leak_bits < 2 || leak_bits > 32)
        return fail(RANC_ERANGE, "leak_bits must be 0 or in [2, 32] (got %d)", d->leak_bits);
    if (reset_bits < 2 || reset_bits > 32)
        return fail(RANC_ERANGE, "reset_bits must be 0 or in [2, 32] (got %d)", d->reset_bits);
    const long long vlo = -(1LL << (d->potential_bits - 1)), vhi = (1LL << (d->potential_bits - 1)) - 1;
    const long long llo = -(1LL << (leak_bits - 1)), lhi = (1LL << (leak_bits - 1)) - 1;
    const long long rlo = std::max(vlo, -(1LL << (reset_bits - 1))), rhi = std::min(vhi, (1LL << (reset_bits - 1)) - 1);
    for (size_t i = 0; i < (size_t)C * N; ++i) {
        if (d->reset[i] < rlo || d->reset[i] > rhi)
            return fail(RANC_ERANGE, "reset[%zu] = %d outside the potential range and the %d-bit reset range", i,
                        d->reset[i], reset_bits);
        if (d->v_init[i] < vlo || d->v_init[i] > vhi)
            return fail(RANC_ERANGE, "v_init[%zu] = %d outside the potential range", i, d->v_init[i]);
        if (d->leak[i] < llo || d->leak[i] > lhi)
            return fail(RANC_ERANGE, "leak[%zu] = %d outside the %d-bit leak range", i, d->leak[i], leak_bits);
        if (d->leak[i] < -(1 << 30) || d->leak[i] > (1 << 30))
            return fail(RANC_ERANGE, "leak[%zu] = %d outside [-2^30, 2^30]", i, d->leak[i]);
        if (d->floor && (d->floor[i] < vlo || d->floor[i] > vhi))
            return fail(RANC_ERANGE, "floor[%zu] = %d outside the potential range", i, d->floor[i]);
        if (d->reset_mode && d->reset_mode[i] > RANC_RESET_LINEAR)
            return fail(RANC_EINVAL, "reset_mode[%zu] = %u unknown", i, d->reset_mode[i]);
        const uint8_t k = d->dest_kind[i];
        if (k > RANC_DEST_OUT)
            return fail(RANC_EINVAL, "dest_kind[%zu] = %u unknown", i, k);
        if (k == RANC_DEST_CORE) {
            const int c = (int)(i / N);
            const long long x = c % d->grid_w + (long long)d->dest_dx[i];
            const long long y = c / d->grid_w + (long long)d->dest_dy[i];
            if (x < 0 || x >= d->grid_w || y < 0 || y >= d->grid_h)
                return fail(RANC_ERANGE, "neuron %zu: destination (%+d, %+d) leaves the %dx%d mesh", i,
                            d->dest_dx[i], d->dest_dy[i], d->grid_w, d->grid_h);
            if (d->dest_axon[i] >= A)
                return fail(RANC_ERANGE, "neuron %zu: dest_axon %u >= num_axons", i, d->dest_axon[i]);
            if (d->dest_delay[i] < 1 || d->dest_delay[i] > d->max_delay)
                return fail(RANC_ERANGE, "neuron %zu: dest_delay %u outside [1, %d]", i, d->dest_delay[i],
                            d->max_delay);
        }
    }
    std::vector<char> seen(C, 0);
    for (int i = 0; i < d->num_input_cores; ++i) {
        const int c = d->input_cores[i];
        if (c < 0 || c >= C)
            return fail(RANC_ERANGE, "input_cores[%d] = %d out of range", i, c);
        if (seen[c])
            return fail(RANC_EINVAL, "input core %d listed twice", c);
        seen[c] = 1;
    }
    return RANC_OK;
}

// Whether the network needs the extended potential update: potentials
// narrower than 32 bits (clamp), a floor above the potential range's lowest
// value, or linear-reset neurons.
bool neuron_model_ext(const ranc_net_desc *d)
{
    if (d->potential_bits < 32)
        return true;
    const size_t CN = (size_t)d->num_cores * d->num_neurons;
    const int32_t vmin = (int32_t)(-(1LL << (d->potential_bits - 1)));
    for (size_t i = 0; i < CN; ++i)
        if ((d->floor && d->floor[i] > vmin) || (d->reset_mode && d->reset_mode[i] == RANC_RESET_LINEAR))
            return true;
    return false;
}

// Levels of the cores when no spike can come back to the core it left
// (directly or through others): a core's level is the longest path to it from
// a core without sources. More than MAX_LEVELS levels, or a cycle: none.
constexpr int MAX_LEVELS = 64;
// Lines of the dispatch, in neurons times samples.
constexpr long long AUTO_MFMA_MIN_NEURONS = 1 << 20;
constexpr long long PLAIN_SOLO_MIN_NEURONS = 1 << 17;
// The byte ring, and so the plain path's launches without a router, up to here
// and to 2 GiB of ring (a byte per axon, sample and slot; its addresses within a
// slot have 28 bits); with 64 samples or more, where the automatic path is
// MFMA, up to 2^22. With a router and without, us per tick: 512 cores of
// 256 x 256 with 63 samples 127 and 59, 4096 with 10 samples 201 and 155, 1024
// of 512 x 512 with 30 samples 402 and 200.
constexpr long long PLAIN_FUSED_MAX_NEURONS = 1 << 26, PLAIN_FUSED_MAX_NEURONS_S64 = 1 << 22;
constexpr long long PLAIN_RING8_MAX_BYTES = 2LL << 30;
// The whole-network form (kern_plain_whole.hip) loads and stores everything
// once per call: 18 us and 1.9 us per tick for 12 cores of 256 x 256, against
// 5 us and 3.4 us per tick.
constexpr int PLAIN_WHOLE_MIN_TICKS = 12;
// Sorted columns (12 words instead of 8 for four types) are kept while they
// stay in cache from tick to tick, and used by a one-tick launch that does
// enough work to be bound by it (128 cores x 23 samples 10.3 us against 10.7)
// rather than by the loads it waits for (45 cores of 512 axons, one sample 4.4
// us against 3.9).
constexpr long long PLAIN_SORTED_MAX_NEURONS = 1 << 18;
constexpr long long PLAIN_SORTED_MIN_WORK = 1 << 18;     // neurons times samples
bool feed_forward_levels(const ranc_net_desc *d, Plan &p)
{
    const int C = p.C, N = p.N;
    std::vector<uint32_t> indeg(C, 0);
    auto dest = [&](size_t i) {
        const int c = (int)(i / N);
        return (c % d->grid_w + d->dest_dx[i]) + (c / d->grid_w + d->dest_dy[i]) * d->grid_w;
    };
    for (size_t i = 0; i < (size_t)C * N; ++i)
        if (d->dest_kind[i] == RANC_DEST_CORE)
            ++indeg[dest(i)];
    std::vector<int32_t> ready, level(C, 0);
    for (int c = 0; c < C; ++c)
        if (!indeg[c])
            ready.push_back(c);
    int top = 0;
    for (size_t r = 0; r < ready.size(); ++r) {
        const int c = ready[r];
        top = std::max(top, level[c]);
        if (top >= MAX_LEVELS)
            return false;
        for (size_t i = (size_t)c * N; i < (size_t)(c + 1) * N; ++i)
            if (d->dest_kind[i] == RANC_DEST_CORE) {
                const int t = dest(i);
                level[t] = std::max(level[t], level[c] + 1);
                if (--indeg[t] == 0)
                    ready.push_back(t);
            }
    }
    if ((int)ready.size() != C)
        return false;
    std::vector<bool> taken((size_t)C * d->num_axons, false);
    p.multi_source = false;
    for (size_t i = 0; i < (size_t)C * N && !p.multi_source; ++i)
        if (d->dest_kind[i] == RANC_DEST_CORE) {
            const size_t at = (size_t)dest(i) * d->num_axons + d->dest_axon[i];
            p.multi_source = taken[at];
            taken[at] = true;
        }
    p.levels = top + 1;
    p.level_first.assign(p.levels + 1, 0);
    for (int c = 0; c < C; ++c)
        ++p.level_first[level[c] + 1];
    for (int l = 0; l < p.levels; ++l)
        p.level_first[l + 1] += p.level_first[l];
    p.order.resize(C);
    std::vector<int32_t> at(p.level_first.begin(), p.level_first.end() - 1);
    for (int c = 0; c < C; ++c)
        p.order[at[level[c]]++] = c;
    p.level = std::move(level);
    return true;
}

// MFMA path: whether workgroups take one tile of 64 samples each
// (kern_mfma_tile.hip), or run a pipeline over several (kern_mfma_unit.h), which
// read their core's B tiles once. One tile each: where the pipelines would leave
// CUs idle; where the B tiles are few beside the potentials, or the pipelined
// form's LDS leaves one workgroup on a CU; and where there are two tiles, unless
// both planes of 256 neurons are read for each. us per tick, pipelined and
// one tile each: 40 cores of 256 x 256 (8 bits) x 300 samples 28.2, 10.1; 2048 x 200
// of 64 x 64 67.2, 59.6, of 128 x 128 (9 bits) 196, 131, of 256 x 256 (8 bits) 223,
// 221; 4096 x 128 of 256 x 128 152, 143, of 512 x 256 (9 bits) 467, 397. The other
// way, 2048 x 200 of 128 x 256 (9 bits) 231, 289, of 256 x 128 (8 bits) 124, 138, of
// 512 x 256 (9 bits) 357, 376; 512 x 128 of 256 x 256 (9 bits) 40, 44.
bool one_tile_per_workgroup(const Plan &p, int tiles)
{
    const bool wide = mfma_width(p.A, p.N, p.two) == 256;
    if (tiles == 1 || (long long)p.C * p.slices * tiles <= 400)
        return true;
    if (wide && p.two)
        return false;
    return tiles == 2 || p.N == 64 || p.A <= 128 || (wide && p.A <= 256);
}

// Plain path: words per axon type of the columns sorted by type, 0: natural order
// (columns so large that they come from memory every tick, or too many words).
int plain_sorted_columns(const ranc_net_desc *d, const Plan &p)
{
    int longest = 0;
    for (int c = 0; c < p.C; ++c) {
        int count[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int a = 0; a < p.A; ++a)
            longest = std::max(longest, ++count[d->axon_type[(size_t)c * p.A + a]]);
    }
    const int pw = plain_sorted_words(p.G, longest);
    return p.G * pw <= 2 * p.W && (long long)p.C * p.N <= PLAIN_SORTED_MAX_NEURONS ? pw : 0;
}

// Whether the MFMA path is the faster with 32 to 63 samples, where its time goes by
// 64-sample tiles and the plain path's by samples. It is from 2^20 neurons times
// samples on for most shapes (us per tick, plain and MFMA, 4 types: 128 cores of 256 x
// 256 (9 bits) x 32 samples 13.5, 11.5; 200 of 128 x 128 x 40 11.5, 8.1; 512 of 64 x 64 x
// 32 11.1, 7.9), but:
// - B tiles large beside a core's axons (64 x 256 and 128 x 512 with two planes, 64 x
//   512 with one) cost: MFMA is 0.8 to 1.0 times as fast at 2^20, 0.95 to 1.14 at
//   1.3 * 2^20, 1.03 and more from 1.5 * 2^20 on. 64 x 512 with two planes fill the GPU
//   with 256 workgroups: up to there 0.7 at 2^20, 0.95 to 1.05 at 1.7 * 2^20, 1.2 to 1.5
//   at 3 * 2^20 (56 samples); past it 0.65 to 0.95 with 32 and 44 samples and 1.1 to 1.5
//   with 56 and 63 from 4.5 * 2^20 on (eight types: from 44 samples on).
// - feed-forward networks of wide cores, whose plain launches of several ticks are
//   cheap: 256 x 256 (9 bits) and 512 x 512 (8 bits) 0.75 to 1.0 at 2^20, 0.93 to 1.2
//   at 1.3 * 2^20. With 512 axons and two planes the MFMA path runs them tick by
//   tick: 512 x 256 1.2 at 2^21 x 63 samples, 1.1 at 3 * 2^20 x 56, 1.1 at 4 * 2^20 x 44;
//   512 x 512 1.05 at 2^21 x 63, 1.1 at 6 * 2^20 x 56, 0.7 with 32.
// The plain path's cost counts as that of a larger network where it is the higher:
// 512 axons of one or two types (1.3 times), and columns in natural order (one AND
// and population count per word and type, where sorted columns take at most 24: 384
// cores of 512 x 512 with 8 types 93 us, sorted 25).
bool mfma_below_a_tile(const ranc_net_desc *d, const Plan &p)
{
    const int planes = p.two ? 2 : 1, spread = p.N * planes / p.A;
    double size = (double)p.C * p.N * p.S;
    if (size < AUTO_MFMA_MIN_NEURONS)
        return false;
    if (p.A == 512 && p.G <= 2)
        size *= 1.3;
    if (!plain_sorted_columns(d, p))
        size *= std::max(1.0, p.W * p.G / 24.0);
    Plan q = p;
    const bool forward = p.RT > 1 && p.N * planes >= 512 && feed_forward_levels(d, q);
    if (forward && !mfma_ticks_supported(p.A, p.N, p.two)) {
        double least = 1 << 21;
        for (int i = 0; i < p.N / 128; ++i)
            least *= 64.0 / p.S;
        return size >= least;
    }
    if (spread > 8 && p.C * mfma_slices(p.A, p.N, p.two) <= 256)
        return size >= 3 << 19;
    if (spread > 8)
        return size >= 9 << 19 && p.S >= (p.G == 8 ? 40 : 52);
    return size >= (spread > 4 || forward ? 5 << 18 : AUTO_MFMA_MIN_NEURONS);
}

// level: what the layout may use memory for. PLAN_FULL: RANC_PATH_AUTO may take
// the MFMA path below 64 samples; PLAN_FORMS: rings for several ticks per launch
// and for launches without a router; PLAN_SMALL: neither.
enum PlanLevel { PLAN_SMALL, PLAN_FORMS, PLAN_FULL };
ranc_status make_plan(const ranc_net_desc *d, int32_t S, int32_t RT, int32_t path, Plan &p, PlanLevel level = PLAN_FULL)
{
    const bool blocks = level >= PLAN_FORMS;
    ranc_status st = validate(d, S, RT, path);
    if (st != RANC_OK)
        return st;
    p.C = d->num_cores;
    p.A = d->num_axons;
    p.N = d->num_neurons;
    p.G = d->num_types;
    p.W = p.A / 32;
    p.NW = p.N / 32;
    p.D = d->max_delay;
    p.Q = p.D + 1;
    p.S = S;
    p.S64 = (S + 63) / 64 * 64;
    p.RT = RT;
    p.Cin = d->num_input_cores;
    p.grid_w = d->grid_w;
    p.grid_h = d->grid_h;
    p.two = d->weight_bits > 8;
    if (path == RANC_PATH_AUTO) {
        // from 64 samples on (one full tile) the MFMA path
        const bool mid = level >= PLAN_FULL && S >= 32 && S < 64 && mfma_below_a_tile(d, p);
        path = (S >= 64 || mid) && mfma_shape_supported(p.A, p.N, p.two) ? RANC_PATH_MFMA : RANC_PATH_PLAIN;
        p.auto_mid = mid && path == RANC_PATH_MFMA;
    }
    if (path == RANC_PATH_MFMA && !mfma_shape_supported(p.A, p.N, p.two))
        return fail(RANC_EUNSUPPORTED, "MFMA path does not support A=%d N=%d with %d-bit weights", p.A, p.N,
                    d->weight_bits);
    if (path == RANC_PATH_SPARSE && !sparse_shape_supported(p.A, p.N, p.G))
        return fail(RANC_EUNSUPPORTED, "sparse path does not support N=%d with G=%d", p.N, p.G);
    p.path = path;
    // segments of at most 32 ticks: the history ring then takes about as much
    // memory as the potentials (one bit per tick against 32); and below 4 GiB
    if (blocks && path == RANC_PATH_MFMA && RT > 1 && mfma_ticks_supported(p.A, p.N, p.two)) {
        const long long slot = (long long)p.C * p.N * (p.S64 / 64) * 8;
        const long long seg = std::min<long long>(std::min(RT, MFMA_BLOCK_TICKS_MAX), ((1LL << 32) - 1) / slot - p.D);
        if (seg > 1 && mfma_ticks_offsets_fit(p.C, p.N, p.S64, p.D + (int)seg, p.C * p.N, (long long)RT * p.Cin * p.W) &&
            feed_forward_levels(d, p)) {
            p.seg_ticks = (int)seg;
            p.Q = p.D + p.seg_ticks;
        }
    }
    // plain path: the byte ring, longer for a feed-forward network
    const long long slot8 = (long long)p.C * p.A * S;
    const bool ring8 = blocks && path == RANC_PATH_PLAIN && (long long)p.C * p.N * S <= (S < 64 ? PLAIN_FUSED_MAX_NEURONS : PLAIN_FUSED_MAX_NEURONS_S64) &&
                       slot8 * (p.D + 2) <= PLAIN_RING8_MAX_BYTES && (long long)p.C * p.A < 1LL << 28;
    if (ring8) {
        p.Q = p.D + 2;
        const int seg = std::min(RT, MFMA_BLOCK_TICKS_MAX);
        if (seg > 1 && slot8 * (p.D + 1 + seg) <= PLAIN_RING8_MAX_BYTES && feed_forward_levels(d, p)) {
            p.seg_ticks = seg;
            p.Q = p.D + 1 + seg;
        }
        p.sorted_words = plain_sorted_columns(d, p);
    }
    p.slices = path == RANC_PATH_MFMA ? mfma_slices(p.A, p.N, p.two)
             : path == RANC_PATH_SPARSE ? p.N / sparse_slice_width(p.N) : 1;
    p.cnt_rows = path == RANC_PATH_PLAIN ? p.N / 64 : p.slices;
    // Samples per workgroup (sample-tiled paths), in 64-sample tiles: aim for
    // >= 2048 workgroups, but keep >= 4 tiles per workgroup where the batch
    // has them (the software pipeline runs over a workgroup's tiles). On the
    // 512-core net at 1024 samples: 256 -> 232.8 us per tick, 512 -> 235.5,
    // 128 -> 263.2.
    {
        const int tiles = (S + 63) / 64;
        const int per_chunk = p.C * p.slices;   // workgroups per sample chunk
        int chunks = (2048 + per_chunk - 1) / per_chunk;
        chunks = std::max(1, std::min(chunks, std::max(1, tiles / 4)));
        const int tiles_per = (tiles + chunks - 1) / chunks;
        const int cap = path == RANC_PATH_SPARSE ? sparse_max_samples_per_wg() : mfma_max_samples_per_wg();
        p.spw = p.spw_pipelined = std::min(64 * tiles_per, std::min(cap, 512));
        if (path == RANC_PATH_MFMA && one_tile_per_workgroup(p, tiles))
            p.spw = 64;
        if (const char *e = getenv("RANC_MFMA_SPW")) {
            const int v = atoi(e);
            if (v > 0 && v % 64 == 0 && v <= cap)
                p.spw = v;
        }
    }
    p.bsrc = -1;
    if (const char *e = getenv("RANC_MFMA_BSRC"))
        p.bsrc = strcmp(e, "planes") == 0 ? 0 : strcmp(e, "compact") == 0 ? 1 : -1;
    long long E = 0, wout = 0, nout = 0;
    for (size_t i = 0; i < (size_t)p.C * p.N; ++i) {
        E += d->dest_kind[i] == RANC_DEST_CORE;
        nout += d->dest_kind[i] == RANC_DEST_OUT;
    }
    {
        // wave-interleaved table: every group of 64 destination words is padded
        // to its longest list
        const size_t CW = (size_t)p.C * p.W;
        std::vector<uint32_t> cnt(CW, 0);
        for (size_t i = 0; i < (size_t)p.C * p.N; ++i)
            if (d->dest_kind[i] == RANC_DEST_CORE) {
                const int c = (int)(i / p.N);
                const int dc = (c % d->grid_w + d->dest_dx[i]) + (c / d->grid_w + d->dest_dy[i]) * d->grid_w;
                ++cnt[(size_t)dc * p.W + d->dest_axon[i] / 32];
            }
        long long words = 0;
        for (size_t g = 0; g < (CW + 63) / 64; ++g) {
            uint32_t mx = 0;
            for (size_t k = g * 64; k < std::min(CW, g * 64 + 64); ++k)
                mx = std::max(mx, cnt[k]);
            words += 64LL * mx;
        }
        p.ell_words = words;
    }
    for (int c = 0; c < p.C; ++c)
        for (int w = 0; w < p.NW; ++w) {
            bool any = false;
            for (int b = 0; b < 32; ++b)
                any |= d->dest_kind[(size_t)c * p.N + 32 * w + b] == RANC_DEST_OUT;
            wout += any;
        }
    p.ecsr_entries = 0;
    if (path == RANC_PATH_SPARSE) {
        // connections per neuron slice, each slice's rows padded
        const int NW = p.N / 32, SW = sparse_slice_width(p.N) / 32, al = sparse_row_align();
        for (int c = 0; c < p.C; ++c)
            for (int sl = 0; sl < p.slices; ++sl) {
                long long k = 0;
                for (int a = 0; a < p.A; ++a)
                    for (int w = sl * SW; w < (sl + 1) * SW; ++w)
                        k += __builtin_popcount(d->crossbar[((size_t)c * p.A + a) * NW + w]);
                p.ecsr_entries += (k + al - 1) / al * al;
            }
    }
    p.E = E;
    p.Wout = (int)wout;
    p.Nout = (int)nout;
    const size_t C = p.C, A = p.A, N = p.N, G = p.G, W = p.W, NW = p.NW;
    const bool mf = p.path == RANC_PATH_MFMA;
    const bool sp = p.path == RANC_PATH_SPARSE;
    const bool tiled = mf || sp;   // sample-tiled paths: spike history, neuron-major raster
    p.size[R_COLBITS] = tiled ? 0 : C * W * N * 4;
    // MFMA path: crossbar column words, then the per-type plane bytes of
    // every neuron, then the axon types (the compact source its kernels build
    // B tiles from; see pack_bsrc)
    p.size[R_BSRC] = mf ? C * W * N * 4 + C * (p.two ? 2 : 1) * 2 * N * 4 + C * A : 0;
    p.size[R_TYPEMASK] = C * G * W * 4;
    p.size[R_WTS] = C * G * N * 4;
    p.size[R_LEAK] = p.size[R_THR] = p.size[R_RST] = p.size[R_VINIT] = p.size[R_FLOOR] = C * N * 4;
    p.size[R_LINMASK] = C * NW * 4;
    p.size[R_ECSRPTR] = sp ? C * p.slices * (A + 1) * 4 : 0;
    p.size[R_ECSRENT] = sp ? std::max<size_t>((size_t)p.ecsr_entries, 8) * 2 : 0;
    p.size[R_COREMASK] = p.size[R_OUTMASK] = p.size[R_OUTWORD] = C * NW * 4;
    p.size[R_ININDEX] = C * 4;
    p.size[R_RTDCNT] = tiled ? 0 : (C * W + 63) / 64 * 64 * route_dmax(p.D) * 2;
    p.size[R_RTGOFF] = tiled ? 0 : (C * W + 63) / 64 * 4;
    p.size[R_RTENT] = tiled ? 0 : std::max<size_t>((size_t)p.ell_words, 1) * 4;
    p.size[R_RTXPTR] = tiled ? (C * A + 1) * 4 : 0;
    p.size[R_RTXENT] = tiled ? std::max<size_t>((size_t)E, 1) * 4 : 0;
    const size_t HG = (size_t)p.S64 / 64;
    // zeros: a history row (HG words), and the A / 32 input words of a core that
    // takes none (kern_mfma_ticks.hip)
    p.size[R_HZERO] = tiled ? std::max<size_t>(HG * 8, W * 4) : 0;
    p.size[R_DEGB] = mf ? C * p.slices * 2 * A : 0;
    p.size[R_OUTIDX] = tiled ? C * N * 4 : 0;
    // int8 weight planes: the B source when a core's samples take several
    // workgroups, of the persistent batch kernel and of the state-resident
    // kernel (otherwise B is built from R_BSRC)
    p.size[R_PLANES] = mf ? C * A * N * (p.two ? 2 : 1) : 0;
    p.size[R_V] = C * (tiled ? (size_t)p.S64 : (size_t)S) * N * 4;
    // plain path: the scheduler ring; sparse path: the scheduler row of the
    // tick being integrated, [C][S64][W], written by the delivery kernel
    p.size[R_RING] = mf ? 0 : sp ? C * (size_t)p.S64 * W * 4 : (size_t)p.Q * S * C * W * 4;
    p.size[R_SPK] = tiled ? 0 : (size_t)S * C * NW * 4;
    p.size[R_HIST] = tiled ? (size_t)p.Q * C * N * HG * 8 : 0;
    p.size[R_RASTER] = tiled ? (size_t)RT * p.Nout * HG * 8 : (size_t)RT * S * p.Wout * 4;
    p.size[R_CNT] = C * p.cnt_rows * S * CNT_N * 8;   // plain: one row per 64 neurons, MFMA and sparse: per slice
    p.size[R_CRING] = (size_t)RT * C * p.cnt_rows * S * 8;   // one packed word per row, sample and tick of a call
    p.size[R_TICK] = 16;
    p.size[R_BATCH] = BATCH_TABLE_BYTES;
    p.size[R_EXT] = (size_t)RT * S * p.Cin * W * 4;
    p.size[R_LINKREC] = C * N * 8;
    // sample-tiled paths: for every (direction, core) difference-array row,
    // the run starts (+1) and ends (-1) that land there, by source neuron
    p.size[R_LINKPTR] = tiled ? (size_t)(4 * C + 1) * 4 : 0;
    p.size[R_LINKENT] = tiled ? std::max<size_t>((size_t)4 * E, 1) * 4 : 0;
    p.size[R_OUTCOL] = tiled ? 0 : std::max<size_t>((size_t)p.Wout, 1) * 8;
    p.size[R_OUTPOS] = tiled ? 0 : std::max<size_t>((size_t)p.Nout, 1) * 4;
    p.size[R_PLAINDST] = ring8 ? C * N * 4 : 0;
    p.size[R_SCOLS] = C * G * p.sorted_words * N * 4;
    p.size[R_SPOS] = C * ((G * p.sorted_words + 1) / 2 * 64) * 2;
    p.size[R_RING8] = ring8 ? (size_t)p.Q * S * C * A : 0;
    p.size[R_LINKD] = (size_t)4 * C * p.S64 * 8;
    p.size[R_RSYNC] = mf ? 8 : 0;   // state-resident loop: arrival counter, give-up flag
    p.size[R_ORDER] = p.levels ? 2 * C * 4 : 0;
    size_t off = 0;
    for (int r = 0; r < R_NREG; ++r) {
        if (r == R_PARAMS_END)
            p.params_bytes = off;
        p.off[r] = off;
        off += align256(p.size[r]);
    }
    p.total = off;
    return RANC_OK;
}

// 32 x 32 bit transpose: bit i of word j becomes bit j of word i, by the recursive
// block exchange of H. S. Warren, Hacker's Delight, section 7-3 (transposing a bit
// matrix), its loop indexes included.
static void transpose_bits(uint32_t (&a)[32])
{
    uint32_t m = 0x0000FFFFu;
    for (int j = 16; j; j >>= 1, m ^= m << j)
        for (int k = 0; k < 32; k = (k + j + 1) & ~j) {
            const uint32_t t = ((a[k] >> j) ^ a[k + j]) & m;
            a[k + j] ^= t;
            a[k] ^= t << j;
        }
}

// Crossbar columns of core c, words [positions/32][N]: bit p % 32 of word p / 32
// of neuron j = the axon at position p connects to j. axon(p) < 0: none.
template <typename Axon> static void pack_columns(const ranc_net_desc *d, const Plan &p, int c, int positions, uint32_t *col, Axon &&axon)
{
    const int N = p.N, NW = p.NW;
    for (int p0 = 0; p0 < positions; p0 += 32) {
        const uint32_t *row[32];
        for (int i = 0; i < 32; ++i) {
            const int a = axon(p0 + i);
            row[i] = a < 0 ? nullptr : d->crossbar + ((size_t)c * p.A + a) * NW;
        }
        for (int w = 0; w < NW; ++w) {
            uint32_t b[32];
            for (int i = 0; i < 32; ++i)
                b[i] = row[i] ? row[i][w] : 0u;
            transpose_bits(b);
            memcpy(col + (size_t)(p0 / 32) * N + 32 * w, b, sizeof b);
        }
    }
}

// Crossbar columns [C][A/32][N] with the axons in natural order.
static void pack_columns(const ranc_net_desc *d, const Plan &p, uint32_t *col)
{
    for (int c = 0; c < p.C; ++c)
        pack_columns(d, p, c, p.A, col + (size_t)c * p.W * p.N, [](int a) { return a; });
}

// Host-side packing of the MFMA path's compact B source (R_BSRC): column
// words [C][W][N] (bit a % 32 of word a / 32 of neuron j: axon a connects to
// j); then [C][planes][2][N] words, byte g % 4 of word g / 4 = the plane
// value of weight(j, g) (two planes: w >> 7, then w & 127; one: w); then the
// axon types [C][A], one byte each.
void pack_bsrc(const ranc_net_desc *d, const Plan &p, std::vector<uint8_t> &buf)
{
    buf.assign(p.size[R_BSRC], 0);
    const int C = p.C, A = p.A, N = p.N, G = p.G, W = p.W, PL = p.two ? 2 : 1;
    uint32_t *col = reinterpret_cast<uint32_t *>(buf.data());
    pack_columns(d, p, col);
    uint32_t *ws = col + (size_t)C * W * N;
    for (int c = 0; c < C; ++c)
        for (int j = 0; j < N; ++j)
            for (int g = 0; g < G; ++g) {
                const int w = d->weight[((size_t)c * N + j) * G + g];
                for (int pl = 0; pl < PL; ++pl) {
                    const uint32_t v = (uint32_t)(PL == 2 ? (pl == 0 ? w >> 7 : w & 127) : w) & 255u;
                    ws[(((size_t)c * PL + pl) * 2 + g / 4) * N + j] |= v << (8 * (g % 4));
                }
            }
    memcpy(reinterpret_cast<uint8_t *>(ws + (size_t)C * PL * 2 * N), d->axon_type, (size_t)C * A);
}

// Host-side packing of the parameter region (bytes [0, params_bytes)).
void pack_params(const ranc_net_desc *d, const Plan &p, std::vector<uint8_t> &buf, std::vector<int> &out_words)
{
    buf.assign(p.params_bytes, 0);
    auto at = [&](Region r) { return buf.data() + p.off[r]; };
    const int C = p.C, A = p.A, N = p.N, G = p.G, W = p.W, NW = p.NW;
    auto conn = [&](int c, int a, int j) -> int {
        return (d->crossbar[((size_t)c * A + a) * NW + j / 32] >> (j % 32)) & 1u;
    };
    if (p.size[R_COLBITS])
        pack_columns(d, p, (uint32_t *)at(R_COLBITS));
    uint32_t *tm = (uint32_t *)at(R_TYPEMASK);
    for (int c = 0; c < C; ++c)
        for (int a = 0; a < A; ++a)
            tm[((size_t)c * G + d->axon_type[(size_t)c * A + a]) * W + a / 32] |= 1u << (a % 32);
    int32_t *wts = (int32_t *)at(R_WTS);
    for (int c = 0; c < C; ++c)
        for (int g = 0; g < G; ++g)
            for (int j = 0; j < N; ++j)
                wts[((size_t)c * G + g) * N + j] = d->weight[((size_t)c * N + j) * G + g];
    memcpy(at(R_LEAK), d->leak, (size_t)C * N * 4);
    memcpy(at(R_THR), d->threshold, (size_t)C * N * 4);
    memcpy(at(R_RST), d->reset, (size_t)C * N * 4);
    memcpy(at(R_VINIT), d->v_init, (size_t)C * N * 4);
    // floor: the lowest potential of the range where none is given (a no-op
    // after the clamp); linear-reset neurons as one bit per neuron
    int32_t *fl = (int32_t *)at(R_FLOOR);
    const int32_t vmin = (int32_t)(-(1LL << (d->potential_bits - 1)));
    for (size_t i = 0; i < (size_t)C * N; ++i)
        fl[i] = d->floor ? std::max(d->floor[i], vmin) : vmin;
    uint32_t *lin = (uint32_t *)at(R_LINMASK);
    if (d->reset_mode)
        for (size_t i = 0; i < (size_t)C * N; ++i)
            lin[i / 32] |= (uint32_t)(d->reset_mode[i] == RANC_RESET_LINEAR) << (i % 32);
    uint32_t *cmask = (uint32_t *)at(R_COREMASK), *omask = (uint32_t *)at(R_OUTMASK);
    int32_t *oword = (int32_t *)at(R_OUTWORD);
    out_words.clear();
    for (int c = 0; c < C; ++c)
        for (int w = 0; w < NW; ++w) {
            uint32_t cm = 0, om = 0;
            for (int b = 0; b < 32; ++b) {
                const uint8_t k = d->dest_kind[(size_t)c * N + 32 * w + b];
                cm |= (uint32_t)(k == RANC_DEST_CORE) << b;
                om |= (uint32_t)(k == RANC_DEST_OUT) << b;
            }
            cmask[(size_t)c * NW + w] = cm;
            omask[(size_t)c * NW + w] = om;
            oword[(size_t)c * NW + w] = om ? (int32_t)(out_words.size() / 2) : -1;
            if (om) {
                out_words.push_back(c);
                out_words.push_back(w);
            }
        }
    if (p.size[R_OUTCOL]) {
        // plain-path raster columns: neuron word and the output index of its
        // first output neuron (output neurons numbered in (core, neuron) order)
        int32_t *oc = (int32_t *)at(R_OUTCOL);
        int base = 0;
        for (size_t ow = 0; ow < out_words.size() / 2; ++ow) {
            const int c = out_words[2 * ow], w = out_words[2 * ow + 1];
            oc[2 * ow] = c * NW + w;
            oc[2 * ow + 1] = base;
            base += __builtin_popcount(omask[(size_t)c * NW + w]);
        }
        int32_t *op = (int32_t *)at(R_OUTPOS);
        int o = 0;
        for (size_t ow = 0; ow < out_words.size() / 2; ++ow) {
            const int c = out_words[2 * ow], w = out_words[2 * ow + 1];
            for (uint32_t m = omask[(size_t)c * NW + w]; m; m &= m - 1u)
                op[o++] = (int32_t)(ow << 5) | __builtin_ctz(m);
        }
    }
    int32_t *inidx = (int32_t *)at(R_ININDEX);
    for (int c = 0; c < C; ++c)
        inidx[c] = -1;
    for (int i = 0; i < p.Cin; ++i)
        inidx[d->input_cores[i]] = i;
    // Inverted routing table, one list per destination axon word, sorted by
    // delay, stored wave-interleaved (see ranc_internal.h).
    if (p.size[R_RTENT]) {
        const size_t CW = (size_t)C * W;
        std::vector<std::vector<uint32_t>> lists(CW);
        for (size_t i = 0; i < (size_t)C * N; ++i)
            if (d->dest_kind[i] == RANC_DEST_CORE) {
                const int c = (int)(i / N);
                const int dc = (c % d->grid_w + d->dest_dx[i]) + (c / d->grid_w + d->dest_dy[i]) * d->grid_w;
                const uint32_t ent = ((uint32_t)i << RT_SRC_SHIFT) |
                                     ((uint32_t)(d->dest_delay[i] - 1) << RT_DELAY_SHIFT) | (d->dest_axon[i] % 32u);
                lists[(size_t)dc * W + d->dest_axon[i] / 32].push_back(ent);
            }
        const int dmax = route_dmax(p.D);
        uint16_t *dcnt = (uint16_t *)at(R_RTDCNT);
        uint32_t *goff = (uint32_t *)at(R_RTGOFF), *ent = (uint32_t *)at(R_RTENT);
        size_t off = 0;
        for (size_t g = 0; g < (CW + 63) / 64; ++g) {
            size_t mx = 0;
            for (size_t k = g * 64; k < std::min(CW, g * 64 + 64); ++k) {
                auto &L = lists[k];
                std::stable_sort(L.begin(), L.end(), [](uint32_t a, uint32_t b) {
                    return ((a >> RT_DELAY_SHIFT) & 15u) < ((b >> RT_DELAY_SHIFT) & 15u);
                });
                for (uint32_t x : L)
                    ++dcnt[k * dmax + ((x >> RT_DELAY_SHIFT) & 15u)];
                mx = std::max(mx, L.size());
                for (size_t e = 0; e < L.size(); ++e)
                    ent[off + e * 64 + (k - g * 64)] = L[e];
            }
            goff[g] = (uint32_t)off;
            off += 64 * mx;
        }
    }
    // MFMA path: the inverted table keyed by destination axon (CSR).
    if (p.size[R_RTXPTR]) {
        uint32_t *ptr = (uint32_t *)at(R_RTXPTR), *ent = (uint32_t *)at(R_RTXENT);
        const size_t CA = (size_t)C * A;
        std::vector<uint32_t> fill(CA + 1, 0);
        auto dest_of = [&](size_t i) -> size_t {
            const int c = (int)(i / N);
            const int dc = (c % d->grid_w + d->dest_dx[i]) + (c / d->grid_w + d->dest_dy[i]) * d->grid_w;
            return (size_t)dc * A + d->dest_axon[i];
        };
        for (size_t i = 0; i < (size_t)C * N; ++i)
            if (d->dest_kind[i] == RANC_DEST_CORE)
                ++fill[dest_of(i) + 1];
        for (size_t k = 0; k < CA; ++k)
            fill[k + 1] += fill[k];
        memcpy(ptr, fill.data(), (CA + 1) * 4);
        for (size_t i = 0; i < (size_t)C * N; ++i)
            if (d->dest_kind[i] == RANC_DEST_CORE)
                ent[fill[dest_of(i)]++] = ((uint32_t)i << 4) | (uint32_t)(d->dest_delay[i] - 1);
    }
    if (p.size[R_ECSRPTR]) {
        // Sparse path: per (core, neuron slice) one row per axon, listing the
        // slice's connected neurons with their weight for the axon's type:
        // entry = neuron within the slice (7 bits) | weight (9 bits) << 7.
        // Row starts are absolute; each slice's rows start on a multiple of
        // sparse_row_align() entries (the padding entries are never read as
        // connections).
        uint32_t *ptr = (uint32_t *)at(R_ECSRPTR);
        uint16_t *ent = (uint16_t *)at(R_ECSRENT);
        const int NS = sparse_slice_width(N), al = sparse_row_align();
        uint32_t off = 0;
        for (int c = 0; c < C; ++c)
            for (int sl = 0; sl < p.slices; ++sl) {
                uint32_t *rp = ptr + ((size_t)c * p.slices + sl) * (A + 1);
                for (int a = 0; a < A; ++a) {
                    rp[a] = off;
                    const int g = d->axon_type[(size_t)c * A + a];
                    for (int jl = 0; jl < NS; ++jl) {
                        const int j = sl * NS + jl;
                        if (conn(c, a, j)) {
                            const int w = d->weight[((size_t)c * N + j) * G + g];
                            ent[off++] = (uint16_t)(jl | ((w & 511) << 7));
                        }
                    }
                }
                rp[A] = off;
                off = (off + al - 1) / al * al;
            }
    }
    if (p.size[R_DEGB]) {
        // connected neurons per axon within each neuron slice, as a low-byte
        // and a high-byte plane: [C][slices][2][A]
        uint8_t *db = at(R_DEGB);
        const int SL = p.slices, WS = NW / SL;
        for (int c = 0; c < C; ++c)
            for (int sl = 0; sl < SL; ++sl)
                for (int a = 0; a < A; ++a) {
                    int k = 0;
                    for (int w = sl * WS; w < (sl + 1) * WS; ++w)
                        k += __builtin_popcount(d->crossbar[((size_t)c * A + a) * NW + w]);
                    const size_t r = (size_t)c * SL + sl;
                    db[(r * 2 + 0) * A + a] = (uint8_t)(k & 255);
                    db[(r * 2 + 1) * A + a] = (uint8_t)(k >> 8);
                }
    }
    if (p.size[R_PLAINDST]) {
        // plain path: each neuron's scheduler byte and delay (C * A < 2^28)
        uint32_t *dst = (uint32_t *)at(R_PLAINDST);
        for (size_t i = 0; i < (size_t)C * N; ++i) {
            const int c = (int)(i / N);
            const int dc = (c % d->grid_w + d->dest_dx[i]) + (c / d->grid_w + d->dest_dy[i]) * d->grid_w;
            dst[i] = d->dest_kind[i] == RANC_DEST_CORE
                         ? ((uint32_t)dc * A + d->dest_axon[i]) << 4 | (uint32_t)d->dest_delay[i]
                         : PLAIN_NO_DEST;
        }
    }
    if (p.size[R_SCOLS]) {
        // axons sorted by type, sorted_words words per type
        const int PW = p.sorted_words, SW = G * PW, P = (SW + 1) / 2 * 64;
        uint32_t *sc = (uint32_t *)at(R_SCOLS);
        uint16_t *sp = (uint16_t *)at(R_SPOS);
        std::fill(sp, sp + (size_t)C * P, (uint16_t)0x8000);
        for (int c = 0; c < C; ++c) {
            int fill[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            for (int a = 0; a < A; ++a) {
                const int g = d->axon_type[(size_t)c * A + a];
                sp[(size_t)c * P + 32 * PW * g + fill[g]++] = (uint16_t)a;
            }
            pack_columns(d, p, c, 32 * SW, sc + (size_t)c * SW * N, [&](int pos) {
                const int a = sp[(size_t)c * P + pos];
                return a < 0x8000 ? a : -1;
            });
        }
    }
    {
        // mesh path ends of each neuron's packets (x first, then y; see
        // kern_links.hip): no hop is -1, else 2 * end core + (negative step)
        int32_t *lr = (int32_t *)at(R_LINKREC);
        for (size_t i = 0; i < (size_t)C * N; ++i) {
            int32_t xc = -1, yc = -1;
            if (d->dest_kind[i] == RANC_DEST_CORE) {
                const int c = (int)(i / N), gw = d->grid_w;
                const int xs = c % gw, ys = c / gw, dx = d->dest_dx[i], dy = d->dest_dy[i];
                const int xd = xs + dx, yd = ys + dy;
                if (dx != 0)
                    xc = 2 * (ys * gw + xd) + (dx < 0);
                if (dy != 0)
                    yc = 2 * (yd * gw + xd) + (dy < 0);
            }
            lr[2 * i] = xc;
            lr[2 * i + 1] = yc;
        }
        if (p.size[R_LINKPTR]) {
            // rows of the difference arrays ([direction][core], direction
            // 0 +x, 1 -x, 2 +y, 3 -y) and the entries each packet adds to
            // them: +1 where a run of links starts, -1 where it ends; entry =
            // source neuron << 1 | (1 for -1), by source neuron within a row
            uint32_t *tp = (uint32_t *)at(R_LINKPTR);
            uint32_t *te = (uint32_t *)at(R_LINKENT);
            std::fill(tp, tp + 4 * (size_t)C + 1, 0u);
            auto visit = [&](auto &&emit) {
                for (size_t i = 0; i < (size_t)C * N; ++i) {
                    const int32_t xc = lr[2 * i], yc = lr[2 * i + 1];
                    const int c = (int)(i / N);
                    if (xc >= 0) {
                        emit((xc & 1) * C + c, i, 0u);
                        emit((xc & 1) * C + (xc >> 1), i, 1u);
                    }
                    if (yc >= 0) {
                        const int dir = 2 + (yc & 1);
                        emit(dir * C + (xc >= 0 ? xc >> 1 : c), i, 0u);
                        emit(dir * C + (yc >> 1), i, 1u);
                    }
                }
            };
            visit([&](int row, size_t, uint32_t) { ++tp[row + 1]; });
            for (size_t r = 0; r < 4 * (size_t)C; ++r)
                tp[r + 1] += tp[r];
            std::vector<uint32_t> fill(tp, tp + 4 * (size_t)C);
            visit([&](int row, size_t g, uint32_t neg) { te[fill[row]++] = (uint32_t)g << 1 | neg; });
        }
    }
    if (p.size[R_OUTIDX]) {
        int32_t *oi = (int32_t *)at(R_OUTIDX);
        int32_t next = 0;
        for (size_t i = 0; i < (size_t)C * N; ++i)
            oi[i] = d->dest_kind[i] == RANC_DEST_OUT ? next++ : -1;
    }
}

}  // namespace

struct EventPair {
    hipEvent_t a, b;
};

struct Profiler {
    bool on = false;
    std::vector<EventPair> pool;          // created on demand, reused
    std::vector<std::pair<int, int>> used; // (pool index, kind 0=integrate 1=route 2=graph 3=resident)
    double ms[4] = {0, 0, 0, 0};           // kind 3: state-resident launches
    int64_t launches[4] = {0, 0, 0, 0};
};

// A captured tick loop: num_ticks ticks reading inputs at `base`. A handle
// keeps at most MAX_CAPTURED_LOOPS of them and drops the least recently
// replayed one to capture a new one (callers that cycle through many input
// buffers would otherwise hold one graph per address forever).
struct CapturedLoop {
    int num_ticks;
    const uint32_t *base;
    hipGraph_t graph;
    hipGraphExec_t exec;
    uint64_t used;   // replay counter of the handle at the last replay
};
constexpr size_t MAX_CAPTURED_LOOPS = 16;

// A batch of networks run together, as last set up by ranc_run_ticks with
// this handle first; its tables are in this handle's workspace.
struct Batch {
    std::vector<ranc_net *> nets;
    std::vector<uint64_t> uids;   // identity of the networks (a freed handle's address may be reused)
    std::vector<const uint32_t *> bases;
    int num_ticks = 0;
    std::vector<BatchEntry> mf, pl;
    // MFMA shape classes (one launch each per tick), unless persistent
    struct Group { int first, num, units, code, ext, compact; MfmaGroupArgs args; };
    std::vector<Group> groups;
    // Phases: networks whose combined per-tick state fits the GPU's last-level
    // cache; all ticks of a phase run before the next phase starts. Groups
    // [g_first, g_first + g_num), plain entries with the byte ring [pf_first,
    // pf_first + pf_num) and without [pl_first, pl_first + pl_num), each
    // numbered from 0 within the phase. One phase when persistent.
    struct Phase { int g_first, g_num, pf_first, pf_num, pf_units, pl_first, pl_num, pl_units, rt_units; };
    // networks (indexes in nets) that run the call's ticks in launches of
    // their own (runs_solo); they are in no other list
    std::vector<int> solo;
    std::vector<char> is_solo;
    std::vector<Phase> phases;
    std::vector<std::vector<int>> phase_links;   // per phase: networks (index in nets) counting mesh links
    std::vector<char> links;                     // links_on of each network when the batch was set up
    std::vector<char> words;                     // and whether it runs through the router (wants_words)
    bool persistent = false;
    int mf_units = 0, pl_units = 0, rt_units = 0, mf_workgroups = 0;
    size_t rt_lds = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

struct ranc_net {
    Plan p{};
    uint64_t uid = 0;   // unique per loaded handle
    Batch batch;
    std::vector<CapturedLoop> loops;
    uint64_t replays = 0;              // captured-loop replays (recency of the cached loops)
    uint64_t loops_dropped = 0;        // captured loops dropped to respect MAX_CAPTURED_LOOPS
    hipStream_t cap_stream = nullptr;  // private stream used only for capture
    // batches led by this handle: streams on which the shape classes' tick
    // chains run side by side, and the fork and join events
    static constexpr int BATCH_BRANCHES = 4;
    hipStream_t br_stream[BATCH_BRANCHES] = {};
    hipEvent_t br_fork = nullptr, br_join[BATCH_BRANCHES] = {};
    RouteCfg rcfg;
    Profiler prof;
    DevNet dn;
    uint8_t *ws;
    hipStream_t last_stream;
    int64_t tick;
    uint64_t version, raster_version;
    std::vector<int> out_words;        // (core, word) pairs of raster columns (plain path)
    std::vector<int> out_neurons;      // (core, neuron) of each output-bus neuron, in index order
    std::vector<uint32_t> raster_host; // mirror of the raster
    uint64_t v_version = 0;
    std::vector<int32_t> v_host;       // mirror of the potentials
    uint64_t cnt_version = 0;
    std::vector<unsigned long long> cnt_host; // mirror of the counters
    LinkArgs lk{nullptr, nullptr, nullptr, nullptr}; // mesh link path ends, rows and counts in the workspace
    const int2 *outcol = nullptr;      // plain path: raster columns (kern_raster.hip)
    const int32_t *opos = nullptr;     // plain path: raster position of each output neuron
    bool links_on = false;             // count packets per mesh link on every tick run
    uint64_t links_version = 0;
    std::vector<long long> links_host; // mirror of the link difference arrays
    int static_dev = -1;               // device whose library-held workspace this handle holds, or -1
    bool state_lost = false;           // a state-resident launch gave up: state undefined until reset
    bool ring_words = false;           // the scheduled spikes are in the bit ring, not the byte ring (enter_ring)
    bool recorded = false;             // a caller's own graph holds runs of this handle
    bool slots_unsure = true;          // any slot of the rings may hold spikes (reset_state)
};

// MFMA path: whether this network's launches build their B tiles from the
// compact crossbar (RANC_MFMA_BSRC=planes|compact at load overrides the
// default choice, mfma_compact_b)
static int mfma_compact(const ranc_net *net)
{
    const Plan &p = net->p;
    return p.bsrc >= 0 ? p.bsrc : mfma_compact_b(net->dn, p.two, p.spw) ? 1 : 0;
}

// Plain path: the form without a router wherever the network has the byte ring.
static int auto_lanes(const ranc_net *net, const RouteCfg &rc)
{
    return net->p.size[R_RING8] ? route_split_lanes() : route_auto_lanes(net->dn, rc);
}

static bool is_recording(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    return s && hipStreamIsCapturing(s, &status) == hipSuccess && status != hipStreamCaptureStatusNone;
}

// Every instance to its initial state. A workspace just loaded, or left by a call
// that failed, may hold spikes in any slot, as may one when a recorded reset is
// replayed.
static hipError_t reset_state(ranc_net *net, hipStream_t s)
{
    const bool recording = is_recording(s), all = net->slots_unsure || recording;
    const hipError_t e =
        launch_reset_state(net->dn, net->lk, net->p.size[R_RING8] ? net->ws + net->p.off[R_RING8] : nullptr, all, s);
    if (e == hipSuccess && !recording)
        net->slots_unsure = false;
    return e;
}

static hipError_t prof_begin(ranc_net *net, int kind, hipStream_t s, int *slot)
{
    *slot = -1;
    if (!net->prof.on)
        return hipSuccess;
    Profiler &pr = net->prof;
    const size_t idx = pr.used.size();
    if (idx == pr.pool.size()) {
        EventPair e;
        hipError_t r = hipEventCreate(&e.a);
        if (r == hipSuccess)
            r = hipEventCreate(&e.b);
        if (r != hipSuccess)
            return r;
        pr.pool.push_back(e);
    }
    pr.used.push_back({(int)idx, kind});
    *slot = (int)idx;
    return hipEventRecord(pr.pool[idx].a, s);
}

static hipError_t prof_end(ranc_net *net, int slot, hipStream_t s)
{
    if (slot < 0)
        return hipSuccess;
    return hipEventRecord(net->prof.pool[slot].b, s);
}

// Fold recorded event pairs into the totals (the stream must be synchronized).
static hipError_t prof_collect(ranc_net *net)
{
    Profiler &pr = net->prof;
    for (auto &u : pr.used) {
        float ms = 0.f;
        hipError_t r = hipEventElapsedTime(&ms, pr.pool[u.first].a, pr.pool[u.first].b);
        if (r != hipSuccess)
            return r;
        pr.ms[u.second] += ms;
        pr.launches[u.second] += 1;
    }
    pr.used.clear();
    return hipSuccess;
}

// A long timed run folds finished event pairs in batches.
static hipError_t prof_fold(ranc_net *net, hipStream_t s)
{
    if (net->prof.used.size() < 4096)
        return hipSuccess;
    const hipError_t r = hipStreamSynchronize(s);
    return r == hipSuccess ? prof_collect(net) : r;
}

// How a call's segment of T ticks of a feed-forward network runs: `block`
// ticks per launch and core (0: tick by tick), the levels one after another
// (each the whole segment) or, `skewed`, all levels in each launch with level
// l one block behind level l - 1.
struct BlockPlan {
    int block = 0;
    bool skewed = false;
};

// The cheapest form by the time of its launches, launch(cores, ticks)
// microseconds each, against `cost` tick by tick.
template <typename Launch> static BlockPlan cheapest_blocks(const Plan &p, int T, double cost, Launch &&launch)
{
    BlockPlan best;
    double seq = 0;
    for (int l = 0; l < p.levels; ++l)
        seq += launch(p.level_first[l + 1] - p.level_first[l], T);
    if (seq < cost) {
        cost = seq;
        best.block = T;
    }
    for (int b = 2; b < T && p.levels > 1; b *= 2) {
        const int nb = (T + b - 1) / b;
        double skew = 0;
        for (int s = 0; s < nb + p.levels - 1; ++s) {
            const int lo = std::max(0, s - nb + 1), hi = std::min(s, p.levels - 1);
            skew += launch(p.level_first[hi + 1] - p.level_first[lo], b);
        }
        if (skew < cost) {
            cost = skew;
            best.block = b;
            best.skewed = true;
        }
    }
    return best;
}

// Plain path (k_plain_ticks): a launch takes about 4 us and 1 us per tick of a
// block while its workgroups fit the GPU. Fitted to cores of 256 x 256; over 16 core
// shapes, 2 to 8 levels of 16 to 200 cores, 1 to 60 samples and 2 to 32 ticks the form
// taken is within 12% of the fastest and at most 6% slower than tick by tick but
// for two ticks of smaller cores (2 levels of 200 cores of 64 x 256 x 40 samples
// 53 us tick by tick, 59; of 256 x 256 73, 67).
static BlockPlan choose_plain_blocks(const Plan &p, int T)
{
    if (T == 2 && (p.A < 256 || p.N < 256))
        return BlockPlan();
    auto launch = [&](long long cores, int ticks) {
        const double rounds = std::max(1.0, (double)cores * p.S * p.N / (256.0 * 1024));
        return 4.0 + rounds * (1.0 * ticks + 1.0);
    };
    return cheapest_blocks(p, T, T * launch(p.C, 1), launch);
}

// MFMA path, in us. A tick by itself: a chain that grows with the axons and the
// B tiles, and per 256 workgroups of 64 samples (a CU each) the potentials (512
// bytes per neuron) and the axons. A launch of several ticks: that chain once, moving
// potentials and B tiles per 512 workgroups of 32 samples, and per tick the time of
// one workgroup on a CU, of two, or of as many rounds of two as there are (of one
// with 512 axons, whose LDS leaves room for no more). Fitted to 14 core shapes
// with one plane and two, 2 to 6 levels of 16 to 200 cores, 64 to 1000 samples and 2
// to 32 ticks: the form taken is on average 0.5% slower than the fastest of
// tick by tick, level after level and skewed, and on 260 random layered networks of 256
// x 256 cores 0.9%, at most 36% (6 levels of 108 cores x 540 samples x 16 ticks, level
// after level 1699 us, skewed 1250); next to tick by tick at most 9% (2 levels of 200
// cores of 512 x 128 x 64 samples x 4 ticks, 54.6 us, 59.4). (Constants measured on 256 x
// 256 cores alone took up to 2.6 times as long as tick by tick: 2 ticks of 2 levels of
// 200 cores of 512 x 64 x 1000 samples 397 us, 152.)
static BlockPlan choose_blocks(const Plan &p, int T)
{
    if (!p.levels || T < 2)
        return BlockPlan();
    if (p.path == RANC_PATH_PLAIN)
        return choose_plain_blocks(p, T);
    const int w = p.N / p.slices;   // neurons of a workgroup
    const bool wide = w == 256;
    const double A = p.A;
    const int held = p.A == 512 ? 256 : 512;   // workgroups the GPU holds
    const double one = 0.7 + 0.0008 * A + (wide ? 0.15 : 0.0) + (p.two ? 0.05 + 0.0006 * A : 0.0);
    const double round = wide ? 1.35 + (p.two ? A / 640 : 0.0) : 0.6 + 0.0011 * A + (p.two && p.A >= 256 ? 0.1 : 0.0);
    const double chain = 3.3 + 0.004 * A + 0.006 * w + (p.two && wide ? 0.2 + 0.006 * A : 0.0);
    auto launch = [&](long long cores, int ticks) {
        const long long units = cores * p.slices * ((p.S + 31) / 32);
        const double tick = units <= 256 ? one : std::max(1.0, round * ((units + held - 1) / held));
        return chain + (1.5 + 0.013 * w + 0.016 * A) * units / 512 + tick * ticks;
    };
    const double per = 0.022 * w + 0.0018 * A + (p.two && wide ? 1.0 : 0.0) + (w == 128 && p.A >= 256 ? 0.7 : 0.0);
    const double units = (double)p.C * p.slices * (p.S64 / 64);
    return cheapest_blocks(p, T, 3.0 + T * (chain + per * std::max(0.0, units - 64) / 256), launch);
}

static void set_plain_args(const ranc_net *net, BlockArgs &a)
{
    const Plan &p = net->p;
    a.ring8 = net->ws + p.off[R_RING8];
    a.dst = (const uint32_t *)(net->ws + p.off[R_PLAINDST]);
    a.cols = (const uint32_t *)(net->ws + p.off[R_SCOLS]);
    a.pos = (const uint16_t *)(net->ws + p.off[R_SPOS]);
    a.sorted_words = p.sorted_words;
    a.spw = 1;
    a.want_spk = net->links_on ? 1 : 0;
}

// Queue ticks [k0, k0 + T) of the call (T <= seg_ticks) in blocks.
static hipError_t queue_blocks(ranc_net *net, const uint32_t *base, int num_ticks, int k0, int T, const BlockPlan &bp,
                               hipStream_t s, ranc_net *timer)
{
    const Plan &p = net->p;
    BlockArgs a;
    a.order = (const int32_t *)(net->ws + p.off[R_ORDER]);
    a.level = a.order + p.C;
    a.block = bp.block;
    a.k0 = k0;
    a.ticks = T;
    a.multi = p.multi_source ? 1 : 0;
    if (p.path == RANC_PATH_PLAIN)
        set_plain_args(net, a);
    a.ext_base = base;
    a.tick_words = (long long)p.Cin * p.W;
    a.ext_sstride = (long long)num_ticks * a.tick_words;
    const int nb = (T + bp.block - 1) / bp.block;
    const int steps = bp.skewed ? nb + p.levels - 1 : p.levels;
    hipError_t e = hipSuccess;
    for (int st = 0; e == hipSuccess && st < steps; ++st) {
        // levels of the launch: every level whose block of this step exists
        const int lo = bp.skewed ? std::max(0, st - nb + 1) : st, hi = bp.skewed ? std::min(st, p.levels - 1) : st;
        a.first = p.level_first[lo];
        a.count = p.level_first[hi + 1] - a.first;
        a.step = st;
        int slot = -1;
        e = timer ? prof_begin(timer, 0, s, &slot) : hipSuccess;
        if (e == hipSuccess)
            e = p.path == RANC_PATH_MFMA ? launch_integrate_mfma_ticks(net->dn, a, p.two, s) : launch_plain_ticks(net->dn, a, s);
        if (e == hipSuccess && timer)
            e = prof_end(timer, slot, s);
    }
    return e;
}

// How a call of num_ticks ticks runs: tick by tick; a feed-forward network's
// blocks of ticks; a small network's whole call in one launch. The last two add
// their counts to the totals themselves. Counting packets per link reads every
// tick's spikes as they stand after that tick. fused: the plain path's form
// without a router is wanted.
enum TickForm { FORM_TICKS, FORM_BLOCKS, FORM_WHOLE };
static TickForm choose_form(const ranc_net *net, int num_ticks, bool fused, BlockPlan &bp)
{
    const Plan &p = net->p;
    bp = BlockPlan();
    if (net->links_on || (p.path == RANC_PATH_PLAIN && !(fused && p.size[R_RING8])))
        return FORM_TICKS;
    if (p.path == RANC_PATH_PLAIN && num_ticks >= PLAIN_WHOLE_MIN_TICKS &&
        plain_whole_supported(p.C, p.A, p.N, p.G, p.D, p.Cin, p.sorted_words))
        return FORM_WHOLE;
    bp = choose_blocks(p, std::min(num_ticks, p.seg_ticks));
    return bp.block ? FORM_BLOCKS : FORM_TICKS;
}

// Queue a call's ticks in the form chosen, if it is not tick by tick (without
// the tick advance).
static hipError_t queue_several(ranc_net *net, const uint32_t *base, int num_ticks, hipStream_t s, ranc_net *timer)
{
    const Plan &p = net->p;
    BlockPlan bp;
    hipError_t e = hipSuccess;
    if (choose_form(net, num_ticks, true, bp) == FORM_WHOLE) {
        BlockArgs a;
        memset(&a, 0, sizeof a);
        set_plain_args(net, a);
        a.ext_base = base;
        a.tick_words = (long long)p.Cin * p.W;
        a.ext_sstride = (long long)num_ticks * a.tick_words;
        for (; e == hipSuccess && a.k0 < num_ticks; a.k0 += a.ticks) {
            a.ticks = std::min(num_ticks - a.k0, PLAIN_WHOLE_TICKS_MAX);
            int slot = -1;
            e = timer ? prof_begin(timer, 0, s, &slot) : hipSuccess;
            if (e == hipSuccess)
                e = launch_plain_whole(net->dn, a, s);
            if (e == hipSuccess && timer)
                e = prof_end(timer, slot, s);
        }
        return e;
    }
    for (int k = 0; e == hipSuccess && k < num_ticks; k += p.seg_ticks) {
        const int T = std::min(p.seg_ticks, num_ticks - k);
        BlockPlan b = bp;
        b.block = std::min(b.block, T);
        e = queue_blocks(net, base, num_ticks, k, T, b, s, timer);
    }
    return e;
}

// Samples per workgroup of k_plain_ticks, one tick per launch: as many as keep
// the launch within what the GPU holds at once (2048 threads on 256 CUs). One
// to three measured the same at 128 cores x 23 samples, six 17% slower.
static int plain_samples_per_wg(const Plan &p)
{
    const long long held = 256LL * 2048 / p.N / p.C;   // samples in one round of workgroups
    const long long spw = held < 1 ? 1 : (p.S + held - 1) / held;
    return (int)std::min<long long>(spw, 32);
}

// Tick k of the call on the plain path without a router (k_plain_ticks).
static hipError_t queue_plain_tick(ranc_net *net, const uint32_t *base, int num_ticks, int k, hipStream_t s)
{
    const Plan &p = net->p;
    BlockArgs a;
    memset(&a, 0, sizeof a);
    a.count = p.C;
    a.block = a.ticks = 1;
    a.k0 = k;
    set_plain_args(net, a);
    a.ext_base = base;
    a.tick_words = (long long)p.Cin * p.W;
    a.ext_sstride = (long long)num_ticks * a.tick_words;
    a.spw = plain_samples_per_wg(p);
    if ((long long)p.C * p.N * p.S < PLAIN_SORTED_MIN_WORK)
        a.sorted_words = 0;
    return launch_plain_ticks(net->dn, a, s);
}

// Queue num_ticks ticks on stream s: per tick the integration (and on the
// plain path the router), then the device tick advance. With `timer`,
// HIP event pairs are recorded around each launch while that handle's profiling is
// on (the handle's own or, in a batch, the first one's). one_tick: tick by tick even
// where several ticks would take one launch.
static ranc_status queue_ticks(ranc_net *net, const uint32_t *base, int num_ticks, hipStream_t s, ranc_net *timer,
                               bool one_tick = false)
{
    const Plan &p = net->p;
    const size_t tick_words = (size_t)p.Cin * p.W;
    if (timer && !timer->prof.on)
        timer = nullptr;
    BlockPlan bp;
    const bool fused = p.size[R_RING8] && net->rcfg.lanes == route_split_lanes();
    if (!one_tick && choose_form(net, num_ticks, fused, bp) != FORM_TICKS) {
        hipError_t e = timer ? prof_fold(timer, s) : hipSuccess;
        if (e == hipSuccess)
            e = queue_several(net, base, num_ticks, s, timer);
        if (e == hipSuccess)
            e = launch_advance_tick(net->dn, num_ticks, s);
        return e == hipSuccess ? RANC_OK : hip_fail(e, "launching integration (several ticks)");
    }
    for (int k = 0; k < num_ticks; ++k) {
        TickArgs ta;
        ta.k = k;
        ta.ext_t = base ? base + (size_t)k * tick_words : nullptr;
        ta.ext_sstride = (long long)num_ticks * tick_words;
        hipError_t e = timer ? prof_fold(timer, s) : hipSuccess;
        if (e != hipSuccess)
            return hip_fail(e, "collecting kernel timings");
        int slot = -1;
        e = timer ? prof_begin(timer, 0, s, &slot) : hipSuccess;
        if (e == hipSuccess)
            e = fused                        ? queue_plain_tick(net, base, num_ticks, k, s)
                : p.path == RANC_PATH_MFMA   ? launch_integrate_mfma(net->dn, ta, p.two, p.spw, mfma_compact(net), s)
                : p.path == RANC_PATH_SPARSE ? launch_integrate_sparse(net->dn, ta, p.spw, s)
                                             : launch_integrate_plain(net->dn, ta, s);
        if (e == hipSuccess && timer)
            e = prof_end(timer, slot, s);
        if (e != hipSuccess)
            return hip_fail(e, "launching integration");
        // The MFMA path delivers spikes inside the next tick's integration
        // (spike history gathered by destination); the plain path routes
        // into the scheduler ring here, unless integration did.
        if (p.path == RANC_PATH_PLAIN && !fused) {
            e = timer ? prof_begin(timer, 1, s, &slot) : hipSuccess;
            if (e == hipSuccess)
                e = launch_route(net->dn, k, net->rcfg, s);
            if (e == hipSuccess && timer)
                e = prof_end(timer, slot, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching routing");
        }
        if (net->links_on) {
            e = launch_link_counts(net->dn, net->lk, k, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching the mesh link count");
        }
    }
    hipError_t e = fused ? hipSuccess : launch_fold_counts(net->dn, num_ticks, s);
    if (e == hipSuccess)
        e = launch_advance_tick(net->dn, num_ticks, s);
    if (e != hipSuccess)
        return hip_fail(e, "advancing the tick");
    return RANC_OK;
}

// Whether a handle with the byte ring runs through the router all the same
// (route_lanes_per_word 1), which works on the bit ring.
static bool wants_words(const ranc_net *net)
{
    return net->p.size[R_RING8] && net->rcfg.lanes != route_split_lanes();
}

// Before a call that finds its scheduled spikes in the bit ring (words) or the
// byte ring: move them there if they are in the other. They stay where a call
// leaves them, so calls of one form after another move nothing (a move at both
// ends of every router call took 6 to 10 us of the 30 to 54 of a one-tick call).
// A call recorded into a caller's own graph may be replayed after calls of the other
// form, so from the first such call on they go back to the byte ring after every
// router call, and every router call starts with a move (one that finds the other
// ring empty changes nothing).
static hipError_t move_ring(ranc_net *net, bool words, hipStream_t s, bool recording)
{
    const hipError_t e = launch_move_ring(net->dn, net->ws + net->p.off[R_RING8], words ? 0 : 1, s);
    if (e == hipSuccess && !recording)
        net->ring_words = words;
    return e;
}
static hipError_t enter_ring(ranc_net *net, bool words, hipStream_t s)
{
    if (!net->p.size[R_RING8])
        return hipSuccess;
    const bool recording = is_recording(s);
    net->recorded = net->recorded || recording;
    const bool move = words ? net->recorded || !net->ring_words : net->ring_words;
    return move ? move_ring(net, words, s, recording) : hipSuccess;
}
static hipError_t leave_ring(ranc_net *net, bool words, hipStream_t s)
{
    return words && net->recorded ? move_ring(net, false, s, is_recording(s)) : hipSuccess;
}

// Whether a batch runs network `net` in launches of its own (queue_ticks): those
// that run several ticks per launch, and plain networks without a router large
// enough that a few of them fill the GPU. k_plain_ticks keeps a core's columns
// in registers for several samples where the batch's kernel reads them for
// each, and the chains run beside each other: the eight networks of a sweep
// with 8 samples (16 thousand to a million neurons times samples) 1405 us for
// 16 ticks in one launch per tick, 1120 with those from 2^20 on alone, 640 from
// 2^18, 633 from 2^16, 697 each alone; five networks with 15 samples 3550,
// 1769, 1171, 1128, 1130.
static bool runs_solo(const ranc_net *net, int num_ticks, bool several)
{
    const Plan &p = net->p;
    BlockPlan bp;
    if (p.path == RANC_PATH_PLAIN && p.size[R_RING8] &&
        (long long)p.C * p.N * p.S >= PLAIN_SOLO_MIN_NEURONS)
        return true;
    return several && choose_form(net, num_ticks, true, bp) != FORM_TICKS;
}

// Run num_ticks ticks as one captured graph: the tick loop is captured once
// per (num_ticks, input address) on a private stream and replayed on s.
// Every launch argument is position-in-call relative (the scheduler slot and
// raster row come from the device tick), so one graph serves every call.
static ranc_status run_captured(ranc_net *net, const uint32_t *base, int num_ticks, hipStream_t s)
{
    CapturedLoop *loop = nullptr;
    for (auto &g : net->loops)
        if (g.num_ticks == num_ticks && g.base == base)
            loop = &g;
    if (!loop) {
        hipError_t e = hipSuccess;
        if (!net->cap_stream)
            e = hipStreamCreateWithFlags(&net->cap_stream, hipStreamNonBlocking);
        if (e != hipSuccess)
            return hip_fail(e, "creating the capture stream");
        e = hipStreamBeginCapture(net->cap_stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess)
            return hip_fail(e, "beginning capture");
        ranc_status st = queue_ticks(net, base, num_ticks, net->cap_stream, nullptr);
        hipGraph_t graph = nullptr;
        e = hipStreamEndCapture(net->cap_stream, &graph);
        if (st != RANC_OK) {
            if (graph)
                hipGraphDestroy(graph);
            return st;
        }
        if (e != hipSuccess)
            return hip_fail(e, "ending capture");
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            hipGraphDestroy(graph);
            return hip_fail(e, "instantiating the tick loop");
        }
        if (net->loops.size() >= MAX_CAPTURED_LOOPS) {
            // drop the least recently used loop; its last replay may still be
            // queued, so wait for the handle's stream first
            e = hipStreamSynchronize(net->last_stream);
            if (e == hipSuccess && net->last_stream != s)
                e = hipStreamSynchronize(s);
            if (e != hipSuccess) {
                hipGraphExecDestroy(exec);
                hipGraphDestroy(graph);
                return hip_fail(e, "synchronizing before dropping a captured tick loop");
            }
            auto old = std::min_element(net->loops.begin(), net->loops.end(),
                                        [](const CapturedLoop &x, const CapturedLoop &y) { return x.used < y.used; });
            hipGraphExecDestroy(old->exec);
            hipGraphDestroy(old->graph);
            net->loops.erase(old);
            ++net->loops_dropped;
        }
        net->loops.push_back({num_ticks, base, graph, exec, 0});
        loop = &net->loops.back();
    }
    loop->used = ++net->replays;
    int slot = -1;
    hipError_t e = prof_begin(net, 2, s, &slot);
    if (e == hipSuccess)
        e = hipGraphLaunch(loop->exec, s);
    if (e == hipSuccess)
        e = prof_end(net, slot, s);
    if (e != hipSuccess)
        return hip_fail(e, "launching the tick loop");
    return RANC_OK;
}

static int device_cu_count();

// Longest wait at a grid barrier of the state-resident loop, in microseconds
// (a normal wait takes a few). RANC_RESIDENT_WAIT_US overrides it (at most
// one hour).
static unsigned long long resident_wait_us()
{
    const char *e = getenv("RANC_RESIDENT_WAIT_US");
    if (e && *e) {
        char *end = nullptr;
        const unsigned long long v = strtoull(e, &end, 10);
        if (end && *end == '\0')
            return std::min(v, 3600000000ull);
    }
    return 2000000ull;
}

// Why the state-resident loop cannot run this handle (nullptr: it can), and
// its grid.
static const char *resident_blocker(const ranc_net *net, int num_ticks, int *grid)
{
    const Plan &p = net->p;
    if (p.path != RANC_PATH_MFMA || p.auto_mid)
        return "the state-resident loop runs MFMA-path handles (64 samples or the path asked for) only";
    if (p.N != 256 || p.slices != 1)
        return "the state-resident loop needs cores of 256 neurons";
    if (p.A > 256)
        return "the state-resident loop needs cores of at most 256 axons";
    if (!net->dn.planes)
        return "the state-resident loop needs the weight planes";
    if (net->links_on)
        return "mesh link counting needs the per-tick loop";
    const int per_cu = resident_blocks_per_cu(p.A, p.two, net->dn.model_ext);
    const int cus = device_cu_count();
    if (per_cu < 1 || cus < 1)
        return "the state-resident kernel cannot be resident on this device";
    const long long max_wg = (long long)per_cu * cus;
    const long long cpw = ((long long)p.C + max_wg - 1) / max_wg;
    if (cpw > resident_max_cores_per_wg())
        return "too many cores to keep resident on this device";
    *grid = (int)((p.C + cpw - 1) / cpw);
    // the arrival counter counts every workgroup at every barrier (one per
    // tick and 64-sample group) in 32 bits
    if ((unsigned long long)(p.S64 / 64) * (unsigned long long)num_ticks * (unsigned long long)*grid >= (1ull << 32))
        return "too many ticks x sample groups for one state-resident launch";
    return nullptr;
}

// All ticks of the call in one cooperative launch (kern_resident.hip), then
// the count fold and tick advance. The launch's give-up flag is read back
// before returning (the call synchronizes `s`).
static ranc_status run_resident(ranc_net *net, const uint32_t *base, int num_ticks, hipStream_t s)
{
    const Plan &p = net->p;
    int grid = 0;
    if (const char *why = resident_blocker(net, num_ticks, &grid))
        return fail(RANC_EUNSUPPORTED, "%s", why);
    int dev = 0, rate_khz = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&rate_khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess || rate_khz < 1)
        return hip_fail(e != hipSuccess ? e : hipErrorInvalidValue, "reading the device wall-clock rate");
    ResidentArgs ra;
    ra.ext_base = base;
    ra.tick_words = (long long)p.Cin * p.W;
    ra.ext_sstride = (long long)num_ticks * ra.tick_words;
    ra.num_ticks = num_ticks;
    unsigned *sync = (unsigned *)(net->ws + p.off[R_RSYNC]);
    ResSync sy;
    sy.ctr = sync;
    sy.abort = sync + 1;
    sy.wait_ticks = resident_wait_us() * (unsigned long long)rate_khz / 1000ull;
    int slot = -1;
    e = prof_begin(net, 3, s, &slot);
    if (e == hipSuccess)
        e = launch_mfma_resident(net->dn, ra, sy, grid, p.two, s);
    if (e == hipSuccess)
        e = prof_end(net, slot, s);
    if (e != hipSuccess)
        return hip_fail(e, "launching the state-resident tick loop");
    e = launch_fold_counts(net->dn, num_ticks, s);
    if (e == hipSuccess)
        e = launch_advance_tick(net->dn, num_ticks, s);
    if (e != hipSuccess)
        return hip_fail(e, "advancing the tick");
    unsigned gave_up = 0;
    e = hipMemcpyAsync(&gave_up, sy.abort, sizeof(gave_up), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess)
        return hip_fail(e, "reading the state-resident loop's give-up flag");
    if (gave_up) {
        net->state_lost = true;
        return fail(RANC_ETIMEOUT, "a grid barrier of the state-resident loop waited longer than %llu us; "
                                   "the state is undefined until ranc_reset_state",
                    resident_wait_us());
    }
    return RANC_OK;
}

// ---------------------------------------------------------------------------
// Batches: several networks (any shapes) advanced together, one launch per
// tick and path for all of them (plus one router launch for the plain path).

static int device_cu_count()
{
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
    }
    return cus;
}

// Build the host tables of a batch: for the persistent MFMA launch one unit
// numbering sorted by decreasing work per unit (largest units handed out
// first); otherwise the MFMA entries by phase and shape class, each class
// split into launches of at most MFMA_GROUP_MAX networks whose descriptions
// travel as kernel arguments; plain entries by phase.
static ranc_status build_batch(ranc_net *const *nets, int num, const uint32_t *const *bases,
                               int num_ticks, bool persistent, Batch &b)
{
    b.persistent = persistent;
    b.groups.clear();
    b.phases.clear();
    // Phase of each network: first fit, largest state first, into phases of
    // at most `budget` bytes of state (a larger network forms its own phase).
    // Networks are independent, so running them phase after phase is exact.
    // Off unless RANC_BATCH_PHASE_MB is set: on the 64-variant sweep, phases
    // of 64 or 160 MB were 0.5-1% slower than one phase.
    size_t budget = 0;
    if (const char *env = getenv("RANC_BATCH_PHASE_MB"))
        budget = (size_t)std::max(0, atoi(env)) << 20;
    std::vector<int> phase_of(num, 0);
    if (!persistent && budget > 0) {
        std::vector<std::pair<size_t, int>> foot;
        for (int i = 0; i < num; ++i) {
            const Plan &p = nets[i]->p;
            foot.push_back({p.params_bytes + p.size[R_PLANES] + p.size[R_BSRC] + p.size[R_V] + p.size[R_HIST] + p.size[R_RING] +
                                p.size[R_SPK] + p.size[R_CNT],
                            i});
        }
        std::stable_sort(foot.begin(), foot.end(), [](const std::pair<size_t, int> &x,
                                                       const std::pair<size_t, int> &y) { return x.first > y.first; });
        std::vector<size_t> fill;
        for (const auto &f : foot) {
            size_t ph = 0;
            while (ph < fill.size() && fill[ph] + f.first > budget)
                ++ph;
            if (ph == fill.size())
                fill.push_back(0);
            fill[ph] += f.first;
            phase_of[f.second] = (int)ph;
        }
    }
    b.solo.clear();
    b.is_solo.clear();
    b.nets.assign(nets, nets + num);
    b.uids.clear();
    for (int i = 0; i < num; ++i)
        b.uids.push_back(nets[i]->uid);
    b.bases.assign(bases, bases + num);
    b.num_ticks = num_ticks;
    b.mf.clear();
    b.pl.clear();
    b.rt_lds = 0;
    int num_mf = 0, num_pl = 0;   // as RANC_PATH_AUTO's rule of 64 samples counts them
    for (int i = 0; i < num; ++i)
        ++(nets[i]->p.path == RANC_PATH_MFMA && !nets[i]->p.auto_mid ? num_mf : num_pl);
    int spare = BATCH_MAX - num_mf;
    for (int i = 0; i < num; ++i) {
        ranc_net *net = nets[i];
        const Plan &p = net->p;
        BatchEntry e;
        memset(&e, 0, sizeof e);
        e.n = net->dn;
        e.ext_base = bases[i];
        e.tick_words = (long long)p.Cin * p.W;
        e.ext_sstride = (long long)num_ticks * e.tick_words;
        e.spw = p.spw == 64 && persistent ? p.spw_pipelined : p.spw;   // (the persistent kernel has the pipelined form)
        e.form = p.path == RANC_PATH_MFMA ? mfma_compact(net) : 0;
        e.phase = phase_of[i];
        if (p.path == RANC_PATH_SPARSE)
            return fail(RANC_EUNSUPPORTED, "nets[%d]: the sparse path runs one network per call", i);
        b.is_solo.push_back(0);
        // (networks below 64 samples that RANC_PATH_AUTO put on the MFMA path
        // take what places the others leave)
        if (runs_solo(net, num_ticks, !persistent && !budget) || (p.auto_mid && --spare < 0)) {
            b.is_solo[i] = 1;
            b.solo.push_back(i);
            continue;
        }
        if (p.path == RANC_PATH_MFMA) {
            e.code = mfma_shape_code(p.A, mfma_width(p.A, p.N, p.two), p.two);
            if (p.spw == 64 && !persistent)
                e.code |= MFMA_TILE | (p.N == 64 ? MFMA_TILE_N64 : 0);
            e.units = p.C * p.slices * ((p.S + e.spw - 1) / e.spw);
            b.mf.push_back(e);
        } else {
            e.code = plain_shape_code(p.W, p.G);
            e.units = p.C * p.S * (p.N / 64);
            if (p.size[R_RING8]) {
                BlockArgs a;
                set_plain_args(net, a);
                e.ring8 = a.ring8;
                e.dst = a.dst;
                e.form = BATCH_BYTES | (a.want_spk ? BATCH_WANT_SPK : 0);
                b.pl.push_back(e);
                continue;
            }
            // batched routing reads the spike bitmaps from L2 (no LDS staging,
            // so the one launch keeps its occupancy for every network)
            RouteCfg rc = net->rcfg;
            rc.stage = 0;
            e.route_code = route_shape_code(rc, p.D);
            if (e.route_code < 0)
                return fail(RANC_EUNSUPPORTED, "nets[%d]: router shape (%d samples per block, max delay %d) "
                            "cannot run in a batch", i, net->rcfg.samples_per_block, p.D);
            e.route_split = net->rcfg.blocks_per_group;
            e.route_units = e.route_split * ((p.S + net->rcfg.samples_per_block - 1) / net->rcfg.samples_per_block);
            b.pl.push_back(e);
        }
    }
    if (num_mf > BATCH_MAX || num_pl > BATCH_MAX)
        return fail(RANC_EUNSUPPORTED, "a batch holds at most %d networks per path", BATCH_MAX);
    auto work = [](const BatchEntry &e) {
        return (double)e.spw * (e.n.N / e.n.slices) * (e.n.A + 64) * ((e.code & 1) ? 2 : 1);
    };
    // (one-tile launches take networks with and without the extended update)
    auto ext = [](const BatchEntry &e) { return (e.code & MFMA_TILE) ? 0 : e.n.model_ext; };
    auto compact = [](const BatchEntry &e) { return e.form; };
    long long mu = 0, pu = 0, ru = 0;
    if (persistent) {
        // one unit numbering, largest units first
        std::stable_sort(b.mf.begin(), b.mf.end(),
                         [&](const BatchEntry &x, const BatchEntry &y) { return work(x) > work(y); });
        for (auto &e : b.mf) {
            e.unit_begin = (int)mu;
            mu += e.units;
        }
    } else {
        // by phase, then shape class (each numbered from 0), largest units first within a class
        std::stable_sort(b.mf.begin(), b.mf.end(), [&](const BatchEntry &x, const BatchEntry &y) {
            if (x.phase != y.phase)
                return x.phase < y.phase;
            if (x.code != y.code)
                return x.code < y.code;
            if (ext(x) != ext(y))
                return ext(x) < ext(y);
            if (compact(x) != compact(y))
                return compact(x) < compact(y);
            return work(x) > work(y);
        });
        for (size_t i = 0; i < b.mf.size(); ++i) {
            BatchEntry &e = b.mf[i];
            if (b.groups.empty() || b.mf[b.groups.back().first].phase != e.phase ||
                b.groups.back().code != e.code || b.groups.back().ext != ext(e) ||
                b.groups.back().compact != compact(e) || b.groups.back().num == MFMA_GROUP_MAX) {
                b.groups.push_back(Batch::Group());
                Batch::Group &g = b.groups.back();
                memset(&g.args, 0, sizeof g.args);
                g.first = (int)i;
                g.num = g.units = 0;
                g.code = e.code;
                g.ext = ext(e);
                g.compact = compact(e);
            }
            Batch::Group &g = b.groups.back();
            if ((long long)g.units + e.units > INT32_MAX)
                return fail(RANC_EUNSUPPORTED, "batch has too many work units");
            e.unit_begin = g.units;
            MfmaGroupEntry &ge = g.args.e[g.num];
            ge.n = e.n;
            ge.ext_base = e.ext_base;
            ge.tick_words = e.tick_words;
            ge.ext_sstride = e.ext_sstride;
            ge.spw = e.spw;
            ge.unit_begin = e.unit_begin;
            g.units += e.units;
            g.num += 1;
            g.args.num = g.num;
            mu += e.units;
        }
    }
    // plain entries by phase, those with the byte ring first
    std::stable_sort(b.pl.begin(), b.pl.end(), [](const BatchEntry &x, const BatchEntry &y) {
        return x.phase != y.phase ? x.phase < y.phase : (x.form & BATCH_BYTES) > (y.form & BATCH_BYTES);
    });
    int nphases = 0;
    for (int i = 0; i < num; ++i)
        nphases = std::max(nphases, phase_of[i] + 1);
    b.phases.assign(nphases, Batch::Phase{});
    b.phase_links.assign(nphases, std::vector<int>());
    b.links.assign(num, 0);
    b.words.assign(num, 0);
    for (int i = 0; i < num; ++i) {
        b.links[i] = nets[i]->links_on ? 1 : 0;
        b.words[i] = b.is_solo[i] && wants_words(nets[i]) ? 1 : 0;   // (the batch's own kernels use the byte ring)
        if (nets[i]->links_on && !b.is_solo[i])
            b.phase_links[phase_of[i]].push_back(i);
    }
    for (size_t g = b.groups.size(); g-- > 0;) {
        Batch::Phase &ph = b.phases[b.mf[b.groups[g].first].phase];
        ph.g_first = (int)g;
        ph.g_num += 1;
    }
    for (size_t i = b.pl.size(); i-- > 0;)
        ((b.pl[i].form & BATCH_BYTES) ? b.phases[b.pl[i].phase].pf_first : b.phases[b.pl[i].phase].pl_first) = (int)i;
    for (auto &e : b.pl) {
        Batch::Phase &ph = b.phases[e.phase];
        if (e.form & BATCH_BYTES) {
            if ((long long)ph.pf_units + e.units > INT32_MAX)
                return fail(RANC_EUNSUPPORTED, "batch has too many work units");
            e.unit_begin = ph.pf_units;
            ph.pf_units += e.units;
            ph.pf_num += 1;
            pu += e.units;
            continue;
        }
        if ((long long)ph.pl_units + e.units > INT32_MAX || (long long)ph.rt_units + e.route_units > INT32_MAX)
            return fail(RANC_EUNSUPPORTED, "batch has too many work units");
        e.unit_begin = ph.pl_units;
        ph.pl_units += e.units;
        e.route_begin = ph.rt_units;
        ph.rt_units += e.route_units;
        ph.pl_num += 1;
        pu += e.units;
        ru += e.route_units;
    }
    if (mu > INT32_MAX || pu > INT32_MAX || ru > INT32_MAX)
        return fail(RANC_EUNSUPPORTED, "batch has too many work units");
    b.mf_units = (int)mu;
    b.pl_units = (int)pu;
    b.rt_units = (int)ru;
    b.mf_workgroups = (int)std::min<long long>(mu, device_cu_count());
    return RANC_OK;
}

static BatchEntry *batch_table(ranc_net *lead, int which)
{
    return (BatchEntry *)(lead->ws + lead->p.off[R_BATCH]) + (which ? BATCH_MAX : 0);
}

static unsigned *batch_queue(ranc_net *lead)
{
    return (unsigned *)(batch_table(lead, 0) + 2 * BATCH_MAX);
}

// Branch form of a batch's ticks: the networks of different shape classes do
// not depend on each other, so each class's launches for all ticks form one
// chain, and the chains (and those of the plain-path networks and of each
// network that runs several ticks per launch) run on the
// lead handle's branch streams side by side, forked from and joined back to
// `s` with events (under stream capture they become parallel branches of the
// graph). Used when nothing orders the classes within a tick: one phase, no
// persistent launch, no link counting, no per-launch timing.
static int batch_chains(const Batch &b)
{
    const Batch::Phase &ph = b.phases[0];
    return ph.g_num + (int)b.solo.size() + (ph.pf_num > 0 ? 1 : 0) + (ph.pl_num > 0 ? 1 : 0);
}

// Estimated work of a chain per tick: bytes of potentials, and a launch's own time as bytes.
static double chain_work(const Batch &b, int c)
{
    const Batch::Phase &ph = b.phases[0];
    auto bytes = [](const DevNet &n) { return 8.0 * n.C * n.N * n.S; };
    double w = 1e7;
    if (c < ph.g_num) {
        const Batch::Group &g = b.groups[ph.g_first + c];
        for (int i = g.first; i < g.first + g.num; ++i)
            w += bytes(b.mf[i].n);
    } else if (c < ph.g_num + (int)b.solo.size()) {
        w += bytes(b.nets[b.solo[c - ph.g_num]]->dn);
    } else {
        const bool pf = ph.pf_num > 0 && c == ph.g_num + (int)b.solo.size();
        const int first = pf ? ph.pf_first : ph.pl_first, num = pf ? ph.pf_num : ph.pl_num;
        for (int i = first; i < first + num; ++i)
            w += bytes(b.pl[i].n);
    }
    return w;
}

static ranc_status queue_batch_branches(ranc_net *lead, const Batch &b, hipStream_t s)
{
    const BatchEntry *tpl = batch_table(lead, 1);
    const Batch::Phase &ph = b.phases[0];
    const int chains = batch_chains(b);
    const int nb = std::min(chains, (int)ranc_net::BATCH_BRANCHES);
    hipError_t e = hipSuccess;
    for (int i = 0; e == hipSuccess && i < nb; ++i) {
        if (!lead->br_stream[i])
            e = hipStreamCreateWithFlags(&lead->br_stream[i], hipStreamNonBlocking);
        if (e == hipSuccess && !lead->br_join[i])
            e = hipEventCreateWithFlags(&lead->br_join[i], hipEventDisableTiming);
    }
    if (e == hipSuccess && !lead->br_fork)
        e = hipEventCreateWithFlags(&lead->br_fork, hipEventDisableTiming);
    if (e == hipSuccess)
        e = hipEventRecord(lead->br_fork, s);
    int forked = 0;
    for (; e == hipSuccess && forked < nb; forked += e == hipSuccess)
        e = hipStreamWaitEvent(lead->br_stream[forked], lead->br_fork, 0);
    ranc_status st_solo = RANC_OK;
    // chains by decreasing work, each on the branch with the least so far (in list
    // order, round robin: six networks x 100 samples 1870 us, now 1745)
    std::vector<std::pair<double, int>> order;
    for (int c = 0; c < chains; ++c)
        order.push_back({chain_work(b, c), c});
    std::stable_sort(order.begin(), order.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
    double load[ranc_net::BATCH_BRANCHES] = {};
    for (int i = 0; e == hipSuccess && st_solo == RANC_OK && i < chains; ++i) {
        const int c = order[i].second;
        const int branch = (int)(std::min_element(load, load + nb) - load);
        load[branch] += order[i].first;
        hipStream_t st = lead->br_stream[branch];
        if (c < ph.g_num) {
            const Batch::Group &g = b.groups[ph.g_first + c];
            for (int k = 0; e == hipSuccess && k < b.num_ticks; ++k)
                e = launch_integrate_mfma_group(g.args, g.units, k, g.code, g.ext, g.compact, st);
            for (int i = g.first; e == hipSuccess && i < g.first + g.num; ++i)
                e = launch_fold_counts(b.mf[i].n, b.num_ticks, st);
        } else if (c < ph.g_num + (int)b.solo.size()) {
            const int i = b.solo[c - ph.g_num];
            st_solo = queue_ticks(b.nets[i], b.bases[i], b.num_ticks, st, nullptr);
        } else if (ph.pf_num > 0 && c == ph.g_num + (int)b.solo.size()) {
            for (int k = 0; e == hipSuccess && k < b.num_ticks; ++k)
                e = launch_plain_ticks_batch(tpl + ph.pf_first, ph.pf_num, ph.pf_units, k, st);
        } else {
            const BatchEntry *tp = tpl + ph.pl_first;
            for (int k = 0; e == hipSuccess && k < b.num_ticks; ++k) {
                e = launch_integrate_plain_batch(tp, ph.pl_num, ph.pl_units, k, st);
                if (e == hipSuccess)
                    e = launch_route_batch(tp, ph.pl_num, ph.rt_units, k, b.rt_lds, st);
            }
            for (int i = ph.pl_first; e == hipSuccess && i < ph.pl_first + ph.pl_num; ++i)
                e = launch_fold_counts(b.pl[i].n, b.num_ticks, st);
        }
    }
    // joined also after an error: what was queued is ordered before what follows on `s`
    for (int i = 0; i < forked; ++i) {
        hipError_t j = hipEventRecord(lead->br_join[i], lead->br_stream[i]);
        if (j == hipSuccess)
            j = hipStreamWaitEvent(s, lead->br_join[i], 0);
        if (e == hipSuccess)
            e = j;
    }
    return st_solo != RANC_OK ? st_solo : e != hipSuccess ? hip_fail(e, "launching batch integration (branches)") : RANC_OK;
}

static ranc_status queue_batch_ticks(ranc_net *lead, const Batch &b, hipStream_t s, bool timed)
{
    const BatchEntry *tmf = batch_table(lead, 0), *tpl = batch_table(lead, 1);
    unsigned *queue = batch_queue(lead);
    timed = timed && lead->prof.on;
    bool any_links = false;
    for (const auto &pl : b.phase_links)
        any_links = any_links || !pl.empty();
    const bool branches = !b.persistent && b.phases.size() == 1 && !any_links && !timed &&
                          batch_chains(b) > 1;
    if (branches) {
        const ranc_status st = queue_batch_branches(lead, b, s);
        if (st != RANC_OK)
            return st;
    }
    for (int i : b.solo) {
        const ranc_status st = branches ? RANC_OK : queue_ticks(b.nets[i], b.bases[i], b.num_ticks, s, timed ? lead : nullptr);
        if (st != RANC_OK)
            return st;
    }
    for (const Batch::Phase &ph : b.phases)
    for (int k = 0; !branches && k < b.num_ticks; ++k) {
        int slot = -1;
        hipError_t e = hipSuccess;
        const bool mf = b.persistent ? !b.mf.empty() : ph.g_num > 0;
        if (mf) {
            e = timed ? prof_begin(lead, 0, s, &slot) : hipSuccess;
            if (e == hipSuccess && b.persistent)
                e = launch_integrate_mfma_batch(tmf, (int)b.mf.size(), b.mf_units, k, queue, b.mf_workgroups, s);
            for (int g = ph.g_first; e == hipSuccess && !b.persistent && g < ph.g_first + ph.g_num; ++g)
                e = launch_integrate_mfma_group(b.groups[g].args, b.groups[g].units, k, b.groups[g].code,
                                                b.groups[g].ext, b.groups[g].compact, s);
            if (e == hipSuccess && timed)
                e = prof_end(lead, slot, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching batch integration (MFMA)");
        }
        if (ph.pf_num > 0) {
            e = timed ? prof_begin(lead, 0, s, &slot) : hipSuccess;
            if (e == hipSuccess)
                e = launch_plain_ticks_batch(tpl + ph.pf_first, ph.pf_num, ph.pf_units, k, s);
            if (e == hipSuccess && timed)
                e = prof_end(lead, slot, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching batch integration (plain)");
        }
        if (ph.pl_num > 0) {
            const BatchEntry *tp = tpl + ph.pl_first;
            e = timed ? prof_begin(lead, 0, s, &slot) : hipSuccess;
            if (e == hipSuccess)
                e = launch_integrate_plain_batch(tp, ph.pl_num, ph.pl_units, k, s);
            if (e == hipSuccess && timed)
                e = prof_end(lead, slot, s);
            if (e == hipSuccess)
                e = timed ? prof_begin(lead, 1, s, &slot) : hipSuccess;
            if (e == hipSuccess)
                e = launch_route_batch(tp, ph.pl_num, ph.rt_units, k, b.rt_lds, s);
            if (e == hipSuccess && timed)
                e = prof_end(lead, slot, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching batch integration (plain)");
        }
        for (int i : b.phase_links[&ph - b.phases.data()]) {
            e = launch_link_counts(b.nets[i]->dn, b.nets[i]->lk, k, s);
            if (e != hipSuccess)
                return hip_fail(e, "launching the mesh link count");
        }
    }
    hipError_t e = hipSuccess;
    for (size_t i = 0; e == hipSuccess && !branches && i < b.nets.size(); ++i)
        if (!b.is_solo[i] && !b.nets[i]->p.size[R_RING8])   // (the others add to the totals themselves)
            e = launch_fold_counts(b.nets[i]->dn, b.num_ticks, s);
    if (e == hipSuccess && !b.mf.empty())
        e = launch_advance_batch(tmf, (int)b.mf.size(), b.num_ticks, queue, s);
    if (e == hipSuccess && !b.pl.empty())
        e = launch_advance_batch(tpl, (int)b.pl.size(), b.num_ticks, queue, s);
    if (e != hipSuccess)
        return hip_fail(e, "advancing batch ticks");
    return RANC_OK;
}

// Run num_ticks ticks of several networks together. The batch set-up (tables
// in the first network's workspace, and the captured graph with
// RANC_RUN_GRAPH) is reused while the same networks, input addresses and
// tick count repeat.
static ranc_status run_batch(ranc_net *const *nets, int num, const uint32_t *const *bases, int num_ticks,
                             bool graph, bool persistent, hipStream_t s)
{
    ranc_net *lead = nets[0];
    Batch &b = lead->batch;
    bool same = b.num_ticks == num_ticks && b.persistent == persistent && (int)b.nets.size() == num &&
                std::equal(b.nets.begin(), b.nets.end(), nets) && std::equal(b.bases.begin(), b.bases.end(), bases);
    for (int i = 0; same && i < num; ++i)
        same = b.uids[i] == nets[i]->uid && b.links[i] == (nets[i]->links_on ? 1 : 0) &&
               b.words[i] == (b.is_solo[i] && wants_words(nets[i]) ? 1 : 0);
    if (!same) {
        if (b.exec)
            hipGraphExecDestroy(b.exec);
        if (b.graph)
            hipGraphDestroy(b.graph);
        b.exec = nullptr;
        b.graph = nullptr;
        b.num_ticks = 0;
        Batch nb;
        ranc_status st = build_batch(nets, num, bases, num_ticks, persistent, nb);
        if (st != RANC_OK)
            return st;
        // the previous tables may still be read by queued work
        hipError_t e = hipStreamSynchronize(s);
        if (e == hipSuccess && !nb.mf.empty())
            e = hipMemcpy(batch_table(lead, 0), nb.mf.data(), nb.mf.size() * sizeof(BatchEntry), hipMemcpyHostToDevice);
        if (e == hipSuccess && !nb.pl.empty())
            e = hipMemcpy(batch_table(lead, 1), nb.pl.data(), nb.pl.size() * sizeof(BatchEntry), hipMemcpyHostToDevice);
        if (e == hipSuccess) {
            const unsigned zero[2] = {0u, 0u};
            e = hipMemcpy(batch_queue(lead), zero, sizeof zero, hipMemcpyHostToDevice);
        }
        if (e != hipSuccess)
            return hip_fail(e, "uploading the batch table");
        b.nets = std::move(nb.nets);
        b.uids = std::move(nb.uids);
        b.bases = std::move(nb.bases);
        b.mf = std::move(nb.mf);
        b.pl = std::move(nb.pl);
        b.groups = std::move(nb.groups);
        b.phases = std::move(nb.phases);
        b.phase_links = std::move(nb.phase_links);
        b.links = std::move(nb.links);
        b.words = std::move(nb.words);
        b.solo = std::move(nb.solo);
        b.is_solo = std::move(nb.is_solo);
        b.persistent = nb.persistent;
        b.mf_units = nb.mf_units;
        b.pl_units = nb.pl_units;
        b.rt_units = nb.rt_units;
        b.mf_workgroups = nb.mf_workgroups;
        b.rt_lds = nb.rt_lds;
        b.num_ticks = num_ticks;
    }
    auto each_ring = [&](hipError_t (*settle)(ranc_net *, bool, hipStream_t)) -> ranc_status {
        for (int i = 0; i < num; ++i) {
            const hipError_t e = settle(nets[i], b.words[i] != 0, s);
            if (e != hipSuccess)
                return hip_fail(e, "moving the scheduled spikes");
        }
        return RANC_OK;
    };
    if (!graph) {
        ranc_status st = each_ring(enter_ring);
        if (st == RANC_OK)
            st = queue_batch_ticks(lead, b, s, true);
        return st == RANC_OK ? each_ring(leave_ring) : st;
    }
    if (!b.exec) {
        hipError_t e = hipSuccess;
        if (!lead->cap_stream)
            e = hipStreamCreateWithFlags(&lead->cap_stream, hipStreamNonBlocking);
        if (e == hipSuccess)
            e = hipStreamBeginCapture(lead->cap_stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess)
            return hip_fail(e, "beginning batch capture");
        ranc_status st = queue_batch_ticks(lead, b, lead->cap_stream, false);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(lead->cap_stream, &g);
        if (st != RANC_OK) {
            if (g)
                hipGraphDestroy(g);
            return st;
        }
        if (e == hipSuccess)
            e = hipGraphInstantiate(&b.exec, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            if (g)
                hipGraphDestroy(g);
            return hip_fail(e, "capturing the batch tick loop");
        }
        b.graph = g;
    }
    ranc_status st = each_ring(enter_ring);
    if (st != RANC_OK)
        return st;
    int slot = -1;
    hipError_t e = prof_begin(lead, 2, s, &slot);
    if (e == hipSuccess)
        e = hipGraphLaunch(b.exec, s);
    if (e == hipSuccess)
        e = prof_end(lead, slot, s);
    if (e != hipSuccess)
        return hip_fail(e, "launching the batch tick loop");
    return each_ring(leave_ring);
}

static void drop_graphs(ranc_net *net);

extern "C" {

const char *ranc_last_error(void) { return g_err.c_str(); }

ranc_status ranc_workspace_bytes(const ranc_net_desc *desc, int32_t num_samples, int32_t max_ticks_per_call,
                                 int32_t path, size_t *bytes)
{
    if (!bytes)
        return fail(RANC_EINVAL, "bytes is NULL");
    Plan p{};
    ranc_status st = make_plan(desc, num_samples, max_ticks_per_call, path, p);
    if (st != RANC_OK)
        return st;
    *bytes = p.total;
    return RANC_OK;
}

ranc_status ranc_load_network(const ranc_net_desc *desc, int32_t num_samples, int32_t max_ticks_per_call,
                              int32_t path, void *workspace, size_t workspace_bytes, void *stream, ranc_net **out)
{
    if (!out)
        return fail(RANC_EINVAL, "out is NULL");
    *out = nullptr;
    Plan p{};
    ranc_status st = make_plan(desc, num_samples, max_ticks_per_call, path, p);
    if (st != RANC_OK)
        return st;
    if (!workspace)
        return fail(RANC_EINVAL, "workspace is NULL");
    if ((uintptr_t)workspace % 256)
        return fail(RANC_EINVAL, "workspace must be 256-byte aligned");
    for (int level = PLAN_FORMS; workspace_bytes < p.total && level >= PLAN_SMALL; --level) {
        // a workspace sized for a layout without these
        Plan q{};
        st = make_plan(desc, num_samples, max_ticks_per_call, path, q, (PlanLevel)level);
        if (st != RANC_OK)
            return st;
        p = std::move(q);
    }
    if (workspace_bytes < p.total)
        return fail(RANC_ENOMEM, "workspace has %zu bytes, needs %zu", workspace_bytes, p.total);
    ranc_net *net = new (std::nothrow) ranc_net();
    if (!net)
        return fail(RANC_ENOMEM, "host allocation failed");
    static std::atomic<uint64_t> next_uid{1};
    net->p = p;
    net->uid = next_uid++;
    net->ws = (uint8_t *)workspace;
    auto reg = [&](Region r) -> uint8_t * { return net->ws + p.off[r]; };
    DevNet &n = net->dn;
    n.C = p.C; n.A = p.A; n.N = p.N; n.G = p.G; n.W = p.W; n.NW = p.NW; n.D = p.D; n.Q = p.Q;
    n.S = p.S; n.S64 = p.S64; n.RT = p.RT; n.Wout = p.Wout; n.Nout = p.Nout; n.Cin = p.Cin;
    n.cnt_rows = p.cnt_rows;
    n.slices = p.slices;
    n.vlayout = p.path == RANC_PATH_MFMA ? VLAYOUT_BRICK : p.path == RANC_PATH_SPARSE ? VLAYOUT_SPARSE : VLAYOUT_CSN;
    n.vmin = (int32_t)(-(1LL << (desc->potential_bits - 1)));
    n.vmax = (int32_t)((1LL << (desc->potential_bits - 1)) - 1);
    n.model_ext = neuron_model_ext(desc) ? 1 : 0;
    n.floor = (const int32_t *)reg(R_FLOOR);
    n.linmask = (const uint32_t *)reg(R_LINMASK);
    // the plain path's column words, or the MFMA path's compact B source
    // (which starts with the same words)
    n.colbits = p.size[R_BSRC] ? (const uint32_t *)reg(R_BSRC)
                : p.size[R_COLBITS] ? (const uint32_t *)reg(R_COLBITS) : nullptr;
    n.typemask = (const uint32_t *)reg(R_TYPEMASK);
    n.wts = (const int32_t *)reg(R_WTS);
    n.leak = (const int32_t *)reg(R_LEAK);
    n.thr = (const int32_t *)reg(R_THR);
    n.rst = (const int32_t *)reg(R_RST);
    n.vinit = (const int32_t *)reg(R_VINIT);
    n.coremask = (const uint32_t *)reg(R_COREMASK);
    n.outmask = (const uint32_t *)reg(R_OUTMASK);
    n.outword = (const int32_t *)reg(R_OUTWORD);
    n.in_index = (const int32_t *)reg(R_ININDEX);
    n.rt_dcnt = (const uint16_t *)reg(R_RTDCNT);
    n.rt_goff = (const uint32_t *)reg(R_RTGOFF);
    n.rt_ent = (const uint32_t *)reg(R_RTENT);
    n.degb = (const uint32_t *)reg(R_DEGB);
    n.outidx = (const int32_t *)reg(R_OUTIDX);
    n.planes = p.size[R_PLANES] ? (const uint4 *)reg(R_PLANES) : nullptr;
    n.V = (int32_t *)reg(R_V);
    n.ring = (uint32_t *)reg(R_RING);
    n.spk = (uint32_t *)reg(R_SPK);
    n.hist = (uint64_t *)reg(R_HIST);
    n.rtx_ptr = (const uint32_t *)reg(R_RTXPTR);
    n.rtx_ent = (const uint32_t *)reg(R_RTXENT);
    n.hist_zero = (const uint64_t *)reg(R_HZERO);
    n.ecsr_ptr = (const uint32_t *)reg(R_ECSRPTR);
    n.ecsr_ent = (const uint16_t *)reg(R_ECSRENT);
    n.raster = (uint32_t *)reg(R_RASTER);
    n.cnt = (unsigned long long *)reg(R_CNT);
    n.cring = (unsigned long long *)reg(R_CRING);
    n.tick = (int *)reg(R_TICK);
    net->lk.rec = (const int2 *)reg(R_LINKREC);
    net->lk.rows = p.size[R_LINKPTR] ? (const uint32_t *)reg(R_LINKPTR) : nullptr;
    net->lk.ents = p.size[R_LINKPTR] ? (const uint32_t *)reg(R_LINKENT) : nullptr;
    net->outcol = p.size[R_OUTCOL] ? (const int2 *)reg(R_OUTCOL) : nullptr;
    net->opos = p.size[R_OUTPOS] ? (const int32_t *)reg(R_OUTPOS) : nullptr;
    net->lk.d = (long long *)reg(R_LINKD);
    std::vector<uint8_t> host;
    pack_params(desc, p, host, net->out_words);
    for (size_t i = 0; i < (size_t)p.C * p.N; ++i)
        if (desc->dest_kind[i] == RANC_DEST_OUT) {
            net->out_neurons.push_back((int)(i / p.N));
            net->out_neurons.push_back((int)(i % p.N));
        }
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(net->ws, host.data(), p.params_bytes, hipMemcpyHostToDevice, s);
    std::vector<uint8_t> bsrc;
    if (e == hipSuccess && p.size[R_BSRC]) {
        pack_bsrc(desc, p, bsrc);
        e = hipMemcpyAsync(reg(R_BSRC), bsrc.data(), bsrc.size(), hipMemcpyHostToDevice, s);
        if (e == hipSuccess && p.size[R_PLANES])
            e = launch_build_planes(n, p.two, (uint4 *)reg(R_PLANES), s);
    }
    if (e == hipSuccess && p.levels) {
        e = hipMemcpyAsync(reg(R_ORDER), p.order.data(), (size_t)p.C * 4, hipMemcpyHostToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(reg(R_ORDER) + (size_t)p.C * 4, p.level.data(), (size_t)p.C * 4, hipMemcpyHostToDevice, s);
    }
    if (e == hipSuccess)
        e = reset_state(net, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        delete net;
        return hip_fail(e, "uploading the network");
    }
    net->rcfg = route_default_cfg(n);
    if (const char *e = getenv("RANC_ROUTE_SB")) {
        const int v = atoi(e);
        if (v == 1 || v == 2 || v == 4 || v == 8)
            net->rcfg.samples_per_block = v;
    }
    if (const char *e = getenv("RANC_ROUTE_SPLIT")) {
        const int v = atoi(e);
        if (v >= 1)
            net->rcfg.blocks_per_group = v;
    }
    if (const char *e = getenv("RANC_ROUTE_STAGE"))
        net->rcfg.stage = atoi(e) != 0;
    if ((size_t)n.C * n.NW * 4 * net->rcfg.samples_per_block > 128 * 1024)
        net->rcfg.stage = 0;
    net->rcfg.lanes = auto_lanes(net, net->rcfg);
    net->last_stream = s;
    net->tick = 0;
    net->version = 1;
    net->raster_version = 0;
    *out = net;
    return RANC_OK;
}

ranc_status ranc_load_network_static(const ranc_net_desc *desc, int32_t num_samples, int32_t max_ticks_per_call,
                                     int32_t path, void *stream, ranc_net **out)
{
    if (!out)
        return fail(RANC_EINVAL, "out is NULL");
    *out = nullptr;
    Plan p{};
    ranc_status st = make_plan(desc, num_samples, max_ticks_per_call, path, p, PLAN_SMALL);
    if (st != RANC_OK)
        return st;
    if (p.total > RANC_STATIC_WORKSPACE_BYTES)
        return fail(RANC_ENOMEM, "the network needs %zu bytes of workspace; the library-held workspace has %zu",
                    p.total, (size_t)RANC_STATIC_WORKSPACE_BYTES);
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e, "querying the current device");
    if (dev < 0 || dev >= STATIC_WS_MAX_DEVICES)
        return fail(RANC_EUNSUPPORTED, "device %d: the library-held workspace exists for devices 0..%d", dev,
                    STATIC_WS_MAX_DEVICES - 1);
    void *ws = nullptr;
    bool held = false;
    e = static_ws_claim(dev, &ws, &held);
    if (e != hipSuccess)
        return hip_fail(e, "looking up the library-held workspace");
    if (held)
        return fail(RANC_ESTATE, "the library-held workspace of device %d is used by a handle not yet freed", dev);
    st = ranc_load_network(desc, num_samples, max_ticks_per_call, path, ws, RANC_STATIC_WORKSPACE_BYTES, stream,
                           out);
    if (st != RANC_OK) {
        static_ws_release(dev);
        return st;
    }
    (*out)->static_dev = dev;
    return RANC_OK;
}

ranc_status ranc_run_ticks(ranc_net *const *nets, int32_t num_nets, const uint32_t *const *inputs, uint32_t flags,
                           int32_t num_ticks, void *stream)
{
    if (!nets || num_nets < 1)
        return fail(RANC_EINVAL, "nets is NULL or num_nets < 1");
    for (int i = 0; i < num_nets; ++i) {
        if (!nets[i])
            return fail(RANC_EINVAL, "nets[%d] is NULL", i);
        if (num_ticks < 1 || num_ticks > nets[i]->p.RT)
            return fail(RANC_EINVAL, "num_ticks %d outside [1, max_ticks_per_call=%d]", num_ticks, nets[i]->p.RT);
    }
    if (flags & ~(RANC_INPUTS_ON_DEVICE | RANC_RUN_GRAPH | RANC_BATCH_PERSISTENT | RANC_RUN_RESIDENT))
        return fail(RANC_EINVAL, "unknown flags 0x%x", flags);
    for (int i = 0; i < num_nets; ++i)
        if (nets[i]->state_lost)
            return fail(RANC_ESTATE, "nets[%d]: a state-resident run gave up; reset the state first", i);
    if (flags & RANC_RUN_RESIDENT) {
        if (num_nets != 1)
            return fail(RANC_EUNSUPPORTED, "RANC_RUN_RESIDENT runs one network per call");
        int grid = 0;
        if (const char *why = resident_blocker(nets[0], num_ticks, &grid))
            return fail(RANC_EUNSUPPORTED, "%s", why);
    }
    for (int i = 0; i < num_nets; ++i)
        for (int j = 0; j < i; ++j)
            if (nets[i] == nets[j])
                return fail(RANC_EINVAL, "nets[%d] and nets[%d] are the same network", j, i);
    hipStream_t s = (hipStream_t)stream;
    std::vector<const uint32_t *> bases(num_nets, nullptr);
    for (int i = 0; i < num_nets; ++i) {
        ranc_net *net = nets[i];
        const Plan &p = net->p;
        const uint32_t *base = inputs ? inputs[i] : nullptr;
        const size_t tick_words = (size_t)p.Cin * p.W;
        if (base && p.Cin > 0 && !(flags & RANC_INPUTS_ON_DEVICE)) {
            uint32_t *stage = (uint32_t *)(net->ws + p.off[R_EXT]);
            hipError_t e = hipMemcpyAsync(stage, base, (size_t)p.S * num_ticks * tick_words * 4,
                                          hipMemcpyHostToDevice, s);
            if (e != hipSuccess)
                return hip_fail(e, "staging inputs");
            base = stage;
        }
        if (p.Cin == 0)
            base = nullptr;
        bases[i] = base;
    }
    if (num_nets > 1) {
        ranc_status st = run_batch(nets, num_nets, bases.data(), num_ticks, (flags & RANC_RUN_GRAPH) != 0,
                                   (flags & RANC_BATCH_PERSISTENT) != 0, s);
        if (st != RANC_OK) {
            for (int i = 0; i < num_nets; ++i)
                nets[i]->slots_unsure = true;
            return st;
        }
    } else {
        const bool words = wants_words(nets[0]);
        hipError_t e = enter_ring(nets[0], words, s);
        if (e != hipSuccess) {
            nets[0]->slots_unsure = true;
            return hip_fail(e, "moving the scheduled spikes");
        }
        ranc_status st = (flags & RANC_RUN_RESIDENT) ? run_resident(nets[0], bases[0], num_ticks, s)
                         : (flags & RANC_RUN_GRAPH)  ? run_captured(nets[0], bases[0], num_ticks, s)
                                                     : queue_ticks(nets[0], bases[0], num_ticks, s, nets[0]);
        if (st == RANC_OK && (e = leave_ring(nets[0], words, s)) != hipSuccess)
            st = hip_fail(e, "moving the scheduled spikes");
        if (st == RANC_ETIMEOUT) {   // the ticks ran partially: the call counts as run
            nets[0]->tick += num_ticks;
            nets[0]->last_stream = s;
            ++nets[0]->version;
        }
        if (st != RANC_OK) {
            nets[0]->slots_unsure = true;
            return st;
        }
    }
    for (int i = 0; i < num_nets; ++i) {
        nets[i]->tick += num_ticks;
        nets[i]->last_stream = s;
        ++nets[i]->version;
    }
    return RANC_OK;
}

static ranc_status sync_net(ranc_net *net)
{
    hipError_t e = hipStreamSynchronize(net->last_stream);
    if (e != hipSuccess)
        return hip_fail(e, "synchronizing");
    return RANC_OK;
}

// Whole-buffer host mirrors, refreshed once per state version: reading many
// samples costs one device-to-host copy.
static ranc_status refresh_mirror(ranc_net *net, const void *src, size_t bytes, void *dst, uint64_t &version,
                                  const char *what)
{
    if (version == net->version)
        return RANC_OK;
    ranc_status st = sync_net(net);
    if (st != RANC_OK)
        return st;
    hipError_t e = hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
    if (e != hipSuccess)
        return hip_fail(e, what);
    version = net->version;
    return RANC_OK;
}

ranc_status ranc_read_spikes(ranc_net *net, int32_t sample, int64_t tick_begin, int64_t tick_end, ranc_spike *out,
                             int64_t capacity, int64_t *count)
{
    if (!net || !count)
        return fail(RANC_EINVAL, "net or count is NULL");
    const Plan &p = net->p;
    if (sample < 0 || sample >= p.S)
        return fail(RANC_EINVAL, "sample %d out of range", sample);
    const int64_t lo = std::max<int64_t>(0, net->tick - p.RT);
    if (tick_begin < lo || tick_end > net->tick || tick_begin > tick_end)
        return fail(RANC_ESTATE, "ticks [%lld, %lld) outside the retained window [%lld, %lld)",
                    (long long)tick_begin, (long long)tick_end, (long long)lo, (long long)net->tick);
    const bool mf = p.path != RANC_PATH_PLAIN;   // sample-tiled paths: neuron-major raster
    const size_t HG = (size_t)p.S64 / 64;
    net->raster_host.resize(mf ? (size_t)p.RT * p.Nout * HG * 2 : (size_t)p.RT * p.S * p.Wout);
    ranc_status st = refresh_mirror(net, net->dn.raster, net->raster_host.size() * 4, net->raster_host.data(),
                                    net->raster_version, "reading the raster");
    if (st != RANC_OK)
        return st;
    int64_t k = 0;
    auto emit = [&](int64_t t, int core, int neuron) {
        if (out && k < capacity) {
            out[k].tick = t;
            out[k].core = core;
            out[k].neuron = neuron;
        }
        ++k;
    };
    if (mf) {
        // neuron-major words of 64 samples; on the MFMA path the bit of a
        // sample inverts the spike-word order sigma(b) = 8((b%16)/4) + 4(b/16)
        // + b%4, on the sparse path it is the sample's index in its tile
        const int i = sample % 32;
        const int bit = p.path == RANC_PATH_SPARSE ? sample % 64
                                                   : 32 * ((sample % 64) / 32) + 16 * ((i % 8) / 4) + 4 * (i / 8) + i % 4;
        const uint64_t *r64 = reinterpret_cast<const uint64_t *>(net->raster_host.data());
        for (int64_t t = tick_begin; t < tick_end; ++t) {
            const uint64_t *row = r64 + (size_t)(t % p.RT) * p.Nout * HG + sample / 64;
            // 64 output neurons at a time: gather their bits into one mask
            // without branches, then emit the set bits in order
            for (int o0 = 0; o0 < p.Nout; o0 += 64) {
                const int n = std::min(64, p.Nout - o0);
                uint64_t m = 0;
                for (int j = 0; j < n; ++j)
                    m |= ((row[(size_t)(o0 + j) * HG] >> bit) & 1u) << j;
                while (m) {
                    const int o = o0 + __builtin_ctzll(m);
                    m &= m - 1;
                    emit(t, net->out_neurons[2 * o], net->out_neurons[2 * o + 1]);
                }
            }
        }
    } else {
        for (int64_t t = tick_begin; t < tick_end; ++t) {
            const uint32_t *row = net->raster_host.data() + ((size_t)(t % p.RT) * p.S + sample) * p.Wout;
            for (int ow = 0; ow < p.Wout; ++ow) {
                uint32_t w = row[ow];
                while (w) {
                    const int b = __builtin_ctz(w);
                    w &= w - 1;
                    emit(t, net->out_words[2 * ow], net->out_words[2 * ow + 1] * 32 + b);
                }
            }
        }
    }
    *count = k;
    if (k > capacity)
        return fail(RANC_ETRUNC, "%lld spikes do not fit capacity %lld", (long long)k, (long long)capacity);
    return RANC_OK;
}

ranc_status ranc_raster_bytes(const ranc_net *net, int64_t num_ticks, uint32_t layout, size_t *bytes)
{
    if (!net || !bytes)
        return fail(RANC_EINVAL, "net or bytes is NULL");
    if (num_ticks < 0)
        return fail(RANC_EINVAL, "num_ticks %lld < 0", (long long)num_ticks);
    const Plan &p = net->p;
    if (layout == RANC_RASTER_BY_NEURON)
        *bytes = (size_t)num_ticks * p.Nout * (p.S64 / 64) * 8;
    else if (layout == RANC_RASTER_BY_SAMPLE)
        *bytes = (size_t)num_ticks * p.S * ((p.Nout + 31) / 32) * 4;
    else
        return fail(RANC_EINVAL, "unknown raster layout %u", layout);
    return RANC_OK;
}

ranc_status ranc_copy_raster(ranc_net *net, int64_t tick_begin, int64_t tick_end, uint32_t layout, void *dst,
                             size_t dst_bytes, void *stream)
{
    if (!net || !dst)
        return fail(RANC_EINVAL, "net or dst is NULL");
    if (layout != RANC_RASTER_BY_NEURON && layout != RANC_RASTER_BY_SAMPLE)
        return fail(RANC_EINVAL, "unknown raster layout %u", layout);
    const Plan &p = net->p;
    const int64_t lo = std::max<int64_t>(0, net->tick - p.RT);
    if (tick_begin < lo || tick_end > net->tick || tick_begin >= tick_end)
        return fail(RANC_ESTATE, "ticks [%lld, %lld) empty or outside the retained window [%lld, %lld)",
                    (long long)tick_begin, (long long)tick_end, (long long)lo, (long long)net->tick);
    size_t need = 0;
    ranc_raster_bytes(net, tick_end - tick_begin, layout, &need);
    if (dst_bytes < need)
        return fail(RANC_ENOMEM, "dst has %zu bytes, needs %zu", dst_bytes, need);
    hipError_t e = launch_pack_raster(net->dn, net->outcol, net->opos, layout == RANC_RASTER_BY_SAMPLE, tick_begin,
                                      (int)(tick_end - tick_begin), dst, (hipStream_t)stream);
    if (e != hipSuccess)
        return hip_fail(e, "packing the output raster");
    return RANC_OK;
}

ranc_status ranc_output_neurons(const ranc_net *net, int32_t *out, int64_t capacity, int64_t *count)
{
    if (!net || !count)
        return fail(RANC_EINVAL, "net or count is NULL");
    const int64_t n = (int64_t)net->out_neurons.size() / 2;
    *count = n;
    if (capacity < n)
        return fail(RANC_ETRUNC, "%lld output neurons do not fit capacity %lld", (long long)n, (long long)capacity);
    if (n && !out)
        return fail(RANC_EINVAL, "out is NULL");
    memcpy(out, net->out_neurons.data(), (size_t)n * 2 * sizeof(int32_t));
    return RANC_OK;
}

ranc_status ranc_read_potentials(ranc_net *net, int32_t sample, int32_t *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    const Plan &p = net->p;
    if (sample < 0 || sample >= p.S)
        return fail(RANC_EINVAL, "sample %d out of range", sample);
    const bool brick = net->dn.vlayout == VLAYOUT_BRICK;
    const size_t SV = net->dn.vlayout == VLAYOUT_CSN ? (size_t)p.S : (size_t)p.S64;
    net->v_host.resize((size_t)p.C * SV * p.N);
    ranc_status st = refresh_mirror(net, net->dn.V, net->v_host.size() * 4, net->v_host.data(), net->v_version,
                                    "reading potentials");
    if (st != RANC_OK)
        return st;
    if (net->dn.vlayout == VLAYOUT_SPARSE) {   // [C][N][S64]
        for (size_t cj = 0; cj < (size_t)p.C * p.N; ++cj)
            out[cj] = net->v_host[cj * SV + sample];
        return RANC_OK;
    }
    if (!brick) {
        for (int c = 0; c < p.C; ++c)
            memcpy(out + (size_t)c * p.N, net->v_host.data() + ((size_t)c * SV + sample) * p.N, (size_t)p.N * 4);
        return RANC_OK;
    }
    // brick (c, nb, g): element (q, lane l, e) = sample 32g + 8q + 4(l/32) + e, neuron 32nb + l%32
    const int NB = p.N / 32;
    const size_t groups = (size_t)p.S64 / 32;
    const int g = sample / 32, i = sample % 32, q = i / 8, hh = (i % 8) / 4, e = i % 4;
    for (int c = 0; c < p.C; ++c)
        for (int nb = 0; nb < NB; ++nb)
            for (int jj = 0; jj < 32; ++jj)
                out[(size_t)c * p.N + nb * 32 + jj] =
                    net->v_host[(((((size_t)c * NB + nb) * groups + g) * 4 + q) * 64 + 32 * hh + jj) * 4 + e];
    return RANC_OK;
}

ranc_status ranc_read_counters(ranc_net *net, int32_t sample, ranc_counters *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    const Plan &p = net->p;
    if (sample < 0 || sample >= p.S)
        return fail(RANC_EINVAL, "sample %d out of range", sample);
    const int rows = p.C * net->dn.cnt_rows;   // counter rows: per core, 64-neuron block (plain) or slice (MFMA)
    net->cnt_host.resize((size_t)rows * p.S * CNT_N);
    ranc_status st = refresh_mirror(net, net->dn.cnt, net->cnt_host.size() * 8, net->cnt_host.data(),
                                    net->cnt_version, "reading counters");
    if (st != RANC_OK)
        return st;
    unsigned long long sum[CNT_N] = {0, 0, 0, 0, 0};
    for (int c = 0; c < rows; ++c)
        for (int k = 0; k < CNT_N; ++k)
            sum[k] += net->cnt_host[((size_t)c * p.S + sample) * CNT_N + k];
    out->emitted = sum[CNT_EMITTED];
    out->routed = sum[CNT_ROUTED];
    out->delivered = sum[CNT_DELIVERED];
    out->out = sum[CNT_OUT];
    out->events = sum[CNT_EVENTS];
    return RANC_OK;
}

ranc_status ranc_link_counts_enable(ranc_net *net, int32_t enable)
{
    if (!net)
        return fail(RANC_EINVAL, "net is NULL");
    if (enable != 0 && enable != 1)
        return fail(RANC_EINVAL, "enable must be 0 or 1");
    if (net->links_on != (enable == 1)) {
        drop_graphs(net);
        net->links_on = enable == 1;
    }
    return RANC_OK;
}

ranc_status ranc_read_links(ranc_net *net, int32_t sample, int64_t *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    const Plan &p = net->p;
    if (sample < 0 || sample >= p.S)
        return fail(RANC_EINVAL, "sample %d out of range", sample);
    net->links_host.resize((size_t)4 * p.C * p.S64);
    ranc_status st = refresh_mirror(net, net->lk.d, net->links_host.size() * 8, net->links_host.data(),
                                    net->links_version, "reading mesh link counts");
    if (st != RANC_OK)
        return st;
    // difference arrays [dir][core][S64] -> counts: prefix sums along each
    // mesh row (+x ascending x, -x descending), column (+y, -y)
    const int gw = p.grid_w, gh = p.grid_h;
    auto dv = [&](int dir, int core) { return net->links_host[((size_t)dir * p.C + core) * p.S64 + sample]; };
    for (int y = 0; y < gh; ++y) {
        long long up = 0, down = 0;
        for (int x = 0; x < gw; ++x) {
            up += dv(RANC_LINK_XPLUS, y * gw + x);
            out[(size_t)(y * gw + x) * 4 + RANC_LINK_XPLUS] = up;
            const int xr = gw - 1 - x;
            down += dv(RANC_LINK_XMINUS, y * gw + xr);
            out[(size_t)(y * gw + xr) * 4 + RANC_LINK_XMINUS] = down;
        }
    }
    for (int x = 0; x < gw; ++x) {
        long long up = 0, down = 0;
        for (int y = 0; y < gh; ++y) {
            up += dv(RANC_LINK_YPLUS, y * gw + x);
            out[(size_t)(y * gw + x) * 4 + RANC_LINK_YPLUS] = up;
            const int yr = gh - 1 - y;
            down += dv(RANC_LINK_YMINUS, yr * gw + x);
            out[(size_t)(yr * gw + x) * 4 + RANC_LINK_YMINUS] = down;
        }
    }
    return RANC_OK;
}

ranc_status ranc_current_tick(const ranc_net *net, int64_t *tick)
{
    if (!net || !tick)
        return fail(RANC_EINVAL, "net or tick is NULL");
    *tick = net->tick;
    return RANC_OK;
}

ranc_status ranc_get_path(const ranc_net *net, int32_t *path)
{
    if (!net || !path)
        return fail(RANC_EINVAL, "net or path is NULL");
    *path = net->p.path;
    return RANC_OK;
}

ranc_status ranc_profile_enable(ranc_net *net, int32_t enable)
{
    if (!net)
        return fail(RANC_EINVAL, "net is NULL");
    if (enable) {
        ranc_status st = sync_net(net);
        if (st != RANC_OK)
            return st;
        net->prof.used.clear();
        for (int k = 0; k < 4; ++k) {
            net->prof.ms[k] = 0;
            net->prof.launches[k] = 0;
        }
    }
    net->prof.on = enable != 0;
    return RANC_OK;
}

ranc_status ranc_profile_read(ranc_net *net, ranc_profile *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    ranc_status st = sync_net(net);
    if (st != RANC_OK)
        return st;
    hipError_t e = prof_collect(net);
    if (e != hipSuccess)
        return hip_fail(e, "reading kernel timings");
    out->integrate_ms = net->prof.ms[0];
    out->route_ms = net->prof.ms[1];
    out->integrate_launches = net->prof.launches[0];
    out->route_launches = net->prof.launches[1];
    out->graph_ms = net->prof.ms[2];
    out->graph_launches = net->prof.launches[2];
    out->graphs_held = (int64_t)net->loops.size();
    out->graphs_dropped = (int64_t)net->loops_dropped;
    out->resident_ms = net->prof.ms[3];
    out->resident_launches = net->prof.launches[3];
    return RANC_OK;
}

ranc_status ranc_reset_state(ranc_net *net, void *stream)
{
    if (!net)
        return fail(RANC_EINVAL, "net is NULL");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = reset_state(net, s);
    if (e != hipSuccess)
        return hip_fail(e, "resetting state");
    net->tick = 0;
    net->last_stream = s;
    ++net->version;
    net->state_lost = false;
    return RANC_OK;
}

// Launch-shape autotuner: time every candidate shape of the handle's path on
// num_ticks ticks of the given inputs and keep the fastest.
static void drop_graphs(ranc_net *net)
{
    for (auto &g : net->loops) {
        hipGraphExecDestroy(g.exec);
        hipGraphDestroy(g.graph);
    }
    net->loops.clear();
    if (net->batch.exec)
        hipGraphExecDestroy(net->batch.exec);
    if (net->batch.graph)
        hipGraphDestroy(net->batch.graph);
    net->batch = Batch();
}

ranc_status ranc_autotune(ranc_net *net, const uint32_t *inputs, uint32_t flags, int32_t num_ticks, void *stream,
                          ranc_tune *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    if (num_ticks < 1 || num_ticks > net->p.RT)
        return fail(RANC_EINVAL, "num_ticks %d outside [1, max_ticks_per_call=%d]", num_ticks, net->p.RT);
    if (flags & ~RANC_INPUTS_ON_DEVICE)
        return fail(RANC_EINVAL, "unknown flags 0x%x", flags);
    hipStream_t s = (hipStream_t)stream;
    Plan &p = net->p;
    struct Cand {
        int spw;
        RouteCfg rc;
    };
    std::vector<Cand> cands;
    if (p.path != RANC_PATH_PLAIN) {
        const int tiles = (p.S + 63) / 64;
        int last_chunks = -1;
        const int cap = p.path == RANC_PATH_SPARSE ? sparse_max_samples_per_wg() : mfma_max_samples_per_wg();
        for (int spw = 64; spw <= cap; spw *= 2) {
            const int chunks = (tiles * 64 + spw - 1) / spw;
            if (chunks == last_chunks)
                break;
            last_chunks = chunks;
            cands.push_back({spw, net->rcfg});
        }
    } else {
        const RouteCfg def = route_default_cfg(net->dn);
        const int dmax = route_dmax(p.D);
        for (int sb = 1; sb <= 8; sb *= 2) {
            if (sb * dmax > 32 || (sb > 1 && sb > p.S))
                continue;
            const size_t bitmap = (size_t)p.C * p.NW * 4 * sb;
            const int groups = (p.S + sb - 1) / sb;
            const int max_split = std::max(1, (p.C * p.W + 255) / 256);
            int base = std::max(1, std::min(max_split, (2048 + groups - 1) / groups));
            for (int f = 0; f < 3; ++f) {
                const int split = f == 0 ? std::max(1, base / 2) : f == 1 ? base : std::min(max_split, base * 2);
                if (f > 0 && split == (f == 1 ? std::max(1, base / 2) : base))
                    continue;
                for (int stage = 0; stage <= 1; ++stage) {
                    if (stage && bitmap > 128 * 1024)
                        continue;
                    if ((p.S + sb - 1) / sb > 65535)
                        continue;
                    RouteCfg rc;
                    rc.samples_per_block = sb;
                    rc.blocks_per_group = split;
                    rc.stage = stage;
                    rc.lanes = 1;
                    cands.push_back({p.spw, rc});
                }
            }
        }
        // without a router, or several lanes per destination word (the fields
        // above do not apply), once
        RouteCfg rc = def;
        rc.lanes = route_split_lanes();
        cands.push_back({p.spw, rc});
    }
    const uint32_t *base = inputs;
    if (base && p.Cin > 0 && !(flags & RANC_INPUTS_ON_DEVICE)) {
        uint32_t *stage = (uint32_t *)(net->ws + p.off[R_EXT]);
        hipError_t e = hipMemcpyAsync(stage, base, (size_t)p.S * num_ticks * p.Cin * p.W * 4,
                                      hipMemcpyHostToDevice, s);
        if (e != hipSuccess)
            return hip_fail(e, "staging inputs");
        base = stage;
    }
    if (p.Cin == 0)
        base = nullptr;
    drop_graphs(net);
    const bool prof_on = net->prof.on;
    net->prof.on = false;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess)
        e = hipEventCreate(&e1);
    double best = -1.0;
    Cand best_c = cands[0];
    ranc_status st = RANC_OK;
    // (samples per workgroup are those of the tick-by-tick launches; several
    // ticks in one launch run the same for every candidate)
    const bool one_tick = p.path != RANC_PATH_PLAIN;
    for (const Cand &c : cands) {
        if (e != hipSuccess || st != RANC_OK)
            break;
        p.spw = c.spw;
        net->rcfg = c.rc;
        // one untimed pass, then a timed pass, each from the initial state
        e = reset_state(net, s);
        if (e == hipSuccess && (st = queue_ticks(net, base, num_ticks, s, nullptr, one_tick)) == RANC_OK)
            e = reset_state(net, s);
        if (e == hipSuccess && st == RANC_OK)
            e = hipEventRecord(e0, s);
        if (e == hipSuccess && st == RANC_OK && (st = queue_ticks(net, base, num_ticks, s, nullptr, one_tick)) == RANC_OK)
            e = hipEventRecord(e1, s);
        if (e == hipSuccess && st == RANC_OK)
            e = hipEventSynchronize(e1);
        float ms = 0.f;
        if (e == hipSuccess && st == RANC_OK)
            e = hipEventElapsedTime(&ms, e0, e1);
        if (e == hipSuccess && st == RANC_OK && (best < 0 || ms < best)) {
            best = ms;
            best_c = c;
        }
    }
    if (e0)
        hipEventDestroy(e0);
    if (e1)
        hipEventDestroy(e1);
    p.spw = best_c.spw;
    net->rcfg = best_c.rc;
    net->prof.on = prof_on;
    if (st != RANC_OK || e != hipSuccess)
        net->slots_unsure = true;
    if (st != RANC_OK)
        return st;
    if (e == hipSuccess)
        e = reset_state(net, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess)
        return hip_fail(e, "autotuning");
    net->tick = 0;
    net->last_stream = s;
    ++net->version;
    const bool tiled = p.path != RANC_PATH_PLAIN;
    out->samples_per_wg = tiled ? p.spw : 0;
    out->route_samples_per_block = tiled ? 0 : net->rcfg.samples_per_block;
    out->route_split = tiled ? 0 : net->rcfg.blocks_per_group;
    out->route_stage = tiled ? 0 : net->rcfg.stage;
    out->ms_per_tick = best / num_ticks;
    out->candidates = (int32_t)cands.size();
    out->route_lanes_per_word = tiled ? 0 : net->rcfg.lanes;
    return RANC_OK;
}

ranc_status ranc_set_launch_shape(ranc_net *net, const ranc_tune *shape)
{
    if (!net || !shape)
        return fail(RANC_EINVAL, "net or shape is NULL");
    const Plan &p = net->p;
    const int v = shape->samples_per_wg;
    const int cap = p.path == RANC_PATH_SPARSE ? sparse_max_samples_per_wg() : mfma_max_samples_per_wg();
    const bool v_ok = v > 0 && v % 64 == 0 && v <= cap;
    // (a handle below 64 samples that RANC_PATH_AUTO put on the MFMA path also
    // takes the shapes of the plain path, which do nothing there)
    if (p.path != RANC_PATH_PLAIN && (!p.auto_mid || v_ok)) {
        if (!v_ok)
            return fail(RANC_EINVAL, "samples_per_wg %d must be a multiple of 64 in [64, %d]", v, cap);
        drop_graphs(net);
        net->p.spw = v;
        return RANC_OK;
    }
    RouteCfg rc;
    rc.samples_per_block = shape->route_samples_per_block;
    rc.blocks_per_group = shape->route_split;
    rc.stage = shape->route_stage != 0;
    const int sb = rc.samples_per_block;
    if ((sb != 1 && sb != 2 && sb != 4 && sb != 8) || sb * route_dmax(p.D) > 32)
        return fail(RANC_EINVAL, "route_samples_per_block %d unsupported with max delay %d", sb, p.D);
    if (rc.blocks_per_group < 1)
        return fail(RANC_EINVAL, "route_split must be >= 1");
    if (rc.stage && (size_t)p.C * p.NW * 4 * sb > 128 * 1024)
        return fail(RANC_EINVAL, "staged spike bitmaps of %d samples exceed the router's LDS", sb);
    if ((p.S + sb - 1) / sb > 65535)
        return fail(RANC_EINVAL, "too many sample groups for the router grid");
    const int lanes = shape->route_lanes_per_word;
    if (lanes != 0 && lanes != 1 && lanes != route_split_lanes())
        return fail(RANC_EINVAL, "route_lanes_per_word %d must be 0 (automatic), 1 or %d", lanes,
                    route_split_lanes());
    rc.lanes = lanes ? lanes : auto_lanes(net, rc);
    drop_graphs(net);
    if (p.path == RANC_PATH_PLAIN)
        net->rcfg = rc;
    return RANC_OK;
}

ranc_status ranc_get_launch_shape(const ranc_net *net, ranc_tune *out)
{
    if (!net || !out)
        return fail(RANC_EINVAL, "net or out is NULL");
    const bool mf = net->p.path != RANC_PATH_PLAIN;
    out->samples_per_wg = mf ? net->p.spw : 0;
    out->route_samples_per_block = mf ? 0 : net->rcfg.samples_per_block;
    out->route_split = mf ? 0 : net->rcfg.blocks_per_group;
    out->route_stage = mf ? 0 : net->rcfg.stage;
    out->ms_per_tick = 0.0;
    out->candidates = 0;
    out->route_lanes_per_word = mf ? 0 : net->rcfg.lanes;
    return RANC_OK;
}

void ranc_free(ranc_net *net)
{
    if (!net)
        return;
    hipStreamSynchronize(net->last_stream);
    drop_graphs(net);
    if (net->cap_stream)
        hipStreamDestroy(net->cap_stream);
    for (int i = 0; i < ranc_net::BATCH_BRANCHES; ++i) {
        if (net->br_stream[i])
            hipStreamDestroy(net->br_stream[i]);
        if (net->br_join[i])
            hipEventDestroy(net->br_join[i]);
    }
    if (net->br_fork)
        hipEventDestroy(net->br_fork);
    for (auto &e : net->prof.pool) {
        hipEventDestroy(e.a);
        hipEventDestroy(e.b);
    }
    if (net->static_dev >= 0)
        static_ws_release(net->static_dev);
    delete net;
}

}  // extern "C"
