// Host side of libssp: configuration checks, device memory layout inside the
// caller's buffers, launch sequencing, hipGraph capture/replay, and the
// extern "C" entry points declared in include/ssp.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/ssp.h"
#include "ssp_f64.h"
#include "ssp_internal.h"
#include "ssp_schedule.h"

using namespace ssp;

namespace {

thread_local std::string g_create_error;
thread_local std::string g_create_warning;

// Sec. 3.1 caps the hop probabilities at 1/2, the construction probability
// per attempt at 1/2 and the destruction probability at 1; at dt / zeta_s =
// 0.1 (Sec. 4.1) none of them binds.  Above dt / zeta_s = 1/4 a hop
// probability 2 (dt / zeta_s) / (1 + e^{2 q y}) can reach 1/2 for y < 0, and
// the step no longer follows the continuous-time rates it discretises: a
// configuration that large is accepted, with a warning.
std::string cap_warning(const ssp_config& k)
{
    const double h = k.dt / k.zeta_s;
    if (!(h > 0.25)) return std::string();
    char buf[256];
    std::snprintf(buf, sizeof buf,
                  "dt/zeta_s = %.4g > 0.25: the 1/2 caps on the hop probabilities%s%s bind (Sec. 3.1 step map)", h,
                  (h / k.n0 > 0.5) ? ", the construction probability" : "",
                  (h >= 1.0) ? " and the destruction probability" : "");
    return std::string(buf);
}

// Most steps of a launch when the caller names none.  Every launch pays for the
// state read and written, the last units of its queue running out, and the
// correlator's histories and accumulators read and written (400 MB each way at
// 16384 chains): 16384 x 32 with the correlator, 5000 steps: 15.9 ms in five
// launches, 14.3 ms in one.
constexpr int64_t kAutoLaunchSteps = 5000;

// Most slots that ssp_write_state checks on the host: copying so few costs less
// than the check kernel's launches (512 slots: 39 against 44 us a call; 41 000 slots:
// 46 against 43; 2 million 610 against 67).
constexpr int64_t kHostCheckSlots = 16384;

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Chain-to-wavefront mapping of one group of chains: segment width W lanes
// and B beads per lane, W * B >= N for every chain of the group.
struct Mapping {
    int W, B;
};

Mapping default_mapping(int n)
{
    if (n <= 8) return {8, 1};
    if (n <= 16) return {16, 1};
    if (n <= 32) return {32, 1};
    if (n <= 64) return {64, 1};
    return {64, 2};
}

// Mappings by number: 1 or 2 beads in 8, 16, 32 or 64 lanes, in the order of the groups.
constexpr int kMappingKinds = 8;
uint8_t mapping_kind(Mapping m) { return (uint8_t)(2 * (__builtin_ctz((unsigned)m.W) - 3) + m.B - 1); }
Mapping mapping_of_kind(int k) { return {8 << (k / 2), k % 2 + 1}; }

bool mapping_supported(int W, int B)
{
    if (B == 1) return W == 8 || W == 16 || W == 32 || W == 64;
    if (B == 2) return W == 16 || W == 32 || W == 64;
    return false;
}

struct Layout {
    // work buffer offsets (bytes)
    size_t ctrl, flags, off, n, elem, gid, tasks, elem_off, thr, samples, hist, acc, pend, acc_v, pend_v, batch,
        series, corr_out, sched, pairs, packed, packed_chains, tables, total;
    size_t host_begin, host_end;  // the tables that creation fills: off .. tables
    // state buffer offsets
    size_t r0, r1, a0, a1, s, state_total;
    int64_t q_cap;
    int32_t chunk;
};

struct Resolved {
    ssp_config cfg;
    std::vector<int32_t> N;
    std::vector<int32_t> elem_off;
    int64_t total_beads = 0;
};

bool resolve(const ssp_config* c, Resolved& r, std::string& err)
{
    if (!c) {
        err = "null config";
        return false;
    }
    r.cfg = *c;
    const ssp_config& k = r.cfg;
    if (k.n_chains < 1) {
        err = "n_chains must be >= 1";
        return false;
    }
    if (k.n_chains > (int64_t)INT32_MAX) {
        err = "n_chains must fit in int32";
        return false;
    }
    if (k.n_elements < 1 || k.n_elements > k.n_chains) {
        err = "n_elements must be in 1..n_chains";
        return false;
    }
    if (k.precision != SSP_FP32 && k.precision != SSP_FP64) {
        err = "precision must be SSP_FP32 or SSP_FP64";
        return false;
    }
    if (!(k.dt > 0.0) || !(k.n0 > 0.0) || !(k.ns > 0.0) || !(k.zeta_s > 0.0) || !std::isfinite(k.dt) ||
        !std::isfinite(k.ns) || !std::isfinite(k.zeta_s)) {
        err = "dt, n0, ns and zeta_s must be positive and finite";
        return false;
    }
    if (k.sample_every < 1) {
        err = "sample_every must be >= 1";
        return false;
    }
    if (k.corr_levels < 0 || k.corr_levels > kMaxCorrLevels) {
        err = "corr_levels must be in 0..16";
        return false;
    }
    if (k.corr_levels > 0 && k.corr_lags != kCorrLags) {
        err = "corr_lags must be 16";
        return false;
    }
    if (k.corr_levels > 0 && (k.corr_batches < 1 || k.corr_batches > 64 || k.corr_batches > k.n_chains)) {
        err = "corr_batches must be in 1..min(64, n_chains)";
        return false;
    }
    if (k.series_capacity < 0) {
        err = "series_capacity must be >= 0";
        return false;
    }
    if (k.max_steps_per_launch < 0) {
        err = "max_steps_per_launch must be >= 0";
        return false;
    }
    if (k.construct_rule != 0 && k.construct_rule != 1) {
        err = "construct_rule must be 0 (K = C - Z) or 1 (K = 1)";
        return false;
    }
    if (k.corr_virtual != 0 && k.corr_virtual != 1) {
        err = "corr_virtual must be 0 or 1";
        return false;
    }
    const int64_t M = k.n_chains;
    r.N.resize(M);
    for (int64_t i = 0; i < M; ++i) {
        const int32_t n = k.n_beads_host ? k.n_beads_host[i] : k.n_beads;
        if (n < 2 || n > SSP_MAX_BEADS) {
            err = "every chain needs 2 <= N <= 128 beads (chain " + std::to_string(i) + ")";
            return false;
        }
        r.N[i] = n;
        r.total_beads += n;
    }
    r.elem_off.resize(k.n_elements + 1);
    if (k.element_offsets_host) {
        for (int e = 0; e <= k.n_elements; ++e) r.elem_off[e] = k.element_offsets_host[e];
        if (r.elem_off[0] != 0 || r.elem_off[k.n_elements] != M) {
            err = "element_offsets must start at 0 and end at n_chains";
            return false;
        }
        for (int e = 0; e < k.n_elements; ++e)
            if (r.elem_off[e + 1] <= r.elem_off[e]) {
                err = "element_offsets must be strictly increasing";
                return false;
            }
    } else {
        for (int e = 0; e <= k.n_elements; ++e) r.elem_off[e] = (int32_t)(M * e / k.n_elements);
        for (int e = 0; e < k.n_elements; ++e)
            if (r.elem_off[e + 1] <= r.elem_off[e]) {
                err = "empty element in equal split";
                return false;
            }
    }
    for (int64_t i = 0; k.chain_ids_host && i < M; ++i)
        if (k.chain_ids_host[i] < 0 || k.chain_ids_host[i] > (int64_t)UINT32_MAX) {
            err = "chain ids must be in 0..2^32-1";
            return false;
        }
    return true;
}

Layout make_layout(const Resolved& r)
{
    const ssp_config& k = r.cfg;
    const int64_t M = k.n_chains;
    Layout L{};
    // steps per launch: bounded so that the per-launch sample buffer stays below
    // about 1 GiB (12 FP64 values per chain and sample).
    int32_t chunk = k.max_steps_per_launch;
    if (chunk == 0) {
        const double per_sample = (double)M * kSampleValues * 8.0;
        int64_t max_q = (int64_t)std::max(1.0, std::floor((1024.0 * 1024.0 * 1024.0) / per_sample));
        int64_t c = std::min<int64_t>(kAutoLaunchSteps, max_q * k.sample_every);
        chunk = (int32_t)std::max<int64_t>(1, c);
    }
    L.chunk = chunk;
    L.q_cap = chunk / k.sample_every + 1;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    L.ctrl = take(sizeof(int64_t) * kCtrlWords);
    L.flags = take(sizeof(uint32_t));
    L.host_begin = o;
    L.off = take(sizeof(int64_t) * M);
    L.n = take(sizeof(int32_t) * M);
    L.elem = take(sizeof(int32_t) * M);
    L.gid = take(sizeof(uint32_t) * M);
    L.tasks = take(sizeof(int32_t) * M);
    L.elem_off = take(sizeof(int32_t) * (k.n_elements + 1));
    L.thr = take(sizeof(uint32_t) * 2 * (kMaxBeads + 1));
    L.tables = take(k.precision == SSP_FP64 ? sizeof(F64Tables) : 0);
    L.host_end = o;
    L.samples = take(sizeof(double) * (size_t)L.q_cap * M * kSampleValues);
    const int lv = k.corr_levels;
    L.hist = take(lv ? sizeof(double) * (size_t)lv * 3 * M * 16 : 0);
    L.acc = take(lv ? sizeof(double) * (size_t)lv * 3 * M * 16 : 0);
    L.pend = take(lv ? sizeof(double) * (size_t)3 * M * 16 * 2 : 0);
    const bool cv = lv && k.corr_virtual;
    L.acc_v = take(cv ? sizeof(double) * (size_t)lv * 3 * M * 16 : 0);
    L.pend_v = take(cv ? sizeof(double) * (size_t)3 * M * 16 : 0);
    L.batch = take(lv ? sizeof(double) * (size_t)k.corr_batches * lv * 16 : 0);
    L.corr_out = take(lv ? sizeof(double) * (size_t)lv * 16 * 2 : 0);
    // persistent schedule: per mapping group a counter and a word per wave task
    // (at most M + 8 words), zeroed as (M + 17) / 2 doubles
    L.sched = take(sizeof(uint32_t) * (size_t)(M + 18));
    L.series = take(sizeof(double) * (size_t)k.n_elements * k.series_capacity * 6);
    L.pairs = take(sizeof(double) * 2 * kSampleValues * (size_t)std::max(k.n_elements, kMeanParts));  // element means
    L.packed = take(sizeof(PackedWave) * (size_t)M);
    L.packed_chains = take(sizeof(int32_t) * (size_t)M);
    L.total = o;
    const size_t beads = (size_t)r.total_beads;
    const size_t v4 = k.precision == SSP_FP32 ? 16 : 32;
    o = 0;
    L.r0 = take(v4 * beads);
    L.r1 = k.precision == SSP_FP32 ? take(v4 * beads) : 0;
    L.a0 = take(v4 * beads);
    L.a1 = k.precision == SSP_FP32 ? take(v4 * beads) : 0;
    L.s = take(sizeof(int32_t) * beads);
    L.state_total = o;
    return L;
}

// Chains packed side by side into wavefronts of 64 lanes with B beads per lane,
// every wavefront's of one element: the longest chain left, then the longest
// that still fits, again and again.  Chains marked in `apart` are left out; the
// others take `lanes`.
struct Packing {
    std::vector<PackedWave> waves;
    std::vector<int32_t> chains;  // of the wavefronts, then the wave tasks of the chains that keep their segments
};
void pack_elements(const Resolved& r, int B, int64_t lanes, const std::vector<char>& apart, Packing& p)
{
    p.waves.clear();
    p.chains.clear();
    p.waves.reserve((size_t)(lanes / kWaveSize * 5 / 4));  // (a fifth of the lanes idle, or more room is taken)
    p.chains.reserve(r.N.size());
    std::vector<int32_t> sorted;  // an element's chains, by the lanes they take
    auto lanes_of = [&](int32_t i) { return (r.N[i] + B - 1) >> (B - 1); };
    for (size_t e = 0; e + 1 < r.elem_off.size(); ++e) {
        const int32_t lo = r.elem_off[e], hi = r.elem_off[e + 1];
        int32_t count[kWaveSize + 1] = {}, next[kWaveSize + 1];
        uint64_t left = 0;  // bit l - 1: some chain of l lanes is left
        for (int32_t i = lo; i < hi; ++i)
            if (!apart[i]) {
                const int l = lanes_of(i);
                ++count[l];
                left |= 1ull << (l - 1);
            }
        int32_t at = 0;
        for (uint64_t m = left; m; m &= m - 1) {
            const int l = __builtin_ctzll(m) + 1;
            next[l] = at;
            at += count[l];
        }
        sorted.resize(at);
        for (int32_t i = lo; i < hi; ++i)
            if (!apart[i]) sorted[next[lanes_of(i)]++] = i;
        for (uint64_t m = left; m; m &= m - 1) {
            const int l = __builtin_ctzll(m) + 1;
            next[l] -= count[l];
        }
        while (left) {
            PackedWave w{0, (uint32_t)p.chains.size(), 0};
            int start = 0;
            uint64_t fits = left;
            for (int c = 0; c < kMaxPacked && fits; ++c) {
                const int l = kWaveSize - __builtin_clzll(fits);
                w.starts |= 1ull << start;
                p.chains.push_back(sorted[next[l]++]);
                if (--count[l] == 0) left &= ~(1ull << (l - 1));
                start += l;
                fits = start < kWaveSize ? left & (~0ull >> start) : 0;
            }
            p.waves.push_back(w);
        }
    }
}

// Integer form of u < p for u = ((w >> 9) + 1/2) 2^-23: (w >> 9) < ceil(p 2^23 - 1/2).
uint32_t threshold(double p)
{
    const double x = std::ceil(p * 8388608.0 - 0.5);
    if (x <= 0.0) return 0u;
    if (x >= 8388608.0) return 8388608u;
    return (uint32_t)x;
}

}  // namespace

struct ssp_handle {
    Resolved res;
    Layout lay;
    int device = 0;
    char* state = nullptr;
    char* work = nullptr;
    using Groups = std::vector<std::pair<Mapping, std::pair<int64_t, int64_t>>>;  // mapping, [task begin, count)
    Groups groups;
    std::vector<uint8_t> chain_map;                                       // mapping of every chain (mapping_kind)
    int packed_B = 0;           // the packed wavefronts' beads per lane (0: none)
    bool set_mapping = false;   // some chain has another mapping than its default: no packing
    int64_t packed_waves = 0;
    Groups packed_groups;       // the packed chains, and the groups of those that keep their segments
    // last recorded window (adjoint)
    struct {
        const void* ptr = nullptr;
        int64_t window = 0, g0 = 0;
        int32_t ckpt = 0;
        bool stored = false;  // the forward stored the trajectory (one segment)
    } rec;
    int cus = 0;            // compute units of the device
    int32_t n_max = 0;      // longest chain
    int64_t n_largest = 0;  // chains of the largest element
    bool initialized = false;
    int64_t steps = 0, corr_samples = 0, series_samples = 0;
    hipStream_t capture_stream = nullptr;
    // Streams for the step kernels of the second and later mapping groups, and
    // the events that fork them from the caller's stream and join them to it.
    std::vector<hipStream_t> side;
    std::vector<hipEvent_t> joined;
    hipEvent_t forked = nullptr;
    std::map<std::pair<int64_t, const double*>, hipGraphExec_t> graphs;
    std::string err;
    std::string warning;  // set at creation (cap_warning)
    bool persistent = true;  // plain steps run the persistent schedule (ssp_set_schedule)
    // device address of the static scratch of the allocation-free reverse
    // pass, looked up at creation (null if the lookup failed; hipError kept)
    double* noalloc = nullptr;
    hipError_t noalloc_err = hipSuccess;
    // kernel timing mode: events bracket every step-kernel launch
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
    double timed_ms = 0.0;
    int64_t timed_launches = 0, timed_bead_steps = 0;

    State st() const
    {
        State s;
        s.r0 = state + lay.r0;
        s.r1 = lay.r1 ? state + lay.r1 : nullptr;
        s.a0 = state + lay.a0;
        s.a1 = lay.a1 ? state + lay.a1 : nullptr;
        if (res.cfg.precision == SSP_FP64) {
            s.r1 = nullptr;
            s.a1 = nullptr;
        }
        s.s = reinterpret_cast<int32_t*>(state + lay.s);
        return s;
    }
    ChainTables ct() const
    {
        ChainTables c;
        c.off = reinterpret_cast<const int64_t*>(work + lay.off);
        c.n = reinterpret_cast<const int32_t*>(work + lay.n);
        c.elem = reinterpret_cast<const int32_t*>(work + lay.elem);
        c.gid = reinterpret_cast<const uint32_t*>(work + lay.gid);
        return c;
    }
    int64_t* ctrl() const { return reinterpret_cast<int64_t*>(work + lay.ctrl); }
    uint32_t* flags() const { return reinterpret_cast<uint32_t*>(work + lay.flags); }
    double* samples() const { return reinterpret_cast<double*>(work + lay.samples); }
    double n_mean() const { return (double)res.total_beads / (double)res.cfg.n_chains; }
    double* pairs() const { return reinterpret_cast<double*>(work + lay.pairs); }
    const int32_t* elem_offsets() const { return reinterpret_cast<const int32_t*>(work + lay.elem_off); }
    bool packs() const { return packed_B != 0 && !set_mapping; }
    const F64Tables* tables() const
    {
        return res.cfg.precision == SSP_FP64 ? reinterpret_cast<const F64Tables*>(work + lay.tables) : nullptr;
    }
    Physics phys() const
    {
        Physics p;
        p.dt = res.cfg.dt;
        p.n0 = res.cfg.n0;
        p.ns = res.cfg.ns;
        p.zeta_s = res.cfg.zeta_s;
        p.key0 = (uint32_t)(res.cfg.seed & 0xffffffffu);
        p.key1 = (uint32_t)(res.cfg.seed >> 32);
        return p;
    }
    StepConsts consts() const
    {
        const ssp_config& k = res.cfg;
        const bool f32 = k.precision == SSP_FP32;  // base-2 logarithm and exponential
        const double sd = std::sqrt(2.0 * k.dt), q = 3.0 / (4.0 * k.ns);
        StepConsts c;
        c.noise = (f32 ? -2.0 * M_LN2 : -2.0) * sd * sd;
        c.bond = 3.0 * k.dt;
        c.spring = 3.0 / k.ns * k.dt;
        c.hop_h2 = 2.0 * k.dt / k.zeta_s;
        c.hop_e2q = f32 ? 2.0 * q * M_LOG2E : 2.0 * q;
        c.anchor = std::sqrt(k.ns / 3.0);
        c.stress = 3.0 / k.ns;
        return c;
    }
};

namespace {

int fail(ssp_handle* h, int code, const std::string& msg)
{
    if (h) h->err = msg;
    return code;
}

#define HIPCHK(h, expr)                                                                                   \
    do {                                                                                                  \
        hipError_t e_ = (expr);                                                                           \
        if (e_ != hipSuccess) return fail((h), SSP_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

// ck_end (optional): where the last launch also writes the final state.
// Outputs of a storing forward (see StepArgs).
struct StoreOut {
    void* traj = nullptr;
    void* traj2 = nullptr;
    void* dlog = nullptr;
    int64_t* dcnt = nullptr;
    int32_t dcap = 0;
};

// Side streams and events for every mapping group after the first; made with
// the groups, so that a step under a caller's capture only records.
int make_sides(ssp_handle* h)
{
    const size_t count = std::max(h->groups.size(), h->packed_groups.size()) - 1;
    if (count && !h->forked) HIPCHK(h, hipEventCreateWithFlags(&h->forked, hipEventDisableTiming));
    while (h->side.size() < count) {
        hipStream_t st = nullptr;
        HIPCHK(h, hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
        h->side.push_back(st);
    }
    while (h->joined.size() < count) {
        hipEvent_t e = nullptr;
        HIPCHK(h, hipEventCreateWithFlags(&e, hipEventDisableTiming));
        h->joined.push_back(e);
    }
    return SSP_OK;
}

int64_t wave_tasks(const std::pair<Mapping, std::pair<int64_t, int64_t>>& g)
{
    const int64_t cpw = kWaveSize / g.first.W;
    return (g.second.second + cpw - 1) / cpw;
}

// The forms of a plain launch's groups, the packed chains first; the result as
// choose_step_forms has it.
constexpr int kMaxGroups = kMappingKinds + 1;
int step_forms(const ssp_handle* h, const ssp_handle::Groups& groups, bool packed, StepGroup (&forms)[kMaxGroups])
{
    for (size_t i = 0; i < groups.size(); ++i)
        forms[i] = {groups[i].first.B, wave_tasks(groups[i]), packed && i == 0, false};
    return choose_step_forms(h->res.cfg.precision == SSP_FP64, h->cus, forms, (int)groups.size());
}

int enqueue_steps(ssp_handle* h, int64_t n, const double* kappa, hipStream_t s, int8_t* rec_s = nullptr,
                  int64_t rec_g0 = 0, const State* ck_end = nullptr, const StoreOut* out = nullptr)
{
    const ssp_config& k = h->res.cfg;
    const int64_t M = k.n_chains;
    for (int64_t done = 0; done < n;) {
        // launches of equal length, none above the limit
        const int64_t left = n - done, launches = (left + h->lay.chunk - 1) / h->lay.chunk;
        const int32_t m = (int32_t)((left + launches - 1) / launches);
        // a plain step (nothing recorded or stored) runs the persistent schedule
        const bool persistent = !rec_s && !ck_end && !out && h->persistent;
        uint32_t* sched = reinterpret_cast<uint32_t*>(h->work + h->lay.sched);
        const bool packed = persistent && h->packs();
        const auto& groups = packed ? h->packed_groups : h->groups;
        StepGroup forms[kMaxGroups];
        const int per_cu = step_forms(h, groups, packed, forms);
        bool queued = false;  // some group takes its units from the queue
        for (size_t i = 0; i < groups.size(); ++i) queued |= persistent && !forms[i].low_latency;
        if (queued) HIPCHK(h, launch_zero(reinterpret_cast<double*>(sched), (M + 16 + 1) / 2, s));
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (h->timing) {
            HIPCHK(h, hipEventCreate(&e0));
            HIPCHK(h, hipEventCreate(&e1));
            HIPCHK(h, hipEventRecord(e0, s));
        }
        // The mapping groups step disjoint chains: with several, each runs on a
        // stream of its own between the same two points of the caller's stream
        // (parallel branches of a captured graph), so that small groups, each
        // bound by its own latency, do not queue up behind each other.
        // (65536 chains of 16..128 beads, 500 steps: 24.5 -> 23.7 ms; 1000 such
        // chains, 300 steps: 2.32 -> 1.09; 256: 2.25 -> 0.75.)
        // Packed chains are one group of their own, the first (launched last:
        // 65536 chains of 16..128 beads 1.4 % slower).
        const size_t sides = groups.size() - 1;
        if (sides) HIPCHK(h, hipEventRecord(h->forked, s));
        // (a launch that fails is reported after the join, so that the caller's
        // stream is ordered after the groups already launched)
        hipError_t launched = hipSuccess;
        for (auto& g : groups) {
            const size_t which = &g - groups.data();
            const hipStream_t gs = which ? h->side[which - 1] : s;
            if (which) HIPCHK(h, hipStreamWaitEvent(gs, h->forked, 0));
            StepArgs a{};
            if (persistent) {  // each group's counter and progress words after the previous group's
                const bool pk = packed && !which;
                a.n_wave_tasks = pk ? h->packed_waves : wave_tasks(g);
                if (pk) {
                    a.packed = reinterpret_cast<const PackedWave*>(h->work + h->lay.packed);
                    a.packed_chains = reinterpret_cast<const int32_t*>(h->work + h->lay.packed_chains);
                }
                a.sched = sched;
                a.low_latency = forms[which].low_latency ? per_cu : 0;
                sched += 1 + a.n_wave_tasks;
                a.chunk = m;  // the launcher picks the chunk length
            }
            a.st = h->st();
            a.ct = h->ct();
            a.tasks = reinterpret_cast<const int32_t*>(h->work + (packed ? h->lay.packed_chains : h->lay.tasks)) + g.second.first;
            a.n_tasks = g.second.second;
            a.kappa = kappa;
            a.thr = reinterpret_cast<const uint32_t*>(h->work + h->lay.thr);
            a.thr_destroy = threshold(std::min(k.dt / k.zeta_s * 1.0, 1.0));
            a.construct_rule = k.construct_rule;
            a.ph = h->phys();
            a.cs = h->consts();
            a.tables = h->tables();
            a.ctrl = h->ctrl();
            a.n_steps = m;
            a.sample_every = k.sample_every;
            a.samples = h->samples();
            a.n_chains = M;
            a.flags = h->flags();
            a.rec_s = rec_s;
            a.rec_g0 = rec_g0;
            if (ck_end && done + m == n) a.ck_end = *ck_end;
            if (out) {
                a.traj = out->traj;
                a.traj2 = out->traj2;
                a.dlog = out->dlog;
                a.dcnt = out->dcnt;
                a.dcap = out->dcap;
            }
            a.total = h->res.total_beads;
            if (launched == hipSuccess) launched = launch_step(k.precision, g.first.W, g.first.B, a, gs);
            if (which) HIPCHK(h, hipEventRecord(h->joined[which - 1], gs));
        }
        for (size_t i = 0; i < sides; ++i) HIPCHK(h, hipStreamWaitEvent(s, h->joined[i], 0));
        HIPCHK(h, launched);
        if (h->timing) {
            HIPCHK(h, hipEventRecord(e1, s));
            h->events.push_back({e0, e1});
            h->timed_bead_steps += h->res.total_beads * (int64_t)m;
        }
        if (k.corr_levels > 0) {
            CorrArgs c{};
            c.samples = h->samples();
            c.hist = reinterpret_cast<double*>(h->work + h->lay.hist);
            c.acc = reinterpret_cast<double*>(h->work + h->lay.acc);
            c.pend = reinterpret_cast<double*>(h->work + h->lay.pend);
            if (k.corr_virtual) {
                c.acc_v = reinterpret_cast<double*>(h->work + h->lay.acc_v);
                c.pend_v = reinterpret_cast<double*>(h->work + h->lay.pend_v);
            }
            c.n_chains = M;
            c.levels = k.corr_levels;
            c.n_steps = m;
            c.sample_every = k.sample_every;
            c.ctrl = h->ctrl();
            HIPCHK(h, launch_corr(c, s));
        }
        if (k.series_capacity > 0) {
            HIPCHK(h, launch_series(h->samples(), reinterpret_cast<const int32_t*>(h->work + h->lay.elem_off),
                                    k.n_elements, M, m, k.sample_every, h->lay.q_cap, h->ctrl(),
                                    reinterpret_cast<double*>(h->work + h->lay.series), k.series_capacity, s));
        }
        HIPCHK(h, launch_advance(h->ctrl(), m, k.sample_every, k.series_capacity, h->flags(), s));
        done += m;
    }
    return SSP_OK;
}

int64_t samples_between(int64_t g0, int64_t n, int32_t every) { return (g0 + n) / every - g0 / every; }

// Groups chains by their mapping (chain order kept inside a group) and
// writes the concatenated task list; h->groups receives the ranges.
void group_tasks(ssp_handle* h, int32_t* tasks)
{
    int64_t next[kMappingKinds] = {};
    for (uint8_t k : h->chain_map) ++next[k];
    h->groups.clear();
    int64_t at = 0;
    for (int k = 0; k < kMappingKinds; ++k) {
        const int64_t count = next[k];
        next[k] = at;
        if (count) h->groups.push_back({mapping_of_kind(k), {at, count}});
        at += count;
    }
    for (size_t i = 0; i < h->chain_map.size(); ++i) tasks[next[h->chain_map[i]]++] = (int32_t)i;
}

// Packs the chains when that is the faster way for plain steps.  In units of a
// wavefront with one bead per lane, a wavefront with two takes kTwoBeads, and a
// packed one kPackedCost times its kind (its chains' lengths and addresses are
// per lane, not scalar).  Below kPackedMinWaves the low-latency form and groups
// side by side are the faster way.  Apart -> packed, 300 steps: 65536 chains of
// 16..128 beads in flow (500 steps) 23.8 -> 19.0 ms, 3000 of them (2750
// wavefronts apart) 1.32 -> 0.94; 65536 x 20 at rest 3.42 -> 2.65, 6000 x 20 (3000
// wavefronts) 0.49 -> 0.45; 65536 x 10 under shear 1.95 -> 1.56; 32768 x 20 FP64 3.84 ->
// 2.93; where lanes are full or waves too few: 40 x 16384 the same, and 1000 chains
// of 16..128 stay apart.
// In FP32 the wavefronts of the segments that hold chains of several elements stay
// as they are, in groups of their own: under flow a row of kappa that any chain
// of a wavefront has renormalises the (hi, lo) pairs of all its flowing anchors,
// and with other neighbours a bead in some 10^6 would differ by a rounding.
void choose_packing(ssp_handle* h, const int32_t* tasks, const int32_t* elem, Packing& p)
{
    const bool f32 = h->res.cfg.precision == SSP_FP32;
    const double kTwoBeads = f32 ? 1.9 : 2.7, kPackedCost = 1.08;
    constexpr int64_t kPackedMinWaves = 2560;
    double now = 0.0;
    int64_t waves = 0;
    for (auto& g : h->groups) {
        const int64_t cpw = kWaveSize / g.first.W, w = (g.second.second + cpw - 1) / cpw;
        waves += w;
        now += (double)w * (g.first.B == 2 ? kTwoBeads : 1.0);
    }
    h->packed_B = 0;
    if (waves < kPackedMinWaves) return;
    const int B = h->n_max > kWaveSize ? 2 : 1;
    // the lanes taken and the elements give the fewest wavefronts possible: worth the
    // packing at all?
    int64_t lanes = 0;
    for (int32_t n : h->res.N) lanes += (n + B - 1) >> (B - 1);
    const double unit = kPackedCost * (B == 2 ? kTwoBeads : 1.0);
    if (unit * (double)lanes / kWaveSize > 0.95 * now) return;
    if (!f32 && unit * h->res.cfg.n_elements > 0.95 * now) return;
    std::vector<char> apart(h->res.N.size(), 0);
    ssp_handle::Groups rest;
    std::vector<int32_t> rest_tasks;
    double rest_cost = 0.0;
    if (f32 && h->res.cfg.n_elements > 1) {
        for (auto& g : h->groups) {
            const int64_t cpw = kWaveSize / g.first.W, end = g.second.first + g.second.second;
            const int64_t from = (int64_t)rest_tasks.size();
            for (int64_t t = g.second.first; t < end; t += cpw) {
                const int64_t to = std::min(t + cpw, end);
                if (elem[tasks[t]] == elem[tasks[to - 1]]) continue;
                rest_tasks.insert(rest_tasks.end(), tasks + t, tasks + to);
                for (int64_t q = t; q < to; ++q) lanes -= (h->res.N[tasks[q]] + B - 1) / B;
                rest_cost += g.first.B == 2 ? kTwoBeads : 1.0;
            }
            const int64_t count = (int64_t)rest_tasks.size() - from;
            if (count) rest.push_back({g.first, {from, count}});
        }
        if (unit * (double)lanes / kWaveSize + rest_cost > 0.95 * now) return;
        for (int32_t i : rest_tasks) apart[i] = 1;
    }
    pack_elements(h->res, B, lanes, apart, p);
    if (p.waves.empty() || (double)p.waves.size() * unit + rest_cost > 0.95 * now) return;
    const int64_t in = (int64_t)p.chains.size();
    h->packed_B = B;
    h->packed_waves = (int64_t)p.waves.size();
    h->packed_groups = {{{kWaveSize, B}, {0, in}}};
    for (auto& g : rest) h->packed_groups.push_back({g.first, {in + g.second.first, g.second.second}});
    p.chains.insert(p.chains.end(), rest_tasks.begin(), rest_tasks.end());
}

int flag_error(ssp_handle* h, uint32_t f)
{
    if (f & kFlagNonFinite) return fail(h, SSP_ENONFINITE, "a non-finite bead position was produced");
    if (f & kFlagInternal) return fail(h, SSP_EHIP, "internal error: slip-spring force gather did not complete");
    return SSP_OK;
}

int check_flags(ssp_handle* h, hipStream_t s)
{
    uint32_t f = 0;
    HIPCHK(h, hipMemcpyAsync(&f, h->flags(), sizeof(f), hipMemcpyDeviceToHost, s));
    HIPCHK(h, hipStreamSynchronize(s));
    return flag_error(h, f);
}

int zero_observables(ssp_handle* h, hipStream_t s)
{
    const ssp_config& k = h->res.cfg;
    const int64_t M = k.n_chains;
    if (k.corr_levels > 0) {
        HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.hist), (int64_t)k.corr_levels * 3 * M * 16, s));
        HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.acc), (int64_t)k.corr_levels * 3 * M * 16, s));
        HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.pend), 3 * M * 16 * 2, s));
        if (k.corr_virtual) {
            HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.acc_v), (int64_t)k.corr_levels * 3 * M * 16, s));
            HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.pend_v), 3 * M * 16, s));
        }
    }
    if (k.series_capacity > 0)
        HIPCHK(h, launch_zero(reinterpret_cast<double*>(h->work + h->lay.series),
                              (int64_t)k.n_elements * k.series_capacity * 6, s));
    HIPCHK(h, launch_zero_ctrl_obs(h->ctrl(), s));
    h->corr_samples = 0;
    h->series_samples = 0;
    return SSP_OK;
}

// Runs a body that takes host memory: no exception may cross the C boundary.
template <typename F> int guarded(std::string& err, F body) noexcept
{
    try {
        return body();
    } catch (...) {
        try {
            err = "out of host memory";
        } catch (...) {
        }
        return SSP_EINVAL;
    }
}

// Frees a handle and what it holds; its device is current.
void release(ssp_handle* h)
{
    for (auto& ev : h->events) {
        (void)hipEventDestroy(ev.first);
        (void)hipEventDestroy(ev.second);
    }
    for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    if (h->capture_stream) (void)hipStreamDestroy(h->capture_stream);
    for (auto st : h->side) (void)hipStreamDestroy(st);
    for (auto ev : h->joined) (void)hipEventDestroy(ev);
    if (h->forked) (void)hipEventDestroy(h->forked);
    delete h;
}

// Fills a new handle and its part of the work buffer; what it holds on an error is
// released by the caller.
int fill_handle(ssp_handle* h, const ssp_config* cfg, void* state_dev, void* work_dev)
{
    if (!resolve(cfg, h->res, g_create_error)) {
        return SSP_EINVAL;
    }
    h->warning = cap_warning(h->res.cfg);
    g_create_warning = h->warning;
    h->res.cfg.n_beads_host = nullptr;
    h->res.cfg.element_offsets_host = nullptr;
    h->res.cfg.chain_ids_host = nullptr;  // (the caller's list is read below)
    h->lay = make_layout(h->res);
    h->state = static_cast<char*>(state_dev);
    h->work = static_cast<char*>(work_dev);
    if (hipGetDevice(&h->device) != hipSuccess ||
        hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess) {
        g_create_error = "reading the device's properties failed";
        return SSP_EHIP;
    }
    h->noalloc_err = noalloc_scratch(h->device, &h->noalloc);
    const int64_t M = h->res.cfg.n_chains;
    // the tables, built in one host copy of their part of the work buffer
    const Layout& L = h->lay;
    const std::unique_ptr<char[]> host(new (std::nothrow) char[L.host_end - L.host_begin]);
    if (!host) {
        g_create_error = "out of host memory";
        return SSP_EINVAL;
    }
    auto table = [&](size_t at, auto type) { return reinterpret_cast<decltype(type)*>(host.get() + (at - L.host_begin)); };
    int64_t* off = table(L.off, int64_t());
    int32_t* n = table(L.n, int32_t());
    int32_t* elem = table(L.elem, int32_t());
    uint32_t* gid = table(L.gid, uint32_t());
    int32_t* tasks = table(L.tasks, int32_t());
    uint32_t* thr = table(L.thr, uint32_t());
    const ssp_config& k = h->res.cfg;
    h->chain_map.resize(M);
    int64_t o = 0;
    for (int64_t i = 0; i < M; ++i) {
        n[i] = h->res.N[i];
        off[i] = o;
        o += n[i];
        gid[i] = (uint32_t)(cfg->chain_ids_host ? cfg->chain_ids_host[i] : i);
        h->n_max = std::max(h->n_max, n[i]);
        h->chain_map[i] = mapping_kind(default_mapping(n[i]));
    }
    for (int e = 0; e < k.n_elements; ++e) {
        std::fill(elem + h->res.elem_off[e], elem + h->res.elem_off[e + 1], e);
        h->n_largest = std::max<int64_t>(h->n_largest, h->res.elem_off[e + 1] - h->res.elem_off[e]);
    }
    std::copy(h->res.elem_off.begin(), h->res.elem_off.end(), table(L.elem_off, int32_t()));
    group_tasks(h, tasks);
    Packing packing;
    choose_packing(h, tasks, elem, packing);
    thr[0] = thr[kMaxBeads + 1] = 0u;
    for (int K = 1; K <= kMaxBeads; ++K) {
        double p = k.dt / (k.zeta_s * k.n0 * (double)K);
        if (p > 0.5) p = 0.5;
        thr[K] = threshold(p);
        thr[kMaxBeads + 1 + K] = threshold(2.0 * p);
    }
    if (k.precision == SSP_FP64) {
        static const F64Tables f64 = [] {
            F64Tables t;
            make_f64_tables(t);
            return t;
        }();
        *table(L.tables, F64Tables()) = f64;
    }
    auto up = [&](size_t at, const void* src, size_t bytes) {
        return hipMemcpy(h->work + at, src, bytes, hipMemcpyHostToDevice);
    };
    if (up(L.host_begin, host.get(), L.host_end - L.host_begin) != hipSuccess ||
        (h->packed_B &&
         (up(L.packed, packing.waves.data(), sizeof(PackedWave) * packing.waves.size()) != hipSuccess ||
          up(L.packed_chains, packing.chains.data(), sizeof(int32_t) * packing.chains.size()) != hipSuccess))) {
        g_create_error = "copying the chain tables to the device failed";
        return SSP_EHIP;
    }
    if (hipStreamCreateWithFlags(&h->capture_stream, hipStreamNonBlocking) != hipSuccess) {
        g_create_error = "hipStreamCreateWithFlags failed";
        return SSP_EHIP;
    }
    if (make_sides(h) != SSP_OK) {
        g_create_error = h->err;
        return SSP_EHIP;
    }
    return SSP_OK;
}

}  // namespace

extern "C" {

int ssp_config_init(ssp_config* c)
{
    if (!c) return SSP_EINVAL;
    std::memset(c, 0, sizeof(*c));
    c->n_chains = 1;
    c->n_elements = 1;
    c->precision = SSP_FP32;
    c->n_beads = 8;
    c->sample_every = 1;
    c->dt = 0.01;
    c->n0 = 4.0;
    c->ns = 0.5;
    c->zeta_s = 0.1;
    c->seed = 1;
    c->corr_levels = 16;
    c->corr_lags = 16;
    c->corr_batches = 16;
    c->series_capacity = 0;
    c->use_graph = 1;
    c->construct_rule = 0;
    c->corr_virtual = 0;
    return SSP_OK;
}

int ssp_query_sizes(const ssp_config* cfg, size_t* state_bytes, size_t* work_bytes)
{
    return guarded(g_create_error, [&]() -> int {
        Resolved r;
        g_create_warning.clear();
        if (!resolve(cfg, r, g_create_error)) return SSP_EINVAL;
        g_create_warning = cap_warning(r.cfg);
        if (cfg->corr_levels > 0 && cfg->corr_batches > cfg->n_chains) {
            g_create_error = "corr_batches exceeds n_chains";
            return SSP_EINVAL;
        }
        const Layout L = make_layout(r);
        if (state_bytes) *state_bytes = L.state_total;
        if (work_bytes) *work_bytes = L.total;
        return SSP_OK;
    });
}

int ssp_create(const ssp_config* cfg, void* state_dev, void* work_dev, ssp_handle** out)
{
    if (!out) {
        g_create_error = "null output handle";
        return SSP_EINVAL;
    }
    *out = nullptr;
    if (!state_dev || !work_dev) {
        g_create_error = "state and work buffers are required";
        return SSP_EINVAL;
    }
    if ((reinterpret_cast<uintptr_t>(state_dev) % kAlign) || (reinterpret_cast<uintptr_t>(work_dev) % kAlign)) {
        g_create_error = "state and work buffers must be 256-byte aligned";
        return SSP_EINVAL;
    }
    ssp_handle* h = new (std::nothrow) ssp_handle();
    if (!h) {
        g_create_error = "out of host memory";
        return SSP_EINVAL;
    }
    const int rc = guarded(g_create_error, [&] { return fill_handle(h, cfg, state_dev, work_dev); });
    if (rc != SSP_OK) {
        release(h);
        return rc;
    }
    *out = h;
    return SSP_OK;
}

int ssp_init_equilibrium(ssp_handle* h, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    HIPCHK(h, launch_reset_ctrl(h->ctrl(), h->flags(), s));
    HIPCHK(h, launch_init(h->res.cfg.precision, h->st(), h->ct(), h->res.cfg.n_chains, h->phys(), s));
    int rc = zero_observables(h, s);
    if (rc) return rc;
    h->steps = 0;
    h->initialized = true;
    return SSP_OK;
}

int ssp_step(ssp_handle* h, int64_t n_steps, const double* kappa_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!h->initialized) return fail(h, SSP_ESTATE, "ssp_step before ssp_init_equilibrium");
    if (n_steps < 0) return fail(h, SSP_EINVAL, "n_steps must be >= 0");
    if (n_steps == 0) return SSP_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    if (h->res.cfg.use_graph && !h->timing) {
        const auto key = std::make_pair(n_steps, kappa_dev);
        auto it = h->graphs.find(key);
        if (it == h->graphs.end()) {
            hipGraph_t graph = nullptr;
            HIPCHK(h, hipStreamBeginCapture(h->capture_stream, hipStreamCaptureModeRelaxed));
            int rc = enqueue_steps(h, n_steps, kappa_dev, h->capture_stream);
            hipError_t ec = hipStreamEndCapture(h->capture_stream, &graph);
            if (rc) return rc;
            if (ec != hipSuccess) return fail(h, SSP_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(ec));
            hipGraphExec_t exec = nullptr;
            ec = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (ec != hipSuccess) return fail(h, SSP_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(ec));
            it = h->graphs.emplace(key, exec).first;
        }
        HIPCHK(h, hipGraphLaunch(it->second, s));
    } else {
        int rc = enqueue_steps(h, n_steps, kappa_dev, s);
        if (rc) return rc;
    }
    const int64_t q = samples_between(h->steps, n_steps, h->res.cfg.sample_every);
    h->steps += n_steps;
    h->corr_samples += q;
    h->series_samples += q;
    return SSP_OK;
}

int ssp_read_stress(ssp_handle* h, double* out_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!h->initialized) return fail(h, SSP_ESTATE, "read before ssp_init_equilibrium");
    if (!out_dev) return fail(h, SSP_EINVAL, "out_dev is required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    HIPCHK(h, launch_stress(h->res.cfg.precision, h->st(), h->ct(), h->res.cfg.n_chains, h->n_mean(), h->res.cfg.ns, out_dev, s));
    return check_flags(h, s);
}

int ssp_read_element_stress(ssp_handle* h, double* out_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!h->initialized) return fail(h, SSP_ESTATE, "read before ssp_init_equilibrium");
    if (!out_dev) return fail(h, SSP_EINVAL, "out_dev is required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    const ssp_config& k = h->res.cfg;
    HIPCHK(h, launch_element_stress(k.precision, h->st(), h->ct(), h->n_mean(), k.ns, h->elem_offsets(), k.n_elements,
                                    h->n_largest, out_dev, h->pairs(), h->flags(), s));
    return check_flags(h, s);
}

int ssp_read_state(ssp_handle* h, double* R_dev, double* A_dev, int32_t* S_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!R_dev || !A_dev || !S_dev) return fail(h, SSP_EINVAL, "R_dev, A_dev and S_dev are required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    HIPCHK(h, launch_read_state(h->res.cfg.precision, h->st(), h->res.total_beads, R_dev, A_dev, S_dev, s));
    return check_flags(h, s);
}

int ssp_write_state(ssp_handle* h, const double* R_dev, const double* A_dev, const int32_t* S_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!R_dev || !A_dev || !S_dev) return fail(h, SSP_EINVAL, "R_dev, A_dev and S_dev are required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    // validate S: it must name a bead of its own chain or be -1
    const int64_t M = h->res.cfg.n_chains;
    int64_t bad = 0;
    if (h->res.total_beads <= kHostCheckSlots) {
        std::vector<int32_t> S(h->res.total_beads);
        HIPCHK(h, hipMemcpyAsync(S.data(), S_dev, sizeof(int32_t) * S.size(), hipMemcpyDeviceToHost, s));
        HIPCHK(h, hipStreamSynchronize(s));
        auto slot = S.begin();
        for (bool ok = true; bad < M; ++bad) {
            const int32_t n = h->res.N[bad];
            for (int32_t j = 0; j < n; ++j, ++slot) ok &= *slot >= -1 && *slot < n;
            if (!ok) break;
        }
    } else {
        int64_t* word = h->ctrl() + kCtrlCheck;
        HIPCHK(h, launch_check_slots(h->ct(), M, S_dev, word, s));
        HIPCHK(h, hipMemcpyAsync(&bad, word, sizeof(bad), hipMemcpyDeviceToHost, s));
        HIPCHK(h, hipStreamSynchronize(s));
    }
    if (bad < M) return fail(h, SSP_EINVAL, "S out of range in chain " + std::to_string(bad));
    if (!h->initialized) {
        HIPCHK(h, launch_reset_ctrl(h->ctrl(), h->flags(), s));
        int rc = zero_observables(h, s);
        if (rc) return rc;
        h->steps = 0;
    }
    HIPCHK(h, launch_write_state(h->res.cfg.precision, h->st(), h->res.total_beads, R_dev, A_dev, S_dev, s));
    h->initialized = true;
    return SSP_OK;
}

int ssp_read_element_series(ssp_handle* h, double* out_dev, int64_t* n_samples_host, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    const ssp_config& k = h->res.cfg;
    if (k.series_capacity == 0) return fail(h, SSP_ESTATE, "element series disabled (series_capacity = 0)");
    if (!out_dev) return fail(h, SSP_EINVAL, "out_dev is required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    HIPCHK(h, hipMemcpyAsync(out_dev, h->work + h->lay.series, sizeof(double) * k.n_elements * k.series_capacity * 6,
                             hipMemcpyDeviceToDevice, s));
    if (n_samples_host) *n_samples_host = std::min(h->series_samples, k.series_capacity);
    return check_flags(h, s);
}

int ssp_read_correlator(ssp_handle* h, double* G_dev, double* G_err_dev, double* tau_host, int64_t* counts_host,
                        ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    const ssp_config& k = h->res.cfg;
    if (k.corr_levels == 0) return fail(h, SSP_ESTATE, "correlator disabled (corr_levels = 0)");
    if (!G_dev || !G_err_dev) return fail(h, SSP_EINVAL, "G_dev and G_err_dev are required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    double* batch = reinterpret_cast<double*>(h->work + h->lay.batch);
    HIPCHK(h, launch_corr_batches(reinterpret_cast<const double*>(h->work + h->lay.acc), k.n_chains, k.corr_levels,
                                  k.corr_batches, batch, s));
    HIPCHK(h, launch_corr_final(batch, k.n_chains, k.corr_levels, k.corr_batches, h->corr_samples, G_dev, G_err_dev, s));
    for (int l = 0; l < k.corr_levels; ++l)
        for (int q = 0; q < 16; ++q) {
            const int64_t len = h->corr_samples >> l;
            if (tau_host) tau_host[l * 16 + q] = (double)q * std::ldexp(1.0, l) * k.sample_every * k.dt;
            if (counts_host) counts_host[l * 16 + q] = len > q ? len - q : 0;
        }
    return check_flags(h, s);
}

int ssp_read_correlator_virtual(ssp_handle* h, double* Gv_dev, double* Gv_err_dev, double* dGv_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    const ssp_config& k = h->res.cfg;
    if (k.corr_levels == 0 || !k.corr_virtual)
        return fail(h, SSP_ESTATE, "virtual-stress correlator disabled (corr_levels = 0 or corr_virtual = 0)");
    if (!Gv_dev || !Gv_err_dev) return fail(h, SSP_EINVAL, "Gv_dev and Gv_err_dev are required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    double* batch = reinterpret_cast<double*>(h->work + h->lay.batch);
    HIPCHK(h, launch_corr_batches(reinterpret_cast<const double*>(h->work + h->lay.acc_v), k.n_chains, k.corr_levels,
                                  k.corr_batches, batch, s));
    HIPCHK(h, launch_corr_final(batch, k.n_chains, k.corr_levels, k.corr_batches, h->corr_samples, Gv_dev, Gv_err_dev,
                                s));
    if (dGv_dev) {
        // G(t) of the same samples into the handle's own output area, then Gv / G
        double* G = reinterpret_cast<double*>(h->work + h->lay.corr_out);
        HIPCHK(h, launch_corr_batches(reinterpret_cast<const double*>(h->work + h->lay.acc), k.n_chains, k.corr_levels,
                                      k.corr_batches, batch, s));
        HIPCHK(h, launch_corr_final(batch, k.n_chains, k.corr_levels, k.corr_batches, h->corr_samples, G,
                                    G + (size_t)k.corr_levels * 16, s));
        HIPCHK(h, launch_grid_ratio(Gv_dev, G, k.corr_levels, h->corr_samples, dGv_dev, s));
    }
    return check_flags(h, s);
}

int ssp_linear_viscoelasticity(ssp_handle* h, const double* G_dev, const double* omega_dev, int32_t n_omega,
                               double t_lo, double t_hi, double* moduli_dev, double* scalars_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    const ssp_config& k = h->res.cfg;
    if (k.corr_levels == 0) return fail(h, SSP_ESTATE, "correlator disabled (corr_levels = 0)");
    if (!G_dev || !scalars_dev) return fail(h, SSP_EINVAL, "G_dev and scalars_dev are required");
    if (n_omega < 0) return fail(h, SSP_EINVAL, "n_omega must be >= 0");
    if (n_omega > 0 && (!omega_dev || !moduli_dev)) return fail(h, SSP_EINVAL, "omega_dev and moduli_dev are required");
    if (!(t_lo <= t_hi)) return fail(h, SSP_EINVAL, "t_lo must not exceed t_hi");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    HIPCHK(h, launch_moduli(G_dev, k.corr_levels, h->corr_samples, k.sample_every * k.dt, omega_dev, n_omega, t_lo, t_hi,
                            moduli_dev, scalars_dev, s));
    return SSP_OK;
}

int ssp_reset_observables(ssp_handle* h, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    return zero_observables(h, s);
}

int ssp_step_count(const ssp_handle* h, int64_t* steps_host)
{
    if (!h || !steps_host) return SSP_EINVAL;
    *steps_host = h->steps;
    return SSP_OK;
}

int ssp_rng_normals(ssp_handle* h, int64_t chain_id, int64_t step, int32_t bead, int32_t count, double* out_dev,
                    ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!out_dev || count < 0 || bead < 0 || bead + (int64_t)count > 65536 || chain_id < 0 ||
        chain_id > (int64_t)UINT32_MAX || step < 0)
        return fail(h, SSP_EINVAL, "invalid ssp_rng_normals arguments");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    const Physics p = h->phys();
    HIPCHK(h, launch_rng_normals(h->res.cfg.precision, h->tables(), p.key0, p.key1, (uint32_t)chain_id, step, bead, count,
                                 out_dev, s));
    return SSP_OK;
}

}  // extern "C"

namespace {

// Regions of a recording buffer: slot rows, checkpoints, replay state and
// control words, segment trajectory, carried adjoint.
struct RecLayout {
    size_t rows, ckpts, ctrl, traj, traj2, dlog, dcnt, lam, total;
    int n_seg;
    int32_t dcap;  // stored window: destruction-log entries per chain
};

// Destruction-log capacity per chain for a stored window.  Destructions are
// at most the initial springs (<= N) plus the creations; creations per step
// have mean K 2 p_K <= 2 dt/(zeta_s N0) under either construction rule (each
// of K attempts creates with probability 2 p_K, p_K = min{dt/(zeta_s N0 K),
// 1/2}; or K attempts when p_K is clamped, K < 2 dt/(zeta_s N0)).  The
// capacity adds 8 standard deviations of a Poisson count of that mean, plus
// 16; a chain that still overflows is reported by ssp_adjoint.
int32_t destruction_log_capacity(const ssp_handle* h, int64_t window)
{
    const ssp_config& k = h->res.cfg;
    const double mean = (double)window * 2.0 * k.dt / (k.zeta_s * k.n0);
    int32_t nmax = 0;
    for (int32_t v : h->res.N) nmax = std::max(nmax, v);
    const double cap = nmax + std::ceil(mean + 8.0 * std::sqrt(mean)) + 16.0;
    return (int32_t)std::min(cap, 1.0e9);
}

RecLayout rec_layout(const ssp_handle* h, int64_t window, int32_t ckpt)
{
    RecLayout L{};
    const size_t beads = (size_t)h->res.total_beads;
    const size_t t = h->res.cfg.precision == SSP_FP32 ? 4 : 8;
    L.n_seg = (int)((window + ckpt - 1) / ckpt);
    const size_t seg = (size_t)std::min<int64_t>(ckpt, window);  // steps of the longest segment
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    L.rows = take((size_t)(window + 1) * beads);
    L.ckpts = take((size_t)L.n_seg * h->lay.state_total);
    L.ctrl = take(sizeof(int64_t) * kCtrlWords);
    const bool store = L.n_seg == 1;  // the forward stores the window's trajectory
    L.traj = take((seg + 1) * beads * 3 * t);
    L.traj2 = take((store ? 1 : seg + 1) * beads * 3 * t);
    L.dcap = store ? destruction_log_capacity(h, window) : 0;
    L.dlog = take((size_t)h->res.cfg.n_chains * (size_t)L.dcap * 3 * t);
    L.dcnt = take(store ? sizeof(int64_t) * (size_t)h->res.cfg.n_chains : 0);
    L.lam = take(beads * 6 * t);
    L.total = o;
    return L;
}

State state_at(const ssp_handle* h, char* base)
{
    State s;
    s.r0 = base + h->lay.r0;
    s.r1 = h->res.cfg.precision == SSP_FP32 ? base + h->lay.r1 : nullptr;
    s.a0 = base + h->lay.a0;
    s.a1 = h->res.cfg.precision == SSP_FP32 ? base + h->lay.a1 : nullptr;
    s.s = reinterpret_cast<int32_t*>(base + h->lay.s);
    return s;
}

}  // namespace

extern "C" {

int ssp_adjoint_bytes(const ssp_handle* h, int64_t window, int32_t ckpt_every, size_t* bytes)
{
    if (!h || !bytes || window < 1 || ckpt_every < 1) return SSP_EINVAL;
    *bytes = rec_layout(h, window, ckpt_every).total;
    return SSP_OK;
}

int ssp_forward_record(ssp_handle* h, int64_t window, int32_t ckpt_every, const double* kappa_dev, void* rec_dev,
                       ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!h->initialized) return fail(h, SSP_ESTATE, "ssp_forward_record before ssp_init_equilibrium");
    if (window < 1 || ckpt_every < 1 || !rec_dev)
        return fail(h, SSP_EINVAL, "window >= 1, ckpt_every >= 1 and rec_dev are required");
    if (reinterpret_cast<uintptr_t>(rec_dev) % kAlign) return fail(h, SSP_EINVAL, "rec_dev must be 256-byte aligned");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    const RecLayout R = rec_layout(h, window, ckpt_every);
    char* rec = static_cast<char*>(rec_dev);
    int8_t* rows = reinterpret_cast<int8_t*>(rec + R.rows);
    const int64_t g0 = h->steps;
    HIPCHK(h, launch_rec_s0(h->st().s, rows, h->res.total_beads, s));
    // A one-segment window stores its trajectory as it runs, and the reverse
    // pass starts from that.  Otherwise checkpoint 0 is a copy of the state,
    // each segment's last launch writes the next checkpoint from its
    // epilogue, and the reverse pass replays each segment from its checkpoint.
    const bool store = R.n_seg == 1;
    StoreOut so;
    if (store) {
        so.traj = rec + R.traj;
        so.traj2 = rec + R.traj2;
        so.dlog = rec + R.dlog;
        so.dcnt = reinterpret_cast<int64_t*>(rec + R.dcnt);
        so.dcap = R.dcap;
        HIPCHK(h, launch_zero(reinterpret_cast<double*>(so.dcnt), h->res.cfg.n_chains, s));  // all-zero bits: 0
    } else {
        HIPCHK(h, launch_copy_bytes(rec + R.ckpts, h->state, h->lay.state_total, s));
    }
    h->rec.ptr = nullptr;  // not a usable recording until the window is complete
    for (int c = 0; c < R.n_seg; ++c) {
        const int64_t m = std::min<int64_t>(ckpt_every, window - (int64_t)c * ckpt_every);
        const State next = state_at(h, rec + R.ckpts + (size_t)(c + 1) * h->lay.state_total);
        int rc = enqueue_steps(h, m, kappa_dev, s, rows, g0, c + 1 < R.n_seg ? &next : nullptr,
                               store ? &so : nullptr);
        if (rc) return rc;
        const int64_t q = samples_between(h->steps, m, h->res.cfg.sample_every);
        h->steps += m;
        h->corr_samples += q;
        h->series_samples += q;
    }
    h->rec.ptr = rec_dev;
    h->rec.window = window;
    h->rec.ckpt = ckpt_every;
    h->rec.g0 = g0;
    h->rec.stored = store;
    return SSP_OK;
}

}  // extern "C"

namespace {

// The reverse pass of ssp_adjoint: per-chain gradients into grad_dev [M][10] and,
// with elem_grad_dev, their element means.  Nothing is in flight when it returns.
int adjoint_pass(ssp_handle* h, const void* rec_dev, const double* kappa_dev, int32_t component, int32_t init_window,
                 double* grad_dev, double* elem_grad_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!rec_dev || rec_dev != h->rec.ptr) return fail(h, SSP_ESTATE, "rec_dev does not hold the last recorded window");
    if (!grad_dev || component < 0 || component > 5)
        return fail(h, SSP_EINVAL, "grad_dev and component 0..5 are required");
    hipStream_t s = static_cast<hipStream_t>(stream);
    HIPCHK(h, hipSetDevice(h->device));
    const ssp_config& k = h->res.cfg;
    const RecLayout R = rec_layout(h, h->rec.window, h->rec.ckpt);
    char* rec = static_cast<char*>(const_cast<void*>(rec_dev));
    const int8_t* rows = reinterpret_cast<const int8_t*>(rec + R.rows);
    int64_t* sctrl = reinterpret_cast<int64_t*>(rec + R.ctrl);
    HIPCHK(h, launch_zero(grad_dev, k.n_chains * 10, s));
    for (int c = R.n_seg - 1; c >= 0; --c) {
        const int64_t m = std::min<int64_t>(h->rec.ckpt, h->rec.window - (int64_t)c * h->rec.ckpt);
        // replay the segment from its checkpoint (read in place, left as it
        // is), storing the trajectory; a one-segment window has it from the
        // forward
        if (!h->rec.stored) {
            HIPCHK(h, launch_set_ctrl_steps(sctrl, h->rec.g0 + (int64_t)c * h->rec.ckpt, s));
            for (auto& g : h->groups) {
                StepArgs a{};
                a.st = state_at(h, rec + R.ckpts + (size_t)c * h->lay.state_total);  // read in place
                a.ct = h->ct();
                a.tasks = reinterpret_cast<const int32_t*>(h->work + h->lay.tasks) + g.second.first;
                a.n_tasks = g.second.second;
                a.kappa = kappa_dev;
                a.thr = reinterpret_cast<const uint32_t*>(h->work + h->lay.thr);
                a.thr_destroy = threshold(std::min(k.dt / k.zeta_s * 1.0, 1.0));
                a.construct_rule = k.construct_rule;
                a.ph = h->phys();
                a.cs = h->consts();
                a.tables = h->tables();
                a.ctrl = sctrl;
                a.n_steps = (int32_t)m;
                a.sample_every = 0;
                a.samples = nullptr;
                a.n_chains = k.n_chains;
                a.flags = h->flags();
                a.total = h->res.total_beads;
                a.traj = rec + R.traj;
                a.traj2 = rec + R.traj2;
                a.replay_s = rows;  // the recorded slot states, replayed
                a.rec_g0 = h->rec.g0;
                HIPCHK(h, launch_step(k.precision, g.first.W, g.first.B, a, s));
            }
        }
        for (auto& g : h->groups) {
            AdjointArgs a{};
            a.ct = h->ct();
            a.tasks = reinterpret_cast<const int32_t*>(h->work + h->lay.tasks) + g.second.first;
            a.n_tasks = g.second.second;
            a.kappa = kappa_dev;
            a.ph = h->phys();
            a.tables = h->tables();
            a.rec_s = rows;
            a.rec_g0 = h->rec.g0;
            a.m0 = (int64_t)c * h->rec.ckpt;
            a.len = (int32_t)m;
            a.traj = rec + R.traj;
            a.traj2 = rec + R.traj2;
            a.lam = rec + R.lam;
            a.grad = grad_dev;
            a.total = h->res.total_beads;
            a.comp = component;
            a.seed_lambda = (c == R.n_seg - 1) ? 1 : 0;
            a.init_terms = (c == 0 && init_window && h->rec.g0 == 0) ? 1 : 0;
            a.flags = h->flags();
            a.stored = h->rec.stored ? 1 : 0;  // a replay checks the rows it re-creates
            a.dlog = rec + R.dlog;
            a.dcnt = reinterpret_cast<const int64_t*>(rec + R.dcnt);
            a.dcap = R.dcap;
            HIPCHK(h, launch_adjoint(k.precision, g.first.W, g.first.B, a, s));
        }
    }
    // (before the flags are read, so that one wait covers both; on an error the
    // means are left unwritten)
    if (elem_grad_dev)
        HIPCHK(h, launch_element_mean(grad_dev, 10, 10, h->elem_offsets(), k.n_elements, h->n_largest, elem_grad_dev,
                                      h->pairs(), h->flags(),
                                      kFlagNonFinite | kFlagInternal | kFlagReplay | kFlagLogOverflow, s));
    // A bad recording leaves the ensemble itself untouched (the replay starts
    // from a checkpoint and writes only the trajectory): report it and clear
    // its flag.
    uint32_t f = 0;
    HIPCHK(h, hipMemcpyAsync(&f, h->flags(), sizeof(f), hipMemcpyDeviceToHost, s));
    HIPCHK(h, hipStreamSynchronize(s));
    if (f & kFlagLogOverflow) {
        f &= ~(uint32_t)(kFlagLogOverflow | kFlagReplay);
        HIPCHK(h, hipMemcpyAsync(h->flags(), &f, sizeof(f), hipMemcpyHostToDevice, s));
        HIPCHK(h, hipStreamSynchronize(s));
        return fail(h, SSP_ESIZE,
                    "a chain destroyed more springs in the stored window than its log holds; gradients are "
                    "invalid (record the window with checkpoints, ckpt_every < window)");
    }
    if (f & kFlagReplay) {
        f &= ~(uint32_t)kFlagReplay;
        HIPCHK(h, hipMemcpyAsync(h->flags(), &f, sizeof(f), hipMemcpyHostToDevice, s));
        HIPCHK(h, hipStreamSynchronize(s));
        return fail(h, SSP_EINVAL,
                    "the recorded slot rows are not a run of this ensemble (recording buffer changed since "
                    "ssp_forward_record, or recorded by another handle); gradients are invalid");
    }
    return flag_error(h, f);
}

}  // namespace

extern "C" {

int ssp_adjoint(ssp_handle* h, const void* rec_dev, const double* kappa_dev, int32_t component, int32_t init_window,
                double* grad_dev, ssp_stream stream)
{
    return adjoint_pass(h, rec_dev, kappa_dev, component, init_window, grad_dev, nullptr, stream);
}

int ssp_adjoint_elements(ssp_handle* h, const void* rec_dev, const double* kappa_dev, int32_t component,
                         int32_t init_window, double* chain_grad_dev, double* elem_grad_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!elem_grad_dev || !chain_grad_dev) return fail(h, SSP_EINVAL, "chain_grad_dev and elem_grad_dev are required");
    return adjoint_pass(h, rec_dev, kappa_dev, component, init_window, chain_grad_dev, elem_grad_dev, stream);
}

int ssp_adjoint_elements_noalloc(ssp_handle* h, const void* rec_dev, const double* kappa_dev, int32_t component,
                                 int32_t init_window, double* elem_grad_dev, ssp_stream stream)
{
    if (!h) return SSP_EINVAL;
    if (!elem_grad_dev) return fail(h, SSP_EINVAL, "elem_grad_dev is required");
    if (h->res.cfg.n_chains > kNoAllocMaxChains)
        return fail(h, SSP_ESIZE, "ssp_adjoint_elements_noalloc handles at most 262144 chains (its static scratch); "
                                  "use ssp_adjoint_elements with a workspace");
    if (!h->noalloc)
        return fail(h, SSP_EHIP, std::string("the static scratch of this device is not available: ") +
                                     hipGetErrorString(h->noalloc_err));
    return adjoint_pass(h, rec_dev, kappa_dev, component, init_window, h->noalloc, elem_grad_dev, stream);
}

int ssp_set_mapping(ssp_handle* h, int32_t n_lo, int32_t n_hi, int32_t lanes_per_chain, int32_t beads_per_lane)
{
    if (!h) return SSP_EINVAL;
    if (n_lo < 2 || n_hi < n_lo || n_hi > SSP_MAX_BEADS) return fail(h, SSP_EINVAL, "need 2 <= n_lo <= n_hi <= 128");
    if (!mapping_supported(lanes_per_chain, beads_per_lane))
        return fail(h, SSP_EINVAL, "unsupported mapping (lanes 8/16/32/64 with 1 bead per lane, 16/32/64 with 2)");
    if (lanes_per_chain * beads_per_lane < n_hi)
        return fail(h, SSP_EINVAL, "lanes_per_chain * beads_per_lane must be >= n_hi");
    HIPCHK(h, hipSetDevice(h->device));
    const int64_t M = h->res.cfg.n_chains;
    const uint8_t kind = mapping_kind({lanes_per_chain, beads_per_lane});
    std::vector<int32_t> tasks;
    int rc = guarded(h->err, [&]() -> int {
        tasks.resize(M);
        return SSP_OK;
    });
    if (rc) return rc;
    for (int64_t i = 0; i < M; ++i)
        if (h->res.N[i] >= n_lo && h->res.N[i] <= n_hi) h->chain_map[i] = kind;
    // Chains are packed while all have their default mapping (what tuning finds for
    // most lengths: 2^18 chains of 16..128 beads, 10^4 steps, tuned: 1.88 -> 1.47 s).
    h->set_mapping = false;
    for (int64_t i = 0; i < M && !h->set_mapping; ++i)
        h->set_mapping = h->chain_map[i] != mapping_kind(default_mapping(h->res.N[i]));
    group_tasks(h, tasks.data());
    rc = make_sides(h);
    if (rc) return rc;
    HIPCHK(h, hipDeviceSynchronize());  // no launch may still read the old task list
    HIPCHK(h, hipMemcpy(h->work + h->lay.tasks, tasks.data(), sizeof(int32_t) * M, hipMemcpyHostToDevice));
    for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    h->graphs.clear();
    return SSP_OK;
}

int ssp_step_plan(const ssp_handle* h, int64_t* packed_chains_host, int64_t* packed_wavefronts_host,
                  int64_t* low_latency_chains_host)
{
    if (!h) return SSP_EINVAL;
    int64_t chains = 0, waves = 0, low_latency = 0;
    if (h->persistent) {
        const bool packed = h->packs();
        const auto& groups = packed ? h->packed_groups : h->groups;
        if (packed) {
            chains = groups[0].second.second;
            waves = h->packed_waves;
        }
        StepGroup forms[kMaxGroups];
        (void)step_forms(h, groups, packed, forms);
        for (size_t i = 0; i < groups.size(); ++i)
            if (forms[i].low_latency) low_latency += groups[i].second.second;
    }
    if (packed_chains_host) *packed_chains_host = chains;
    if (packed_wavefronts_host) *packed_wavefronts_host = waves;
    if (low_latency_chains_host) *low_latency_chains_host = low_latency;
    return SSP_OK;
}

int ssp_set_schedule(ssp_handle* h, int persistent)
{
    if (!h) return SSP_EINVAL;
    if ((persistent != 0) != h->persistent) {
        HIPCHK(h, hipSetDevice(h->device));
        HIPCHK(h, hipDeviceSynchronize());
        for (auto& kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
        h->graphs.clear();
        h->persistent = persistent != 0;
    }
    return SSP_OK;
}

int ssp_set_kernel_timing(ssp_handle* h, int enable)
{
    if (!h) return SSP_EINVAL;
    h->timing = enable != 0;
    return SSP_OK;
}

int ssp_kernel_time(ssp_handle* h, double* ms_host, int64_t* launches_host, int64_t* bead_steps_host)
{
    if (!h) return SSP_EINVAL;
    HIPCHK(h, hipSetDevice(h->device));
    for (auto& ev : h->events) {
        HIPCHK(h, hipEventSynchronize(ev.second));
        float ms = 0.f;
        HIPCHK(h, hipEventElapsedTime(&ms, ev.first, ev.second));
        h->timed_ms += ms;
        ++h->timed_launches;
        (void)hipEventDestroy(ev.first);
        (void)hipEventDestroy(ev.second);
    }
    h->events.clear();
    if (ms_host) *ms_host = h->timed_ms;
    if (launches_host) *launches_host = h->timed_launches;
    if (bead_steps_host) *bead_steps_host = h->timed_bead_steps;
    h->timed_ms = 0.0;
    h->timed_launches = 0;
    h->timed_bead_steps = 0;
    return SSP_OK;
}

int ssp_destroy(ssp_handle* h)
{
    if (!h) return SSP_OK;
    (void)hipSetDevice(h->device);
    release(h);
    return SSP_OK;
}

const char* ssp_last_error(const ssp_handle* h) { return h ? h->err.c_str() : g_create_error.c_str(); }

const char* ssp_warning(const ssp_handle* h)
{
    const std::string& w = h ? h->warning : g_create_warning;
    return w.empty() ? nullptr : w.c_str();
}

}  // extern "C"
