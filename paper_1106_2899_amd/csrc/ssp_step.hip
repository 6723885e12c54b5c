// The slip-spring ensemble step (three-substep scheme of Sec. 3.1 with the
// K = C - Z reconstruction of Sec. 3.2), one persistent launch for n steps.
//
// Mapping: a wavefront holds 64 / W chains; chain c of the wave owns the
// lane segment [W c, W c + W).  Lane li of a segment owns beads and slots
// li*B .. li*B + B - 1 (slot capacity C = N, one slot per bead).  The whole
// chain state stays in VGPRs for the n steps; it is read from HBM once at
// launch start and written once at the end.
//
// Cross-lane data paths:
//   - neighbour bonds: DPP wave shifts (VALU, no LDS traffic);
//   - per-bead records {R hi, R lo, bond right, bond left} are staged in a
//     wave-private LDS array after the move; slots read the record of their
//     bead for the hop, for new anchors and for the anchor offsets;
//   - the slot -> bead force scatter is a deterministic gather: every spring
//     sets its slot's bit in its bead's LDS mask and each bead adds the
//     offsets d of its set bits (read from LDS) in increasing slot order; no
//     float atomics, so runs are bitwise reproducible;
//   - stress sums: every lane writes its FP64 partial sums to LDS and the
//     lanes of the segment add one column each in lane order (deterministic).
//
// Per step, in the paper's order:
//   1. forces at time t: bond forces and slip-spring forces,
//   2. Euler-Maruyama move of beads and affine advection of anchors,
//   3. hops decided from the post-move positions (one uniform per spring),
//   4. destruction at the ends and K = C - Z construction attempts (integer
//      thresholds, identical in every precision),
//   5. anchor offsets recomputed from the stored positions, and the stress /
//      virtual stress of the new state every sample_every steps.
//
// k_replay is the same step with the slot decisions of 3 and 4 read from a
// recording: the adjoint's reverse pass re-creates each checkpoint segment's
// positions with it.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ssp_device.h"
#include "ssp_internal.h"

namespace ssp {

namespace {

template <typename T> struct Vec4 {
    using type = float4;
};
template <> struct Vec4<double> {
    using type = double4;
};

template <typename T> __device__ __forceinline__ v3<T> ld3(const void* base, int64_t idx)
{
    const typename Vec4<T>::type v = reinterpret_cast<const typename Vec4<T>::type*>(base)[idx];
    return {v.x, v.y, v.z};
}
template <typename T> __device__ __forceinline__ void st3(void* base, int64_t idx, v3<T> v)
{
    typename Vec4<T>::type o;
    o.x = v.x;
    o.y = v.y;
    o.z = v.z;
    o.w = T(0);
    reinterpret_cast<typename Vec4<T>::type*>(base)[idx] = o;
}

// Row length of the stress sums in LDS (see the sampling).
constexpr int kSumStride = kWaveSize + 1;

// Per-bead record staged in LDS: R hi, R lo, bond to the right, bond from the left.
template <typename T> struct alignas(16) BeadRec {
    T v[12];
};
template <typename T> struct alignas(16) Off4 {
    T v[4];
};
template <typename T> __device__ __forceinline__ v3<T> unpack3(const Off4<T>& o) { return {o.v[0], o.v[1], o.v[2]}; }

template <typename T>
__device__ __forceinline__ void rec_put(BeadRec<T>& r, v3<T> rh, v3<T> rl, v3<T> br, v3<T> bl)
{
    BeadRec<T> t;
    t.v[0] = rh.x; t.v[1] = rh.y; t.v[2] = rh.z;
    t.v[3] = rl.x; t.v[4] = rl.y; t.v[5] = rl.z;
    t.v[6] = br.x; t.v[7] = br.y; t.v[8] = br.z;
    t.v[9] = bl.x; t.v[10] = bl.y; t.v[11] = bl.z;
    r = t;
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wavefront-ordered LDS accesses of the slot masks.
template <typename M> __device__ __forceinline__ void lmask_store(M* p, M v)
{
    __hip_atomic_store(p, v, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename M> __device__ __forceinline__ M lmask_load(M* p)
{
    return __hip_atomic_load(p, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename M> __device__ __forceinline__ void lmask_or(M* p, M v)
{
    __hip_atomic_fetch_or(p, v, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Index of the lowest set bit, or -1 (all bits set) when there is none, as
// the hardware's find-first-bit gives it.
__device__ __forceinline__ uint32_t first_bit(uint32_t x)
{
    uint32_t r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// The slots of a segment anchored at one bead: bit j of the mask for slot j,
// in 32-bit words.
template <int kCap> struct SlotMask {
    static constexpr int kWords = (kCap + 31) / 32;
    uint32_t w[kWords];

    __device__ __forceinline__ bool any() const
    {
        uint32_t o = 0;
#pragma unroll
        for (int q = 0; q < kWords; ++q) o |= w[q];
        return o != 0;
    }
    // lowest slot in the mask, -1 when it is empty
    __device__ __forceinline__ int lowest() const
    {
        uint32_t r = first_bit(w[0]);
#pragma unroll
        for (int q = 1; q < kWords; ++q) r = min(r, first_bit(w[q]) | (32u * q));  // -1 stays -1
        return (int)r;
    }
    // removes the lowest slot
    __device__ __forceinline__ void drop()
    {
        bool below = true;  // no slot in the words below
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            const uint32_t v = w[q];
            if (q == 0)
                w[q] = v & (v - 1);  // no change when zero
            else
                w[q] = below ? (v & (v - 1)) : v;
            below = below && v == 0;
        }
    }
};

__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0; }

// Ballot bits of the W-lane segment starting at lane sb.
template <int W> __device__ __forceinline__ uint64_t seg_mask(int sb)
{
    if constexpr (W == 64)
        return ~0ull;
    else
        return ((1ull << W) - 1ull) << sb;
}

template <typename T> __device__ __forceinline__ bool finite3(v3<T> v)
{
    return isfinite(v.x) && isfinite(v.y) && isfinite(v.z);
}

// Wave-private LDS: the bead records double as the transpose buffer of the
// stress sums ([12][65] FP64), which is used only after the records of
// a step have been consumed, and as the beads' slot masks of the force
// gather, which is done before the step's records are written.
// SAMP: room for the stress-sample partials (a replay samples nothing, and
// without them its LDS no longer limits the waves per SIMD).
// MASKS: the slot masks have room of their own (they are built while a step's
// records are still read).
template <typename T, int W, int B, bool SAMP, bool MASKS, bool PACKED = false> struct WaveLds {
    static constexpr int kRecBytes = (int)sizeof(BeadRec<T>) * kWaveSize * B;
    static constexpr int kSumBytes = SAMP ? (int)sizeof(double) * kSumStride * kSampleValues : 0;
    static constexpr int kShared = kRecBytes > kSumBytes ? kRecBytes : kSumBytes;
    alignas(16) unsigned char shared[kShared];
    // per segment (chain): a zero entry, then the slots
    Off4<T> off[PACKED ? kWaveSize * B + kMaxPacked : (kWaveSize / W) * (W * B + 1)];
    T kdt[(kWaveSize / W) * 9];                   // per segment: dt kappa (flow variants)
    uint32_t masks[MASKS ? kWaveSize * B * SlotMask<W * B>::kWords : 1];
};

// What the drawing waves hand the stepping wave for one step: the scaled noise
// and the hop uniform of every bead/slot, and the normals of a new anchor with
// the reconstruction word's 23 bits.
template <typename T, int B> struct DrawnStep {
    Off4<T> noise_u[kWaveSize * B];
    Off4<T> anchor_w[kWaveSize * B];
};
template <typename T> using word_of = std::conditional_t<std::is_same<T, float>::value, uint32_t, uint64_t>;
template <typename T> __device__ __forceinline__ T pack_word(uint32_t w) { return __builtin_bit_cast(T, (word_of<T>)w); }
template <typename T> __device__ __forceinline__ uint32_t unpack_word(T v)
{
    return (uint32_t)__builtin_bit_cast(word_of<T>, v);
}

// The step, for the kernels below.  K1: construction by the K = 1 rule (one
// attempt per chain and step, by the lowest empty slot) instead of K = C - Z;
// a template parameter so that neither kernel carries the other rule's work.
// RP: replay of a recorded run: the slot state after each step is read from
// the recorded rows instead of being decided (no hop or construction draws or
// probabilities); positions and anchors follow bit for bit.
// ST: a recorded forward that also stores the trajectory the replay would
// (positions every step, the anchors the adjoint cannot rebuild), so that the
// reverse pass of a one-segment window needs no replay.  Its destroyed-spring
// anchors go to a compact per-chain log instead of a dense plane.
// FL: compiled with the flow terms (a velocity gradient table is given); a
// run at rest (no table) uses the variant without them, whose registers are
// not shared with the flow code.  The two give identical trajectories at
// kappa = 0.
// DW > 0: the low-latency form for launches that leave most of the chip's
// wavefront slots empty: the workgroup is one stepping wave and DW waves that
// draw its random numbers ahead of it (see k_step_pair).
// PK: chains packed side by side in the wavefront's lanes wherever they fit
// (a.packed), instead of one to each segment of W lanes; all of one element.
template <typename T, int W, int B, bool K1, bool RP, bool ST, bool FL, bool PS, int DW, bool PK = false>
__device__ __forceinline__ void step_body()
{
    static_assert(!PK || (PS && W == kWaveSize), "packed wavefronts run the queue's plain steps");
    constexpr bool LL = DW > 0;
    static_assert(!LL || (!RP && !ST && !PS), "the low-latency form runs plain steps only");
    // The launch arguments, read from the kernel argument segment where they
    // are used (scalar loads), instead of a copy held in scalar registers.
    using ArgPtr = const __attribute__((address_space(4))) StepArgs*;
    const ArgPtr kernarg = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const auto& a = *kernarg;
    constexpr bool kComp = std::is_same<T, float>::value;  // (hi, lo) position sums
    constexpr int kChainsPerWave = kWaveSize / W;
    constexpr int kCap = W * B;  // bead capacity of a segment

    __shared__ WaveLds<T, W, B, !RP, LL, PK> lds[LL ? 1 : kWavesPerGroup];
    // two drawn step pairs: one is stepped through while the other is drawn
    __shared__ DrawnStep<T, B> drawn[LL ? 4 : 1];
    // creation thresholds for p_K and 2 p_K, K = 0..kMaxBeads, read every step
    __shared__ uint32_t thr[2 * (kMaxBeads + 1)];
    __shared__ std::conditional_t<kComp, NoTables, F64Tables> tab;
    constexpr int kThreads = LL ? kWaveSize * (1 + DW) : kGroupThreads;
    load_tables(tab, a.tables, threadIdx.x, kThreads);
    for (int q = threadIdx.x; q < 2 * (kMaxBeads + 1); q += kThreads) thr[q] = a.thr[q];
    __syncthreads();

    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wv = wave_uniform((int)(threadIdx.x / kWaveSize));  // (scalar: whole waves branch on it)

    // One unit of work: the chains of wave task `wtask` for n_steps steps from
    // global step g0, their samples from index q0 of the launch's sample
    // buffer on.  State is read from HBM at the start and written back at the
    // end, so units of one wave task may run on different wavefronts.
    auto run = [&](const int64_t wtask, const int64_t g0, const int32_t n_steps, const int64_t q0) {
    int li = lane % W, seg = lane / W, sb = lane - li;  // sb: first lane of the segment
    uint64_t smask = seg_mask<W>(sb);                   // its lanes
    int64_t task = wtask * kChainsPerWave + seg;
    bool valid = task < a.n_tasks;
    int chain = 0;
    if constexpr (PK) {
        const PackedWave pw = {a.packed[wtask].starts, a.packed[wtask].first, 0u};
        const uint64_t upto = ~0ull >> (kWaveSize - 1 - lane);  // lanes up to this one
        const uint64_t next = pw.starts & ~upto;
        seg = __popcll(pw.starts & upto) - 1;
        sb = kWaveSize - 1 - __builtin_clzll(pw.starts & upto);  // (a chain starts at lane 0)
        li = lane - sb;
        smask = ~0ull << sb;
        if (next) smask &= (next & (0ull - next)) - 1ull;
        valid = true;
        chain = a.packed_chains[pw.first + seg];
    } else {
        chain = valid ? a.tasks[task] : 0;
    }
    int n = valid ? a.ct.n[chain] : 0;
    int64_t off = valid ? a.ct.off[chain] : 0;
    uint32_t gid = valid ? a.ct.gid[chain] : 0u;
    int elem = valid ? a.ct.elem[chain] : 0;
    if constexpr (PK) {
        elem = wave_uniform(elem);
    } else if constexpr (W == kWaveSize) {
        // one chain per wavefront: its table entries go to scalar registers,
        // and the addresses built from them stay scalar
        chain = wave_uniform(chain);
        n = wave_uniform(n);
        off = wave_uniform(off);
        gid = wave_uniform(gid);
        elem = wave_uniform(elem);
    }
    BeadRec<T>* rec = reinterpret_cast<BeadRec<T>*>(lds[wv].shared);
    double* sums = reinterpret_cast<double*>(lds[wv].shared);
    const int lbase = PK ? sb * B : seg * kCap;  // this segment's first entry in the LDS arrays
    // this segment's slot offsets: slot j at offs[j], a zero entry at offs[-1]
    Off4<T>* offs = lds[wv].off + lbase + seg + 1;
    if (li == 0) offs[-1] = Off4<T>{};
    constexpr int kMaskWords = SlotMask<kCap>::kWords;
    static_assert(4 * kMaskWords <= (int)sizeof(BeadRec<T>), "the slot masks fit in the records");
    uint32_t* lmask = LL ? lds[wv].masks : reinterpret_cast<uint32_t*>(lds[wv].shared);
    // word w of a bead's mask: the wavefront's words w side by side, so that
    // the lanes' accesses to their own beads fall in distinct banks
    auto mask_at = [&](int bead, int w) { return w * (kWaveSize * B) + lbase + bead; };
    uint32_t mbit[B];  // this lane's slots: their bit and word in a mask
    int mbit_word[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        mbit[b] = 1u << ((li * B + b) % 32);
        mbit_word[b] = (li * B + b) / 32;
    }

    // Step constants (StepConsts), in vector registers: see in_vgpr.  The FP32
    // kernels at rest work them out themselves, which the compiler schedules
    // better there (16384 x 32, 5000 steps: 15.8 against 16.1 ms); those under
    // flow would spill for it (65536 x 32: 11.5 against 11.8 ms per 1000).
    T cnoise, cbond, cspring, hop_h2, hop_e2q, asd;
    double kstress;
    if constexpr (FL || LL || !kComp) {
        cnoise = in_vgpr(T(a.cs.noise));
        cbond = in_vgpr(T(a.cs.bond));
        cspring = in_vgpr(T(a.cs.spring));
        hop_h2 = in_vgpr(T(a.cs.hop_h2));
        hop_e2q = in_vgpr(T(a.cs.hop_e2q));
        asd = T(a.cs.anchor);
        kstress = a.cs.stress;
    } else {
        cnoise = normal_scale<T>(sqrt(2.0 * a.ph.dt));
        cbond = T(3.0 * a.ph.dt);
        cspring = T(3.0 / a.ph.ns * a.ph.dt);
        hop_h2 = T(2.0 * a.ph.dt / a.ph.zeta_s);
        hop_e2q = glauber_exp_scale<T>(3.0 / (4.0 * a.ph.ns));
        asd = T(sqrt(a.ph.ns / 3.0));
        kstress = 3.0 / a.ph.ns;
    }
    uint32_t k0 = a.ph.key0, k1 = a.ph.key1;

    T kdt_v[9];  // dt kappa of the chain's element
    uint32_t kmask = 0;  // entries of kappa that are nonzero in some chain of the wavefront
    bool chain_flow = false;  // this lane's chain has a nonzero kappa
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        kdt_v[q] = T(0);
        if constexpr (FL) {
            const double kq = valid ? a.kappa[9 * elem + q] : 0.0;
            kdt_v[q] = T(a.ph.dt * kq);
            // one chain per wavefront: its element's kappa is wave-uniform
            if constexpr (W == kWaveSize) kdt_v[q] = wave_uniform(kdt_v[q]);
            if (wave_any(kq != 0.0)) kmask |= 1u << q;
            chain_flow |= kq != 0.0;
        }
    }
    const bool flow = FL && kmask != 0;
    // Shape of kappa in this wavefront: simple shear (xy alone) and elongation
    // (the diagonal alone) take straight-line code with their one or three
    // entries in registers; any other pattern tests its entries one by one.
    // Both shapes are what the rheometer flows of the model are made of, and
    // the general form costs 27 scalar branches and a wait on LDS for each
    // entry in use at every step.
    constexpr uint32_t kShearBits = 1u << 1, kDiagBits = (1u << 0) | (1u << 4) | (1u << 8);
    const bool flow_xy = FL && kmask == kShearBits;
    const bool flow_diag = flow && (kmask & ~kDiagBits) == 0u;
    T kfl[3] = {T(0), T(0), T(0)};  // the entries of a shear (one) or a diagonal (three)
    if constexpr (FL) {
        kfl[0] = flow_xy ? kdt_v[1] : kdt_v[0];
        kfl[1] = kdt_v[4];
        kfl[2] = kdt_v[8];
    }
    // elongation (a positive diagonal entry of kappa) stretches chains without
    // bound above the Rouse instability: such chains take the error-free move
    const bool chain_stretch = chain_flow && (kdt_v[0] > T(0) || kdt_v[4] > T(0) || kdt_v[8] > T(0));
    // With several chains per wavefront dt kappa differs between segments:
    // it is kept in LDS (a row per segment) and read where the general flow
    // terms use it, instead of holding nine registers per lane across the steps.
    constexpr bool kKdtLds = FL && W < kWaveSize;
    T* const kdt_lds = lds[wv].kdt + seg * 9;
    if constexpr (kKdtLds) {
        if (li == 0) {
#pragma unroll
            for (int q = 0; q < 9; ++q) kdt_lds[q] = kdt_v[q];
        }
    }
    const T* kdt;
    if constexpr (kKdtLds)
        kdt = kdt_lds;
    else
        kdt = kdt_v;

    v3<T> rh[B], rl[B], ah[B], al[B], d[B], br[B], bl[B];
    int s[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int i = li * B + b;
        const bool act = i < n;
        rh[b] = act ? ld3<T>(a.st.r0, off + i) : zero3<T>();
        ah[b] = act ? ld3<T>(a.st.a0, off + i) : zero3<T>();
        if constexpr (kComp) {
            rl[b] = act ? ld3<T>(a.st.r1, off + i) : zero3<T>();
            al[b] = act ? ld3<T>(a.st.a1, off + i) : zero3<T>();
        } else {
            rl[b] = zero3<T>();
            al[b] = zero3<T>();
        }
        s[b] = act ? a.st.s[off + i] : -1;
    }

    // Bonds to the right neighbour (br) and from the left neighbour (bl) of
    // every bead owned by the lane (zero past the chain ends), then the bead
    // records in LDS.
    auto bonds_and_records = [&]() {
        const v3<T> nh = from_next3(rh[0]);
        const v3<T> nl = from_next3(rl[0]);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = li * B + b;
            const v3<T> h = (b + 1 < B) ? rh[b + 1 < B ? b + 1 : b] : nh;
            const v3<T> l = (b + 1 < B) ? rl[b + 1 < B ? b + 1 : b] : nl;
            const v3<T> v = (h - rh[b]) + (l - rl[b]);  // computed everywhere, then selected
            br[b] = sel(i < n - 1, v, zero3<T>());
        }
        // The bond from the left needs no mask: the lane before the first lane
        // of a segment holds the previous segment's last bead (or is lane 0 of
        // the wave, which DPP fills with 0), and its right bond is zero since
        // it lies at or past that chain's end; past the end of this chain
        // the right bonds are zero as well.
        const v3<T> left = from_prev3(br[B - 1]);
#pragma unroll
        for (int b = 0; b < B; ++b) bl[b] = (b > 0) ? br[b > 0 ? b - 1 : 0] : left;
#pragma unroll
        for (int b = 0; b < B; ++b) rec_put(rec[lbase + li * B + b], rh[b], rl[b], br[b], bl[b]);
        wave_sync();
    };

    // Anchor offsets d_j = R_{S_j} - A_j of the occupied slots, always
    // recomputed from the stored positions (never carried across a step) so
    // that a trajectory does not depend on how steps are split into launches;
    // also staged in LDS for the next force gather.
    auto refresh_offsets = [&]() {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int t = s[b] > 0 ? s[b] : 0;
            const BeadRec<T> r = rec[lbase + t];
            const v3<T> Rh = {r.v[0], r.v[1], r.v[2]};
            const v3<T> Rl = {r.v[3], r.v[4], r.v[5]};
            d[b] = (s[b] >= 0) ? ((Rh - ah[b]) + (Rl - al[b])) : zero3<T>();
            Off4<T> o;
            o.v[0] = d[b].x;
            o.v[1] = d[b].y;
            o.v[2] = d[b].z;
            o.v[3] = T(0);
            offs[li * B + b] = o;
        }
        wave_sync();
    };

    // Slip-spring force, sum of d_j over the springs of each bead in increasing
    // slot order.  Every occupied slot sets its bit in its bead's slot mask (LDS
    // atomics of one wavefront complete in order, so the clearing stores land
    // first); each bead then reads its mask and adds the staged offsets of its
    // set bits lowest first.
    auto read_masks = [&](SlotMask<kCap> (&mw)[B]) {
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int w = 0; w < kMaskWords; ++w) lmask_store(&lmask[mask_at(li * B + b, w)], 0u);
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (s[b] >= 0) lmask_or(&lmask[mask_at(s[b], mbit_word[b])], mbit[b]);
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int w = 0; w < kMaskWords; ++w) mw[b].w[w] = lmask_load(&lmask[mask_at(li * B + b, w)]);
    };
    // The first two springs of every bead (read unconditionally: a missing one
    // reads the zero entry), then the rare beads with more.  The sum is never
    // -0, so adding +0 for a missing spring changes nothing.
    v3<T> acc[B];
    auto gather = [&](SlotMask<kCap> (&mw)[B]) {
        bool more = false;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const v3<T> o0 = unpack3(offs[mw[b].lowest()]);
            mw[b].drop();
            const v3<T> o1 = unpack3(offs[mw[b].lowest()]);
            mw[b].drop();
            acc[b] = (zero3<T>() + o0) + o1;
            more |= mw[b].any();
        }
        if (wave_any(more)) {
            do {
                more = false;
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    if (mw[b].any()) {
                        acc[b] = acc[b] + unpack3(offs[mw[b].lowest()]);
                        mw[b].drop();
                    }
                    more |= mw[b].any();
                }
            } while (wave_any(more));
        }
    };

    bonds_and_records();
    refresh_offsets();
    if constexpr (LL) {
        SlotMask<kCap> mw[B];
        read_masks(mw);
        gather(mw);
    }

    // Trajectory output: R after every step (row 0: the state before the
    // first step), FP32 positions rounded from hi + lo.  Anchors are written
    // only where the adjoint cannot recover them by running the advection
    // backwards: for every slot at the launch end, and for each spring
    // destroyed in a step (a replay: at that step's row; a storing forward:
    // appended to the chain's log).  A replay counts rows from its launch (one
    // segment); a storing forward from the recorded window's start, however
    // the window is split into launches.
    constexpr bool kTraj = RP || ST;
    const int64_t trow0 = RP ? 0 : g0 - a.rec_g0;
    // (the chain's row base and the lane's bead index are kept apart, so that
    // with one chain per wavefront the 64-bit part of the address is scalar)
    auto store_r = [&](int row) {
        T* base = reinterpret_cast<T*>(a.traj) + 3 * ((trow0 + row) * a.total + off);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = li * B + b;
            if (i < n) {  // streamed out once, read back once by the adjoint: non-temporal
                const v3<T> v = rh[b] + rl[b];
                T* q = base + 3u * (uint32_t)i;
                __builtin_nontemporal_store(v.x, q);
                __builtin_nontemporal_store(v.y, q + 1);
                __builtin_nontemporal_store(v.z, q + 2);
            }
        }
    };
    auto store_a = [&](int row, int b) {
        v3<T>* base = reinterpret_cast<v3<T>*>(a.traj2) + ((trow0 + row) * a.total + off);
        base[(uint32_t)(li * B + b)] = ah[b] + al[b];
    };
    if constexpr (kTraj) store_r(0);
    int64_t dcount = 0;  // storing forward: entries in this chain's destruction log
    if constexpr (ST) dcount = valid ? a.dcnt[chain] : 0;
    auto log_destroyed = [&](const bool (&destroyed)[B]) {
        bool any = false;
#pragma unroll
        for (int b = 0; b < B; ++b) any |= destroyed[b];
        if (!wave_any(any)) return;
        // entries of one step in slot order (slot li B + b), whatever the mapping:
        // a slot's rank counts the destroyed slots of lower lanes and its own lower b
        const uint64_t below = (1ull << lane) - 1ull;
        int tot = 0, lower = 0;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const uint64_t m = __ballot(destroyed[b]) & smask;
            tot += __popcll(m);
            lower += __popcll(m & below);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (destroyed[b]) {
                const int64_t q = dcount + lower;
                if (q < a.dcap) reinterpret_cast<v3<T>*>(a.dlog)[(int64_t)chain * a.dcap + q] = ah[b] + al[b];
                ++lower;
            }
        }
        dcount += tot;
    };

    bool finite_ok = true;

    // Random streams come in step pairs (2k, 2k+1), three Philox blocks per
    // bead/slot index and pair (counter step word k):
    //   NOISE  -> Box-Muller pairs (x0,x1), (x2,x3): noise (c, s, c) of step 2k
    //             and the first normal of step 2k+1 (carried);
    //   NOISE2 -> hop / reconstruction words y2, y3 of step 2k; y0, y1 (carried)
    //             make the Box-Muller pair of the other two normals of 2k+1;
    //   SLOT   -> hop / reconstruction words z0, z1 of step 2k+1 (carried).
    // In FP64 the even step draws all three together: they share the first
    // round's products and the round keys in vector registers (philox_blocks),
    // and three independent chains hide each other's latency at 3 waves per
    // SIMD (8191 x 27, 1000 steps: 6.72 -> 5.90 ms).  So does a replay, which
    // needs no SLOT block (65536 x 64, checkpointed gradient of 400 steps: 28.4
    // -> 27.5 ms).  In FP32 each block is drawn where it is needed: NOISE2 and
    // SLOT run while the bead records go through LDS, which the joint draw
    // leaves exposed (16384 x 32 at rest 15.8 against 16.4 ms per 5000 steps).
    // A launch that starts at an odd step draws the pair's blocks in its
    // prologue.
    constexpr bool kJointDraws = RP || !kComp;
    constexpr int kDraws = RP ? 2 : 3;
    T carry_n[B];
    uint32_t carry_w0[B], carry_w1[B], carry_h[B], carry_r[B];
    auto draw_pair = [&](int b, int64_t k, uint4 (&w)[3]) {
        const uint32_t i = (uint32_t)(li * B + b);
        uint4 c[kDraws];
        c[0] = counter(kNoise, i, gid, k);
        c[1] = counter(kNoise2, i, gid, k);
        if constexpr (!RP) c[kDraws - 1] = counter(kSlot, i, gid, k);
        philox_blocks<kDraws>(c, k0, k1);
        w[0] = c[0];
        w[1] = c[1];
        w[2] = c[kDraws - 1];
        carry_w0[b] = c[1].x;
        carry_w1[b] = c[1].y;
        carry_h[b] = w[2].x;
        carry_r[b] = w[2].y;
    };
#pragma unroll
    for (int b = 0; b < B; ++b) {
        carry_n[b] = T(0);
        carry_w0[b] = carry_w1[b] = carry_h[b] = carry_r[b] = 0u;
        if (g0 & 1) {
            uint4 w[3];
            draw_pair(b, g0 >> 1, w);
            T c;
            box_muller(tab, w[0].z, w[0].w, cnoise, c, carry_n[b]);
        }
    }
    // arguments read in the step loop (held: a scalar load there is waited for)
    const uint32_t thr_destroy = a.thr_destroy;
    const int32_t sample_every = RP ? 0 : a.sample_every;  // a replay samples nothing
    int8_t* const rec_s = PS ? nullptr : a.rec_s;
    // sampling phase: step g is sampled when (g + 1) % sample_every == 0
    int phase = sample_every > 0 ? (int)((g0 + 1) % sample_every) : 1;
    // row of the launch's sample buffer that this unit's next sample goes to
    const int64_t sample_row = a.n_chains * kSampleValues;
    double* sample_out = RP ? nullptr : a.samples + q0 * sample_row;

    // Replay: the recorded slot row of a step is loaded one step ahead, so that
    // its latency runs under the previous step.
    int replay_next[B], replay_ahead[B];
    auto replay_load = [&](int64_t gs, int (&dst)[B]) {
        const int8_t* row = a.replay_s + ((gs + 1 - a.rec_g0) * a.total + off);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = li * B + b;
            dst[b] = (j < n) ? (int)row[(uint32_t)j] : -1;
        }
    };
    if constexpr (RP) {
        if (n_steps > 0) replay_load(g0, replay_ahead);
    }

    // Low-latency form: a step's random numbers are read at the end of the step
    // before, behind the barrier that ends a pair's drawing.
    Off4<T> next_noise[B];
    uint32_t next_word[B];
    auto read_drawn = [&](int64_t gs) {
        if (gs == g0 || (gs & 1) == 0) __syncthreads();
        const DrawnStep<T, B>& ds = drawn[(int)(gs & 3)];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            next_noise[b] = ds.noise_u[b * kWaveSize + lane];
            next_word[b] = unpack_word(ds.anchor_w[b * kWaveSize + lane].v[3]);
        }
    };
    if constexpr (LL) read_drawn(g0);

    for (int step = 0; step < n_steps; ++step) {
        // the flow terms test the bits of kmask every step; recomputing those
        // tests (scalar ops) is cheaper than keeping nine hoisted conditions
        // in scalar registers across the loop, which spilled
        if constexpr (FL) asm volatile("" : "+s"(kmask));
        const int64_t g = g0 + step;
        if constexpr (RP) {
#pragma unroll
            for (int b = 0; b < B; ++b) replay_next[b] = replay_ahead[b];
            if (step + 1 < n_steps) replay_load(g + 1, replay_ahead);
        }
        const bool even = (g & 1) == 0;  // wave-uniform
        const int64_t kp = g >> 1;       // step pair: counter step word of the random streams

        // The counts that substep 3 takes from the post-hop state: a hop moves
        // a spring but never fills or frees a slot, so they are those of the
        // state before the step, and the thresholds' LDS reads are issued here.
        int z = 0;
        int first_empty = kCap;  // lowest empty slot of the chain (K = 1 rule)
#pragma unroll
        for (int b = 0; b < B && !RP; ++b) {
            z += __popcll(__ballot(s[b] >= 0) & smask);
            if constexpr (K1) {
                const uint64_t m = __ballot(s[b] < 0 && li * B + b < n) & smask;
                if (m) first_empty = min(first_empty, ((int)__builtin_ctzll(m) - sb) * B + b);
            }
        }
        const int K = K1 ? (z < n ? 1 : 0) : n - z;
        const uint32_t t1 = thr[K < 0 ? 0 : K];
        const uint32_t t2 = thr[kMaxBeads + 1 + (K < 0 ? 0 : K)];

        // ---- substep 1a: slip-spring force.  The mask round trip is issued
        // before the step's noise is computed (it does not depend on it), so
        // that its latency runs under that arithmetic.  The low-latency form
        // gathered at the end of the step before.
        SlotMask<kCap> mw[B];
        if constexpr (!LL) read_masks(mw);

        // ---- substep 1b, first part: sqrt(2 dt) w of this step, and its hop and
        // reconstruction words.
        v3<T> noise[B];
        uint32_t whop[B], wrec[B];
        T uhop[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if constexpr (LL) {  // read at the end of the step before
                noise[b] = unpack3(next_noise[b]);
                uhop[b] = next_noise[b].v[3];
                wrec[b] = next_word[b];
            } else if (even) {
                uint4 w[3];
                if constexpr (kJointDraws)
                    draw_pair(b, kp, w);
                else
                    w[0] = draw(kNoise, (uint32_t)(li * B + b), gid, kp, k0, k1);
                box_muller(tab, w[0].x, w[0].y, cnoise, noise[b].x, noise[b].y);
                box_muller(tab, w[0].z, w[0].w, cnoise, noise[b].z, carry_n[b]);
                if constexpr (kJointDraws) {
                    whop[b] = w[1].z;
                    wrec[b] = w[1].w;
                }
            } else {
                noise[b].x = carry_n[b];
                box_muller(tab, carry_w0[b], carry_w1[b], cnoise, noise[b].y, noise[b].z);
                whop[b] = carry_h[b];
                wrec[b] = carry_r[b];
            }
        }

        // ---- substep 1a, completion.
        if constexpr (!LL) gather(mw);

        // ---- substep 1b: Euler-Maruyama for beads, advection for anchors.
        // FP32 under flow: positions drift and stretch far from the origin
        // while bonds near the chain ends and anchor offsets stay O(1), so the
        // terms of the move that scale with |R| must keep their low bits:
        //  - beads: the flow term takes dt kappa (hi + lo); the low part's
        //    product is small but systematic and would add up over the steps;
        //  - anchors: advected error-free (flow_row, cadd_big); under shear an
        //    anchor's increment dt gamma_dot A_y is the same number every
        //    step, so its rounding error would add up linearly;
        //  - chains under elongation (a positive diagonal entry of kappa),
        //    which stretch to bonds of hundreds: the bead's flow term and its
        //    bond force, taken from the compensated positions, split into a
        //    binary32 value and its exact rounding error (flow_row,
        //    two_prod); the large part enters hi through an exact TwoSum
        //    (cadd_big), so that only O(1) quantities are ever rounded.
        // Which form a chain takes depends only on its own element, and chains
        // without flow keep the plain binary32 step, so trajectories do not
        // depend on the launch split, nor on the mapping but for one thing: a
        // row of kappa that is zero for a flowing chain renormalises its
        // anchors' pairs where another chain of the wavefront has that row,
        // which changes a bead in some 10^6 by a rounding.
        auto plain_inc = [&](int b) {
            v3<T> inc = noise[b];
            inc = fma3(cbond, br[b] - bl[b], inc);
            return fma3(-cspring, acc[b], inc);
        };
        if constexpr (kComp) {
            // (R_{i+1} - R_i) - (R_i - R_{i-1}) of every bead from the compensated
            // parts, and the error-free move of the stretched chains; row(r, h, l,
            // big, small) gives row r of their flow term.
            auto move_stretched = [&](auto&& row) {
                const v3<T> nh = from_next3(rh[0]), nl = from_next3(rl[0]);
                const v3<T> ph = from_prev3(rh[B - 1]), pl = from_prev3(rl[B - 1]);
                v3<T> lap[B];  // every bead reads its in-lane neighbours before any moves
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const int i = li * B + b;
                    const v3<T> h1 = (b + 1 < B) ? rh[b + 1 < B ? b + 1 : b] : nh;
                    const v3<T> l1 = (b + 1 < B) ? rl[b + 1 < B ? b + 1 : b] : nl;
                    const v3<T> h0 = (b > 0) ? rh[b > 0 ? b - 1 : 0] : ph;
                    const v3<T> l0 = (b > 0) ? rl[b > 0 ? b - 1 : 0] : pl;
                    const bool right = i < n - 1, left = i > 0;
                    lap[b] = (sel(right, h1 - rh[b], zero3<T>()) - sel(left, rh[b] - h0, zero3<T>())) +
                             (sel(right, l1 - rl[b], zero3<T>()) - sel(left, rl[b] - l0, zero3<T>()));
                }
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    if (li * B + b < n && chain_stretch) {
                        const v3<T> rest = fma3(-cspring, acc[b], noise[b]);
                        v3<T> big, small;
                        row(std::integral_constant<int, 0>{}, rh[b], rl[b], big.x, small.x);
                        row(std::integral_constant<int, 1>{}, rh[b], rl[b], big.y, small.y);
                        row(std::integral_constant<int, 2>{}, rh[b], rl[b], big.z, small.z);
                        cadd_force(rh[b].x, rl[b].x, big.x, small.x, cbond, lap[b].x, rest.x);
                        cadd_force(rh[b].y, rl[b].y, big.y, small.y, cbond, lap[b].y, rest.y);
                        cadd_force(rh[b].z, rl[b].z, big.z, small.z, cbond, lap[b].z, rest.z);
                    }
                }
            };
            // (wave-uniform tests)
            if (flow_xy) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const T f = fmat(kfl[0], rl[b].y, kfl[0] * rh[b].y);
                    v3<T> inc = plain_inc(b);
                    inc.x = inc.x + f;  // a chain at rest adds zero
                    if (li * B + b < n) cadd3(rh[b], rl[b], inc);
                    if (s[b] >= 0 && chain_flow) {
                        T big, small;
                        flow_entry(kfl[0], ah[b].y, al[b].y, big, small);
                        cadd_big(ah[b].x, al[b].x, big, small);
                    }
                }
            } else if (!flow) {
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (li * B + b < n) cadd3(rh[b], rl[b], plain_inc(b));
            } else if (flow_diag) {
                if (wave_any(chain_stretch))
                    move_stretched([&](auto R, v3<T> h, v3<T> l, T& big, T& small) {
                        constexpr int r = decltype(R)::value;
                        flow_entry(kfl[r], r == 0 ? h.x : (r == 1 ? h.y : h.z), r == 0 ? l.x : (r == 1 ? l.y : l.z), big,
                                   small);
                    });
                if (wave_any(!chain_stretch)) {
#pragma unroll
                    for (int b = 0; b < B; ++b) {
                        if (li * B + b < n && !chain_stretch) {
                            v3<T> inc = plain_inc(b);
                            inc.x = inc.x + fmat(kfl[0], rl[b].x, kfl[0] * rh[b].x);
                            inc.y = inc.y + fmat(kfl[1], rl[b].y, kfl[1] * rh[b].y);
                            inc.z = inc.z + fmat(kfl[2], rl[b].z, kfl[2] * rh[b].z);
                            cadd3(rh[b], rl[b], inc);
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    // (rows that no chain of the wavefront has are left as they
                    // are, as in the general form: adding a zero renormalises
                    // the pair)
                    if (s[b] >= 0 && chain_flow) {
                        v3<T> big, small;
                        flow_entry(kfl[0], ah[b].x, al[b].x, big.x, small.x);
                        flow_entry(kfl[1], ah[b].y, al[b].y, big.y, small.y);
                        flow_entry(kfl[2], ah[b].z, al[b].z, big.z, small.z);
                        if (any_bits(kmask, 0x001u)) cadd_big(ah[b].x, al[b].x, big.x, small.x);
                        if (any_bits(kmask, 0x010u)) cadd_big(ah[b].y, al[b].y, big.y, small.y);
                        if (any_bits(kmask, 0x100u)) cadd_big(ah[b].z, al[b].z, big.z, small.z);
                    }
                }
            } else {
                if (wave_any(chain_stretch))
                    move_stretched([&](auto R, v3<T> h, v3<T> l, T& big, T& small) {
                        flow_row<decltype(R)::value>(kdt, kmask, h, l, big, small);
                    });
                // The tests of kmask (wave-uniform) stay outside the
                // per-lane conditions: nested inside them they would be
                // turned into lane masks and vector selects.
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const v3<T> f = masked_mat3(kdt, kmask, rh[b], rl[b]);
                    if (li * B + b < n && !chain_stretch) {
                        v3<T> inc = plain_inc(b);
                        if (chain_flow) inc = inc + f;
                        cadd3(rh[b], rl[b], inc);
                    }
                }
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const bool adv = s[b] >= 0 && chain_flow;
                    v3<T> big, small;
                    if (any_bits(kmask, 0x007u)) {
                        flow_row<0>(kdt, kmask, ah[b], al[b], big.x, small.x);
                        if (adv) cadd_big(ah[b].x, al[b].x, big.x, small.x);
                    }
                    if (any_bits(kmask, 0x038u)) {
                        flow_row<1>(kdt, kmask, ah[b], al[b], big.y, small.y);
                        if (adv) cadd_big(ah[b].y, al[b].y, big.y, small.y);
                    }
                    if (any_bits(kmask, 0x1C0u)) {
                        flow_row<2>(kdt, kmask, ah[b], al[b], big.z, small.z);
                        if (adv) cadd_big(ah[b].z, al[b].z, big.z, small.z);
                    }
                }
            }
        } else {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                v3<T> inc = plain_inc(b);
                // wave-uniform branches; fma(0, r, x) = x keeps chains without flow bit-identical
                if (flow_xy)
                    inc.x = fmat(kfl[0], rh[b].y, inc.x);
                else if (flow_diag)
                    inc = {fmat(kfl[0], rh[b].x, inc.x), fmat(kfl[1], rh[b].y, inc.y), fmat(kfl[2], rh[b].z, inc.z)};
                else if (flow)
                    inc = fma_mat3(kdt, rh[b], inc);
                if (li * B + b < n) rh[b] = rh[b] + inc;
            }
            if (flow) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const v3<T> A = ah[b];
                    // (fused operations written out: left to the compiler, the
                    // kernels fused the general form's products in different
                    // orders; a product on its own is rounded before it is added,
                    // as the general form's sums are)
                    v3<T> inc = zero3<T>();
                    if (flow_xy)
                        inc.x = rounded_mul(kfl[0], A.y);
                    else if (flow_diag)
                        inc = {rounded_mul(kfl[0], A.x), rounded_mul(kfl[1], A.y), rounded_mul(kfl[2], A.z)};
                    else
                        inc = {fmat(kdt[2], A.z, fmat(kdt[1], A.y, rounded_mul(kdt[0], A.x))),
                               fmat(kdt[5], A.z, fmat(kdt[4], A.y, rounded_mul(kdt[3], A.x))),
                               fmat(kdt[8], A.z, fmat(kdt[7], A.y, rounded_mul(kdt[6], A.x)))};
                    if (s[b] >= 0) ah[b] = ah[b] + inc;
                }
            }
        }
        bonds_and_records();

        // ---- substep 2: hops from the post-move positions.
        int s_rec[B];  // replay: the recorded slot state after this step
        if constexpr (RP) {
            bool bad = false;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int j = li * B + b;
                s_rec[b] = -1;
                if (j < n) {
                    const int v = replay_next[b];
                    // a creation lands on an end; a destruction leaves an end after the hop, so
                    // a bead within one of it; anything else moves by at most one bead
                    const bool ok = s[b] >= 0 ? (v == -1 ? (s[b] <= 1 || s[b] >= n - 2)
                                                         : (v >= s[b] - 1 && v <= s[b] + 1 && v < n))
                                              : (v == -1 || v == 0 || v == n - 1);
                    bad |= !ok;
                    s_rec[b] = ok ? v : s[b];
                }
            }
            if (bad) atomicOr(a.flags, kFlagReplay);
        }
#pragma unroll
        for (int b = 0; b < B && !RP; ++b) {
            if constexpr (!kJointDraws && !LL) {
                const uint32_t i = (uint32_t)(li * B + b);
                if (even) {
                    const uint4 y = draw(kNoise2, i, gid, kp, k0, k1);
                    whop[b] = y.z;
                    wrec[b] = y.w;
                    carry_w0[b] = y.x;
                    carry_w1[b] = y.y;
                } else {
                    const uint4 z = draw(kSlot, i, gid, kp, k0, k1);
                    whop[b] = z.x;
                    wrec[b] = z.y;
                }
            }
            const int t = s[b] > 0 ? s[b] : 0;
            const BeadRec<T> r = rec[lbase + t];
            const v3<T> Rh = {r.v[0], r.v[1], r.v[2]};
            const v3<T> Rl = {r.v[3], r.v[4], r.v[5]};
            const v3<T> bp = {r.v[6], r.v[7], r.v[8]};      // R_{S+1} - R_S
            const v3<T> bm = {-r.v[9], -r.v[10], -r.v[11]};  // R_{S-1} - R_S
            const v3<T> dd = (Rh - ah[b]) + (Rl - al[b]);
            // (R_{S+-1} - A)^2 - (R_S - A)^2 = b (b + 2 d) with b = R_{S+-1} - R_S
            const T up = dot(bp, bp + T(2) * dd);
            const T dn = dot(bm, bm + T(2) * dd);
            T pp = (t < n - 1) ? glauber(tab, up, hop_e2q, hop_h2) : T(0);
            T pm = (t > 0) ? glauber(tab, dn, hop_e2q, hop_h2) : T(0);
            // an energy that overflowed to inf - inf gives 1/2, as fmin and the FP32
            // form have it (FP64 holds the exponent's argument to +-700, which loses
            // it); in the low-latency form without a branch, which takes 2 % of a step
            // there, elsewhere with one, since the selects take 5 %
            if constexpr (!kComp && LL) {
                pp = t < n - 1 && up != up ? T(0.5) : pp;
                pm = t > 0 && dn != dn ? T(0.5) : pm;
            } else if constexpr (!kComp) {
                if (__builtin_expect(wave_any(__builtin_isunordered(up, dn)), 0)) {
                    if (t < n - 1 && up != up) pp = T(0.5);
                    if (t > 0 && dn != dn) pm = T(0.5);
                }
            }
            const T u = LL ? uhop[b] : u01<T>(whop[b]);
            const bool up_hop = s[b] >= 0 && u < pp;
            const bool dn_hop = s[b] >= 0 && !(u < pp) && u < pp + pm;
            if constexpr (LL) {
                // the positions of both neighbours are read with the bead's own
                // record, so that the new offset waits on no second LDS read
                const BeadRec<T>& rp = rec[lbase + (t + 1 < kCap ? t + 1 : t)];
                const BeadRec<T>& rm = rec[lbase + (t > 0 ? t - 1 : 0)];
                const v3<T> Ph = {rp.v[0], rp.v[1], rp.v[2]}, Pl = {rp.v[3], rp.v[4], rp.v[5]};
                const v3<T> Mh = {rm.v[0], rm.v[1], rm.v[2]}, Ml = {rm.v[3], rm.v[4], rm.v[5]};
                const v3<T> Nh = sel(up_hop, Ph, sel(dn_hop, Mh, Rh)), Nl = sel(up_hop, Pl, sel(dn_hop, Ml, Rl));
                d[b] = (Nh - ah[b]) + (Nl - al[b]);
            }
            if (up_hop)
                s[b] = t + 1;
            else if (dn_hop)
                s[b] = t - 1;
        }

        // ---- substep 3: destruction at the ends and construction, all from the
        // post-hop state.  K = C - Z attempts (every empty slot once), or with
        // the K = 1 rule a single attempt by the segment's lowest empty slot
        // (both counted at the start of the step).
        int create_at[B];
        bool destroyed[B];
        bool any_create = false;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = li * B + b;
            const uint32_t uw = LL ? wrec[b] : wrec[b] >> 9;
            create_at[b] = -1;
            destroyed[b] = false;
            if constexpr (RP) {
                if (s[b] < 0) {
                    create_at[b] = s_rec[b];
                } else {
                    destroyed[b] = s_rec[b] < 0;
                    s[b] = s_rec[b];
                }
            } else if constexpr (LL) {  // without branches
                const bool occ = s[b] >= 0;
                destroyed[b] = occ & ((s[b] == 0) | (s[b] == n - 1)) & (uw < thr_destroy);
                const bool tries = !occ & (j < n) & (!K1 || j == first_empty);
                create_at[b] = (tries & (uw < t2)) ? (uw < t1 ? 0 : n - 1) : -1;
                s[b] = destroyed[b] ? -1 : s[b];
            } else if (j < n) {
                if (s[b] >= 0) {
                    if ((s[b] == 0 || s[b] == n - 1) && uw < thr_destroy) {
                        s[b] = -1;
                        destroyed[b] = true;
                    }
                } else if (!K1 || j == first_empty) {
                    if (uw < t1)
                        create_at[b] = 0;
                    else if (uw < t2)
                        create_at[b] = n - 1;
                }
            }
            any_create |= create_at[b] >= 0;
        }
        if (wave_any(any_create)) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int j = li * B + b;
                if (create_at[b] >= 0) {
                    const BeadRec<T> r = rec[lbase + create_at[b]];
                    const v3<T> Rh = {r.v[0], r.v[1], r.v[2]};
                    const v3<T> Rl = {r.v[3], r.v[4], r.v[5]};
                    v3<T> gn;
                    if constexpr (LL)
                        gn = unpack3(drawn[(int)(g & 3)].anchor_w[b * kWaveSize + lane]);
                    else
                        gn = anchor_normals<T>(tab, draw(kAnchor, (uint32_t)j, gid, g, k0, k1));
                    const v3<T> off3 = asd * gn;
                    if constexpr (kComp) {
                        ah[b] = Rh;
                        al[b] = Rl;
                        cadd3(ah[b], al[b], off3);
                    } else {
                        ah[b] = Rh + off3;
                    }
                    s[b] = create_at[b];
                    if constexpr (LL) d[b] = (Rh - ah[b]) + (Rl - al[b]);
                }
            }
        }
        if constexpr (LL) {
            read_masks(mw);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                d[b] = sel(s[b] >= 0, d[b], zero3<T>());
                Off4<T> o;
                o.v[0] = d[b].x;
                o.v[1] = d[b].y;
                o.v[2] = d[b].z;
                o.v[3] = T(0);
                offs[li * B + b] = o;
            }
            wave_sync();
            if (step + 1 < n_steps) read_drawn(g + 1);
            gather(mw);  // for the next step's move
        } else {
            refresh_offsets();
        }

        if (rec_s) {
            int8_t* row = rec_s + (g + 1 - a.rec_g0) * a.total + off;
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (li * B + b < n) row[li * B + b] = (int8_t)s[b];
        }
        if constexpr (kTraj) {
            store_r(step + 1);
            if constexpr (RP) {
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (destroyed[b]) store_a(step + 1, b);
            } else {
                log_destroyed(destroyed);
            }
        }

        // ---- observables of the new state.
        if (sample_every > 0 && phase == 0) {
            // Every lane leaves its twelve FP64 sums in LDS, value q of lane l at
            // [q][l] with rows of 65: the writes of a value and the reads of a
            // row both fall in distinct banks, at constant offsets from one
            // address each.  They are formed in two groups of six, so that
            // the twelve are never live together (otherwise the sampling step
            // sets the kernel's register peak).  The lanes of a segment then add
            // them up, twelve lanes for every 16 rows (a fixed order): 16 x 32
            // lanes in turn took 3400 cycles of a step alone on its SIMD, with
            // 16-way bank conflicts on the writes.
            auto put = [&](int q0, const double (&p)[6]) {
#pragma unroll
                for (int q = 0; q < 6; ++q) sums[(q0 + q) * kSumStride + lane] = p[q];
            };
            {
                double p[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const double bx = br[b].x, by = br[b].y, bz = br[b].z;  // zero past the end
                    p[0] += bx * bx;
                    p[1] += by * by;
                    p[2] += bz * bz;
                    p[3] += bx * by;
                    p[4] += by * bz;
                    p[5] += bz * bx;
                }
                put(0, p);
            }
            {
                double p[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const double dx = d[b].x, dy = d[b].y, dz = d[b].z;  // zero when empty
                    p[0] += dx * dx;
                    p[1] += dy * dy;
                    p[2] += dz * dz;
                    p[3] += dx * dy;
                    p[4] += dy * dz;
                    p[5] += dz * dx;
                }
                put(6, p);
            }
            int z2 = 0;
#pragma unroll
            for (int b = 0; b < B; ++b) z2 += __popcll(__ballot(s[b] >= 0) & smask);
            wave_sync();
            if constexpr (PK) {
                // as below for a chain of nl lanes: up to four parts of twelve
                // lanes, or, with fewer than twelve, several values a lane
                const int nl = (n + B - 1) / B;
                const int parts = min(4, max(1, nl / kSampleValues)), rows = (nl + parts - 1) / parts;
                const int part = parts > 1 ? li / kSampleValues : 0;
                for (int v0 = 0; wave_any(v0 < kSampleValues && (v0 == 0 || nl < kSampleValues)); v0 += nl) {
                    const int v = v0 + li - part * kSampleValues;
                    double tot = 0.0;
                    const bool adds = li < nl && part < parts && v < kSampleValues;
                    if (adds)
                        for (int r = part * rows; r < min(nl, (part + 1) * rows); ++r) tot += sums[v * kSumStride + sb + r];
#pragma unroll
                    for (int q = 1; q < 4; ++q) {
                        const double other = lane_read(tot, min(lane + q * kSampleValues, kWaveSize - 1));
                        if (q < parts && part == 0) tot += other;
                    }
                    const double corr = (v < 3) ? (double)n : (v >= 6 && v < 9) ? (double)z2 : 0.0;
                    if (adds && part == 0)
                        sample_out[(int64_t)chain * kSampleValues + v] = (v < 6 ? 3.0 : kstress) * tot - corr;
                }
            } else {
                constexpr int kParts = W >= 64 ? 4 : (W >= 32 ? 2 : 1), kRows = W / kParts;
                const int part = li / kSampleValues;
#pragma unroll
                for (int v0 = 0; v0 < (W < kSampleValues ? kSampleValues : 1); v0 += W) {
                    const int v = v0 + li - part * kSampleValues;  // (kParts > 1 only with W > kSampleValues)
                    double tot = 0.0;
                    if (part < kParts && v < kSampleValues) {
                        const double* col = sums + v * kSumStride + sb + part * kRows;
                        double odd = 0.0;
#pragma unroll
                        for (int r = 0; r < kRows; r += 2) {
                            tot += col[r];
                            odd += col[r + 1];
                        }
                        tot += odd;
                    }
                    if constexpr (kParts == 4) tot += lane_read(tot, lane + 2 * kSampleValues);
                    if constexpr (kParts >= 2) tot += lane_read(tot, lane + kSampleValues);
                    const double corr = (v < 3) ? (double)n : (v >= 6 && v < 9) ? (double)z2 : 0.0;
                    if (valid && part == 0 && v < kSampleValues)
                        sample_out[(int64_t)chain * kSampleValues + v] = (v < 6 ? 3.0 : kstress) * tot - corr;
                }
            }
            sample_out += sample_row;
            wave_sync();  // the records are rewritten by the next step
        }
        if (sample_every > 0) phase = (phase + 1 == sample_every) ? 0 : phase + 1;
    }

    // The final state goes back to the state buffer, except from a replay,
    // which reads its checkpoint in place and leaves it for later reverse
    // passes (its output is the trajectory).
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int i = li * B + b;
        if (i < n) {
            finite_ok &= finite3(rh[b]);
            if constexpr (!RP) {
                st3<T>(a.st.r0, off + i, rh[b]);
                st3<T>(a.st.a0, off + i, ah[b]);
                if constexpr (kComp) {
                    st3<T>(a.st.r1, off + i, rl[b]);
                    st3<T>(a.st.a1, off + i, al[b]);
                }
                a.st.s[off + i] = s[b];
            }
        }
    }
    // a second copy of the final state when asked (the next checkpoint of a
    // recorded window)
    if (!RP && a.ck_end.r0) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = li * B + b;
            if (i < n) {
                st3<T>(a.ck_end.r0, off + i, rh[b]);
                st3<T>(a.ck_end.a0, off + i, ah[b]);
                if constexpr (kComp) {
                    st3<T>(a.ck_end.r1, off + i, rl[b]);
                    st3<T>(a.ck_end.a1, off + i, al[b]);
                }
                a.ck_end.s[off + i] = s[b];
            }
        }
    }
    if constexpr (RP) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (li * B + b < n) store_a(n_steps, b);
    }
    if constexpr (ST) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (li * B + b < n) reinterpret_cast<v3<T>*>(a.traj2)[off + li * B + b] = ah[b] + al[b];
        if (valid && li == 0) a.dcnt[chain] = dcount;
    }
    if (!finite_ok) atomicOr(a.flags, kFlagNonFinite);
    };  // run

    if constexpr (LL) {
        const int64_t g0 = a.ctrl[kCtrlSteps];
        const int32_t n_steps = a.n_steps;
        if (wv == 0) {
            __builtin_amdgcn_s_setprio(3);  // ahead of the drawing waves of its SIMD
            run((int64_t)blockIdx.x, g0, n_steps, 0);
            return;
        }
        // The drawing waves, one step pair ahead of the stepping wave: one draws
        // noise and words, one (the same, with a single drawing wave) the
        // anchor normals.  Both sides pass one barrier per pair: at the barrier
        // of pair k its numbers are drawn, and the stepping wave is done with
        // pair k - 1, whose room pair k + 1 takes.
        const int li = lane % W;
        const int64_t task = (int64_t)blockIdx.x * kChainsPerWave + lane / W;
        const uint32_t gid = task < a.n_tasks ? a.ct.gid[a.tasks[task]] : 0u;
        const T cnoise = in_vgpr(T(a.cs.noise));
        const uint32_t k0 = a.ph.key0, k1 = a.ph.key1;
        const int64_t p0 = g0 >> 1, p1 = (g0 + n_steps - 1) >> 1;
        for (int64_t k = p0; k <= p1; ++k) {
            DrawnStep<T, B>&even = drawn[(int)(2 * k & 3)], &odd = drawn[(int)(2 * k & 3) + 1];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const uint32_t i = (uint32_t)(li * B + b);
                const int at = b * kWaveSize + lane;
                if (wv == 1) {
                    uint4 c[3] = {counter(kNoise, i, gid, k), counter(kNoise2, i, gid, k), counter(kSlot, i, gid, k)};
                    philox_blocks<3>(c, k0, k1);
                    Off4<T> e, o;
                    box_muller(tab, c[0].x, c[0].y, cnoise, e.v[0], e.v[1]);
                    box_muller(tab, c[0].z, c[0].w, cnoise, e.v[2], o.v[0]);
                    box_muller(tab, c[1].x, c[1].y, cnoise, o.v[1], o.v[2]);
                    e.v[3] = u01<T>(c[1].z);
                    o.v[3] = u01<T>(c[2].x);
                    even.noise_u[at] = e;
                    odd.noise_u[at] = o;
                    even.anchor_w[at].v[3] = pack_word<T>(c[1].w >> 9);
                    odd.anchor_w[at].v[3] = pack_word<T>(c[2].y >> 9);
                }
                if (wv == DW) {
                    uint4 c[2] = {counter(kAnchor, i, gid, 2 * k), counter(kAnchor, i, gid, 2 * k + 1)};
                    philox_blocks<2>(c, k0, k1);
                    const v3<T> ge = anchor_normals<T>(tab, c[0]), go = anchor_normals<T>(tab, c[1]);
                    even.anchor_w[at].v[0] = ge.x;
                    even.anchor_w[at].v[1] = ge.y;
                    even.anchor_w[at].v[2] = ge.z;
                    odd.anchor_w[at].v[0] = go.x;
                    odd.anchor_w[at].v[1] = go.y;
                    odd.anchor_w[at].v[2] = go.z;
                }
            }
            __syncthreads();
        }
    } else if constexpr (PS) {
        static_assert(!RP && !ST, "the persistent schedule runs plain steps only");
        {
            // Persistent schedule (a plain step launch): the units (time chunk
            // c, wave task w) are taken in the order c * n_wt + w from one
            // counter, and a unit waits until unit (c - 1, w) has stored its
            // chains' state.  Every unit's predecessor was taken earlier, by a
            // wavefront that is running, and the earliest unfinished unit
            // never waits, so the queue drains; all wavefronts stay busy to
            // the end instead of the last round of a one-wave-per-task launch
            // running part-full.
            const int64_t g0 = a.ctrl[kCtrlSteps];
            const int64_t n_wt = a.n_wave_tasks;
            const int32_t L = a.chunk;
            const int64_t n_chunks = (a.n_steps + L - 1) / L;
            const int64_t total = n_wt * n_chunks;
            uint32_t* progress = a.sched + 1;  // [n_wt] chunks finished per wave task
            for (;;) {
                uint32_t u = 0;
                if (lane == 0) u = atomicAdd(a.sched, 1u);
                u = __builtin_amdgcn_readfirstlane(u);
                if ((int64_t)u >= total) break;
                const int64_t c = (int64_t)u / n_wt, w = (int64_t)u % n_wt;
                if (c > 0) {
                    // bounded wait (the bound only guards against a hang: the
                    // predecessor is running and finishes within one unit)
                    for (uint32_t spin = 0;; ++spin) {
                        const uint32_t done = __hip_atomic_load(&progress[w], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                        if (__builtin_amdgcn_readfirstlane(done) >= (uint32_t)c) break;
                        if (spin > (1u << 22)) {
                            if (lane == 0) atomicOr(a.flags, kFlagInternal);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(8);
                    }
                }
                const int64_t gs = g0 + c * L;
                const int32_t ns = (int32_t)min((int64_t)L, (int64_t)a.n_steps - c * L);
                // samples of steps g0 .. gs - 1 precede this unit's: steps g with (g + 1) % n_s == 0
                const int64_t q0 = a.sample_every > 0 ? gs / a.sample_every - g0 / a.sample_every : 0;
                run(w, gs, ns, q0);
                __hip_atomic_store(&progress[w], (uint32_t)(c + 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else {
        run((int64_t)blockIdx.x * kWavesPerGroup + wv, a.ctrl[kCtrlSteps], a.n_steps, 0);
    }
}

// Waves per SIMD the register budget must allow.  The step is held one wave
// above what its registers would give: FP32 with one bead per lane at 5 waves
// (96 VGPRs instead of 106), with two at 4 (128 instead of 138), FP64 with
// one at 3 (168 instead of ~225).  The compiler spills a few values, mostly
// reloaded in the sampling step and the launch epilogue; the extra wave hides
// more of the LDS round trips (16384 x 32 FP32: 18.1 -> 17.5 ms per 5000-step
// launch; 16384 x 128 at 64 x 2: 31.9 -> 27.0 ms per 2000 steps; 16384 x 32
// FP64: 13.9 -> 12.7 ms per 1000 steps).  Two-bead FP64 cannot reach 3
// waves and is left to the compiler.
template <typename T, int B>
constexpr int kStepWavesPerEu = std::is_same<T, float>::value ? (B == 1 ? 5 : 4) : (B == 1 ? 3 : 1);

template <typename T, int W, int B, bool K1, bool ST, bool FL>
__global__ void __launch_bounds__(kGroupThreads) __attribute__((amdgpu_waves_per_eu(kStepWavesPerEu<T, B>)))
k_step(StepArgs)
{
    step_body<T, W, B, K1, false, ST, FL, false, 0>();
}

// The same step under the persistent schedule (plain steps: nothing recorded
// or stored), a kernel of its own so that the queue's registers do not weigh
// on the other variants.
template <typename T, int W, int B, bool K1, bool FL>
__global__ void __launch_bounds__(kGroupThreads) __attribute__((amdgpu_waves_per_eu(kStepWavesPerEu<T, B>)))
k_step_queue(StepArgs)
{
    step_body<T, W, B, K1, false, false, FL, true, 0>();
}

// The queue with chains packed side by side (plain steps).
template <typename T, int B, bool K1, bool FL>
__global__ void __launch_bounds__(kGroupThreads) __attribute__((amdgpu_waves_per_eu(kStepWavesPerEu<T, B>)))
k_step_packed(StepArgs)
{
    step_body<T, kWaveSize, B, K1, false, false, FL, true, 0, true>();
}

// Drawing waves per stepping wave: in FP64 one for the noise and one for the
// anchors (1024 x 32, 1000 steps: 1066 us, with one drawing wave 1206).
template <typename T> constexpr int kDrawWaves = std::is_same<T, float>::value ? 1 : 2;

// The step for launches with few wave tasks (plain steps).  With no more than a
// few waves per SIMD a step takes as long as its own instruction chain (some
// 2100 cycles of one wave, at a quarter of the issue rate).  The random numbers,
// new anchors' normals among them, do not depend on the state: other waves of
// the workgroup draw them a step pair ahead and pass them through LDS, at a lower
// wave priority (without the priority the gain is gone from two workgroups per
// CU on).  The stepping wave also builds its slot masks while the new offsets
// are formed, reads both neighbours' positions with a bead's own record, and
// decides the slots without branches.  Per 1000 steps, queue form -> this one:
// 2048 x 32 at rest 915 -> 751 us, under shear 1046 -> 916; 512 x 128 2042 -> 1504;
// 64 x 8 FP64, sampled every step, 1992 -> 1307; 512 x 32 FP64 1476 -> 1021.
template <typename T, int W, int B, bool K1, bool FL>
__global__ void __launch_bounds__(kWaveSize * (1 + kDrawWaves<T>)) __attribute__((amdgpu_waves_per_eu(std::is_same<T, float>::value && B == 1 ? 4 : 2)))
k_step_pair(StepArgs)
{
    step_body<T, W, B, K1, false, false, FL, false, kDrawWaves<T>>();
}

// Replay of recorded slot rows (the adjoint's reverse pass re-creates each
// segment's trajectory this way).  It samples no stress.  FP32 with one bead
// per lane is held at 5 waves per SIMD (84 VGPRs, no spills): at 6 it spills
// a few values, and every reload from scratch waits for all of the wave's
// memory operations in flight, the trajectory stores included.
template <typename T, int W, int B, bool FL>
__global__ void __launch_bounds__(kGroupThreads) __attribute__((amdgpu_waves_per_eu(std::is_same<T, float>::value && B == 1 ? 5 : 1)))
k_replay(StepArgs)
{
    step_body<T, W, B, false, true, false, FL, false, 0>();
}

// Workgroups of a queue kernel that fit on the device at once (occupancy x
// CUs), looked up once per kernel.
template <typename K> int resident_groups(K kern, int& cached)
{
    if (cached == 0) {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kGroupThreads, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        cached = per_cu * cus;
    }
    return cached;
}

// Shortest time chunk of the persistent schedule, in steps.
constexpr int kMinChunkSteps = 200;

// Launches a queue kernel of which r workgroups fit at once.
template <typename K> hipError_t launch_queue(K kern, int r, const StepArgs& a, hipStream_t s)
{
    StepArgs p = a;
    // time chunks per wave task: the count (1..16, chunks of at least
    // kMinChunkSteps) with the shortest estimated run, in units of the
    // launch's length.  The slots take ceil(units / slots) rounds of units
    // of 1/nc of the steps, but a wave task's chunks run one after
    // another, so never fewer than nc rounds; each chunk is also charged a
    // little for re-reading and writing the state.  With fewer wave tasks
    // than slots this keeps one chunk: more would only park wavefronts
    // that wait for their chains' previous chunk.
    const double slots = (double)std::max(1, r) * kWavesPerGroup;
    int best = 1;
    double best_t = 1e30;
    for (int nc = 1; nc <= 16; ++nc) {
        if (nc > 1 && (a.n_steps + nc - 1) / nc < kMinChunkSteps) break;
        const double rounds = std::max(std::ceil((double)(a.n_wave_tasks * nc) / slots), (double)nc);
        const double t = rounds / nc + 0.002 * nc;
        if (t < best_t - 1e-12) {
            best_t = t;
            best = nc;
        }
    }
    p.chunk = (a.n_steps + best - 1) / best;
    if (p.chunk < 1) p.chunk = 1;
    const int64_t units = a.n_wave_tasks * ((a.n_steps + p.chunk - 1) / p.chunk);
    const int64_t need = (units + kWavesPerGroup - 1) / kWavesPerGroup;
    const dim3 pg((unsigned)std::max<int64_t>(1, std::min<int64_t>(r > 0 ? r : need, need)));
    hipLaunchKernelGGL(kern, pg, dim3(kGroupThreads), 0, s, p);
    return hipGetLastError();
}

template <typename T, int W, int B, bool FL> hipError_t launch_f(const StepArgs& a, dim3 grid, hipStream_t s)
{
    if (a.sched && a.low_latency) {
        const dim3 pg((unsigned)a.n_wave_tasks), pb(kWaveSize * (1 + kDrawWaves<T>));
        // LDS asked for beyond the kernel's own, so that no more workgroups fit
        // on a CU than an even spread puts there, those of other groups counted in
        // (4096 x 16: 791 -> 764 us per 1000 steps, 4096 x 32: 1107 -> 1075).  One
        // workgroup per CU spreads by itself.
        constexpr int kLdsBytes = 160 * 1024, kGranule = 1280;
        const int own = (int)(sizeof(WaveLds<T, W, B, true, true>) + 4 * sizeof(DrawnStep<T, B>)) +
                        (int)sizeof(uint32_t) * 2 * (kMaxBeads + 1) +
                        (std::is_same<T, float>::value ? 0 : (int)sizeof(F64Tables));
        const int per_cu = a.low_latency;
        const int share = kLdsBytes / (per_cu + 1) + kGranule;  // per_cu of these fit, per_cu + 1 do not
        const unsigned pad = per_cu >= 2 && share > own && per_cu * share <= kLdsBytes ? (unsigned)(share - own) : 0u;
        if (a.construct_rule == 1)
            hipLaunchKernelGGL((k_step_pair<T, W, B, true, FL>), pg, pb, pad, s, a);
        else
            hipLaunchKernelGGL((k_step_pair<T, W, B, false, FL>), pg, pb, pad, s, a);
        return hipGetLastError();
    }
    if (a.sched && !a.replay_s && !a.traj) {
        // persistent: as many groups as fit, each wave taking units from the queue
        static int fit[2] = {0, 0};
        const bool k1 = a.construct_rule == 1;
        auto kern = k1 ? k_step_queue<T, W, B, true, FL> : k_step_queue<T, W, B, false, FL>;
        return launch_queue(kern, resident_groups(kern, fit[k1]), a, s);
    }
    if (a.replay_s)
        hipLaunchKernelGGL((k_replay<T, W, B, FL>), grid, dim3(kGroupThreads), 0, s, a);
    else if (a.traj && a.construct_rule == 1)
        hipLaunchKernelGGL((k_step<T, W, B, true, true, FL>), grid, dim3(kGroupThreads), 0, s, a);
    else if (a.traj)
        hipLaunchKernelGGL((k_step<T, W, B, false, true, FL>), grid, dim3(kGroupThreads), 0, s, a);
    else if (a.construct_rule == 1)
        hipLaunchKernelGGL((k_step<T, W, B, true, false, FL>), grid, dim3(kGroupThreads), 0, s, a);
    else
        hipLaunchKernelGGL((k_step<T, W, B, false, false, FL>), grid, dim3(kGroupThreads), 0, s, a);
    return hipGetLastError();
}

template <typename T, int W, int B, bool FL> hipError_t launch_t(const StepArgs& a, hipStream_t s)
{
    constexpr int kChainsPerGroup = kWavesPerGroup * (kWaveSize / W);
    const int64_t groups = (a.n_tasks + kChainsPerGroup - 1) / kChainsPerGroup;
    if (groups == 0) return hipSuccess;
    return launch_f<T, W, B, FL>(a, dim3((unsigned)groups), s);
}

template <typename T, int B, bool FL> hipError_t launch_packed(const StepArgs& a, hipStream_t s)
{
    static int fit[2] = {0, 0};
    const bool k1 = a.construct_rule == 1;
    auto kern = k1 ? k_step_packed<T, B, true, FL> : k_step_packed<T, B, false, FL>;
    return launch_queue(kern, resident_groups(kern, fit[k1]), a, s);
}

template <typename T, bool FL> hipError_t launch_p(int W, int B, const StepArgs& a, hipStream_t s)
{
    if (a.packed) return B == 1 ? launch_packed<T, 1, FL>(a, s) : launch_packed<T, 2, FL>(a, s);
    if (B == 1) {
        switch (W) {
        case 8: return launch_t<T, 8, 1, FL>(a, s);
        case 16: return launch_t<T, 16, 1, FL>(a, s);
        case 32: return launch_t<T, 32, 1, FL>(a, s);
        case 64: return launch_t<T, 64, 1, FL>(a, s);
        }
    } else if (B == 2) {
        switch (W) {
        case 16: return launch_t<T, 16, 2, FL>(a, s);
        case 32: return launch_t<T, 32, 2, FL>(a, s);
        case 64: return launch_t<T, 64, 2, FL>(a, s);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

// This file is compiled once per part, 2 * (FP64) + (flow): each holds the
// kernels of one precision at rest or under flow.
#if SSP_STEP_PART == 0
hipError_t launch_step_f32_rest(int W, int B, const StepArgs& a, hipStream_t s) { return launch_p<float, false>(W, B, a, s); }

// A null velocity-gradient table means a run at rest: the variant without the
// flow terms.
hipError_t launch_step(int precision, int W, int B, const StepArgs& a, hipStream_t s)
{
    if (precision == 0) return a.kappa ? launch_step_f32_flow(W, B, a, s) : launch_step_f32_rest(W, B, a, s);
    return a.kappa ? launch_step_f64_flow(W, B, a, s) : launch_step_f64_rest(W, B, a, s);
}
#elif SSP_STEP_PART == 1
hipError_t launch_step_f32_flow(int W, int B, const StepArgs& a, hipStream_t s) { return launch_p<float, true>(W, B, a, s); }
#elif SSP_STEP_PART == 2
hipError_t launch_step_f64_rest(int W, int B, const StepArgs& a, hipStream_t s) { return launch_p<double, false>(W, B, a, s); }
#elif SSP_STEP_PART == 3
hipError_t launch_step_f64_flow(int W, int B, const StepArgs& a, hipStream_t s) { return launch_p<double, true>(W, B, a, s); }
#else
#error "SSP_STEP_PART must be 0..3"
#endif

}  // namespace ssp
