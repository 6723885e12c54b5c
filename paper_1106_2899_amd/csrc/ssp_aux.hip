// Setup, observable and reduction kernels of libssp: the equilibrium
// initial-state sampler, the multiple-tau correlator update, compensated
// chain/element reductions, and canonical state views.
#include <algorithm>
#include <type_traits>

#include "ssp_device.h"
#include "ssp_internal.h"

namespace ssp {

namespace {

constexpr int kBlock = 256;

inline unsigned blocks_for(int64_t n, int per = kBlock) { return (unsigned)((n + per - 1) / per); }

// Neumaier compensated accumulation.
struct Neumaier {
    double s = 0.0, c = 0.0;
    __device__ void add(double x)
    {
        const double t = s + x;
        c += (fabs(s) >= fabs(x)) ? ((s - t) + x) : ((x - t) + s);
        s = t;
    }
    __device__ double value() const { return s + c; }
};

// ---------------------------------------------------------------- init -----
// Equilibrium sampler (Sec. 3.1): R_0 = 0, bonds N(0, 1/3); Z from
// Poisson(N/N_0) truncated to 0..N; slots 0..Z-1 occupied with S uniform and
// A = R_S + N(0, N_s/3).  One thread per chain, FP64 arithmetic for both
// precisions (setup is not on the hot path); the FP32 state keeps the FP64
// value as hi + lo.
template <typename T>
__global__ void k_init(State st, ChainTables ct, int64_t M, Physics ph)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= M) return;
    const int n = ct.n[k];
    const int64_t o = ct.off[k];
    const uint32_t gid = ct.gid[k];
    const double bsd = sqrt(1.0 / 3.0), asd = sqrt(ph.ns / 3.0);
    double R[3] = {0.0, 0.0, 0.0};
    auto put_r = [&](int i, const double* x) {
        if constexpr (sizeof(T) == 4) {
            float4 h, l;
            h.x = (float)x[0]; h.y = (float)x[1]; h.z = (float)x[2]; h.w = 0.f;
            l.x = (float)(x[0] - (double)h.x); l.y = (float)(x[1] - (double)h.y); l.z = (float)(x[2] - (double)h.z); l.w = 0.f;
            reinterpret_cast<float4*>(st.r0)[o + i] = h;
            reinterpret_cast<float4*>(st.r1)[o + i] = l;
        } else {
            reinterpret_cast<double4*>(st.r0)[o + i] = make_double4(x[0], x[1], x[2], 0.0);
        }
    };
    auto put_a = [&](int j, const double* x) {
        if constexpr (sizeof(T) == 4) {
            float4 h, l;
            h.x = (float)x[0]; h.y = (float)x[1]; h.z = (float)x[2]; h.w = 0.f;
            l.x = (float)(x[0] - (double)h.x); l.y = (float)(x[1] - (double)h.y); l.z = (float)(x[2] - (double)h.z); l.w = 0.f;
            reinterpret_cast<float4*>(st.a0)[o + j] = h;
            reinterpret_cast<float4*>(st.a1)[o + j] = l;
        } else {
            reinterpret_cast<double4*>(st.a0)[o + j] = make_double4(x[0], x[1], x[2], 0.0);
        }
    };
    put_r(0, R);
    for (int i = 0; i + 1 < n; ++i) {
        const v3<double> g = normals3_f64(draw(kInitBond, (uint32_t)i, gid, 0, ph.key0, ph.key1));
        R[0] += bsd * g.x;
        R[1] += bsd * g.y;
        R[2] += bsd * g.z;
        put_r(i + 1, R);
    }
    // truncated Poisson by inverse CDF
    const double lam = (double)n / ph.n0;
    const double u = u01<double>(draw(kInitZ, 0u, gid, 0, ph.key0, ph.key1).x);
    double pmf = exp(-lam), total = 0.0;
    for (int z = 0; z <= n; ++z) {
        if (z > 0) pmf = pmf * lam / (double)z;
        total += pmf;
    }
    int Z = n;
    pmf = exp(-lam);
    double cdf = 0.0;
    for (int z = 0; z <= n; ++z) {
        if (z > 0) pmf = pmf * lam / (double)z;
        cdf += pmf;
        if (u < cdf / total) {
            Z = z;
            break;
        }
    }
    for (int j = 0; j < n; ++j) {
        double A[3] = {0.0, 0.0, 0.0};
        int sj = -1;
        if (j < Z) {
            const uint32_t w = draw(kInitS, (uint32_t)j, gid, 0, ph.key0, ph.key1).x;
            sj = (int)(((uint64_t)w * (uint64_t)n) >> 32);
            // R_S: re-read the stored bead (hi + lo reproduces the FP64 value)
            double Rs[3];
            if constexpr (sizeof(T) == 4) {
                const float4 h = reinterpret_cast<const float4*>(st.r0)[o + sj];
                const float4 l = reinterpret_cast<const float4*>(st.r1)[o + sj];
                Rs[0] = (double)h.x + (double)l.x;
                Rs[1] = (double)h.y + (double)l.y;
                Rs[2] = (double)h.z + (double)l.z;
            } else {
                const double4 h = reinterpret_cast<const double4*>(st.r0)[o + sj];
                Rs[0] = h.x;
                Rs[1] = h.y;
                Rs[2] = h.z;
            }
            const v3<double> g = normals3_f64(draw(kInitAnchor, (uint32_t)j, gid, 0, ph.key0, ph.key1));
            A[0] = Rs[0] + asd * g.x;
            A[1] = Rs[1] + asd * g.y;
            A[2] = Rs[2] + asd * g.z;
        }
        put_a(j, A);
        st.s[o + j] = sj;
    }
}

__global__ void k_reset_ctrl(int64_t* ctrl, uint32_t* flags)
{
    const int t = threadIdx.x;
    if (t < kCtrlWords) ctrl[t] = 0;
    if (t == 0) *flags = 0u;
}

__global__ void k_zero(double* p, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.0;
}

__global__ void k_zero_ctrl_obs(int64_t* ctrl)
{
    if (threadIdx.x == 0) {
        ctrl[kCtrlCorrSamples] = 0;
        ctrl[kCtrlSeriesSamples] = 0;
    }
}

__device__ __forceinline__ int64_t samples_in(int64_t g0, int32_t n, int32_t every)
{
    return every > 0 ? (g0 + n) / every - g0 / every : 0;
}

__global__ void k_advance(int64_t* ctrl, int32_t n_steps, int32_t every, int64_t series_cap, uint32_t* flags)
{
    if (threadIdx.x != 0) return;
    const int64_t q = samples_in(ctrl[kCtrlSteps], n_steps, every);
    ctrl[kCtrlSteps] += n_steps;
    ctrl[kCtrlCorrSamples] += q;
    if (series_cap > 0 && ctrl[kCtrlSeriesSamples] + q > series_cap) atomicOr(flags, kFlagSeriesOverflow);
    ctrl[kCtrlSeriesSamples] += q;
}

// ------------------------------------------------------- correlator --------
// One 16-lane row per (chain, component) with lane k holding lag k at every
// level.  A new level-l value (x_l, y_l) shifts the y history of level l by
// one lane, adds x_l * y_l(n - k) to lane k, and is either parked as the
// first of a pair or averaged with the parked value into a level-(l+1) value.
// Histories start at zero, so unfilled lags add nothing; the number of
// products per lag is known from the sample count.  With the virtual-stress
// channel (V), x_v = sigma^v_ab(t) is paired with the same y history and
// block-averaged like x.
//
// The row is a DPP row (16 lanes): the history shift is row_shr:1 and the
// parked pair of level l is read with row_newbcast:l, so the level loop runs
// without LDS traffic (DPP controls are immediates: the level loop is fully
// unrolled).
__device__ __forceinline__ double row_shr1(double v)
{
    const int2 p = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(p.x, 0x111, 0xf, 0xf, true),
                                                __builtin_amdgcn_mov_dpp(p.y, 0x111, 0xf, 0xf, true)));
}
template <int L> __device__ __forceinline__ double row_bcast(double v)
{
    const int2 p = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(p.x, 0x150 + L, 0xf, 0xf, true),
                                                __builtin_amdgcn_mov_dpp(p.y, 0x150 + L, 0xf, 0xf, true)));
}
// row_bcast<l> for a level index that is a constant once the level loop is
// unrolled (the switch folds away).
__device__ __forceinline__ double row_bcast_level(double v, int l)
{
    switch (l) {
    case 0: return row_bcast<0>(v);
    case 1: return row_bcast<1>(v);
    case 2: return row_bcast<2>(v);
    case 3: return row_bcast<3>(v);
    case 4: return row_bcast<4>(v);
    case 5: return row_bcast<5>(v);
    case 6: return row_bcast<6>(v);
    case 7: return row_bcast<7>(v);
    case 8: return row_bcast<8>(v);
    case 9: return row_bcast<9>(v);
    case 10: return row_bcast<10>(v);
    case 11: return row_bcast<11>(v);
    case 12: return row_bcast<12>(v);
    case 13: return row_bcast<13>(v);
    case 14: return row_bcast<14>(v);
    default: return row_bcast<15>(v);
    }
}

template <bool V> __global__ void __launch_bounds__(kBlock) k_corr(CorrArgs a)
{
    const int64_t rows = 3 * a.n_chains;
    const int k = threadIdx.x & 15;
    const int64_t r = (int64_t)blockIdx.x * (kBlock / 16) + (threadIdx.x >> 4);
    const bool live = r < rows;
    const int64_t rr = live ? r : 0;
    const int64_t chain = rr / 3;
    const int comp = (int)(rr % 3);

    double yh[kMaxCorrLevels], C[kMaxCorrLevels], Cv[V ? kMaxCorrLevels : 1];
#pragma unroll
    for (int l = 0; l < kMaxCorrLevels; ++l) {
        yh[l] = (l < a.levels) ? a.hist[((int64_t)l * rows + rr) * 16 + k] : 0.0;
        C[l] = (l < a.levels) ? a.acc[((int64_t)l * rows + rr) * 16 + k] : 0.0;
        if constexpr (V) Cv[l] = (l < a.levels) ? a.acc_v[((int64_t)l * rows + rr) * 16 + k] : 0.0;
    }
    double px = a.pend[(rr * 16 + k) * 2 + 0];
    double py = a.pend[(rr * 16 + k) * 2 + 1];
    double pv = V ? a.pend_v[rr * 16 + k] : 0.0;

    const int64_t g0 = a.ctrl[kCtrlSteps];
    const int64_t s0 = a.ctrl[kCtrlCorrSamples];
    const int64_t Q = samples_in(g0, a.n_steps, a.sample_every);
    // the values of the next two samples are in flight while one is processed
    auto load = [&](int64_t q, double& x, double& v) {
        if (q < Q) {
            const double* smp = a.samples + (q * a.n_chains + chain) * kSampleValues;
            x = smp[3 + comp];
            v = smp[9 + comp];
        }
    };
    double nx0 = 0.0, nv0 = 0.0, nx1 = 0.0, nv1 = 0.0;
    load(0, nx0, nv0);
    load(1, nx1, nv1);
    for (int64_t q = 0; q < Q; ++q) {
        double xl = nx0;
        double xv = nv0;
        nx0 = nx1;
        nv0 = nv1;
        load(q + 2, nx1, nv1);
        double yl = xl + xv;
        const int64_t cnt1 = s0 + q + 1;  // 1-based index of this sample
        bool go = true;
#pragma unroll
        for (int l = 0; l < kMaxCorrLevels; ++l) {
            if (go && l < a.levels) {
                const double prev = row_shr1(yh[l]);
                yh[l] = (k == 0) ? yl : prev;
                C[l] += xl * yh[l];
                if constexpr (V) Cv[l] += xv * yh[l];
                if ((cnt1 >> l) & 1) {  // first of a pair at this level: park it
                    if (k == l) {
                        px = xl;
                        py = yl;
                        if constexpr (V) pv = xv;
                    }
                    go = false;
                } else {
                    const double qx = row_bcast_level(px, l);
                    const double qy = row_bcast_level(py, l);
                    xl = (qx + xl) * 0.5;
                    yl = (qy + yl) * 0.5;
                    if constexpr (V) xv = (row_bcast_level(pv, l) + xv) * 0.5;
                }
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int l = 0; l < kMaxCorrLevels; ++l) {
        if (l < a.levels) {
            a.hist[((int64_t)l * rows + r) * 16 + k] = yh[l];
            a.acc[((int64_t)l * rows + r) * 16 + k] = C[l];
            if constexpr (V) a.acc_v[((int64_t)l * rows + r) * 16 + k] = Cv[l];
        }
    }
    a.pend[(r * 16 + k) * 2 + 0] = px;
    a.pend[(r * 16 + k) * 2 + 1] = py;
    if constexpr (V) a.pend_v[r * 16 + k] = pv;
}

// Batch sums of the accumulators: out[b][l][k] = sum over the chains of batch
// b (contiguous, equal split) and the three components, Neumaier-compensated.
// One block per (batch, level); thread t takes lag t % 16 and every 64th row, four
// rows in flight (reading the accumulators is the bound; with 16 rows at once
// 16384 chains took 90 us).
constexpr int kBatchThreads = 1024, kBatchRows = kBatchThreads / 16;
__global__ void __launch_bounds__(kBatchThreads) k_corr_batches(const double* acc, int64_t n_chains, int32_t levels,
                                                                int32_t batches, double* out)
{
    const int b = blockIdx.x / levels;
    const int l = blockIdx.x % levels;
    const int64_t rows = 3 * n_chains;
    const int64_t c0 = n_chains * b / batches, c1 = n_chains * (b + 1) / batches;
    const int k = threadIdx.x & 15, sub = threadIdx.x >> 4;
    const double* at = acc + (int64_t)l * rows * 16 + k;
    Neumaier nm;
    int64_t r = 3 * c0 + sub;
    for (; r + 3 * kBatchRows < 3 * c1; r += 4 * kBatchRows) {
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = at[(r + q * kBatchRows) * 16];
#pragma unroll
        for (int q = 0; q < 4; ++q) nm.add(v[q]);
    }
    for (; r < 3 * c1; r += kBatchRows) nm.add(at[r * 16]);
    __shared__ double ps[kBatchThreads], pc[kBatchThreads];
    ps[threadIdx.x] = nm.s;
    pc[threadIdx.x] = nm.c;
    __syncthreads();
    if (sub < 8) {  // eight threads a lag, then one
        Neumaier tot;
        double cc = 0.0;
        for (int q = sub; q < kBatchRows; q += 8) {
            tot.add(ps[q * 16 + k]);
            cc += pc[q * 16 + k];
        }
        ps[threadIdx.x] = tot.s;  // row sub, which no other thread has read
        pc[threadIdx.x] = tot.c + cc;
    }
    __syncthreads();
    if (sub == 0) {
        Neumaier tot;
        double cc = 0.0;
        for (int q = 0; q < 8; ++q) {
            tot.add(ps[q * 16 + k]);
            cc += pc[q * 16 + k];
        }
        out[((int64_t)b * levels + l) * 16 + k] = tot.value() + cc;
    }
}

// G = sum_b S_b / (3 M cnt); G_err = standard error of the batch means.  One
// block per level: its threads bring the batch sums into LDS, one a lag adds
// them in order.
constexpr int kMaxBatches = 64;
__global__ void __launch_bounds__(kBlock) k_corr_final(const double* bs, int64_t n_chains, int32_t levels,
                                                       int32_t batches, int64_t samples, double* G, double* G_err)
{
    const int l = blockIdx.x, k = threadIdx.x % 16;
    const int64_t len = samples >> l;
    const int64_t cnt = len > k ? len - k : 0;
    __shared__ double sum[kMaxBatches][16], mean_of[kMaxBatches][16];
    for (int b = threadIdx.x / 16; b < batches; b += kBlock / 16) {
        const int64_t mb = n_chains * (b + 1) / batches - n_chains * b / batches;
        const double v = bs[((int64_t)b * levels + l) * 16 + k];
        sum[b][k] = v;
        mean_of[b][k] = v / (3.0 * (double)mb * (double)(cnt > 0 ? cnt : 1));
    }
    __syncthreads();
    if (threadIdx.x >= 16) return;
    const int t = l * 16 + k;
    if (cnt == 0) {
        G[t] = 0.0;
        G_err[t] = 0.0;
        return;
    }
    Neumaier tot;
    for (int b = 0; b < batches; ++b) tot.add(sum[b][k]);
    G[t] = tot.value() / (3.0 * (double)n_chains * (double)cnt);
    if (batches < 2) {
        G_err[t] = 0.0;
        return;
    }
    double mean = 0.0;
    for (int b = 0; b < batches; ++b) mean += mean_of[b][k];
    mean /= batches;
    double var = 0.0;
    for (int b = 0; b < batches; ++b) {
        const double v = mean_of[b][k] - mean;
        var += v * v;
    }
    G_err[t] = sqrt(var / (batches - 1) / batches);
}

// ---------------------------------------------------- element series -------
// series[e][t][c] = sum over the chains of element e of sigma_c (c < 6) for
// the samples of the launch just finished; Neumaier-compensated, fixed order.
// The sample rows are read once, so reading them is the bound (96 B a chain
// and sample move, of which 48 are used).  G wavefronts take one element and
// sample: 21 chains at a time, three lanes a chain with two components (16 B)
// each, and the 21 G partial sums of a component are added in lane order.  With
// one thread per (element, sample, component), as before, one element of 4096
// chains took 1277 us for 100 samples.  G = 4 from 84 chains (one round of the
// lanes) per element on.
template <int G>
__global__ void __launch_bounds__(kBlock) k_series(const double* samples, const int32_t* elem_off, int32_t E, int64_t M,
                                                   int32_t n_steps, int32_t every, int64_t q_most, const int64_t* ctrl,
                                                   double* series, int64_t cap)
{
    constexpr int kGroups = kBlock / (kWaveSize * G);  // (element, sample) pairs of a block
    constexpr int kRound = 21;                         // chains a wavefront reads at once
    __shared__ double ps[kBlock / kWaveSize][6][kRound], pc[kBlock / kWaveSize][6][kRound];
    __shared__ double ws[kBlock / kWaveSize][6], wc[kBlock / kWaveSize][6];
    const int lane = threadIdx.x % kWaveSize, wv = threadIdx.x / kWaveSize;
    const int64_t item = (int64_t)blockIdx.x * kGroups + wv / G;
    const int64_t q = item % q_most;
    const int e = (int)(item / q_most);
    const int64_t Q = samples_in(ctrl[kCtrlSteps], n_steps, every);
    const int64_t pos = ctrl[kCtrlSeriesSamples] + q;
    const bool live = e < E && q < Q && pos < cap;
    const int part = lane / 3, pair = lane % 3;
    if (live && part < kRound) {
        Neumaier n0, n1;
        const double2* row = reinterpret_cast<const double2*>(samples + q * M * kSampleValues) + pair;
        const int64_t end = elem_off[e + 1];
        int64_t k = elem_off[e] + (wv % G) * kRound + part;
        constexpr int kAtOnce = 4;  // rows in flight
        for (; k + (kAtOnce - 1) * kRound * G < end; k += kAtOnce * kRound * G) {
            double2 v[kAtOnce];
#pragma unroll
            for (int r = 0; r < kAtOnce; ++r) v[r] = row[(k + r * kRound * G) * (kSampleValues / 2)];
#pragma unroll
            for (int r = 0; r < kAtOnce; ++r) {
                n0.add(v[r].x);
                n1.add(v[r].y);
            }
        }
        for (; k < end; k += kRound * G) {
            const double2 v = row[k * (kSampleValues / 2)];
            n0.add(v.x);
            n1.add(v.y);
        }
        ps[wv][2 * pair][part] = n0.s;
        pc[wv][2 * pair][part] = n0.c;
        ps[wv][2 * pair + 1][part] = n1.s;
        pc[wv][2 * pair + 1][part] = n1.c;
    }
    __syncthreads();
    if (live && lane < 6) {
        Neumaier tot;
        double cc = 0.0;
        for (int r = 0; r < kRound; ++r) {
            tot.add(ps[wv][lane][r]);
            cc += pc[wv][lane][r];
        }
        ws[wv][lane] = tot.s;
        wc[wv][lane] = tot.c + cc;
    }
    __syncthreads();
    if (live && lane < 6 && wv % G == 0) {
        Neumaier tot;
        double cc = 0.0;
        for (int r = 0; r < G; ++r) {
            tot.add(ws[wv + r][lane]);
            cc += wc[wv + r][lane];
        }
        series[((int64_t)e * cap + pos) * 6 + lane] = tot.value() + cc;
    }
}

// ---------------------------------------------------------- stress ---------
template <typename T> __device__ __forceinline__ void load_pos(const State& st, int64_t i, bool anchor, double* x)
{
    if constexpr (sizeof(T) == 4) {
        const float4 h = reinterpret_cast<const float4*>(anchor ? st.a0 : st.r0)[i];
        const float4 l = reinterpret_cast<const float4*>(anchor ? st.a1 : st.r1)[i];
        x[0] = (double)h.x + (double)l.x;
        x[1] = (double)h.y + (double)l.y;
        x[2] = (double)h.z + (double)l.z;
    } else {
        const double4 h = reinterpret_cast<const double4*>(anchor ? st.a0 : st.r0)[i];
        x[0] = h.x;
        x[1] = h.y;
        x[2] = h.z;
    }
}

// Per-chain sigma and sigma^v of the current state (Sec. 2.1 stress, Appendix B
// virtual stress), FP64 from the canonical positions: W lanes take a chain, a
// bead and slot each (longer chains in rounds of W), leave their products' sums in
// LDS rows of 65 (distinct banks) and twelve lanes of every 16 rows add them up
// in lane order; with W < 16 each lane adds kVals of the rows up.  x[q] is the value
// v = li + q W (sigma for v < 6, then sigma^v) of the segment's chain, in the lanes
// with v < 12.  Reading the state once is the bound
// (68 B a bead in FP32); one thread per chain, as before, strode through it at
// 1.8 TB/s and left small ensembles to a few serial threads (65536 x 64 155 us,
// 512 x 128 97 us).
constexpr int kStressStride = kWaveSize + 1;
template <int W> constexpr int kStressVals = W >= 16 ? 1 : (kSampleValues + W - 1) / W;
template <typename T, int W>
__device__ __forceinline__ void chain_stress(const State& st, int n, int64_t o, double ns, int lane, double* sums,
                                             double (&x)[kStressVals<W>])
{
    const int li = lane % W, sb = lane - li;
    const uint64_t seg = W == 64 ? ~0ull : ((1ull << W) - 1ull) << sb;
    double p[kSampleValues];
#pragma unroll
    for (int q = 0; q < kSampleValues; ++q) p[q] = 0.0;
    int z = 0;
    for (int i0 = 0; __ballot(i0 < n) != 0; i0 += W) {
        const int i = i0 + li;
        int sj = -1;
        double r[3];
        if (i < n) {
            sj = st.s[o + i];
            load_pos<T>(st, o + i, false, r);
        }
        if (i + 1 < n) {
            double u[3];
            load_pos<T>(st, o + i + 1, false, u);
            const double bx = u[0] - r[0], by = u[1] - r[1], bz = u[2] - r[2];
            p[0] += bx * bx;
            p[1] += by * by;
            p[2] += bz * bz;
            p[3] += bx * by;
            p[4] += by * bz;
            p[5] += bz * bx;
        }
        if (sj >= 0) {
            double u[3], a[3];
            load_pos<T>(st, o + sj, false, u);
            load_pos<T>(st, o + i, true, a);
            const double dx = u[0] - a[0], dy = u[1] - a[1], dz = u[2] - a[2];
            p[6] += dx * dx;
            p[7] += dy * dy;
            p[8] += dz * dz;
            p[9] += dx * dy;
            p[10] += dy * dz;
            p[11] += dz * dx;
        }
        z += __popcll(__ballot(sj >= 0) & seg);
    }
#pragma unroll
    for (int q = 0; q < kSampleValues; ++q) sums[q * kStressStride + lane] = p[q];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    constexpr int kParts = W >= 16 ? W / 16 : 1, kRows = W / kParts;
#pragma unroll
    for (int q = 0; q < kStressVals<W>; ++q) {
        const int part = W >= 16 ? li / kSampleValues : 0, v = W >= 16 ? li % kSampleValues : li + q * W;
        double tot = 0.0;
        if (part < kParts && v < kSampleValues) {
            const double* col = sums + v * kStressStride + sb + part * kRows;
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
        const double less = v < 3 ? (double)n : (v >= 6 && v < 9) ? (double)z : 0.0;
        x[q] = (v < 6 ? 3.0 : 3.0 / ns) * tot - less;
    }
    __builtin_amdgcn_wave_barrier();  // the rows are free again
}

template <typename T, int W>
__global__ void __launch_bounds__(kBlock) k_stress(State st, ChainTables ct, int64_t M, double ns, double* out)
{
    __shared__ double sums[kBlock / kWaveSize][kSampleValues * kStressStride];
    const int lane = threadIdx.x % kWaveSize, wv = threadIdx.x / kWaveSize, li = lane % W;
    const int64_t k = ((int64_t)blockIdx.x * (kBlock / kWaveSize) + wv) * (kWaveSize / W) + lane / W;
    const bool live = k < M;
    double x[kStressVals<W>];
    chain_stress<T, W>(st, live ? ct.n[k] : 0, live ? ct.off[k] : 0, ns, lane, sums[wv], x);
#pragma unroll
    for (int q = 0; q < kStressVals<W>; ++q)
        if (live && li + q * W < kSampleValues) out[k * kSampleValues + li + q * W] = x[q];
}

template <typename T> __global__ void k_read_state(State st, int64_t total, double* R, double* A, int32_t* S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    double x[3];
    load_pos<T>(st, i, false, x);
    R[3 * i] = x[0];
    R[3 * i + 1] = x[1];
    R[3 * i + 2] = x[2];
    load_pos<T>(st, i, true, x);
    A[3 * i] = x[0];
    A[3 * i + 1] = x[1];
    A[3 * i + 2] = x[2];
    S[i] = st.s[i];
}

template <typename T>
__global__ void k_write_state(State st, int64_t total, const double* R, const double* A, const int32_t* S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    for (int which = 0; which < 2; ++which) {
        const double* src = which ? A : R;
        const double x0 = src[3 * i], x1 = src[3 * i + 1], x2 = src[3 * i + 2];
        if constexpr (sizeof(T) == 4) {
            float4 h, l;
            h.x = (float)x0; h.y = (float)x1; h.z = (float)x2; h.w = 0.f;
            l.x = (float)(x0 - (double)h.x); l.y = (float)(x1 - (double)h.y); l.z = (float)(x2 - (double)h.z); l.w = 0.f;
            reinterpret_cast<float4*>(which ? st.a0 : st.r0)[i] = h;
            reinterpret_cast<float4*>(which ? st.a1 : st.r1)[i] = l;
        } else {
            reinterpret_cast<double4*>(which ? st.a0 : st.r0)[i] = make_double4(x0, x1, x2, 0.0);
        }
    }
    st.s[i] = S[i];
}

template <typename T>
__global__ void k_rng_normals(const F64Tables* tables, uint32_t k0, uint32_t k1, uint32_t gid, int64_t step,
                              int32_t bead, int32_t count, double* out)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    // the step-pair layout of the step kernel: NOISE pairs give (c, s, c) at
    // the even step 2k; the odd step takes the last sine and the NOISE2 pair
    const uint32_t idx = (uint32_t)(bead + t);
    const T c = normal_scale<T>(1.0);
    const uint4 x = draw(kNoise, idx, gid, step >> 1, k0, k1);
    T g[6];
    box_muller_at(tables, x.x, x.y, c, g[0], g[1]);
    box_muller_at(tables, x.z, x.w, c, g[2], g[3]);
    if (step & 1) {
        const uint4 y = draw(kNoise2, idx, gid, step >> 1, k0, k1);
        box_muller_at(tables, y.x, y.y, c, g[4], g[5]);
    }
    const int o = (step & 1) ? 3 : 0;
    out[3 * t] = (double)g[o];
    out[3 * t + 1] = (double)g[o + 1];
    out[3 * t + 2] = (double)g[o + 2];
}

// ----------------------------------------------------- element means -------
// out[e][c] = (1 / M_e) sum over the chains k of element e of a per-chain value
// c < ncols: the ensemble average of the quantity within one fluid element (the
// average of Sec. 2.1 over the element's chains).  `parts` blocks take an
// element, each a contiguous range of its chains: the lanes' Neumaier sums are
// added in lane and wavefront order, and either divided by M_e (one part) or
// left for k_mean_final as (sum, correction) pairs, which adds the parts in
// order; the result does not depend on timing.
constexpr int kMeanCols = 12;
constexpr int kMeanRows = 32;  // most rows of sums in a block

__device__ __forceinline__ void part_of(const int32_t* elem_off, int e, int part, int parts, int64_t& lo, int64_t& hi)
{
    const int64_t first = elem_off[e], n = elem_off[e + 1] - first;
    lo = first + n * part / parts;
    hi = first + n * (part + 1) / parts;
}

// Adds the sums that `rows` threads of the block hold for each column (a thread row
// r's for the columns c, c + step, ... below ncols) and writes the columns' results
// or pairs.
template <int kHeld>
__device__ __forceinline__ void finish_mean(const Neumaier (&nm)[kHeld], int r, int c, int step, int rows, int ncols,
                                            int64_t e, int part, int parts, double count,
                                            double (&ps)[kMeanCols][kMeanRows], double (&pc)[kMeanCols][kMeanRows],
                                            double* out, double* pairs)
{
#pragma unroll
    for (int q = 0; q < kHeld; ++q)
        if (r < rows && c + q * step < ncols) {
            ps[c + q * step][r] = nm[q].s;
            pc[c + q * step][r] = nm[q].c;
        }
    __syncthreads();
    if ((int)threadIdx.x < ncols) {
        Neumaier tot;
        double cc = 0.0;
        for (int t = 0; t < rows; ++t) {
            tot.add(ps[threadIdx.x][t]);
            cc += pc[threadIdx.x][t];
        }
        if (parts == 1) {
            out[e * ncols + threadIdx.x] = (tot.value() + cc) / count;
        } else {
            double* p = pairs + ((e * parts + part) * ncols + threadIdx.x) * 2;
            p[0] = tot.s;
            p[1] = tot.c + cc;
        }
    }
}

// Means of rows[k][c] (rows of `stride` values): ncols neighbouring threads read
// a row.  Nothing is written when a flag of `skip` is up (the rows are invalid).
__global__ void __launch_bounds__(kBlock) k_element_mean(const double* rows, int64_t stride, int32_t ncols,
                                                         const int32_t* elem_off, int32_t parts, double* out,
                                                         double* pairs, const uint32_t* flags, uint32_t skip)
{
    __shared__ double ps[kMeanCols][kMeanRows], pc[kMeanCols][kMeanRows];
    if (*flags & skip) return;
    const int e = blockIdx.x / parts, part = blockIdx.x % parts;
    const int at_once = min(kBlock / ncols, kMeanRows), r = threadIdx.x / ncols, c = threadIdx.x % ncols;
    int64_t lo, hi;
    part_of(elem_off, e, part, parts, lo, hi);
    Neumaier nm[1];
    if (r < at_once)
        for (int64_t k = lo + r; k < hi; k += at_once) nm[0].add(rows[k * stride + c]);
    finish_mean(nm, r, c, 0, at_once, ncols, e, part, parts, (double)(elem_off[e + 1] - elem_off[e]), ps, pc,
                out, pairs);
}

// Means of the chains' stress, straight from the state.
template <typename T, int W>
__global__ void __launch_bounds__(kBlock) k_element_stress(State st, ChainTables ct, double ns, const int32_t* elem_off,
                                                           int32_t parts, double* out, double* pairs)
{
    __shared__ double sums[kBlock / kWaveSize][kSampleValues * kStressStride];
    __shared__ double ps[kMeanCols][kMeanRows], pc[kMeanCols][kMeanRows];
    const int e = blockIdx.x / parts, part = blockIdx.x % parts;
    const int lane = threadIdx.x % kWaveSize, wv = threadIdx.x / kWaveSize, li = lane % W;
    constexpr int kSegs = kBlock / W;  // chains of a block at once
    static_assert(kSegs <= kMeanRows, "a row of sums for each");
    const int r = threadIdx.x / W;
    int64_t lo, hi;
    part_of(elem_off, e, part, parts, lo, hi);
    Neumaier nm[kStressVals<W>];
    for (int64_t k0 = lo; k0 < hi; k0 += kSegs) {
        const int64_t k = k0 + r;
        const bool live = k < hi;
        double x[kStressVals<W>];
        chain_stress<T, W>(st, live ? ct.n[k] : 0, live ? ct.off[k] : 0, ns, lane, sums[wv], x);
#pragma unroll
        for (int q = 0; q < kStressVals<W>; ++q)
            if (live) nm[q].add(x[q]);
    }
    finish_mean(nm, r, li, W, kSegs, kSampleValues, e, part, parts,
                (double)(elem_off[e + 1] - elem_off[e]), ps, pc, out, pairs);
}

// One block per element; thread r * ncols + c adds the parts r, r + at_once, ...
__global__ void __launch_bounds__(kBlock) k_mean_final(const double* pairs, int32_t ncols, const int32_t* elem_off,
                                                       int32_t parts, double* out, const uint32_t* flags, uint32_t skip)
{
    __shared__ double ps[kMeanCols][kMeanRows], pc[kMeanCols][kMeanRows];
    if (*flags & skip) return;
    const int e = blockIdx.x;
    const int at_once = min(kBlock / ncols, kMeanRows), r = threadIdx.x / ncols, c = threadIdx.x % ncols;
    Neumaier nm[1];
    double cc = 0.0;
    if (r < at_once)
        for (int p = r; p < parts; p += at_once) {
            const double* v = pairs + (((int64_t)e * parts + p) * ncols + c) * 2;
            nm[0].add(v[0]);
            cc += v[1];
        }
    nm[0].c += cc;
    finish_mean(nm, r, c, 0, at_once, ncols, e, 0, 1, (double)(elem_off[e + 1] - elem_off[e]), ps, pc, out,
                nullptr);
}

// Parts of an element whose largest has n chains: blocks of `per_block` chains,
// bounded so that all elements' parts stay within kMeanParts (or one each).
int mean_parts(int64_t n_largest, int32_t n_elements, int per_block)
{
    const int64_t want = (n_largest + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(want, kMeanParts / n_elements));
}

// Whether every slot names a bead of its own chain or is empty: the lowest chain
// where one does not goes to *bad.
__global__ void __launch_bounds__(kBlock) k_check_slots(ChainTables ct, int64_t M, const int32_t* S, unsigned long long* bad)
{
    const int64_t k = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / 16;  // 16 lanes a chain
    if (k >= M) return;
    const int n = ct.n[k];
    const int64_t o = ct.off[k];
    bool ok = true;
    for (int j = threadIdx.x % 16; j < n; j += 16) ok &= S[o + j] >= -1 && S[o + j] < n;
    if (!ok) atomicMin(bad, (unsigned long long)k);
}

__global__ void k_set_word(unsigned long long* w, unsigned long long v)
{
    if (threadIdx.x == 0) *w = v;
}

// ratio[t] = num[t] / den[t] on the multiple-tau grid where the lag has data
// and den != 0, NaN elsewhere (the relative contribution of the virtual
// stress to G(t), Sec. 4.1).
__global__ void k_grid_ratio(const double* num, const double* den, int32_t levels, int64_t samples, double* ratio)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= levels * 16) return;
    const int l = t / 16, k = t % 16;
    const int64_t len = samples >> l;
    ratio[t] = (len > k && den[t] != 0.0) ? num[t] / den[t] : __builtin_nan("");
}

}  // namespace

hipError_t launch_element_mean(const double* rows, int64_t stride, int32_t ncols, const int32_t* elem_off,
                               int32_t n_elements, int64_t n_largest, double* out, double* pairs,
                               const uint32_t* flags, uint32_t skip, hipStream_t s)
{
    if (ncols < 1 || ncols > kMeanCols || n_elements < 1) return hipErrorInvalidValue;
    // 16 rounds of a block's rows: 65536 rows of one element 441 -> 12 us
    const int parts = mean_parts(n_largest, n_elements, 16 * (kBlock / kMeanCols));
    hipLaunchKernelGGL(k_element_mean, dim3((unsigned)n_elements * parts), dim3(kBlock), 0, s, rows, stride, ncols,
                       elem_off, parts, out, pairs, flags, skip);
    if (parts > 1)
        hipLaunchKernelGGL(k_mean_final, dim3((unsigned)n_elements), dim3(kBlock), 0, s, pairs, ncols, elem_off, parts,
                           out, flags, skip);
    return hipGetLastError();
}

namespace {
// Lanes per chain of the stress kernels: the narrowest segment that takes a chain of
// the mean length at once; a wider one for the longest chain leaves most lanes idle
// (a read of 262144 chains of 4 beads beside one of 128: 175 us with 64 lanes a chain,
// 56 with 8; all of 4 beads: 67 us with 16, 42 with 4).
template <typename T, int W>
hipError_t stress_w(const State& st, const ChainTables& ct, int64_t M, double ns, double* out, hipStream_t s)
{
    hipLaunchKernelGGL((k_stress<T, W>), dim3(blocks_for(M, kBlock / W)), dim3(kBlock), 0, s, st, ct, M, ns, out);
    return hipGetLastError();
}
template <typename T, int W>
hipError_t element_stress_w(const State& st, const ChainTables& ct, double ns, const int32_t* elem_off,
                            int32_t n_elements, int64_t n_largest, double* out, double* pairs, const uint32_t* flags,
                            hipStream_t s)
{
    const int parts = mean_parts(n_largest, n_elements, 4 * (kBlock / W));  // four rounds of a block
    hipLaunchKernelGGL((k_element_stress<T, W>), dim3((unsigned)n_elements * parts), dim3(kBlock), 0, s, st, ct, ns,
                       elem_off, parts, out, pairs);
    if (parts > 1)
        hipLaunchKernelGGL(k_mean_final, dim3((unsigned)n_elements), dim3(kBlock), 0, s, pairs, kSampleValues, elem_off,
                           parts, out, flags, 0u);
    return hipGetLastError();
}
template <typename F> hipError_t by_length(double n_mean, F f)
{
    if (n_mean <= 8.0) return f(std::integral_constant<int, 8>{});
    if (n_mean <= 16.0) return f(std::integral_constant<int, 16>{});
    if (n_mean <= 32.0) return f(std::integral_constant<int, 32>{});
    return f(std::integral_constant<int, 64>{});
}
}  // namespace

hipError_t launch_element_stress(int precision, const State& st, const ChainTables& ct, double n_mean, double ns,
                                 const int32_t* elem_off, int32_t n_elements, int64_t n_largest, double* out,
                                 double* pairs, const uint32_t* flags, hipStream_t s)
{
    auto run = [&](auto t) {
        using T = decltype(t);
        return by_length(n_mean, [&](auto w) {
            return element_stress_w<T, decltype(w)::value>(st, ct, ns, elem_off, n_elements, n_largest, out, pairs, flags,
                                                             s);
        });
    };
    return precision == 0 ? run(float{}) : run(double{});
}

hipError_t launch_check_slots(const ChainTables& ct, int64_t M, const int32_t* S, int64_t* bad, hipStream_t s)
{
    auto* w = reinterpret_cast<unsigned long long*>(bad);
    hipLaunchKernelGGL(k_set_word, dim3(1), dim3(64), 0, s, w, (unsigned long long)M);
    hipLaunchKernelGGL(k_check_slots, dim3(blocks_for(M, kBlock / 16)), dim3(kBlock), 0, s, ct, M, S, w);
    return hipGetLastError();
}

hipError_t launch_grid_ratio(const double* num, const double* den, int32_t levels, int64_t samples, double* ratio,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_grid_ratio, dim3(blocks_for(levels * 16)), dim3(kBlock), 0, s, num, den, levels, samples,
                       ratio);
    return hipGetLastError();
}

hipError_t launch_init(int precision, const State& st, const ChainTables& ct, int64_t M, Physics ph, hipStream_t s)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_init<float>, dim3(blocks_for(M, 64)), dim3(64), 0, s, st, ct, M, ph);
    else
        hipLaunchKernelGGL(k_init<double>, dim3(blocks_for(M, 64)), dim3(64), 0, s, st, ct, M, ph);
    return hipGetLastError();
}

hipError_t launch_reset_ctrl(int64_t* ctrl, uint32_t* flags, hipStream_t s)
{
    hipLaunchKernelGGL(k_reset_ctrl, dim3(1), dim3(64), 0, s, ctrl, flags);
    return hipGetLastError();
}

hipError_t launch_zero(double* p, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(count)), dim3(kBlock), 0, s, p, count);
    return hipGetLastError();
}

hipError_t launch_zero_ctrl_obs(int64_t* ctrl, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_ctrl_obs, dim3(1), dim3(64), 0, s, ctrl);
    return hipGetLastError();
}

hipError_t launch_advance(int64_t* ctrl, int32_t n_steps, int32_t sample_every, int64_t series_cap, uint32_t* flags,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, ctrl, n_steps, sample_every, series_cap, flags);
    return hipGetLastError();
}

hipError_t launch_corr(const CorrArgs& a, hipStream_t s)
{
    const int64_t rows = 3 * a.n_chains;
    if (a.acc_v)
        hipLaunchKernelGGL(k_corr<true>, dim3(blocks_for(rows, kBlock / 16)), dim3(kBlock), 0, s, a);
    else
        hipLaunchKernelGGL(k_corr<false>, dim3(blocks_for(rows, kBlock / 16)), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_corr_batches(const double* acc, int64_t n_chains, int32_t levels, int32_t batches, double* out,
                               hipStream_t s)
{
    hipLaunchKernelGGL(k_corr_batches, dim3((unsigned)(batches * levels)), dim3(kBatchThreads), 0, s, acc, n_chains, levels,
                       batches, out);
    return hipGetLastError();
}

hipError_t launch_corr_final(const double* batch_sums, int64_t n_chains, int32_t levels, int32_t batches,
                             int64_t corr_samples, double* G, double* G_err, hipStream_t s)
{
    hipLaunchKernelGGL(k_corr_final, dim3((unsigned)levels), dim3(kBlock), 0, s, batch_sums, n_chains, levels,
                       batches, corr_samples, G, G_err);
    return hipGetLastError();
}

hipError_t launch_series(const double* samples, const int32_t* elem_off, int32_t n_elements, int64_t n_chains,
                         int32_t n_steps, int32_t sample_every, int64_t q_cap, const int64_t* ctrl, double* series,
                         int64_t series_cap, hipStream_t s)
{
    // samples of a launch of n_steps: one more or less with the phase it starts at
    const int64_t q_most = std::min<int64_t>(q_cap, n_steps / sample_every + 1);
    const int64_t items = (int64_t)n_elements * q_most;
    if (n_chains >= (int64_t)84 * n_elements)
        hipLaunchKernelGGL(k_series<4>, dim3((unsigned)items), dim3(kBlock), 0, s, samples, elem_off, n_elements,
                           n_chains, n_steps, sample_every, q_most, ctrl, series, series_cap);
    else
        hipLaunchKernelGGL(k_series<1>, dim3(blocks_for(items, kBlock / kWaveSize)), dim3(kBlock), 0, s, samples,
                           elem_off, n_elements, n_chains, n_steps, sample_every, q_most, ctrl, series, series_cap);
    return hipGetLastError();
}

hipError_t launch_stress(int precision, const State& st, const ChainTables& ct, int64_t M, double n_mean, double ns,
                         double* out, hipStream_t s)
{
    auto run = [&](auto t) {
        using T = decltype(t);
        if (n_mean <= 4.0) return stress_w<T, 4>(st, ct, M, ns, out, s);
        return by_length(n_mean, [&](auto w) { return stress_w<T, decltype(w)::value>(st, ct, M, ns, out, s); });
    };
    return precision == 0 ? run(float{}) : run(double{});
}

hipError_t launch_read_state(int precision, const State& st, int64_t total, double* R, double* A, int32_t* S,
                             hipStream_t s)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_read_state<float>, dim3(blocks_for(total)), dim3(kBlock), 0, s, st, total, R, A, S);
    else
        hipLaunchKernelGGL(k_read_state<double>, dim3(blocks_for(total)), dim3(kBlock), 0, s, st, total, R, A, S);
    return hipGetLastError();
}

hipError_t launch_write_state(int precision, const State& st, int64_t total, const double* R, const double* A,
                              const int32_t* S, hipStream_t s)
{
    if (precision == 0)
        hipLaunchKernelGGL(k_write_state<float>, dim3(blocks_for(total)), dim3(kBlock), 0, s, st, total, R, A, S);
    else
        hipLaunchKernelGGL(k_write_state<double>, dim3(blocks_for(total)), dim3(kBlock), 0, s, st, total, R, A, S);
    return hipGetLastError();
}

hipError_t launch_rng_normals(int precision, const F64Tables* tables, uint32_t key0, uint32_t key1, uint32_t gid,
                              int64_t step, int32_t bead, int32_t count, double* out, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    if (precision == 0)
        hipLaunchKernelGGL(k_rng_normals<float>, dim3(blocks_for(count)), dim3(kBlock), 0, s, tables, key0, key1, gid, step,
                           bead, count, out);
    else
        hipLaunchKernelGGL(k_rng_normals<double>, dim3(blocks_for(count)), dim3(kBlock), 0, s, tables, key0, key1, gid, step,
                           bead, count, out);
    return hipGetLastError();
}

}  // namespace ssp
