// wm_blackwell.hip -- the Blackwell stage-centric family (Section IV-A) on
// the same batched machinery as the CDNA model: forward sweep, adjoint /
// loss-gradient sweep with a float64 pass for descriptors near the
// compute / I-O switch or near T = m, fixed-order float64 reductions, and the
// device Adam step (calibration loops are captured as HIP graphs by the API
// layer).  Descriptors are structure-of-arrays: 5 int32 (bM, bN, bK, CTAs,
// flags) and 3 float32 (K-steps, compression ratio, output element bytes),
// 32 bytes each.
#include "bw_launch.hpp"
#include "wm_device.hpp"

namespace wm {

// row base + k (base wave-uniform, off = lane_offset(k))
__device__ inline BwDesc load_bw_desc(const BwDescPtrs& d, int64_t base, uint32_t off)
{
    BwDesc x;
    x.bM = ntload_at(d.bM + base, off);
    x.bN = ntload_at(d.bN + base, off);
    x.bK = ntload_at(d.bK + base, off);
    x.G = ntload_at(d.G + base, off);
    x.fl = ntload_at(d.flags + base, off);
    x.Kt = ntload_at(d.Kt + base, off);
    x.CR = ntload_at(d.CR + base, off);
    x.ob = ntload_at(d.ob + base, off);
    return x;
}

__device__ inline BwDesc load_bw_desc(const BwDescPtrs& d, int64_t i)
{
    BwDesc x;
    x.bM = ntload(d.bM + i);
    x.bN = ntload(d.bN + i);
    x.bK = ntload(d.bK + i);
    x.G = ntload(d.G + i);
    x.fl = ntload(d.flags + i);
    x.Kt = ntload(d.Kt + i);
    x.CR = ntload(d.CR + i);
    x.ob = ntload(d.ob + i);
    return x;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_bw_predict(BwDescPtrs d, int64_t n, BwSet S,
                                                     float* __restrict__ T, int32_t* __restrict__ cta)
{
    const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (i >= n) return;
    BwEval<float> E;
    evaluate_bw<float, false>(S.st, S.cf, load_bw_desc(d, i), E);
    __builtin_nontemporal_store(E.T, T + i);
    if (cta) __builtin_nontemporal_store(E.cta, cta + i);
}

// mode 0: weight dL/dT; mode 1: measured m (MRE loss).  False if the
// descriptor does not contribute.
template <int MODE, typename R>
__device__ inline bool bw_weight(R T, float wi, double& w, double& lt)
{
    if (MODE == 1) {
        if (!(wi > 0.0f && wi < __builtin_huge_valf())) return false;
        const double m = wi, im = 1.0 / m, Td = (double)T;
        lt = __builtin_fabs(Td - m) * im;
        w = Td > m ? im : (Td < m ? -im : 0.0);
    } else {
        w = wi;
        lt = 0.0;
    }
    return true;
}

// float32 pass: the descriptor's terms go into the lane's float32 partial
// sums unless it sits within 1e-5 of the compute / I-O switch or (mode 1) of
// T = m (returns true: left to the float64 pass)
template <int MODE>
__device__ inline bool bw_grad_fast(const BwSet& S, const BwDesc& x, float wi, float* acc)
{
    BwEval<float> E;
    evaluate_bw<float, true>(S.st, S.cf, x, E);
    if (!(E.T < __builtin_huge_valf())) return false;
    float w = wi;
    if (MODE == 1) {
        if (!(wi > 0.0f && wi < __builtin_huge_valf())) return false;
        const float r0 = __builtin_amdgcn_rcpf(wi);
        if (E.near_kink || __builtin_fabsf(E.T * r0 - 1.0f) <= 1e-5f) return true;
        const float r = r0 * (2.0f - wi * r0);
        w = E.T > wi ? r : (E.T < wi ? -r : 0.0f);
        acc[0] += __builtin_fabsf(E.T - wi) * r;
        acc[1] += 1.0f;
    } else if (E.near_kink) {
        return true;
    }
    bw_accumulate<float, float>(S.cf, E, w, acc);
    return false;
}

template <int MODE>
__device__ inline void bw_grad_exact(const BwSet& S, const BwDesc& x, float wi, double* acc)
{
    BwEval<double> E;
    evaluate_bw<double, false>(S.st, S.cd, x, E);
    if (!(E.T < __builtin_huge_val())) return;
    double w, lt;
    if (!bw_weight<MODE>(E.T, wi, w, lt)) return;
    if (MODE == 1) {
        acc[0] += lt;
        acc[1] += 1.0;
    }
    bw_accumulate<double, double>(S.cd, E, w, acc);
}

// Phase 1: wave-aligned groups of 64 descriptors, one ballot word of redo
// flags per group (written exactly once).
// Bound: vector instructions (244 per 64 descriptors, 251 with the grid doubled;
// 0.95 to 1.0 per CU-cycle)
// and the 36 B of each descriptor, both near their rates.  At 2^24 descriptors
// the sweep took 168 us with the dtype's tensor rate an indexed load from the
// kernel arguments (its latency inside the evaluation) and a 64-bit vector add
// per address, 120 without; with the next group's loads issued before a group
// is evaluated, at seven waves per SIMD for their nine registers, 108 (at six 109,
// at five 132; 120 where the compiler is not held to seven).  The calibration's
// sweep loads nothing ahead and takes seven waves of its eight (bw_grid_t).
template <int MODE, bool PTR, int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(PTR ? 1 : 7, PTR ? 8 : 7))) void k_bw_grad(BwDescPtrs d, int64_t n, const float* __restrict__ wv,
                                                  BwSet sv, const BwSet* __restrict__ sp,
                                                  double* __restrict__ partials,
                                                  uint64_t* __restrict__ flags, uint32_t* __restrict__ ticket)
{
    __shared__ double red[16 * kAcc];
    if (ticket && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0u;   // counted by the float64 pass
    const BwSet& S = PTR ? *sp : sv;
    float acc[kAcc];   // the lane's partial sums; float64 from the wave reduction on
#pragma unroll
    for (int j = 0; j < kAcc; ++j) acc[j] = 0.0f;
    const uint32_t lane = threadIdx.x & 63u;
    // a wave's group of 64 descriptors starts at a wave-uniform row, so that
    // its loads take a scalar base and one 32-bit lane offset
    const int64_t first = (int64_t)blockIdx.x * BLOCK + __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u));
    const int64_t stride = (int64_t)gridDim.x * BLOCK;
    BwDesc next = {};
    float w_next = 0.0f;
    const auto load = [&](int64_t base) {
        if (lane < n - base) {   // n - base may be negative: nothing left
            const uint32_t off = lane_offset(lane);
            next = load_bw_desc(d, base, off);
            w_next = ntload_at(wv + base, off);
        }
    };
    if (!PTR) load(first);
    for (int64_t base = first; base < n; base += stride) {
        bool redo = false;
        if (PTR) load(base);
        const BwDesc x = next;
        const float w = w_next;
        if (!PTR) load(base + stride);
        if (lane < n - base) redo = bw_grad_fast<MODE>(S, x, w, acc);
        const uint64_t m = __ballot(redo);
        if (lane == 0) flags[base >> 6] = m;
    }
    double a64[kAcc];
#pragma unroll
    for (int j = 0; j < kAcc; ++j) a64[j] = (double)acc[j];
    block_reduce_acc(a64, red, partials + (int64_t)blockIdx.x * kAcc);
}

// One Adam step on log(theta); thread 0 rebuilds the set's constants.
struct BwFinishAdam {
    CalibState* st;
    AdamOpts o;
    BwSet* S;
    double* loss_hist;
    typedef AdamLane Ahead;
    __device__ Ahead ahead() const { return AdamLane(st, o); }
    __device__ void operator()(const double* tot, const Ahead& a) const
    {
        __shared__ double th[kTheta];
        if (threadIdx.x >= 64) return;
        if (adam_theta_step(st, a, tot, o, loss_hist, th) && threadIdx.x == 0) {
            make_bw_const<float>(th, S->st, S->cf);
            make_bw_const<double>(th, S->st, S->cd);
        }
    }
};

// Phase 2: fold the phase-1 rows (fixed order), redo flagged descriptors in
// float64; the last block to finish sums the rows and ends the call.
template <int MODE, bool PTR, bool ONE, typename FIN>   // ONE: a single block, n <= kOneBlockRows
__global__ __launch_bounds__(256) void k_bw_grad_redo(BwDescPtrs d, int64_t n,
                                                       const float* __restrict__ wv, BwSet sv,
                                                       const BwSet* sp,
                                                       const uint64_t* __restrict__ flags,
                                                       const double* __restrict__ rows1, int nrows1,
                                                       double* rows2, uint32_t* ticket, FIN fin)
{
    __shared__ double red[4 * kAcc], part[kRowGroups * kAcc], tot[kAcc];
    __shared__ int64_t queue[4][kFlagQueue];
    const BwSet& S = PTR ? *sp : sv;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const typename FIN::Ahead ahead = fin.ahead();
    const FlagWalk<ONE> walk(flags, (n + 63) >> 6, ((int64_t)blockIdx.x * 4 + wid) * 64, (int64_t)gridDim.x * 256);
    column_parts<false, 4>(rows1, nrows1, (int)blockIdx.x, (int)gridDim.x, kAcc, part);
    double acc[kAcc];
#pragma unroll
    for (int j = 0; j < kAcc; ++j) acc[j] = 0.0;
    for_flagged(walk, queue[wid], [&](int64_t i) { bw_grad_exact<MODE>(S, load_bw_desc(d, i), wv[i], acc); });
    const double t = block_reduce_value(acc, red);
    if (finish_rows(t, part, rows2, kAcc, ticket, tot)) fin(tot, ahead);
}

template <int BLOCK>
static void bw_predict_t(const BwDescPtrs& d, int64_t n, const BwSet& S, float* T, int32_t* cta,
                         hipStream_t s)
{
    const int64_t blocks = (n + BLOCK - 1) / BLOCK;
    k_bw_predict<BLOCK><<<(unsigned)blocks, BLOCK, 0, s>>>(d, n, S, T, cta);
}

hipError_t launch_bw_predict(const BwDescPtrs& d, int64_t n, const BwSet& S, float* T, int32_t* cta,
                             const LaunchCfg& c, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    switch (c.block) {
    case 64: bw_predict_t<64>(d, n, S, T, cta, s); break;
    case 128: bw_predict_t<128>(d, n, S, T, cta, s); break;
    case 512: bw_predict_t<512>(d, n, S, T, cta, s); break;
    default: bw_predict_t<256>(d, n, S, T, cta, s); break;
    }
    return hipGetLastError();
}

template <int MODE, bool PTR>
static int bw_grid_t(int64_t n, int grid_mult)
{
    const GradLayout L = grad_layout(n);
    const int64_t want = (n + 255) / 256;
    // The calibration's sweep has room for eight waves per SIMD and takes seven: a
    // lane's rows, and with them the last digits that a fitted theta repeats, are
    // those of the seven that its registers once left.  100 steps at 2^20 / 2^22
    // / 2^23 descriptors 2.76 / 4.94 / 7.15 ms, with eight 2.82 / 5.26 / 7.46.
    int64_t r = (int64_t)resident_blocks(reinterpret_cast<const void*>(&k_bw_grad<MODE, PTR, 256>), 256, PTR ? 7 : 8) *
                (grid_mult < 1 ? 1 : grid_mult);
    r = r < want ? r : want;
    r = r < L.nb ? r : L.nb;
    return (int)(r < 1 ? 1 : r);
}

template <int MODE, bool PTR, typename FIN>
static hipError_t bw_grad_t(const BwDescPtrs& d, int64_t n, const float* w, const BwSet& S, const BwSet* S_dev,
                            double* partials, uint64_t* flags, const GradLayout& L, const LaunchCfg& c,
                            const FIN& fin, hipStream_t s)
{
    const int nb = bw_grid_t<MODE, PTR>(n, c.grid_mult);
    const RedoLayout r = redo_layout(L, nb, partials);
    k_bw_grad<MODE, PTR, 256><<<nb, 256, 0, s>>>(d, n, w, S, S_dev, partials, flags, r.ticket);
    double* rows2 = partials + (int64_t)nb * kAcc;
    if (r.nb2 == 1 && n <= kOneBlockRows)
        k_bw_grad_redo<MODE, PTR, true><<<1, 256, 0, s>>>(d, n, w, S, S_dev, flags, partials, nb, rows2, r.ticket, fin);
    else
        k_bw_grad_redo<MODE, PTR, false><<<r.nb2, 256, 0, s>>>(d, n, w, S, S_dev, flags, partials, nb, rows2, r.ticket,
                                                               fin);
    return hipGetLastError();
}

hipError_t launch_bw_grad(int mode, const BwDescPtrs& d, int64_t n, const float* w, const BwSet& S,
                          double* partials, uint64_t* flags, const GradLayout& L, const LaunchCfg& c,
                          double* out, hipStream_t s)
{
    if (mode == 1) return bw_grad_t<1, false>(d, n, w, S, nullptr, partials, flags, L, c, FinishOut<1>{out}, s);
    return bw_grad_t<0, false>(d, n, w, S, nullptr, partials, flags, L, c, FinishOut<0>{out}, s);
}

hipError_t launch_bw_grad_adam(const BwDescPtrs& d, int64_t n, const float* meas, const GradLayout& L,
                               const LaunchCfg& c, double* partials, uint64_t* flags, CalibState* st,
                               const AdamOpts& o, BwSet* S, double* loss_hist, hipStream_t s)
{
    return bw_grad_t<1, true>(d, n, meas, BwSet{}, S, partials, flags, L, c, BwFinishAdam{st, o, S, loss_hist}, s);
}

}  // namespace wm
