// wm_device.hpp -- device-side helpers shared by the kernel files: streaming
// loads of one descriptor row and its float64 image, the fixed-order FP64
// block reductions, and the Adam step on log(theta).
#pragma once

#include "wm_launch.hpp"

namespace wm {

template <typename T>
__device__ inline T ntload(const T* p) { return __builtin_nontemporal_load(p); }

// Element k of the array at p (wave-uniform) with k < 2^30, as a load from a
// scalar base and a 32-bit lane offset.  off = lane_offset(k) has to be formed
// in the loop body that loads: hoisted out as a 64-bit value, it costs a 64-bit
// vector add per array.
__device__ inline uint32_t lane_offset(uint32_t k)
{
    uint32_t off = k * 4u;
    asm volatile("" : "+v"(off));
    return off;
}

template <typename T>
__device__ inline T ntload_at(const T* p, uint32_t off)
{
    return ntload((const T*)((const char*)p + off));
}

// Parameters read through a pointer into memory that stays constant while
// the kernel runs (a by-value kernel argument in the kernel-argument
// segment, or a set in device memory), laundered so that the optimiser cannot
// see through it: inside a sweep loop each parameter use is then a scalar
// load, served by the scalar cache.  Kept in scalar registers across the loop
// instead, the sixty-odd parameters overflow the 102 scalar registers; the
// compiler spills them to vector-register lanes and reloads each with one
// VALU instruction per descriptor.
template <typename T>
__device__ inline const T& uniform_const(const T* p)
{
    typedef __attribute__((address_space(4))) const T* CP;
    CP q = (CP)p;
    asm volatile("" : "+s"(q));
    return *(const T*)q;
}

// The address of by-value kernel argument `member` in the kernel-argument
// segment.  The arguments lie there in declaration order at their natural
// alignment, as the members of a struct (Mirror) that declares the kernel's
// parameters up to that argument do.  (A mismatch would feed every
// evaluation wrong parameters, which each parity test would show.)
#define WM_KERNARG_PTR(Mirror, member)                                                   \
    reinterpret_cast<const decltype(Mirror::member)*>(                                  \
        (const char*)__builtin_amdgcn_kernarg_segment_ptr() + __builtin_offsetof(Mirror, member))

__device__ inline Desc<float> load_desc(const DescPtrs& d, int64_t i)
{
    Desc<float> x;
    x.F = ntload(d.F + i);
    x.B = ntload(d.B + i);
    x.r1 = ntload(d.r1 + i);
    x.r2 = ntload(d.r2 + i);
    x.r3 = ntload(d.r3 + i);
    x.K = ntload(d.K + i);
    x.u = ntload(d.u + i);
    x.W = ntload(d.W + i);
    x.v = ntload(d.vgpr + i);
    x.s = ntload(d.lds + i);
    x.gp = ntload(d.gpack + i);
    x.G = ntload(d.grid + i);
    return x;
}

__device__ inline Desc<double> widen(const Desc<float>& x)
{
    Desc<double> y;
    y.F = x.F; y.B = x.B; y.r1 = x.r1; y.r2 = x.r2; y.r3 = x.r3; y.K = x.K; y.u = x.u; y.W = x.W;
    y.v = x.v; y.s = x.s; y.gp = x.gp; y.G = x.G;
    return y;
}

// ---------------------------------------------------------------------------
// block reduction of the 26 FP64 accumulators (fixed order)
// ---------------------------------------------------------------------------
// One step of the wave's recursive halving over lane bit M: a lane keeps the
// upper half of its H x 2 remaining columns if its bit M is set, else the
// lower half, and adds the partner lane's copy of the half it keeps.  Bits 32
// and 16 swap half the lane rows of column j with the other half of column j +
// H (v_permlane*_swap), after which the two registers hold exactly the two
// addends; bits 8, 4 and 2 fetch the partner's copy by DPP moves inside the row
// of 16 (i ^ 4 as the mirrors i ^ 3 and i ^ 7).
template <int CTRL>
__device__ inline double row_move(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int M, int H>
__device__ inline void halve_columns(double* v, int lane)
{
#pragma unroll
    for (int j = 0; j < H; ++j) {
        if constexpr (M == 32 || M == 16) {
            const uint64_t a = __builtin_bit_cast(uint64_t, v[j]), b = __builtin_bit_cast(uint64_t, v[j + H]);
            uint32_t al, ah, bl, bh;
            if constexpr (M == 32) {
                const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
                al = lo[0]; bl = lo[1]; ah = hi[0]; bh = hi[1];
            } else {
                const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
                al = lo[0]; bl = lo[1]; ah = hi[0]; bh = hi[1];
            }
            v[j] = __builtin_bit_cast(double, ((uint64_t)ah << 32) | al) +
                   __builtin_bit_cast(double, ((uint64_t)bh << 32) | bl);
        } else {
            static_assert(M == 8 || M == 4 || M == 2, "lane bits 32 .. 2");
            const bool up = (lane & M) != 0;
            const double send = up ? v[j] : v[j + H];
            const double keep = up ? v[j + H] : v[j];
            if constexpr (M == 8) v[j] = keep + row_move<0x128>(send);
            else if constexpr (M == 4) v[j] = keep + row_move<0x141>(row_move<0x1B>(send));
            else v[j] = keep + row_move<0x4E>(send);
        }
    }
}

// Block sum of the 26 per-thread accumulators (fixed order).  Within a wave
// the columns are halved over lane bits 5..1 (32 doubles cross lanes, not
// 26 x 6 for one butterfly per column), after which lanes 2c and 2c + 1
// hold column c over 32 lanes each; then the waves' rows are added in LDS.
// Exchanging the doubles by 64 ds_bpermute per wave instead held the tail of
// a sweep of few rows per lane to the LDS pipe.
// Must be called by every thread of the block; thread j < 26 returns column
// j's sum (other threads 0).  acc is clobbered.
__device__ inline double block_reduce_value(double* acc, double* lds /* [waves][26] */)
{
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
    static_assert(kAcc <= 32, "the halving covers 32 columns");
    double v[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = j < kAcc ? acc[j] : 0.0;
    halve_columns<32, 16>(v, lane);
    halve_columns<16, 8>(v, lane);
    halve_columns<8, 4>(v, lane);
    halve_columns<4, 2>(v, lane);
    halve_columns<2, 1>(v, lane);
    const double s = v[0] + row_move<0xB1>(v[0]);
    const int col = lane >> 1;
    if ((lane & 1) == 0 && col < kAcc) lds[wid * kAcc + col] = s;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < kAcc) {
        const int nw = blockDim.x >> 6;
        for (int w = 0; w < nw; ++w) t += lds[w * kAcc + threadIdx.x];
    }
    __syncthreads();
    return t;
}

__device__ inline void block_reduce_acc(double* acc, double* lds /* [waves][26] */, double* out)
{
    const double t = block_reduce_value(acc, lds);
    if (threadIdx.x < kAcc) out[threadIdx.x] = t;
}

// ---------------------------------------------------------------------------
// rows handed to the last block of a grid
// ---------------------------------------------------------------------------
// A block's row of column sums stored where every other block can read it
// within the launch: the eight XCDs' L2 caches are not coherent with one
// another, so the values go by agent-scope atomic stores (written through) and
// come back by agent-scope atomic loads.
__device__ inline void store_shared(double* p, double v)
{
    __hip_atomic_store((unsigned long long*)p, __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline double load_shared(const double* p)
{
    return __builtin_bit_cast(double, __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}

// True on every thread of the block that finishes last, after wave 0 of each
// block has stored its row by store_shared.  *ticket counts finished blocks (0
// before the launch).  The wait makes the row's stores complete before the
// count shows the block as finished, so the last block's load_shared see
// every row.  An agent-scope release and acquire around the count would write
// back and invalidate whole L2 caches for the same guarantee: measured slower
// than a separate launch for the final reduction.  Only what goes by store_shared
// and load_shared is ordered so: a plain store read by the last block would race.
__device__ inline bool last_block(uint32_t* ticket, uint32_t nblocks)
{
    __shared__ uint32_t last;
    if (threadIdx.x < 64) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0)
            last = nblocks <= 1u || __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT) == nblocks - 1u;
    }
    __syncthreads();
    return last != 0u;
}

// Column sums of rows first, first + step, ... below nrows (`stride` doubles
// apart), by a block of 256: thread COLS g + c adds column c of every G-th row
// from the g-th (G groups of COLS threads), LOADS of them in flight, so that
// consecutive threads read consecutive doubles (one row per thread would spread
// each load over 64 rows); its sum goes to part[COLS g + c].  SHARED: rows stored
// by store_shared in this launch.
constexpr int kRowGroups = 256 / kAcc;   // 9 x 26 of the 256 threads
template <bool SHARED, int LOADS, int COLS = kAcc>
__device__ inline void column_parts(const double* rows, int nrows, int first, int step, int64_t stride, double* part)
{
    constexpr int G = 256 / COLS;
    const int g = (int)threadIdx.x / COLS, c = (int)threadIdx.x - g * COLS;
    if (g >= G) return;
    double v = 0.0;
    const int64_t hop = (int64_t)step * G;
    for (int64_t r0 = first + (int64_t)step * g; r0 < nrows; r0 += hop * LOADS) {
        double x[LOADS];
#pragma unroll
        for (int k = 0; k < LOADS; ++k) {
            const int64_t r = r0 + hop * k;
            x[k] = 0.0;
            if (r < nrows) x[k] = SHARED ? load_shared(rows + r * stride + c) : rows[r * stride + c];
        }
#pragma unroll
        for (int k = 0; k < LOADS; ++k) v += x[k];
    }
    part[threadIdx.x] = v;
}

template <int COLS = kAcc>
__device__ inline double add_parts(const double* part)   // threads 0 .. COLS - 1, after a barrier
{
    double v = 0.0;
#pragma unroll
    for (int g = 0; g < 256 / COLS; ++g) v += part[g * COLS + threadIdx.x];
    return v;
}

// The end of a float64 pass: this block's row of column sums (thread j < COLS:
// t, plus the parts of the sweep's rows) goes to rows2, and the last block to
// finish sums the rows.  True on the threads of that block, with tot[j] in LDS.
template <int COLS = kAcc>
__device__ inline bool finish_rows(double t, double* part /* [256] */, double* rows2, int64_t stride, uint32_t* ticket,
                                   double* tot)
{
    static_assert(COLS <= 64, "a row is stored by one wave");
    const double row = threadIdx.x < COLS ? t + add_parts<COLS>(part) : 0.0;
    if (gridDim.x == 1) {   // a block that is alone has the totals (1 us less: 12.5 -> 11.5 at 16000 descriptors)
        if (threadIdx.x < COLS) tot[threadIdx.x] = row;
        __syncthreads();
        return true;
    }
    if (threadIdx.x < COLS) store_shared(rows2 + (int64_t)blockIdx.x * stride + threadIdx.x, row);
    if (!last_block(ticket, gridDim.x)) return false;
    column_parts<true, 15, COLS>(rows2, (int)gridDim.x, 0, 1, stride, part);
    __syncthreads();
    if (threadIdx.x < COLS) tot[threadIdx.x] = add_parts<COLS>(part);
    __syncthreads();
    return true;
}

// ---------------------------------------------------------------------------
// flagged rows of a bit-per-row flag array, packed over a wave's lanes
// ---------------------------------------------------------------------------
// Orders this wave's LDS stores before its later LDS loads from other lanes
// (the LDS executes one wave's operations in issue order; the fences keep
// the compiler from moving accesses across this point).
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr int kFlagQueue = 128;   // row indices queued per wave

constexpr int64_t kOneBlockRows = 4 * 64 * 64;   // a flag word per lane of a block

// This lane's first two words of a walk over the flag words w0 .. w0 + 63, w0 +
// stride ..., up to nwords (w0 and stride multiples of 64, wave-uniform),
// loaded ahead of other work.  ONE: a block that is alone, whose four waves share
// the words of at most kOneBlockRows rows equally: with 64 to the first wave, 5000
// rows that are all flagged were two waves' work, 100 us a call where it takes 45.
// Larger grids leave at most one block short, and keep the division off the pass's
// chain of latencies.
template <bool ONE = false>
struct FlagWalk {
    const uint64_t* flags;
    int64_t nwords, base, stride;
    uint64_t m, next;
    __device__ inline uint64_t word(int64_t b) const
    {
        const int64_t w = b + (threadIdx.x & 63);
        return w < nwords ? flags[w] : 0ull;
    }
    __device__ inline FlagWalk(const uint64_t* f, int64_t nw, int64_t w0, int64_t st)
        : flags(f), nwords(nw), base(w0), stride(st)
    {
        if (ONE) {
            const int64_t share = (nw + 3) >> 2;
            base = (w0 >> 6) * share;
            stride = nw;   // one step
            nwords = base + share < nw ? base + share : nw;
        }
        m = word(base);
        next = ONE ? 0ull : word(base + stride);
    }
};

// f(row) for every set bit of the walk's words (every lane active).
// Flags are sparse (a few per thousand rows) and f is a long float64 chain,
// so rows are queued in LDS, lowest bit of each lane's word first, and f runs
// with a row on every lane; called on the words' own lanes it would run once
// for nearly every word, a lane or two at a time.
template <bool ONE, typename F>
__device__ inline void for_flagged(FlagWalk<ONE> w, int64_t* queue /* [kFlagQueue], the wave's own */, F f)
{
    const int lane = threadIdx.x & 63;
    int qn = 0;
    for (;;) {
        uint64_t any = __ballot(w.m != 0ull);
        while (qn < 64 && (any != 0ull || w.base + w.stride < w.nwords)) {
            if (any != 0ull) {
                if (w.m != 0ull) {
                    queue[qn + (int)lanes_below(any)] = ((w.base + lane) << 6) + __builtin_ctzll(w.m);
                    w.m &= w.m - 1;
                }
                qn += __builtin_popcountll(any);
            } else {
                w.base += w.stride;
                w.m = w.next;
                w.next = w.word(w.base + w.stride);
            }
            any = __ballot(w.m != 0ull);
        }
        if (qn == 0) return;
        wave_lds_sync();
        if (lane < qn) f(queue[lane]);
        const int left = qn > 64 ? qn - 64 : 0;   // at most 63
        const int64_t moved = lane < left ? queue[64 + lane] : 0;
        wave_lds_sync();
        if (lane < left) queue[lane] = moved;
        qn = left;
    }
}

// ---------------------------------------------------------------------------
// the end of a gradient call: what the last block of the float64 pass does
// with the 26 totals in LDS; ahead() is loaded at the pass's start
// ---------------------------------------------------------------------------
template <int MODE>
struct FinishOut {   // mode 0: the 24 gradient sums; mode 1: loss, count and gradient over the count
    double* out;
    struct Ahead {};
    __device__ Ahead ahead() const { return Ahead(); }
    __device__ void operator()(const double* tot, const Ahead&) const
    {
        if (threadIdx.x >= kAcc) return;
        const double v = tot[threadIdx.x];
        if (MODE == 1) {
            const double c = tot[1];
            out[threadIdx.x] = (threadIdx.x == 1 || c == 0.0) ? v : v / c;
        } else if (threadIdx.x >= 2) {
            out[threadIdx.x - 2] = v;
        }
    }
};

// ---------------------------------------------------------------------------
// device Adam on log(theta)
// ---------------------------------------------------------------------------
// Closest non-decreasing (INC) or non-increasing sequence, in the least-
// squares sense, to the values of lanes base .. base + 3; lane base + i gets
// element i, other lanes keep v.  Element i of the isotonic fit is
// max over a <= i of min over b >= i of the mean of y[a..b] (non-decreasing;
// min and max swap for non-increasing).  Called by all 64 lanes, converged.
template <bool INC>
__device__ inline double isotonic4(double v, int lane, int base)
{
    double y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = __shfl(v, base + k, 64);
    const int i = lane - base;
    if (i < 0 || i > 3) return v;
    double best = INC ? -HUGE_VAL : HUGE_VAL;
    for (int a = 0; a <= i; ++a) {
        double inner = INC ? HUGE_VAL : -HUGE_VAL, sum = 0.0;
        for (int b = a; b < 4; ++b) {
            sum += y[b];
            if (b < i) continue;
            const double mean = sum / (double)(b - a + 1);
            inner = INC ? fmin(inner, mean) : fmax(inner, mean);
        }
        best = INC ? fmax(best, inner) : fmin(best, inner);
    }
    return best;
}

// What lane j < 24 of a wave needs of the step, loaded ahead of the totals (at
// the start of the kernel that ends in the step, where the loads cost nothing;
// after the totals they were 2 us of its chain).
struct AdamLane {
    int32_t step_index, was_diverged;
    double theta, phi, m, v, lo_log, hi_log;
    double lr, c1, c2;   // the step's schedule
    __device__ inline AdamLane(const CalibState* st, const AdamOpts& o)
    {
        const int lane = threadIdx.x & 63;
        const int j = lane < kTheta ? lane : 0;
        step_index = st->t;
        was_diverged = st->diverged;
        theta = st->theta[j];
        phi = st->phi[j];
        m = st->m[j];
        v = st->v[j];
        lo_log = o.lo_log[j];
        hi_log = o.hi_log[j];
        // from the host's table where there is one, else formed here (three
        // pow calls on the wave's critical path)
        if (o.sched && step_index < o.steps) {
            lr = o.sched[3 * step_index];
            c1 = o.sched[3 * step_index + 1];
            c2 = o.sched[3 * step_index + 2];
        } else {
            adam_schedule(o, step_index, &lr, &c1, &c2);
        }
    }
};

__device__ inline bool adam_theta_step(CalibState* st, const AdamLane& a, const double* tot, const AdamOpts& o,
                                       double* loss_hist, double* th_out /* LDS [kTheta] */)
{
    // Called by the 64 lanes of one wave, converged; lane j < 24 updates
    // theta_j.  The step index lives in device memory so one captured graph
    // serves every chunk of steps.  Returns true (on every lane) when theta
    // changed; th_out then holds the new theta, visible to the whole wave,
    // and the caller rebuilds its constants from it.
    const int lane = threadIdx.x & 63;
    const double cnt = tot[1];
    const double loss = cnt > 0.0 ? tot[0] / cnt : 0.0;
    if (lane == 0) {
        st->t = a.step_index + 1;
        if (loss_hist && a.step_index < o.steps)
            loss_hist[a.step_index] = a.was_diverged ? __builtin_nan("") : loss;
    }
    if (a.was_diverged) return false;
    const bool mine = lane < kTheta;
    const double g = mine && cnt > 0.0 ? tot[2 + lane] / cnt : 0.0;
    if (!__builtin_isfinite(loss) || __ballot(!__builtin_isfinite(g)) != 0) {
        if (lane == 0) st->diverged = 1;
        return false;
    }
    const double th = mine ? a.theta : 1.0;
    if (mine) st->theta_ok[lane] = th;
    const double lr = a.lr, c1 = a.c1, c2 = a.c2;
    double th_new = th;
    bool ok = true;
    const bool fit = mine && ((o.free_mask >> lane) & 1u);
    double phi = fit ? a.phi : 0.0;
    if (fit) {
        const double gp = th * g;
        const double m = o.beta1 * a.m + (1.0 - o.beta1) * gp;
        const double v = o.beta2 * a.v + (1.0 - o.beta2) * gp * gp;
        st->m[lane] = m;
        st->v[lane] = v;
        const double mh = m / c1;
        const double vh = v / c2;
        phi -= lr * mh / (sqrt(vh) + o.eps);
    }
    // constraints: the level orderings (every slot of an ordered group is
    // fitted), then the boxes
    if (o.order & 1) phi = isotonic4<false>(phi, lane, 0);
    if (o.order & 2) phi = isotonic4<true>(phi, lane, 4);
    if (fit) {
        phi = fmin(fmax(phi, a.lo_log), a.hi_log);
        st->phi[lane] = phi;
        th_new = exp(phi);
        ok = __builtin_isfinite(th_new) && th_new > 0.0;
    }
    if (__ballot(!ok) != 0) {
        if (lane == 0) st->diverged = 1;
        return false;
    }
    if (mine) {
        st->theta[lane] = th_new;
        th_out[lane] = th_new;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return true;
}


}  // namespace wm
