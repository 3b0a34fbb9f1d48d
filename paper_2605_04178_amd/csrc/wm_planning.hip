// wm_planning.hip -- per-group calibration multipliers and kernel-fusion
// planning on top of the model.
//
// Multipliers (Section IV-D: optional per-case multipliers with train /
// holdout separation): for each group of rows, the multiplier that minimises
// the training mean relative error of mult * T is a weighted median of the
// ratios m/T (weights T/m).  Groups of up to 64 rows are sorted across a
// wave's lanes, two groups per wave where they fit; in larger ones every
// candidate's cumulative weight is compared with all the group's rows.
//
// Fusion (Section IV-B: a fused kernel is modelled with the combined flops
// and bytes plus tau_fusion): a chain of kernels is cut into runs of at most
// R consecutive kernels.  One thread per row extends the fusion sums of the
// runs starting there one row at a time (float64 sums) and evaluates each
// run's combined descriptor in float32; a group of lanes per chain runs the
// prefix dynamic programme over those costs in float64.  Chains where float32
// could decide differently from float64 (a decision within a small relative
// margin, or a run float32 cannot represent) are redone in float64, so plans
// match a float64 evaluation except at its own ties.
#include "wm_device.hpp"
#include "wm_plan_rows.hpp"

namespace wm {

// ---------------------------------------------------------------------------
// multipliers
// ---------------------------------------------------------------------------
// finite and > 0, both
__device__ inline bool mult_ok(float T, float m)
{
    return __builtin_amdgcn_classf(T, 0x180) & __builtin_amdgcn_classf(m, 0x180);
}

// 1 / d for a positive double, two Newton steps from the hardware estimate,
// and n / d from it with one remainder step: the sequence of an IEEE division
// without its scaling and special cases, which operands and quotients made of
// a few float32 values (2^-278 .. 2^278) do not need.  d = 0 or infinity: NaN.
__device__ inline double recip_f32range(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
}

__device__ inline double quot_f32range(double n, double d, double rd)
{
    const double q = n * rd;
    return __builtin_fma(__builtin_fma(-d, q, n), rd, q);
}

template <int NA>
__device__ inline void wave_sum(double* acc)
{
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        double v = acc[j];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
        acc[j] = v;
    }
}

// The wave's index in the grid, in a form the compiler sees as the same on
// every lane (so that what depends on it stays in scalar registers and
// loops over it are scalar-controlled).
__device__ inline int64_t wave_id()
{
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    return (int64_t)blockIdx.x * (int64_t)(blockDim.x >> 6) + w;
}

// Lane k's value of x (k wave-uniform); every lane active.
__device__ inline int64_t read_lane64(int64_t x, int k)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, k);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)x >> 32), k);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ inline double read_lane_f64(double x, int k)
{
    return __builtin_bit_cast(double, read_lane64(__builtin_bit_cast(int64_t, x), k));
}

__device__ inline float read_lane_f32(float x, int k)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, x), k));
}

// Rows i in [a, b) of one group: the training loss and count, the held-out
// loss and count (float64, per lane), and T_scaled = mu T_i.
__device__ inline void mult_apply(double mu, float t, float m, bool tr, int64_t i,
                                  float* __restrict__ T_scaled, double* st)
{
    T_scaled[i] = (float)(mu * (double)t);
    if (!mult_ok(t, m)) return;
    const double e = __builtin_fabs(mu * (double)t - (double)m) / (double)m;
    if (tr) {
        st[0] += e;
        st[1] += 1.0;
    } else {
        st[2] += e;
        st[3] += 1.0;
    }
}

// A group of any size on the whole wave.  Candidate k (a valid training row)
// is the multiplier when its cumulative weight C_k = sum of w_i over valid
// training rows with (x_i, i) <= (x_k, k) reaches half the total and no
// smaller candidate does; the smallest such (x_k, k) wins.  Lanes take 64
// candidates at a time and the group's rows 64 at a time: a lane prepares
// its row once (x_i = m/T in float32 and float64, w_i = T/m in float64, 0
// for rows that do not count), then every row is broadcast to the lanes by
// lane reads.  The order (x_i, i) <= (x_k, k) is decided on the float32
// ratios, which round monotonically, and on the float64 ratios where the
// float32 ones tie; C_k and the total are float64 sums in row order.
__device__ inline void fit_group_scan(int64_t g, int64_t a, int64_t b, const float* __restrict__ T,
                                      const float* __restrict__ meas, const uint8_t* __restrict__ train,
                                      double* __restrict__ mult, float* __restrict__ T_scaled, double* st)
{
    const int lane = threadIdx.x & 63;
    const double dinf = __builtin_huge_val();
    const float finf = __builtin_huge_valf();
    double Wt = 0.0;   // total training weight, row order
    double bx = dinf;
    int64_t bk = INT64_MAX;
    for (int64_t k0 = a; k0 < b; k0 += 64) {
        // this lane's candidate
        const int64_t k = k0 + lane;
        float xfk = finf;
        double xdk = dinf, wk = 0.0;
        if (k < b) {
            const float tk = T[k], mk = meas[k];
            if (train[k] && mult_ok(tk, mk)) {
                xfk = mk / tk;
                xdk = (double)mk / (double)tk;
                wk = (double)tk / (double)mk;
            }
        }
        double C = 0.0;
        for (int64_t i0 = a; i0 < b; i0 += 64) {
            // this lane's row (the candidate's own when the chunks coincide)
            const int64_t i = i0 + lane;
            float xfi = xfk;
            double xdi = xdk, wi = wk;
            if (i0 != k0) {
                xfi = finf;
                xdi = dinf;
                wi = 0.0;
                if (i < b) {
                    const float ti = T[i], mi = meas[i];
                    if (train[i] && mult_ok(ti, mi)) {
                        xfi = mi / ti;
                        xdi = (double)mi / (double)ti;
                        wi = (double)ti / (double)mi;
                    }
                }
            }
            const int cnt = b - i0 < 64 ? (int)(b - i0) : 64;
            for (int r = 0; r < cnt; ++r) {
                const float xf = read_lane_f32(xfi, r);
                const double w = read_lane_f64(wi, r);
                if (k0 == a) Wt += w;
                bool before = xf < xfk;
                const bool tie = xf == xfk;
                if (__ballot(tie) != 0ull) {
                    const double xd = read_lane_f64(xdi, r);
                    if (tie) before = xd < xdk || (xd == xdk && i0 + r <= k);
                }
                C += before ? w : 0.0;
            }
        }
        if (xdk < dinf && C >= 0.5 * Wt && (xdk < bx || (xdk == bx && k < bk))) {
            bx = xdk;
            bk = k;
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const double ox = __shfl_xor(bx, m, 64);
        const int64_t ok = __shfl_xor(bk, m, 64);
        if (ox < bx || (ox == bx && ok < bk)) {
            bx = ox;
            bk = ok;
        }
    }
    const double mu = bk == INT64_MAX ? 1.0 : bx;
    if (lane == 0) mult[g] = mu;
    for (int64_t i = a + lane; i < b; i += 64) mult_apply(mu, T[i], meas[i], train[i] != 0, i, T_scaled, st);
}

// Lane l's partner value at lane l ^ X inside a row of 16 lanes, by DPP (one
// move; two for X = 4, whose mirrors 3 and 7 compose to it).
template <int X>
__device__ inline uint32_t row_xor(uint32_t v)
{
    static_assert(X == 1 || X == 2 || X == 3 || X == 4 || X == 7 || X == 8 || X == 15, "DPP patterns");
    constexpr int ctrl = X == 1 ? 0xB1 : X == 2 ? 0x4E : X == 3 ? 0x1B : X == 8 ? 0x128 : X == 15 ? 0x140 : 0x141;
    // every lane has a partner: no old value to keep, so no copy before the move
    if constexpr (X == 4) v = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x1B, 0xF, 0xF, true);
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xF, 0xF, true);
}

__device__ inline double f64_of(uint32_t lo, uint32_t hi)
{
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// One compare-exchange step of the sort over lanes l and l ^ X: the lane keeps
// the smaller of the two keys if keep_min, else the larger.  X = 16 and 32
// swap half the rows of two copies of the key (v_permlane*_swap), after which
// every lane of a pair holds both keys.
template <int X>
__device__ inline void sort_step(uint32_t& lo, uint32_t& hi, bool keep_min)
{
    if constexpr (X == 16 || X == 32) {
        uint32_t l0, l1, h0, h1;
        if constexpr (X == 16) {
            const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
            const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
            l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
        } else {
            const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
            l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
        }
        const bool second = (f64_of(l1, h1) < f64_of(l0, h0)) == keep_min;
        lo = second ? l1 : l0;
        hi = second ? h1 : h0;
    } else {
        const uint32_t pl = row_xor<X>(lo), ph = row_xor<X>(hi);
        const bool take = (f64_of(pl, ph) < f64_of(lo, hi)) == keep_min;
        lo = take ? pl : lo;
        hi = take ? ph : hi;
    }
}

// Lanes of the wave whose bits b of the lane index are clear, as a 64-bit
// lane mask (b a power of two up to 32).
constexpr uint64_t lanes_clear(int b)
{
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l) m |= (uint64_t)((l & b) == 0) << l;
    return m;
}

// A constant lane mask as a predicate, its halves moved into scalar registers
// where it is used: left to the compiler, a loop's masks all stay in scalar
// registers, overflow into vector-register lanes and cost a VALU instruction
// each to read back.
template <uint64_t MASK>
__device__ inline bool in_lanes()
{
    uint32_t lo, hi;
    asm volatile("s_mov_b32 %0, %1" : "=s"(lo) : "i"((int)(uint32_t)MASK));
    asm volatile("s_mov_b32 %0, %1" : "=s"(hi) : "i"((int)(uint32_t)(MASK >> 32)));
    return __builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo);
}

// The key of each lane sorted ascending over segments of W lanes.  Blocks of
// 2, 4, 8 and 16 lanes are merged by mirrored steps (every block ascending,
// so a merge starts by comparing lane i with the block's mirror of i); the
// odd rows of 16 (and, for W = 64, the odd halves) are sorted descending, so
// that the last merges start with the plain exchange 16 (32) lanes apart.
template <int W>
__device__ inline void sort_lanes(uint32_t& lo, uint32_t& hi)
{
    constexpr uint64_t k1 = lanes_clear(1), k2 = lanes_clear(2), k4 = lanes_clear(4), k8 = lanes_clear(8),
                       k16 = lanes_clear(16), k32 = lanes_clear(32);
    sort_step<1>(lo, hi, in_lanes<k1>());
    sort_step<3>(lo, hi, in_lanes<k2>());
    sort_step<1>(lo, hi, in_lanes<k1>());
    sort_step<7>(lo, hi, in_lanes<k4>());
    sort_step<2>(lo, hi, in_lanes<k2>());
    sort_step<1>(lo, hi, in_lanes<k1>());
    // rows of 16: ascending where lane bit 16 is clear
    sort_step<15>(lo, hi, in_lanes<~(k8 ^ k16)>());
    sort_step<4>(lo, hi, in_lanes<~(k4 ^ k16)>());
    sort_step<2>(lo, hi, in_lanes<~(k2 ^ k16)>());
    sort_step<1>(lo, hi, in_lanes<~(k1 ^ k16)>());
    // halves of 32: ascending, or (W = 64) where lane bit 32 is clear
    constexpr uint64_t up = W == 32 ? ~0ull : k32;
    sort_step<16>(lo, hi, in_lanes<~(k16 ^ up)>());
    sort_step<8>(lo, hi, in_lanes<~(k8 ^ up)>());
    sort_step<4>(lo, hi, in_lanes<~(k4 ^ up)>());
    sort_step<2>(lo, hi, in_lanes<~(k2 ^ up)>());
    sort_step<1>(lo, hi, in_lanes<~(k1 ^ up)>());
    if constexpr (W == 64) {
        sort_step<32>(lo, hi, in_lanes<k32>());
        sort_step<16>(lo, hi, in_lanes<k16>());
        sort_step<8>(lo, hi, in_lanes<k8>());
        sort_step<4>(lo, hi, in_lanes<k4>());
        sort_step<2>(lo, hi, in_lanes<k2>());
        sort_step<1>(lo, hi, in_lanes<k1>());
    }
}

// x plus the value CTRL brings in from an earlier lane; lanes it brings none
// (outside the shift's row, or in a row ROWS masks off) add 0.
template <int CTRL, int ROWS = 0xF>
__device__ inline double add_dpp(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
    if constexpr (ROWS == 0xF) {
        lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true);
        hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWS, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWS, 0xF, false);
    }
    return x + f64_of((uint32_t)lo, (uint32_t)hi);
}

// Inclusive prefix sum over segments of W lanes: inside rows of 16 by shifts
// of 1, 2, 4, 8 lanes, then the totals of the rows (halves) before.
template <int W>
__device__ inline double prefix_lanes(double c)
{
    c = add_dpp<0x111>(c);
    c = add_dpp<0x112>(c);
    c = add_dpp<0x114>(c);
    c = add_dpp<0x118>(c);
    c = add_dpp<0x142, 0xA>(c);                        // row 0 -> 1, 2 -> 3
    if constexpr (W == 64) c = add_dpp<0x143, 0xC>(c);   // rows 0, 1 -> 2, 3
    return c;
}

// Two groups sorted side by side on a wave.  W = 32: one per half of 32 lanes;
// W = 64: laid end to end over the lanes (group 0 on lanes 0 .. n0 - 1, n0 + n1
// <= 64; n1 = 0 for a group alone).  The caller loads the lane's row: its time
// t, measurement m and training mark tr, in = the lane holds a row (row `at`).
// A key is the float64 ratio x = m / t with its last six bits replaced by the
// lane, so that one 64-bit value orders by (x, row) and names its row; with W =
// 64 group 1's keys carry 640 more in the exponent, which keeps them after
// group 0's (x lies within 2^-278 .. 2^278 for float32 t and m); rows that do
// not count sort last.  The keys are sorted across the lanes, each takes its
// row's weight, and an inclusive float64 prefix sum gives the cumulative
// weights; a group's multiplier is its first sorted ratio whose cumulative
// weight reaches half the group's total.
// The prefix sum adds in tree order, so C can differ from the row-order sum
// in the last bits; where that moves the choice, the two ratios' objectives
// are equal to rounding (the objective is flat between them when C equals
// half the total).
// Bound: latency.  Counted over the launch the kernel issues 0.42 vector
// instructions per CU-cycle with 11 waves per CU on average (of 28): the sort is
// 21 dependent steps, and a pair with a group beyond 32 rows (36 % of them at 1-40
// rows per group) waits for its rows, which are not loaded ahead.  At 2^16 groups /
// 1.34 M rows k_fit_mult takes 28.6 us; with (x, row) pairs exchanged by
// ds_bpermute (45 per wave) it was held by the LDS pipe and took 53.3.  DPP moves
// and lane-row swaps leave five VALU instructions per step.
template <int W>
__device__ inline void fit_pair_sorted(int64_t g0, bool has1, int n0, bool in, uint32_t at, float t, float m,
                                       bool tr, double* __restrict__ mult, float* __restrict__ T_scaled,
                                       double* st, uint32_t& n_tr, uint32_t& n_held)
{
    const int lane = threadIdx.x & 63;
    const bool seg = W == 32 ? lane >= 32 : lane >= n0;   // the lane's row is group 1's
    const bool ok = in && mult_ok(t, m);
    const double td = t, md = m;
    const double im = recip_f32range(md);
    const double x = quot_f32range(md, td, recip_f32range(td)), w = quot_f32range(td, md, im);   // where ok
    const bool use = ok && tr;
    constexpr uint64_t kLast = 0x7fe0000000000000ull;   // finite, above every key that counts
    constexpr uint64_t kShift = (uint64_t)640 << 52;
    uint64_t key = __builtin_bit_cast(uint64_t, x) + (W == 64 && seg ? kShift : 0ull);
    key = ((use ? key : kLast) & ~63ull) | (uint64_t)lane;
    uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
    sort_lanes<W>(lo, hi);
    int src = (int)(lo & 63u);   // the lane whose row sorted to this lane
    const bool counts = hi < (uint32_t)(kLast >> 32);
    // Ratios that agree in all but the replaced bits are in row order, not
    // yet in the order of those bits: exchange neighbours until none is out
    // of place (odd-even transposition over runs of such ratios; rare).
    const uint32_t plo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0x138, 0xF, 0xF, true);
    const uint32_t phi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0x138, 0xF, 0xF, true);
    const bool run = counts && (lane & (W - 1)) != 0 && phi == hi && ((plo ^ lo) & ~63u) == 0u;
    const uint64_t runs = __ballot(run);   // lane l continues lane l - 1's run
    if (runs != 0ull) {
        double xs = __shfl(x, src, 64);
        for (int pass = 0; pass < 64; ++pass) {
            const double xp = __shfl_up(xs, 1, 64);
            if (__ballot(run && xp > xs) == 0ull) break;
#pragma unroll 1
            for (int par = 0; par < 2; ++par) {
                const bool second = ((lane ^ par) & 1) != 0;   // the upper lane of its pair
                const int pl = second ? lane - 1 : lane + 1;
                const double xo = __shfl(xs, pl & 63, 64);
                const int so = __shfl(src, pl & 63, 64);
                const bool pair = ((second ? runs >> lane : (lane < 63 ? runs >> (lane + 1) : 0ull)) & 1ull) != 0;
                const bool less = xo < xs || (xo == xs && so < src);
                // the lower lane takes the smaller of the pair, the upper the larger
                if (pair && less != second) {
                    xs = xo;
                    src = so;
                }
            }
        }
    }
    double mu0, mu1;
    {
        const double ws = __shfl(use ? w : 0.0, src, 64);
        double c, tot;
        uint64_t h0, h1;
        if constexpr (W == 32) {
            c = prefix_lanes<32>(ws);
            const double t0 = read_lane_f64(c, 31), t1 = read_lane_f64(c, 63);
            tot = seg ? t1 : t0;
            const uint64_t hit = __ballot(counts && c >= 0.5 * tot);
            h0 = hit & 0xFFFFFFFFull;
            h1 = hit & 0xFFFFFFFF00000000ull;
        } else {
            // group 0's counting rows come first; each group's own prefix sum
            const bool first = src < n0;
            const double c0 = prefix_lanes<64>(first ? ws : 0.0), c1 = prefix_lanes<64>(first ? 0.0 : ws);
            const double t0 = read_lane_f64(c0, 63), t1 = read_lane_f64(c1, 63);
            h0 = __ballot(counts && first && c0 >= 0.5 * t0);
            h1 = __ballot(counts && !first && c1 >= 0.5 * t1);
        }
        const int r0 = __builtin_amdgcn_readlane(src, h0 != 0ull ? __builtin_ctzll(h0) : 0);
        const int r1 = __builtin_amdgcn_readlane(src, h1 != 0ull ? __builtin_ctzll(h1) : 0);
        const double x0 = read_lane_f64(x, r0), x1 = read_lane_f64(x, r1);
        mu0 = h0 != 0ull ? x0 : 1.0;
        mu1 = h1 != 0ull ? x1 : 1.0;
    }
    const double mu = seg ? mu1 : mu0;
    if (lane == 0) mult[g0] = mu0;
    if (lane == 1 && has1) mult[g0 + 1] = mu1;
    if (in) T_scaled[at] = (float)(mu * td);
    const double e = __builtin_fabs(__builtin_fma(mu, td, -md)) * im;
    st[0] += use ? e : 0.0;
    st[2] += ok && !tr ? e : 0.0;
    n_tr += (uint32_t)__builtin_popcountll(__ballot(use));
    n_held += (uint32_t)__builtin_popcountll(__ballot(ok && !tr));
}

// One wave per pair of consecutive groups (persistent): two groups of at
// most 32 rows share the wave by halves, two of at most 64 rows together share
// its 64 lanes, others up to 64 rows take it in turn; groups beyond 64 rows
// follow in a second loop, by the candidate scan.  The next pair's rows are
// loaded while this pair is sorted.  Group bounds are
// clamped into [0, n].  Per wave the stats (training loss, count, held-out
// loss, count) accumulate in float64 and each block writes their sums to
// its row.
__device__ inline void group_bounds(const int32_t* __restrict__ off, int64_t g, int64_t n, int64_t& a, int64_t& b)
{
    a = off[g];
    b = off[g + 1];
    a = a < 0 ? 0 : (a > n ? n : a);
    b = b < a ? a : (b > n ? n : b);
}

// A wave's pair of groups: the bounds (wave-uniform) and, where both groups
// have at most 32 rows and group 1 follows group 0 (as non-decreasing offsets
// have it), this lane's row of its half's group, `at` rows after group 0's first.
struct MultPair {
    int32_t a0, b0, a1, b1;   // offsets are 32-bit
    bool joined, fits, in;
    uint32_t at;
    float t, m;
    uint8_t tr;
    __device__ inline void load(int64_t q, int64_t npairs, int64_t n_groups, int64_t n,
                                const int32_t* __restrict__ off, const float* __restrict__ T,
                                const float* __restrict__ meas, const uint8_t* __restrict__ train)
    {
        fits = in = joined = false;
        at = 0;
        t = m = 0.0f;
        tr = 0;
        a0 = b0 = a1 = b1 = 0;
        if (q >= npairs) return;
        int64_t a, b;
        group_bounds(off, 2 * q, n, a, b);
        a0 = (int32_t)a;
        b0 = a1 = b1 = (int32_t)b;
        if (2 * q + 1 < n_groups) {
            group_bounds(off, 2 * q + 1, n, a, b);
            a1 = (int32_t)a;
            b1 = (int32_t)b;
        }
        joined = a1 == b0;
        fits = joined && b0 - a0 <= 32 && b1 - a1 <= 32;
        const uint32_t lane = threadIdx.x & 63u;
        const uint32_t n0 = (uint32_t)(b0 - a0);
        at = lane < 32u ? lane : lane - 32u + n0;
        in = fits && at < (lane < 32u ? n0 : (uint32_t)(b1 - a0));
        if (in) {
            t = (T + a0)[at];
            m = (meas + a0)[at];
            tr = (train + a0)[at];
        }
    }
};

// threads per block of the multiplier sweep: seven blocks per CU (512: 31.6 us
// against 31.2, three blocks of eight waves)
constexpr int kFitBlock = 256;

__global__ __launch_bounds__(kFitBlock) void k_fit_mult(const float* __restrict__ T,
                                                   const float* __restrict__ meas,
                                                   const int32_t* __restrict__ off,
                                                   int64_t n_groups, int64_t n,
                                                   const uint8_t* __restrict__ train,
                                                   double* __restrict__ mult,
                                                   float* __restrict__ T_scaled,
                                                   double* __restrict__ rows)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = wave_id();
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t npairs = (n_groups + 1) >> 1;
    double st[4] = {0.0, 0.0, 0.0, 0.0};
    MultPair cur, nxt;
    cur.load(wave, npairs, n_groups, n, off, T, meas, train);
    bool big = false;   // the wave met a group of more than 64 rows
    uint32_t n_tr = 0, n_held = 0;   // rows of the sorted groups (wave-uniform, below 2^31)
    for (int64_t q = wave; q < npairs; q += nwaves) {
        nxt.load(q + nwaves, npairs, n_groups, n, off, T, meas, train);
        if (cur.fits) {
            fit_pair_sorted<32>(2 * q, 2 * q + 1 < n_groups, 0, cur.in, cur.at, cur.t, cur.m, cur.tr != 0, mult,
                                T_scaled + cur.a0, st, n_tr, n_held);
        } else {
            const int64_t n0 = (int64_t)cur.b0 - cur.a0, n1 = (int64_t)cur.b1 - cur.a1;
            big = big || n0 > 64 || n1 > 64;
            const bool both = cur.joined && n0 + n1 <= 64;
#pragma unroll 1
            for (int h = 0; h < (both ? 1 : 2); ++h) {
                const int64_t g = 2 * q + h, a = h ? cur.a1 : cur.a0;
                const int64_t len = h ? n1 : n0;
                if (g >= n_groups || len > 64) continue;
                const uint32_t rows = (uint32_t)(both ? n0 + n1 : len), at = (uint32_t)lane;
                const bool in = at < rows;
                float t = 0.0f, m = 0.0f;
                bool tr = false;
                if (in) {
                    t = (T + a)[at];
                    m = (meas + a)[at];
                    tr = (train + a)[at] != 0;
                }
                fit_pair_sorted<64>(g, both && g + 1 < n_groups, (int)len, in, at, t, m, tr, mult, T_scaled + a, st,
                                    n_tr, n_held);
            }
        }
        cur = nxt;
    }
    if (lane == 0) {
        st[1] += (double)n_tr;
        st[3] += (double)n_held;
    }
    if (big) {
        for (int64_t q = wave; q < npairs; q += nwaves) {
#pragma unroll 1
            for (int64_t g = 2 * q; g < 2 * q + 2 && g < n_groups; ++g) {
                int64_t a, b;
                group_bounds(off, g, n, a, b);
                if (b - a > 64) fit_group_scan(g, a, b, T, meas, train, mult, T_scaled, st);
            }
        }
    }
    // the block's waves, then one row per block (fixed order)
    __shared__ double red[kFitBlock / 64][4];
    wave_sum<4>(st);
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) red[threadIdx.x >> 6][j] = st[j];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double v = 0.0;
        for (int w = 0; w < kFitBlock / 64; ++w) v += red[w][threadIdx.x];
        rows[(int64_t)blockIdx.x * 4 + threadIdx.x] = v;
    }
}

// Column sums of the blocks' rows (at most kFitMultMaxBlocks of four): thread
// (g, c) adds column c of rows g, g + 64, ..., sixteen loads in flight at a
// time (consecutive threads read consecutive doubles), then the 64 partials of
// a column in g order.  One block, latency only: 3.9 us (5.5 with one thread
// adding a row's four columns and no loads in flight).
__global__ __launch_bounds__(256) void k_fit_mult_reduce(const double* __restrict__ rows, int nrows,
                                                          double* __restrict__ out)
{
    __shared__ double part[256];
    constexpr int K = 16;
    const int g = threadIdx.x >> 2, c = threadIdx.x & 3;
    double v = 0.0;
    for (int r0 = 0; r0 < nrows; r0 += 64 * K) {
        double x[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int r = r0 + 64 * k + g;
            x[k] = r < nrows ? rows[(int64_t)r * 4 + c] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) v += x[k];
    }
    // lanes 4 g' + c of a wave hold column c: add over g', then the waves
#pragma unroll
    for (int m = 4; m <= 32; m <<= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63) < 4) part[(threadIdx.x >> 6) * 4 + c] = v;
    __syncthreads();
    if (threadIdx.x < 4) out[threadIdx.x] = (part[c] + part[4 + c]) + (part[8 + c] + part[12 + c]);
}

// a pair of groups per wave; every block resident at once
int fit_mult_grid(int64_t n_groups)
{
    constexpr int64_t per_block = kFitBlock / 64;
    const int64_t want = ((n_groups + 1) / 2 + per_block - 1) / per_block;
    int64_t b = (int64_t)resident_blocks(reinterpret_cast<const void*>(&k_fit_mult), kFitBlock);
    b = b < want ? b : want;
    b = b < kFitMultMaxBlocks ? b : kFitMultMaxBlocks;
    return (int)(b < 1 ? 1 : b);
}

hipError_t launch_fit_multipliers(const float* T, const float* meas, const int32_t* off,
                                  int64_t n_groups, int64_t n, const uint8_t* train, double* mult,
                                  float* T_scaled, double* rows, double* stats, hipStream_t s)
{
    const int nb = fit_mult_grid(n_groups);
    k_fit_mult<<<nb, kFitBlock, 0, s>>>(T, meas, off, n_groups, n, train, mult, T_scaled, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_fit_mult_reduce<<<1, 256, 0, s>>>(rows, nb, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fusion planning
// ---------------------------------------------------------------------------
// One descriptor row through the caches: the fusion kernels read each row
// once per run that holds it, so these loads are not marked streaming.
__device__ inline Desc<float> load_row(const DescPtrs& d, int64_t i)
{
    Desc<float> x;
    x.F = d.F[i];
    x.B = d.B[i];
    x.r1 = d.r1[i];
    x.r2 = d.r2[i];
    x.r3 = d.r3[i];
    x.K = d.K[i];
    x.u = d.u[i];
    x.W = d.W[i];
    x.v = d.vgpr[i];
    x.s = d.lds[i];
    x.gp = d.gpack[i];
    x.G = d.grid[i];
    return x;
}

// The float64 sums and integer maxima of a run of rows.
struct FuseSum {
    double F = 0.0, Bs = 0.0, E = 0.0, r1 = 0.0, r2 = 0.0, r3 = 0.0, K = 0.0, Ws = 0.0, tc = 0.0, Fmax = -1.0;
    int32_t v = 0, s = 0, g = 0, G = 0, nc = 0, nd = 0, ns = 0, dt = 0;
};

__device__ inline void fuse_ints(FuseSum& a, double F, int32_t v, int32_t s, int32_t gp, int32_t G)
{
    if (F > a.Fmax) {
        a.Fmax = F;
        a.dt = (gp >> 11) & 7;
    }
    a.v = v > a.v ? v : a.v;
    a.s = s > a.s ? s : a.s;
    a.g = (gp & 2047) > a.g ? (gp & 2047) : a.g;
    a.G = G > a.G ? G : a.G;
    a.nc = ((gp >> 14) & 7) > a.nc ? ((gp >> 14) & 7) : a.nc;
    a.nd = ((gp >> 17) & 7) > a.nd ? ((gp >> 17) & 7) : a.nd;
    a.ns += (gp >> 21) & 15;
}

// The combined descriptor of a run (two or more rows) from its sums, float64:
//   F = sum F;  B = max(sum B - 2 sum edges, 0);  r_l byte-weighted;
//   K = sum K;  W = max(sum W - sum edges, 0);  dtype of the first row with
//   the largest F;  u keeps the summed compute time F_k / (u_k P_k) (capped
//   at 1, 1 when F = 0);  VGPRs, LDS, workgroup size, grid, concurrent
//   kernels and devices the largest;  host syncs summed (<= 15);  fused.
__device__ inline void fuse_form(const FuseSum& a, const double* peak, Desc<double>& o)
{
#pragma clang fp contract(off)
    o.F = a.F;
    o.B = a.Bs - 2.0 * a.E > 0.0 ? a.Bs - 2.0 * a.E : 0.0;
    o.r1 = a.Bs > 0.0 ? a.r1 / a.Bs : 0.0;
    o.r2 = a.Bs > 0.0 ? a.r2 / a.Bs : 0.0;
    o.r3 = a.Bs > 0.0 ? a.r3 / a.Bs : 0.0;
    o.K = a.K;
    o.W = a.Ws - a.E > 0.0 ? a.Ws - a.E : 0.0;
    if (a.F > 0.0) {
        const double u = a.F / (peak[a.dt] * a.tc);
        o.u = u < 1.0 ? u : 1.0;
    } else {
        o.u = 1.0;
    }
    o.v = a.v;
    o.s = a.s;
    o.G = a.G;
    const int32_t ns = a.ns < 15 ? a.ns : 15;
    o.gp = a.g | (a.dt << 11) | (a.nc << 14) | (a.nd << 17) | (1 << 20) | (ns << 21);
}

// The combined descriptor of rows a .. a+len-1 (len >= 2).  Returns false if a
// row or an edge is invalid.
__device__ inline bool fuse_rows(const DescPtrs& d, const float* __restrict__ edge,
                                 const double* peak, int64_t a, int32_t len, Desc<double>& o)
{
#pragma clang fp contract(off)
    FuseSum f;
    for (int32_t q = 0; q < len; ++q) {
        const int64_t k = a + q;
        const Desc<float> x = load_row(d, k);
        if (!desc_valid(x)) return false;
        if (q < len - 1) {
            const float ek = edge[k];
            if (!(ek >= 0.0f && ek < __builtin_huge_valf())) return false;
            f.E += (double)ek;
        }
        const double Fk = x.F, Bk = x.B;
        f.F += Fk;
        f.Bs += Bk;
        f.r1 += (double)x.r1 * Bk;
        f.r2 += (double)x.r2 * Bk;
        f.r3 += (double)x.r3 * Bk;
        f.K += (double)x.K;
        f.Ws += (double)x.W;
        if (Fk > 0.0) f.tc += Fk / ((double)x.u * peak[(x.gp >> 11) & 7]);
        fuse_ints(f, Fk, x.v, x.s, x.gp, x.G);
    }
    fuse_form(f, peak, o);
    return true;
}

struct Peaks {
    double p[5];
};

// Coverage byte per row: bits 0-5 the number of runs costed from the row
// (at most 32), bit 7 set when one of them is uncertain in float32.
constexpr uint8_t kPlanCount = 0x3f;
constexpr uint8_t kPlanUncertain = 0x80;

// One thread per row s: the runs of 1 .. m rows starting at s, m = min(R,
// rows left in s's chain), their fusion sums extended one row per step in
// float64 and each fused descriptor evaluated in float32 (the row itself for
// the run of one); cost[(s + len - 1) * R + len - 1] gets the time (+inf for
// runs holding an invalid row or edge and for NaN).  A run is uncertain when
// float32 cannot stand for float64: its float32 time is not finite while its
// rows are valid (and the kernel is not simply infeasible), the time is
// negative, or its working set lies within 1e-6 of the LLC capacity, where
// the hit rate of Table "hlcc-piecewise" jumps.
//
// A block's 256 rows and the R - 1 behind them are loaded once, a row per
// thread, which costs the run of one and leaves in LDS what the sums add per
// row (bytes-weighted hit rates, compute time, validity): up to R runs hold a
// row, and each used to load, convert, multiply, divide and test it again.
// The chains of the block's rows are bracketed by two 64-way searches of the
// offsets (three dependent loads for 2^16 chains; a binary search per row has
// sixteen).
// Bound: VALU issue while the chip is full, uneven waves at the end (over the
// launch 0.66 vector instructions per CU-cycle with 14 waves per CU on average, of
// 24; lanes wait for their wave's longest start, 5.1 of 8 steps used -- ordering
// the block's starts by run count saved the steps and lost as much to the uneven
// waves).  At 2^16 chains / 589 K rows, R =
// 8: 46.2 us; 51.4 with the model's quotients on integers and its selects as
// branches, 68.0 with the rows loaded, converted and tested per run as well.
struct FuseArgs {   // k_fuse_costs's parameters, in order
    DescPtrs d;
    const float* edge;
    const int32_t* off;
    int64_t n_chains, n;
    int32_t R;
    Set S;
    Peaks pk;
    PlanBufs wb;
};

constexpr int kFuseBlock = 256;   // k_fuse_costs' block: one row per thread
constexpr int kFuseTileR = 8;     // run lengths up to this many are staged in LDS

template <int ROWS>   // rows of a block's runs
struct FuseLds {
    double r1[ROWS], r2[ROWS], r3[ROWS];                // hit rates times bytes
    float F[ROWS], B[ROWS], K[ROWS], W[ROWS], tc[ROWS],
        E[ROWS];                                        // E < 0: the edge behind the row is invalid
    int32_t v[ROWS], s[ROWS], gp[ROWS], G[ROWS];        // gp < 0: the row is invalid
    double peak[5];
    int64_t chain[2];   // chains of the block's first and last row
};

// A run's float32 time is uncertain.
__device__ inline bool run_uncertain(float t, int32_t occ, double Wd, const Set& P)
{
    const bool fin = __builtin_isfinite(t);
    bool unc = (!fin && occ != 0) || (fin && t < 0.0f);
    if (P.st.n_levels == 4 && Wd > 0.0) {
        const double c_llc = P.cd.c_llc;
        const double dw = Wd * (1.0 / 1048576.0) - c_llc;
        unc = unc || (dw < 0.0 ? -dw : dw) <= 1e-6 * c_llc;
    }
    return unc;
}

// The last chain c in [lo, hi) with at(c) <= s, given at(lo) <= s, by the
// whole wave: 64 probes per step.
template <typename AT>
__device__ inline int64_t last_chain(int64_t lo, int64_t hi, int64_t s, const AT& at)
{
    const int lane = threadIdx.x & 63;
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + 63) >> 6;
        const int64_t c = lo + step * lane;
        const uint64_t m = __ballot(lane == 0 || (c < hi && at(c) <= s));
        const int64_t at_lane = 63 - __builtin_clzll(m);
        lo = lo + step * at_lane;
        hi = lo + step < hi ? lo + step : hi;
    }
    return lo;
}

template <bool STAGED>   // R <= kFuseTileR
__global__ __launch_bounds__(kFuseBlock) void k_fuse_costs(DescPtrs d, const float* __restrict__ edge,
                                                     const int32_t* __restrict__ off,
                                                     int64_t n_chains, int64_t n, int32_t R, Set S,
                                                     Peaks pk, PlanBufs wb)
{
#pragma clang fp contract(off)
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    // parameters read in place (scalar loads at each use), not held in
    // scalar registers across the run loop
    const Set* sc = WM_KERNARG_PTR(FuseArgs, S);
    const int tl = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * kFuseBlock;
    const int64_t s = s0 + tl;
    if (s == 0) *wb.n_redo = 0u;   // the queue of the planning pass that follows
    constexpr int RMAX = STAGED ? kFuseTileR : kPlanMaxRun;
    __shared__ FuseLds<kFuseBlock + RMAX - 1> L;
    // STAGED: the block's costs are staged in LDS and written out
    // row by row (consecutive lanes, consecutive addresses); a lane's own
    // stores to rows s .. s + R - 1 at entry q would touch R * 8-byte pieces
    // of 64 lines each and leave the L2 as that many partial writes
    __shared__ float tile[STAGED ? (kFuseBlock + kFuseTileR - 1) * kFuseTileR : 1];
    __shared__ uint8_t m_s[kFuseBlock], h0_s[kFuseBlock];
    if (tl < 5) L.peak[tl] = tl == 0 ? pk.p[0] : tl == 1 ? pk.p[1] : tl == 2 ? pk.p[2] : tl == 3 ? pk.p[3] : pk.p[4];
    // the chain holding s: the last c with off[c] <= s (offsets clamped into
    // [0, n] and non-decreasing)
    auto at = [&](int64_t c) -> int64_t {
        const int64_t v = off[c];
        return v < 0 ? 0 : (v > n ? n : v);
    };
    const int64_t s_last = s0 + kFuseBlock <= n ? s0 + kFuseBlock - 1 : n - 1;
    const int wid = __builtin_amdgcn_readfirstlane(tl >> 6);
    if (wid < 2 && n > 0) {
        const int64_t sx = wid ? s_last : s0;
        const int64_t c = at(0) <= sx ? last_chain(0, n_chains, sx, at) : -1;
        if ((tl & 63) == 0) L.chain[wid] = c;
    }
    // this thread's row, and the rows behind the block's last
    Desc<float> x;
    float e = 0.0f;
    if (s < n) {
        x = load_row(d, s);
        e = edge[s];
    }
    __syncthreads();
    const float inf = __builtin_huge_valf();
    // row terms to LDS at position pos
    auto stage = [&](const Desc<float>& y, float ey, int pos) -> bool {
        const bool ok = desc_valid(y);
        const double Bk = y.B;
        float tk = 0.0f;
        if (ok && y.F > 0.0f) tk = y.F / (y.u * (float)L.peak[(y.gp >> 11) & 7]);
        L.F[pos] = y.F;
        L.B[pos] = y.B;
        L.r1[pos] = (double)y.r1 * Bk;
        L.r2[pos] = (double)y.r2 * Bk;
        L.r3[pos] = (double)y.r3 * Bk;
        L.K[pos] = y.K;
        L.W[pos] = y.W;
        L.tc[pos] = tk;
        L.E[pos] = ey >= 0.0f && ey < inf ? ey : -1.0f;
        L.v[pos] = y.v;
        L.s[pos] = y.s;
        L.gp[pos] = ok ? y.gp : -1;
        L.G[pos] = y.G;
        return ok;
    };
    // h0: row s's entries q >= h0 would end runs that start before its chain
    // (never read; written +inf when staged, so that the rows go out whole)
    int32_t m = 0, h0 = 0;
    bool ok = false, unc = false;
    if (s < n) {
        ok = stage(x, e, tl);
        int64_t lo = L.chain[0], hi = L.chain[1] + 1;
        if (lo < 0 && hi > 0 && at(0) <= s) lo = 0;
        if (lo >= 0) {
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (at(mid) <= s) lo = mid; else hi = mid;
            }
            const int64_t b = at(lo + 1);
            if (s < b) {
                m = (int32_t)(b - s < (int64_t)R ? b - s : (int64_t)R);
                const int64_t back = s - at(lo) + 1;
                h0 = back < (int64_t)R ? (int32_t)back : R;
            }
        }
        if (tl < R - 1 && s + kFuseBlock < n) stage(load_row(d, s + kFuseBlock), edge[s + kFuseBlock], kFuseBlock + tl);
        if (m > 0) {
            float t = inf;
            if (ok) {
                const Set& P = uniform_const(sc);
                Eval<float> Ev;
                evaluate<float, false>(P.st, P.cf, x, Ev);
                unc = run_uncertain(Ev.T, Ev.occ, (double)x.W, P);
                t = Ev.T == Ev.T ? Ev.T : inf;
            }
            if (STAGED) tile[tl * R] = t;
            else wb.cost[s * R] = (double)t;
        }
    }
    __syncthreads();
    if (m > 1) {
        double F = x.F, Bs = x.B, r1 = L.r1[tl], r2 = L.r2[tl], r3 = L.r3[tl], K = x.K, Ws = x.W, tc = L.tc[tl],
               Es = 0.0;
        float Fmax = x.F;
        int32_t v = x.v, sl = x.s, G = x.G, dt = (x.gp >> 11) & 7, nd = (x.gp >> 17) & 7, ns = (x.gp >> 21) & 15;
        us2 gc = {(unsigned short)(x.gp & 2047), (unsigned short)((x.gp >> 14) & 7)};   // threads, concurrent kernels
        for (int32_t q = 1; q < m; ++q) {
            const int k = tl + q;
            const float ek = L.E[k - 1], Fk = L.F[k];
            const int32_t gp = L.gp[k];
            ok = ok && ek >= 0.0f && gp >= 0;
            float t = inf;
            if (ok) {
                const Set& P = uniform_const(sc);
                Es += (double)ek;
                F += (double)Fk;
                Bs += (double)L.B[k];
                r1 += L.r1[k];
                r2 += L.r2[k];
                r3 += L.r3[k];
                K += (double)L.K[k];
                Ws += (double)L.W[k];
                tc += (double)L.tc[k];
                if (Fk > Fmax) {   // dtype of the first row with the most flops
                    Fmax = Fk;
                    dt = (gp >> 11) & 7;
                }
                const int32_t vk = L.v[k], sk = L.s[k], Gk = L.G[k], ndk = (gp >> 17) & 7;
                v = vk > v ? vk : v;
                sl = sk > sl ? sk : sl;
                G = Gk > G ? Gk : G;
                gc = __builtin_elementwise_max(gc, us2{(unsigned short)(gp & 2047), (unsigned short)((gp >> 14) & 7)});
                nd = ndk > nd ? ndk : nd;
                ns += (gp >> 21) & 15;
                // the combined descriptor as fuse_rows forms it, rounded to float32
                Desc<float> o;
                o.F = (float)F;
                o.B = (float)(Bs - 2.0 * Es > 0.0 ? Bs - 2.0 * Es : 0.0);
                const double iB = Bs > 0.0 ? quot_f32range(1.0, Bs, recip_f32range(Bs)) : 0.0;
                o.r1 = (float)(r1 * iB);
                o.r2 = (float)(r2 * iB);
                o.r3 = (float)(r3 * iB);
                o.K = (float)K;
                const double Wd = Ws - Es > 0.0 ? Ws - Es : 0.0;
                o.W = (float)Wd;
                o.u = 1.0f;
                if (F > 0.0) {
                    // (an infinite compute time is redone in float64; with a
                    // zero one u is 1, as for any not below 1)
                    const double den = L.peak[dt] * tc, u = quot_f32range(F, den, recip_f32range(den));
                    o.u = (float)(u < 1.0 ? u : 1.0);
                }
                o.v = v;
                o.s = sl;
                o.G = G;
                o.gp = (int32_t)gc[0] | (dt << 11) | ((int32_t)gc[1] << 14) | (nd << 17) | (1 << 20) |
                       ((ns < 15 ? ns : 15) << 21);
                Eval<float> Ev;
                evaluate<float, false, kFused>(P.st, P.cf, o, Ev);
                unc = unc || run_uncertain(Ev.T, Ev.occ, Wd, P) || !(tc < __builtin_huge_val());
                t = Ev.T == Ev.T ? Ev.T : inf;
            }
            if (STAGED) tile[k * R + q] = t;
            else wb.cost[(s + q) * R + q] = (double)t;
        }
    }
    if (s < n) wb.cov[s] = (uint8_t)(m | (unc ? kPlanUncertain : 0));
    if (!STAGED) return;
    if (s < n)
        for (int32_t q = h0; q < R; ++q) tile[tl * R + q] = inf;
    m_s[tl] = (uint8_t)m;
    h0_s[tl] = (uint8_t)h0;
    __syncthreads();
    // Entry (r, q) of a row here comes from the run starting at r - q: from
    // this tile when q <= r (a run of a start here, or row r's +inf when that
    // run leaves its chain) or when q >= h0[r] (+inf); the previous block
    // writes the rest (runs that start in its rows).  r = idx / R exactly
    // (idx < 2^12, R <= 8: the float quotient is at least 1/16 from an integer).
    const float inv_r = 1.0f / (float)R;
    const int64_t left = n - s0;
    const int nrow = left < kFuseBlock ? (int)left : kFuseBlock;
    for (int idx = tl; idx < nrow * R; idx += kFuseBlock) {
        const int r = (int)(((float)idx + 0.5f) * inv_r), q = idx - r * R;
        if (q <= r || q >= (int)h0_s[r]) wb.cost[s0 * R + idx] = (double)tile[idx];
    }
    // runs that start here and end in the next block's first R - 1 rows
    for (int idx = tl; idx < (R - 1) * R; idx += kFuseBlock) {
        const int i = (int)(((float)idx + 0.5f) * inv_r), q = idx - i * R;
        const int st = kFuseBlock + i - q;   // their start, a row here when q > i
        if (q > i && q < (int)m_s[st] && s0 + kFuseBlock + i < n)
            wb.cost[(s0 + kFuseBlock + i) * R + q] = (double)tile[(kFuseBlock + i) * R + q];
    }
}

// Decision margin below which a float32 plan is re-decided in float64.  A
// decision compares two sums of run times, each off by at most the float32
// model's relative error e relative to itself, so it can only flip within
// 2e; the largest e measured on fused runs against the float64 model is
// about 3e-7, so 1e-5 is some 17 times 2e (a test holds it to at least 4).
constexpr double kPlanWindow = 1e-5;

// The dynamic programme runs on groups of G lanes (2 G the power of two >= R,
// at least 2), one chain per group: lane gl of a group stands for the runs of 2
// gl + 1 and 2 gl + 2 rows ending at the current row j and holds prev[] = best
// over the rows before each, so that a step is two adds, a group minimum
// (shortest run on ties, as a sequential scan with strict improvement picks)
// that carries the runner-up along, and a shift of prev by one run.  Groups of
// one wave step together over their chains.  With a lane per run the lane
// exchanges and selects of a step, which every lane repeats, took 2.3 times the
// instructions per chain: k_plan 35.9 us at 2^16 chains, R = 8, now 22.4, of
// which about half is the 37.7 MB cost table coming in and the rest the
// programme's steps.
template <int G>
struct PlanGroup {
    int gl;        // lane in group
    int64_t c;     // chain (or -1)
    int64_t a;     // first row
    int32_t L;     // rows (offsets are 32-bit)
};

template <int G>
__device__ inline PlanGroup<G> plan_group(int64_t c, int64_t n_chains, const int32_t* off, int64_t n)
{
    PlanGroup<G> g;
    const int lane = threadIdx.x & 63;
    g.gl = lane & (G - 1);
    g.c = c >= 0 && c < n_chains ? c : -1;
    g.a = 0;
    g.L = 0;
    if (g.c >= 0) {
        int64_t a = off[c], b = off[c + 1];
        a = a < 0 ? 0 : (a > n ? n : a);
        b = b < a ? a : (b > n ? n : b);
        g.a = a;
        g.L = (int32_t)(b - a);
    }
    return g;
}

template <int G>
__device__ inline uint64_t group_mask(const PlanGroup<G>& g)
{
    static_assert(G < 64, "a group is part of the wave");
    return ((1ull << G) - 1ull) << ((threadIdx.x & 63) - g.gl);
}

// Lane moves inside a row of 16 lanes (DPP): CTRL 0x140 mirrors the row,
// 0x141 mirrors each half row, 0x4E and 0xB1 swap lanes 2 and 1 apart in each
// quad; 0x138 shifts the wave up by one lane (the lane shifted in is never
// used, so no old value is kept: that would cost a copy per move).
template <int CTRL>
__device__ inline int32_t dpp32(int32_t x)
{
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ inline double dpp64(double x)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    return f64_of((uint32_t)dpp32<CTRL>((int32_t)(uint32_t)u), (uint32_t)dpp32<CTRL>((int32_t)(uint32_t)(u >> 32)));
}

// A group's best run so far: value, length and the runner-up's value.
struct PlanBest {
    double v, second;
    int32_t len;
};

// One step of the group reduction, each doubling the lanes a value covers:
// the row mirror (G >= 16), the half-row mirror (G >= 8), then 2 and 1 apart.
template <int CTRL, bool MARGIN>
__device__ inline void best_step(PlanBest& b)
{
    const double ov = dpp64<CTRL>(b.v);
    const int32_t ol = dpp32<CTRL>(b.len);
    const bool take = (ov < b.v) | ((ov == b.v) & (ol < b.len));
    if (MARGIN) {
        const double os = dpp64<CTRL>(b.second), lose = take ? b.v : ov, s = os < b.second ? os : b.second;
        b.second = lose < s ? lose : s;
    }
    b.v = take ? ov : b.v;
    b.len = take ? ol : b.len;
}

template <int G, bool MARGIN>
__device__ inline void group_best(PlanBest& b)
{
    if constexpr (G >= 16) best_step<0x140, MARGIN>(b);
    if constexpr (G >= 8) best_step<0x141, MARGIN>(b);
    if constexpr (G >= 4) best_step<0x4E, MARGIN>(b);
    if constexpr (G >= 2) best_step<0xB1, MARGIN>(b);
}

struct PlanState {
    double prev[2], single, best;   // single: the all-singles sum (first lane)
    uint64_t cut[2];                // the batch's cut lengths, rows 0-7 and 8-15
};

// The programme over the group's chain, costs from wb.cost.  With COV, the
// chain's coverage bytes are read with the first batch of costs and `run`
// is narrowed to covered chains without an uncertain run (covered and unc
// report them); without, `run` is taken as given.  With MARGIN, `close` is set
// when a decision's runner-up is within kPlanWindow.
template <int G, bool MARGIN, bool COV>
__device__ inline void plan_run(const PlanGroup<G>& g, bool& run, int32_t R, const PlanBufs& wb,
                                PlanState& ps, bool& close, bool& covered, bool& unc)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    const double inf = __builtin_huge_val();
    const int32_t q0 = 2 * g.gl;   // the lane's runs have q0 + 1 and q0 + 2 rows
    ps.prev[0] = ps.prev[1] = ps.single = ps.best = 0.0;
    ps.cut[0] = ps.cut[1] = 0ull;
    covered = true;
    unc = false;
    const double* at = wb.cost + g.a * R + q0;   // this lane's cost entries of the next row
    for (PlanRows rows(g.L); __ballot(run && rows.more()) != 0ull; rows.next()) {
        const int32_t left = run ? rows.left() : 0;
        if (rows.at > 0u && left > 0) {   // the last batch's cut lengths make room
            for (int r = g.gl; r < kPlanBatch; r += G)
                wb.cut[g.a + (int64_t)(rows.at - kPlanBatch) + r] =
                    (uint8_t)((r < 8 ? ps.cut[0] : ps.cut[1]) >> (8 * (r & 7)));
            ps.cut[0] = ps.cut[1] = 0ull;
        }
        double t[kPlanBatch][2];
        // runs longer than the rows so far or than R do not exist
        const int32_t before = rows.at < (uint32_t)kPlanMaxRun ? (int32_t)rows.at : kPlanMaxRun;
#pragma unroll
        for (int k = 0; k < kPlanBatch; ++k) {
            d2 x = {inf, inf};
            if (k < left && q0 < R) {
                if ((R & 1) == 0) x = *(const d2*)at;   // rows of an even length: 16-byte aligned pairs
                else {
                    x[0] = at[0];
                    if (q0 + 1 < R) x[1] = at[1];
                }
            }
            at += R;
            t[k][0] = q0 <= k + before ? x[0] : inf;
            t[k][1] = q0 + 1 <= k + before && q0 + 1 < R ? x[1] : inf;
        }
        if (COV && rows.at == 0u) {
            // coverage and uncertain runs, G rows at a time (loads in flight
            // with the costs above)
            const uint64_t gm = group_mask(g);
            bool bad = false, u = false;
            for (uint32_t i = (uint32_t)g.gl; i < rows.L; i += G) {
                const uint8_t cv = wb.cov[g.a + i];
                const uint32_t want = rows.L - i < (uint32_t)R ? rows.L - i : (uint32_t)R;
                bad = bad || (uint32_t)(cv & kPlanCount) != want;
                u = u || (cv & kPlanUncertain) != 0;
            }
            covered = (__ballot(bad) & gm) == 0ull;
            unc = (__ballot(u) & gm) != 0ull;
            run = run && covered && !unc;
        }
#pragma unroll
        for (int k = 0; k < kPlanBatch; ++k) {
            const bool live = run && k < left;
            if (__ballot(live) == 0ull) break;
            const double v0 = ps.prev[0] + t[k][0], v1 = ps.prev[1] + t[k][1];
            if (live) ps.single += t[k][0];   // (the first lane's run is the row alone)
            const bool second = v1 < v0;
            PlanBest b{second ? v1 : v0, second ? v0 : v1, second ? q0 + 2 : q0 + 1};
            group_best<G, MARGIN>(b);
            if (MARGIN) close = close | (live & (b.second < inf) & (b.second - b.v <= kPlanWindow * b.second));
            const double up = dpp64<0x138>(ps.prev[1]);   // lane - 1's longer run
            ps.prev[1] = ps.prev[0];
            ps.prev[0] = g.gl == 0 ? b.v : up;
            if (live) {
                ps.cut[k >> 3] |= (uint64_t)(uint32_t)b.len << (8 * (k & 7));
                ps.best = b.v;
            }
        }
    }
}

// Start flags of the chosen plan: the run starts found by following the cut
// lengths back from the chain's end, batch by batch.  `live` marks groups that
// write their chain's flags.
template <int G>
__device__ inline void plan_starts(const PlanGroup<G>& g, bool live, const PlanState& ps,
                                   const uint8_t* __restrict__ cut, uint8_t* __restrict__ start)
{
    const int32_t L = live ? g.L : 0;
    // cut bytes of earlier batches were stored by the group's lanes: make them
    // visible to the loads below
    if (__ballot(L > kPlanBatch) != 0ull) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    uint64_t c0 = ps.cut[0], c1 = ps.cut[1];
    int32_t jj = L;   // the next run start found (row in the chain)
    for (int32_t w0 = last_batch(L); __ballot(w0 >= 0) != 0ull; w0 -= kPlanBatch) {
        if (w0 < 0) {
            w0 = 0;   // (stays negative after the step)
            continue;
        }
        if (batch_stored(w0, L)) {
            __builtin_memcpy(&c0, cut + g.a + w0, 8);
            __builtin_memcpy(&c1, cut + g.a + w0 + 8, 8);
        }
        uint32_t flags = jj < L && jj >= w0 ? 1u << (jj - w0) : 0u;   // found from a later batch
        while (jj > w0) {
            const int r = jj - 1 - w0;
            const int32_t len = (int32_t)((r < 8 ? c0 : c1) >> (8 * (r & 7))) & 0xff;
            jj -= len > 0 ? len : 1;
            if (jj >= w0) flags |= 1u << (jj - w0);
        }
        for (int r = g.gl; r < kPlanBatch; r += G)
            if (r < L - w0) start[g.a + w0 + r] = (uint8_t)((flags >> r) & 1u);
    }
}

// Float32 pass: one group per chain steps through the costs of
// k_fuse_costs.  A chain whose rows were not all costed as its own (offsets
// that are not non-decreasing) gets NaN totals and no start flags; a chain
// holding an uncertain run or a close decision is queued for the float64
// redo; the rest get their totals and start flags.
constexpr int kPlanBlock = 256;    // threads per block of the planning pass (4 blocks per CU)

template <int G>
__global__ __launch_bounds__(kPlanBlock) void k_plan(const int32_t* __restrict__ off,
                                                      int64_t n_chains, int64_t n, int32_t R,
                                                      PlanBufs wb, double* __restrict__ total,
                                                      double* __restrict__ unfused,
                                                      uint8_t* __restrict__ start)
{
    __shared__ uint32_t wave_q[kPlanBlock / 64 + 1];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t gid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
    const PlanGroup<G> g = plan_group<G>(gid, n_chains, off, n);
    const uint64_t gm = group_mask(g);
    PlanState ps;
    bool run = g.c >= 0, close = false, covered, unc;
    plan_run<G, true, true>(g, run, R, wb, ps, close, covered, unc);
    close = unc || (__ballot(close) & gm) != 0ull;
    const bool done = g.c >= 0 && covered && !close;
    // queue slots: one atomic per block, the waves' shares by a prefix in LDS
    const bool queue = g.c >= 0 && covered && close && g.gl == 0;
    const uint64_t qm = __ballot(queue);
    if (lane == 0) wave_q[wid] = (uint32_t)__builtin_popcountll(qm);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0u;
        for (int w = 0; w < kPlanBlock / 64; ++w) {
            const uint32_t c = wave_q[w];
            wave_q[w] = sum;
            sum += c;
        }
        wave_q[kPlanBlock / 64] = sum != 0u ? atomicAdd(wb.n_redo, sum) : 0u;
    }
    __syncthreads();
    const uint32_t slot = wave_q[kPlanBlock / 64] + wave_q[wid] +
                          (uint32_t)__builtin_popcountll(qm & ((1ull << lane) - 1ull));
    if (g.c >= 0 && g.gl == 0) {
        if (!covered) {
            total[g.c] = __builtin_nan("");
            unfused[g.c] = __builtin_nan("");
        } else if (done) {
            total[g.c] = ps.best;
            unfused[g.c] = ps.single;
        } else if ((int64_t)slot < n) {
            // non-empty chains that partition the rows number at most n
            wb.redo[slot] = g.c;
        } else {
            total[g.c] = __builtin_nan("");
            unfused[g.c] = __builtin_nan("");
        }
    }
    plan_starts(g, done, ps, wb.cut, start);
}

// The queue's length, clamped to what the queue can hold.
__device__ inline int64_t redo_count(const PlanBufs& wb, int64_t n_chains, int64_t n)
{
    int64_t nq = *wb.n_redo;
    nq = nq < n_chains ? nq : n_chains;
    return nq < n ? nq : n;
}

// Float64 redo.  Wave w takes entries w, w + waves, ... of the queue, as many at
// once as it runs programmes side by side (64 / G), so that a chain has a wave to
// itself until the queue is longer than the waves.  Chains of up to kRedoRows rows
// together are loaded once, a row per lane, into LDS with what the sums add per
// row (products, compute time, validity), and their candidate runs, chain by
// chain and (length, end) in order of length, are laid end to end over the lanes;
// a longer chain goes alone, through memory row by row.  Each run is formed in
// the order and arithmetic of fuse_rows and evaluated with the float64 model, and
// the costs replace the chains' float32 ones; after all of the wave's costs,
// groups of G lanes run its chains' programmes over them (in one loop with the
// costs, the model's constants stay in registers across the programme: 25 to 77
// spilled, 10 us of the call).
// Bound: latency with a short queue (one chain of loads, sums, one or two float64
// evaluations and the programme per wave), float64 issue with a long one, as
// chains of repeated kernels make it.  The call over 2^16 chains of 2-16 rows, R =
// 8, 4 % of them queued: 96 us, as with a wave per chain at any length of the
// queue; half of them repeated kernels (29 % queued) 182 -> 141, all queued 395
// -> 231; all queued with 2 rows, R = 2, 187 -> 38.5, and 2-5 rows, R = 8, 240 ->
// 88 (57 and 143 with separate cost and programme launches).
constexpr int kRedoRows = 64;

struct RedoArgs {   // k_redo's parameters, in order
    DescPtrs d;
    const float* edge;
    const int32_t* off;
    int64_t n_chains, n;
    int32_t R;
    Set S;
    Peaks pk;
};

struct RedoLds {
    double F[kRedoRows], B[kRedoRows], r1[kRedoRows], r2[kRedoRows], r3[kRedoRows], K[kRedoRows], W[kRedoRows],
        tc[kRedoRows], E[kRedoRows];   // E < 0: the edge behind the row is invalid
    int32_t v[kRedoRows], s[kRedoRows], gp[kRedoRows], G[kRedoRows];   // gp < 0: the row is invalid
    // the chains at hand: first row, rows, and how many rows and runs they and
    // those before them have (a chain of more than kRedoRows rows counts one row
    // more than that and no runs)
    int32_t first[64], len[64], rows_to[64], runs_to[64];
};

__device__ inline void redo_stage(RedoLds& L, const DescPtrs& d, const float* __restrict__ edge, const double* peak,
                                  int64_t row, bool has_edge, int pos)
{
#pragma clang fp contract(off)
    const Desc<float> x = load_row(d, row);
    const float e = has_edge ? edge[row] : 0.0f;
    const bool ok = desc_valid(x);
    const double Bk = x.B, Fk = x.F;
    L.F[pos] = Fk;
    L.B[pos] = Bk;
    L.r1[pos] = (double)x.r1 * Bk;
    L.r2[pos] = (double)x.r2 * Bk;
    L.r3[pos] = (double)x.r3 * Bk;
    L.K[pos] = (double)x.K;
    L.W[pos] = (double)x.W;
    L.tc[pos] = ok && Fk > 0.0 ? Fk / ((double)x.u * peak[(x.gp >> 11) & 7]) : 0.0;
    L.E[pos] = e >= 0.0f && e < __builtin_huge_valf() ? (double)e : -1.0;
    L.v[pos] = x.v;
    L.s[pos] = x.s;
    L.gp[pos] = ok ? x.gp : -1;
    L.G[pos] = x.G;
}

// fuse_rows over staged rows p .. p + len - 1
__device__ inline bool fuse_staged(const RedoLds& L, const double* peak, int p, int32_t len, Desc<double>& o)
{
#pragma clang fp contract(off)
    FuseSum a;
    bool ok = true;
    for (int32_t q = 0; q < len; ++q) {
        const int k = p + q;
        const int32_t gp = L.gp[k];
        const double e = q < len - 1 ? L.E[k] : 0.0;
        ok = ok && gp >= 0 && e >= 0.0;
        a.E += e;
        a.F += L.F[k];
        a.Bs += L.B[k];
        a.r1 += L.r1[k];
        a.r2 += L.r2[k];
        a.r3 += L.r3[k];
        a.K += L.K[k];
        a.Ws += L.W[k];
        a.tc += L.tc[k];
        fuse_ints(a, L.F[k], L.v[k], L.s[k], gp, L.G[k]);
    }
    if (ok) fuse_form(a, peak, o);
    return ok;
}

// sum of v over the lanes up to this one (every lane active)
__device__ inline int32_t lanes_sum(int32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t o = __shfl_up(v, d, 64);
        v += lane >= d ? o : 0;
    }
    return v;
}

// the first k in [k0, k1) with to[k] above x, to[] not decreasing and to[k1 - 1] > x
__device__ inline int first_above(const int32_t* to, int32_t x, int k0, int k1)
{
    int hi = k1 - 1;
    while (k0 < hi) {
        const int mid = (k0 + hi) >> 1;
        if (to[mid] > x) hi = mid;
        else k0 = mid + 1;
    }
    return k0;
}

template <int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_redo(DescPtrs d, const float* __restrict__ edge,
                                               const int32_t* __restrict__ off, int64_t n_chains, int64_t n,
                                               int32_t R, Set S, Peaks pk, PlanBufs wb,
                                               double* __restrict__ total, double* __restrict__ unfused,
                                               uint8_t* __restrict__ start)
{
    __shared__ RedoLds lds[4];
    const int lane = threadIdx.x & 63;
    const int64_t wave = wave_id();
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    RedoLds& L = lds[__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))];
    const double inf = __builtin_huge_val();
    const int64_t nq = redo_count(wb, n_chains, n);
    constexpr int kSide = 64 / G;   // programmes side by side
    // the wave's chains are entries wave, wave + nwaves, ... of the queue; lane k
    // (or group k) takes the k-th of the next kSide
    const auto entry = [&](int64_t e, int k) -> int64_t {
        const int64_t i = e + k * nwaves;
        return k < kSide && i < nq ? wb.redo[i] : -1;
    };
    for (int64_t e = wave; e < nq; e += kSide * nwaves) {
        int m;   // chains at hand
        {
            const int64_t id = entry(e, lane);
            m = __popcll(__ballot(id >= 0));
            const PlanGroup<64> c = plan_group<64>(id, n_chains, off, n);
            const int32_t r = c.L < R ? c.L : R;
            const int32_t rows = c.L <= kRedoRows ? c.L : kRedoRows + 1;
            const int32_t runs = c.L <= kRedoRows ? r * c.L - r * (r - 1) / 2 : 0;   // sum over len <= r of L - len + 1
            L.first[lane] = (int32_t)c.a;
            L.len[lane] = c.L;
            L.rows_to[lane] = m > 1 ? lanes_sum(rows) : rows;
            L.runs_to[lane] = m > 1 ? lanes_sum(runs) : runs;
        }
        wave_lds_sync();
        const double* peak = uniform_const(WM_KERNARG_PTR(RedoArgs, pk)).p;
        for (int k0 = 0, row0 = 0, run0 = 0; k0 < m;) {   // row0, run0: of the chains before k0
            // chains k0 .. k1 - 1: as many as fit, or one that does not
            const int fit = __popcll(__ballot(lane >= k0 && lane < m && L.rows_to[lane] - row0 <= kRedoRows));
            const bool staged = fit > 0;
            const int k1 = k0 + (staged ? fit : 1);
            int64_t runs = __builtin_amdgcn_readfirstlane(L.runs_to[k1 - 1]) - run0;
            if (staged) {
                if (row0 + lane < L.rows_to[k1 - 1]) {
                    const int k = first_above(L.rows_to, row0 + lane, k0, k1);
                    const int32_t j = row0 + lane - (k > 0 ? L.rows_to[k - 1] : 0);
                    redo_stage(L, d, edge, peak, (int64_t)L.first[k] + j, j + 1 < L.len[k], lane);
                }
                wave_lds_sync();
            } else {   // longer than R
                runs = (int64_t)R * __builtin_amdgcn_readfirstlane(L.len[k0]) - R * (R - 1) / 2;
            }
            for (int64_t q = lane; q < runs; q += 64) {
                const int k = staged ? first_above(L.runs_to, run0 + (int32_t)q, k0, k1) : k0;
                const int64_t a = L.first[k];
                const int32_t len_c = L.len[k];
                // its place x among the chain's runs -> (len, j): lengths in
                // increasing order, ends j = len - 1 .. len_c - 1
                int64_t x = q;
                if (k > k0) x -= L.runs_to[k - 1] - run0;
                int32_t len = 1;
                while (len < R && x >= len_c - len + 1) {
                    x -= len_c - len + 1;
                    ++len;
                }
                const int64_t s = a + x;   // the run's first row
                double* out = wb.cost + (s + len - 1) * R + (len - 1);
                asm("" : "+v"(out));   // formed before the evaluation, which leaves no register for its parts
                Desc<double> y;
                bool ok;
                if (len == 1) {
                    y = widen(load_row(d, s));
                    ok = true;
                } else if (staged) {
                    ok = fuse_staged(L, peak, (k > 0 ? L.rows_to[k - 1] : 0) - row0 + (int)x, len, y);
                } else {
                    ok = fuse_rows(d, edge, peak, s, len, y);
                }
                double t = inf;
                if (ok) {
                    const Set& P = uniform_const(WM_KERNARG_PTR(RedoArgs, S));
                    Eval<double> E;
                    evaluate<double, false>(P.st, P.cd, y, E);
                    t = E.T == E.T ? E.T : inf;
                }
                *out = t;
            }
            row0 = __builtin_amdgcn_readfirstlane(L.rows_to[k1 - 1]);
            run0 = __builtin_amdgcn_readfirstlane(L.runs_to[k1 - 1]);
            wave_lds_sync();   // the rows are rewritten next
            k0 = k1;
        }
        wave_lds_sync();   // the chains at hand are rewritten next
    }
    // the wave's costs, read back by other lanes of it
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    for (int64_t e = wave; e < nq; e += kSide * nwaves) {
        const int k = lane / G;
        const int64_t c = entry(e, k);
        PlanGroup<G> g;
        if (wave + kSide * nwaves < nq) {
            g = plan_group<G>(c, n_chains, off, n);
        } else {   // still in LDS
            g.gl = lane & (G - 1);
            g.c = c;
            g.a = L.first[k];
            g.L = L.len[k];   // 0 past the chains at hand
        }
        PlanState ps;
        bool run = g.c >= 0, unused = false, covered, unc;
        plan_run<G, false, false>(g, run, R, wb, ps, unused, covered, unc);
        if (g.c >= 0 && g.gl == 0) {
            total[g.c] = ps.best;
            unfused[g.c] = ps.single;
        }
        plan_starts(g, g.c >= 0, ps, wb.cut, start);
    }
}

struct PlanCall {
    DescPtrs d;
    const float* edge;
    const int32_t* off;
    int64_t n_chains, n;
    int32_t R;
    Peaks pk;
    PlanBufs wb;
    double *total, *unfused;
    uint8_t* start;
};

// the programme over the float32 costs, then the queued chains in float64
template <int G>
static hipError_t plan_launch(const PlanCall& p, const Set& S, hipStream_t s)
{
    const int64_t per_block = kPlanBlock / G;   // chains per block
    const int64_t nb = (p.n_chains + per_block - 1) / per_block;
    k_plan<G><<<(unsigned)nb, kPlanBlock, 0, s>>>(p.off, p.n_chains, p.n, p.R, p.wb, p.total, p.unfused, p.start);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t want = (p.n_chains + 3) / 4;   // a chain per wave
    int64_t b = (int64_t)resident_blocks(reinterpret_cast<const void*>(&k_redo<G>), 256);
    b = b < want ? b : want;
    k_redo<G><<<(unsigned)(b < 1 ? 1 : b), 256, 0, s>>>(p.d, p.edge, p.off, p.n_chains, p.n, p.R, S, p.pk, p.wb, p.total,
                                                       p.unfused, p.start);
    return hipGetLastError();
}

hipError_t launch_plan_fusion(const DescPtrs& d, const float* edge, const int32_t* off,
                              int64_t n_chains, int64_t n, int32_t R, const Set& S,
                              const double* peaks, const PlanBufs& wb, double* total,
                              double* unfused, uint8_t* start, hipStream_t s)
{
    if (n_chains <= 0) return hipSuccess;
    PlanCall p{d, edge, off, n_chains, n, R, {}, wb, total, unfused, start};
    for (int t = 0; t < 5; ++t) p.pk.p[t] = peaks[t];
    // at least one block, so that the queue's length is cleared even with no rows
    const int64_t nb = n > 0 ? (n + kFuseBlock - 1) / kFuseBlock : 1;
    if (R <= kFuseTileR)
        k_fuse_costs<true><<<(unsigned)nb, kFuseBlock, 0, s>>>(d, edge, off, n_chains, n, R, S, p.pk, wb);
    else
        k_fuse_costs<false><<<(unsigned)nb, kFuseBlock, 0, s>>>(d, edge, off, n_chains, n, R, S, p.pk, wb);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // lanes per chain: the power of two holding R runs, two per lane (R <= 32)
    if (R <= 2) return plan_launch<1>(p, S, s);
    if (R <= 4) return plan_launch<2>(p, S, s);
    if (R <= 8) return plan_launch<4>(p, S, s);
    if (R <= 16) return plan_launch<8>(p, S, s);
    return plan_launch<16>(p, S, s);
}

}  // namespace wm
