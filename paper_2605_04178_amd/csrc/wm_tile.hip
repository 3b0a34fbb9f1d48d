// wm_tile.hip -- gfx950 kernel of occupancy-driven tile selection (Section
// IV-B, adaptive tile selection): every candidate GEMM tile of a shape becomes
// a kernel descriptor whose predicted time is its cost, and the cheapest wins.
//
// Layout: shapes are structure-of-arrays, candidate codes one flat uint32
// array with CSR offsets per shape.  A wave takes a run of consecutive shapes
// and lays their candidate lists end to end over its lanes (float32 costs kept
// in LDS); the float64 re-evaluations of the near-minimum windows queue up in
// LDS and run on all lanes of the block.
#include "wm_device.hpp"
#include "wm_shares.hpp"

namespace wm {

// GEMM tile -> descriptor.  Tile sizes are powers of two, so the grid, the
// K steps and the panel sizes are shifts of 32-bit integers (every padded
// extent is below 2^32).  Flops and bytes are formed in double from those exact
// integers: exact while below 2^53, and never overflowing.
__device__ inline bool derive_tile(int32_t M, int32_t N, int32_t Kd, int32_t t, uint32_t code,
                                   int wave_shift, Desc<double>& x)
{
#pragma clang fp contract(off)
    const uint32_t kdc = (code >> 4) & 3u;
    if ((code >> 9) != 0u || kdc == 3u || M < 1 || N < 1 || Kd < 1 || t < 0 || t > 3) return false;
    const uint32_t lmt = 5u + (code & 3u), lnt = 5u + ((code >> 2) & 3u), lkd = 4u + kdc;
    const uint32_t wpw = ((code >> 6) & 7u) + 1u;
    const uint32_t le = 3u - (uint32_t)t;          // element bytes 8, 4, 2, 1
    const uint32_t eo = t == 3 ? 2u : (1u << le);  // fp8 writes 16-bit results
    const uint32_t acc = t == 0 ? 2u : 1u;
    const uint32_t gm = ((uint32_t)M + (1u << lmt) - 1u) >> lmt;
    const uint32_t gn = ((uint32_t)N + (1u << lnt) - 1u) >> lnt;
    const uint32_t Ks = ((uint32_t)Kd + (1u << lkd) - 1u) >> lkd;
    const uint64_t G = (uint64_t)gm * gn;
    const uint32_t g = wpw << wave_shift;
    if (G > 0x7fffffffull || g > 1024u) return false;
    const uint32_t pan = ((1u << lmt) + (1u << lnt)) << (lkd + le);   // (mt + nt) kd e <= 2^18
    const double fM = (double)(uint32_t)M, fN = (double)(uint32_t)N, fK = (double)(uint32_t)Kd;
    const double Bi = (double)(uint32_t)G * (double)Ks * (double)pan + fM * fN * (double)eo;
    const double Ui = (fM * fK + fK * fN) * (double)(1u << le) + fM * fN * (double)eo;
    x.F = (double)2 * (double)(gm << lmt) * (double)(gn << lnt) * (double)(Ks << lkd);
    x.B = Bi;
    const double r2 = (double)1 - Ui * Ar<double>::rcp(Bi);
    x.r2 = r2 > (double)0 ? r2 : (double)0;
    x.r1 = (double)0;
    x.r3 = (double)0;
    x.K = (double)Ks;
    x.u = (double)1;
    x.W = (double)0;
    // VGPRs: accumulators and the panel share per thread (numerators below
    // 2^19, divisors at most 4096: udiv21 is exact)
    x.v = (int32_t)(udiv21((acc << (lmt + lnt)) + g - 1u, g) + udiv21(pan + 4u * g - 1u, 4u * g) + 16u);
    x.s = (int32_t)(2u * pan);
    x.gp = (int32_t)g | (t << 11);
    x.G = (int32_t)G;
    return true;
}

// float64 cost of one candidate; invalid codes and infeasible tiles cost +inf
__device__ inline double exact_cost(const Set& S, int32_t M, int32_t N, int32_t K, int32_t t, uint32_t code)
{
    const double inf = __builtin_huge_val();
    Desc<double> x;
    if (!derive_tile(M, N, K, t, code, S.st.wave_shift, x)) return inf;
    Eval<double> E;
    evaluate<double, false, kTile>(S.st, S.cd, x, E);
    return E.T == E.T ? E.T : inf;
}

// ---------------------------------------------------------------------------
// float32 cost of one candidate: the same terms in the form that costs the
// fewest vector instructions: 2^16 shapes with 3.4e6 candidates took 16.5e6 of them
// and 33.2 us with the descriptor formed and evaluated as any other, and take 9.7e6
// and 28.2 us.
//   - Tile sizes and everything that follows from them alone are powers of two:
//     their float forms are built from their exponents.
//   - What only the shape decides (compulsory traffic, the dtype's peak) sits in
//     the shape's record.
//   - The quotients run in float as in occupancy(), VGPRs per thread included, and
//     one reciprocal of the waves per workgroup serves four of them.
// Invalid codes and infeasible tiles cost +inf.  No term can be NaN: parameters
// are finite with positive bandwidths and peaks, and products stay below 2^108.
// ---------------------------------------------------------------------------
struct TileConst {
    float waves_half, pan_scale, pan_half;    // 2^-(s+1), 2^-(s+2), 2^-(s+3), s = log2 of the wave
    float neff_max;                           // the smaller of MWP and CWP that is set
    uint32_t acc_exp;                         // exponent field of 2^(10 - s)
};

static TileConst tile_const(const Struct& st)
{
    TileConst k;
    const float w = 1.0f / (float)(1 << st.wave_shift);
    k.waves_half = w / 2.0f;
    k.pan_scale = w / 4.0f;
    k.pan_half = w / 8.0f;
    // workgroups times waves per CU stay below 2^14, so a bound of 2^20 bounds nothing
    int32_t m = 1 << 20;
    if (st.mwp > 0 && st.mwp < m) m = st.mwp;
    if (st.cwp > 0 && st.cwp < m) m = st.cwp;
    k.neff_max = (float)m;
    k.acc_exp = 127u + 10u - (uint32_t)st.wave_shift;
    return k;
}

// A shape as its candidates read it.  M5 = (M - 1) / 32 and so on: a tile of
// 32 << c then covers M in (M5 >> c) + 1 steps.  e: exponent field of kd e at the
// smallest kd in place, and that of the smallest accumulator tile over the wave
// in the low byte.  D: index of its first code less its first batch position.
// Once the batch's costs are known, the first words hold the window threshold,
// the rank among the batch's shapes with a finite minimum and the first batch
// position instead.
struct alignas(16) TileShape {
    union {
        struct { int32_t M5, N5, K4; float U; };
        struct { float thr; int32_t rank, P; };
    };
    float MN, ip;
    uint32_t e;
    int32_t D;
};

__device__ inline TileShape tile_shape(const Const<float>& c, const TileConst& k, int32_t M, int32_t N, int32_t K,
                                       int32_t t)
{
    TileShape z;
    const bool ok = M >= 1 && N >= 1 && K >= 1 && t >= 0 && t <= 3;
    const uint32_t le = ok ? 3u - (uint32_t)t : 0u;    // element bytes 8, 4, 2, 1
    const uint32_t eo = t == 3 ? 2u : (1u << le);      // fp8 writes 16-bit results
    const float fM = (float)M, fN = (float)N, fK = (float)K;
    z.M5 = ok ? (M - 1) >> 5 : 0;
    z.N5 = ok ? (N - 1) >> 5 : 0;
    z.K4 = ok ? (K - 1) >> 4 : 0;
    z.MN = fM * fN * (float)eo;
    z.U = (fM * fK + fK * fN) * (float)(1u << le) + z.MN;
    const float p0 = vreg(c.inv_peak[0]), p1 = vreg(c.inv_peak[1]), p2 = vreg(c.inv_peak[2]), p3 = vreg(c.inv_peak[3]);
    float ip = t == 1 ? p1 : p0;
    ip = t == 2 ? p2 : ip;
    ip = t == 3 ? p3 : ip;
    z.MN = ok ? z.MN : 0.0f;
    z.U = ok ? z.U : 0.0f;
    z.ip = ok ? ip : __builtin_huge_valf();            // an invalid shape costs +inf
    z.e = ((127u + 4u + le) << 23) | (k.acc_exp + (t == 0 ? 1u : 0u));
    z.D = 0;
    return z;
}

__device__ inline float pow2_bits(uint32_t b) { return __uint_as_float(b); }

__device__ inline float tile_cost(const Struct& st, const Const<float>& c, const TileConst& k, const TileShape& z,
                                  uint32_t code)
{
    const uint32_t mt = code & 3u, nt = (code >> 2) & 3u, kd = (code >> 4) & 3u, mn = mt + nt;
    const float fw = (float)((code >> 6) + 1u);        // waves per workgroup
    const float rw = __builtin_amdgcn_rcpf(fw);
    const uint32_t gm = ((uint32_t)z.M5 >> mt) + 1u, gn = ((uint32_t)z.N5 >> nt) + 1u;
    const float fK = (float)(((uint32_t)z.K4 >> kd) + 1u);
    // (mt + nt) kd e, the bytes of a K step's panels
    const float pan = (pow2_bits((mt << 23) + 0x42000000u) + pow2_bits((nt << 23) + 0x42000000u)) *
                      pow2_bits((kd << 23) + (z.e & 0xff800000u));
    // VGPRs: accumulators and the panel share per thread
    const float va = __builtin_floorf((pow2_bits((mn + z.e) << 23) + (fw - k.waves_half)) * rw);
    const float vp = __builtin_floorf((__builtin_fmaf(pan, k.pan_scale, fw) - k.pan_half) * rw);
    const float vu = __builtin_ceilf((va + vp + 16.0f) * st.inv_vgran);
    const float w = least(__builtin_floorf(st.vgpr_units * __builtin_amdgcn_rcpf(vu)), st.waves_simd);
    const float ow = __builtin_fmaf(w, st.n_simd, 0.5f) * rw;
    const float lds = pan * 2.0f;
    float ol = st.lds_units * __builtin_amdgcn_rcpf(__builtin_ceilf(lds * st.inv_lgran));
    if (st.lds_cu >= (1 << 21)) ol = lds_limit_wide(st, (uint32_t)lds);
    const float o = __builtin_floorf(least(ow, ol));
    bool ok = code < 512u && kd != 3u && o > 0.0f;

    // rounds of workgroups over the chip
    const float pr = st.n_cu * o;
    float G = (float)gm * (float)gn;
    float nr = __builtin_floorf((G + (pr - 0.5f)) * __builtin_amdgcn_rcpf(pr));
    // from 2^21 on an exact division (and the grid limit), as in rounds()
    const bool big = G + pr >= 2097152.0f;
    if (__builtin_expect(__ballot(big) != 0, 0)) {
        if (big) {
            const uint64_t Gi = (uint64_t)gm * gn;
            const uint32_t p = (uint32_t)st.n_cu * (uint32_t)o;
            ok = ok && Gi <= 0x7fffffffull;
            G = (float)Gi;
            nr = ok ? (float)(((uint32_t)Gi + p - 1u) / p) : 1.0f;
        }
    }
    const float GK = G * fK;
    const float B = __builtin_fmaf(GK, pan, z.MN);
    const float sh = least(z.U * __builtin_amdgcn_rcpf(B), 1.0f), s2 = 1.0f - sh;
    const float S = __builtin_fmaf(s2, c.bw[1], sh * c.bw[3]);
    const float Lf = __builtin_fmaf(s2, c.latf[1], sh * c.latf[3]);
    const float Tc = GK * pow2_bits((mn + kd + 142u) << 23) * z.ip;
    const float Tb = B * __builtin_amdgcn_rcpf(S);
    const float Tlat = nr * B * (__builtin_amdgcn_rcpf(G) * rw) * c.inv_lw * Lf;
    const float Tov = __builtin_fmaf(c.ov[2], nr * fK, __builtin_fmaf(c.ov[1], G, c.ov[0]));
    const float Tm = most(Tb, Tlat);
    float step;
    if (st.combine == 0) {
        step = most(Tc, Tm);
    } else {
        const float neff = least(o * fw, k.neff_max);
        const float aT = (neff - 1.0f) * Tc;
        float eta = aT >= Tm ? 1.0f : aT * __builtin_amdgcn_rcpf(Tm);
        eta = neff == 1.0f ? 0.0f : eta;
        const float num = Tm + Tc;
        step = num == 0.0f ? 0.0f : num * __builtin_amdgcn_rcpf(1.0f + eta);
    }
    return ok ? Tov + step : __builtin_huge_valf();
}

// float64 minimum, its lowest local index and the second-smallest value of
// a multiset, accumulated in candidate order (exact ties keep the first)
struct Best2 {
    double c1, c2;
    int32_t j1;
    __device__ inline void add(double cd, int32_t jl)
    {
        if (cd < c1 || (cd == c1 && jl < j1)) {
            c2 = c1;
            c1 = cd;
            j1 = jl;
        } else if (cd < c2) {
            c2 = cd;
        }
    }
};

__device__ inline void write_best(const Best2& r, int64_t i, int32_t* best, double* best_cost,
                                  uint8_t* near_tie)
{
    const double dinf = __builtin_huge_val();
    const bool fin = r.c1 < dinf;
    best[i] = fin ? r.j1 : -1;
    best_cost[i] = r.c1;
    near_tie[i] = (fin && r.c2 < dinf && (r.c2 - r.c1) <= 1e-6 * r.c1) ? 1 : 0;
}

constexpr int kTileQueue = 128;   // queued float64 window candidates per wave
constexpr int kTileSlots = 64;    // shapes per queue (one lane each at the end)
constexpr int kTileBatch = 32;    // consecutive shapes whose candidates share wavefronts, at most
constexpr int kTileSpan = 704;    // candidates a batch may hold (11 rounds of 64)

// Per-wave LDS: the current batch's shapes and float32 costs, and the queue
// of float64 window re-evaluations, shared across batches.  Queue entries
// are appended in (slot, local index) order.
struct TileQueue {
    TileShape bs[kTileBatch];        // the batch's shapes that have candidates
    float cost32[kTileSpan];
    uint64_t ends[kTileSpan / 64];   // bit v: the list at batch position v ends there
    uint32_t bmin[kTileBatch];       // bits of the float32 minimum per batch shape
    int64_t shape[kTileSlots];
    uint32_t key[kTileQueue];        // slot << 24 | local candidate index
    uint32_t cand[kTileQueue];       // index into the candidate-code array; once the
                                     // costs are in, the first entry of each slot
    double cost[kTileQueue];
};

// sum of v over the lanes up to this one, within the lanes 0..31
__device__ inline int32_t sum_upto(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    return v;
}

// The batch shape that a round's lane works on: the lists that end before it.
// `before` counts those of earlier rounds.
__device__ inline int lane_slot(const TileQueue& q, int round, int& before)
{
    const uint64_t e = q.ends[round];
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)e);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(e >> 32));
    const int sl = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, (uint32_t)before));
    before += __popc(lo) + __popc(hi);
    return sl;
}

struct TileArgs {
    ShapePtrs sh;
    const int32_t* off;
    const uint32_t* code;
    int64_t n, n_cand, per;
    int32_t* best;
    double* best_cost;
    uint8_t* near_tie;
    TileConst tk;
    Set S;
};

// The kernel's arguments, read again from here on: what only a batch's start,
// the results and the float64 evaluations need would otherwise be fetched at
// the kernel's start and held in, or spilled from, the scalar registers of pass 1
// (64 spills).
typedef const TileArgs __attribute__((address_space(4))) * TileArgsPtr;
__device__ inline const TileArgs& late_args()
{
    TileArgsPtr p = (TileArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const TileArgs*)p;
}

__device__ inline void clamp_list(int64_t n_cand, int64_t& a, int64_t& b)
{
    // offsets are caller data: clamp them into the candidate array
    a = a < 0 ? 0 : (a > n_cand ? n_cand : a);
    b = b < a ? a : (b > n_cand ? n_cand : b);
}

// A shape's extents and dtype in a loop over its candidates, of which a lane has
// one or two: nothing formed of them is held across the float64 cost, where it
// would spill (and a kernel with scratch memory starts later).
struct ShapeDims {
    int32_t M, N, K, t;
    __device__ inline ShapeDims(const ShapePtrs& sh, int64_t i)   // i wave-uniform
        : M(__builtin_amdgcn_readfirstlane(sh.M[i])), N(__builtin_amdgcn_readfirstlane(sh.N[i])),
          K(__builtin_amdgcn_readfirstlane(sh.K[i])), t(__builtin_amdgcn_readfirstlane(sh.dtype[i]))
    {
    }
    __device__ inline ShapeDims late() const
    {
        ShapeDims x = *this;
        asm volatile("" : "+s"(x.M), "+s"(x.N), "+s"(x.K), "+s"(x.t));
        return x;
    }
};

// shape i's result from the lanes' shares of its window
__device__ inline void write_best_of_wave(const TileArgs& C, Best2 r, int64_t i, int lane)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const double oc1 = __shfl_xor(r.c1, m, 64);
        const double oc2 = __shfl_xor(r.c2, m, 64);
        const int32_t oj1 = __shfl_xor(r.j1, m, 64);
        if (oc1 < r.c1 || (oc1 == r.c1 && oj1 < r.j1)) {
            r.c2 = r.c1 < oc2 ? r.c1 : oc2;
            r.c1 = oc1;
            r.j1 = oj1;
        } else {
            r.c2 = oc1 < r.c2 ? oc1 : r.c2;
        }
    }
    if (lane == 0) write_best(r, i, C.best, C.best_cost, C.near_tie);
}

// A shape of the batch whose window is too large for the queue, on the whole
// wave: record z, window by the float32 costs in LDS.
__device__ inline void wide_window(const TileArgs& C, const TileQueue& q, const TileShape& z, int64_t i, int lane)
{
    const ShapeDims s(C.sh, i);
    int64_t a = C.off[i], b = C.off[i + 1];
    clamp_list(C.n_cand, a, b);
    const int32_t P = z.P, len = (int32_t)(b - a);
    Best2 r{__builtin_huge_val(), __builtin_huge_val(), 0x7fffffff};
    for (int32_t j = lane; j < len; j += 64) {
        if (!(q.cost32[P + j] <= z.thr)) continue;
        const ShapeDims x = s.late();
        r.add(exact_cost(C.S, x.M, x.N, x.K, x.t, C.code[a + j]), j);
    }
    write_best_of_wave(C, r, i, lane);
}

// One shape on the whole wave, without LDS: float32 minimum over its list, then
// the float64 window evaluated lane-parallel and reduced across the wave.  For
// lists too long for LDS.
__device__ inline void direct_shape(const TileArgs& C, int64_t i, int lane)
{
    const Set& S = C.S;
    const TileConst& tk = C.tk;
    const double dinf = __builtin_huge_val();
    const float finf = __builtin_huge_valf();
    const ShapeDims s(C.sh, i);
    int64_t a = C.off[i], b = C.off[i + 1];
    clamp_list(C.n_cand, a, b);
    const TileShape z = tile_shape(S.cf, tk, s.M, s.N, s.K, s.t);
    float c32 = finf;
    for (int64_t j = a + lane; j < b; j += 64)
        c32 = __builtin_fminf(c32, tile_cost(S.st, S.cf, tk, z, C.code[j]));
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) c32 = __builtin_fminf(c32, __shfl_xor(c32, m, 64));
    Best2 r{dinf, dinf, 0x7fffffff};
    if (c32 < finf) {
        const float thr = c32 * (1.0f + kTileWindow);
        for (int64_t j = a + lane; j < b; j += 64) {
            if (!(tile_cost(S.st, S.cf, tk, z, C.code[j]) <= thr)) continue;
            const ShapeDims x = s.late();
            r.add(exact_cost(S, x.M, x.N, x.K, x.t, C.code[j]), (int32_t)(j - a));
        }
    }
    write_best_of_wave(C, r, i, lane);
}

// A wave takes `per` consecutive shapes, in batches of as many as fit the LDS
// (at most kTileBatch shapes and kTileSpan candidates), and lays a batch's
// candidate lists end to end over its lanes, so that short lists leave no lane
// idle.  Pass 1 writes each candidate's float32 cost to LDS and takes each
// shape's minimum.  Every candidate within kTileWindow of its shape's minimum is
// queued for a float64 re-evaluation by a second pass that counts as it appends
// (a queue that overflows is evaluated and the window appended again); the queue
// fills across batches.  At the end the waves of a block evaluate their queues
// together: a wave's own holds some 16 entries, and a float64 evaluation costs the
// same however many of the 64 lanes have one.  The result per shape is
// the smallest float64 cost (the lowest index winning exact ties) and the
// second-smallest, for the near-tie flag.  A shape of more than kTileSpan
// candidates goes without the queue, and where a batch's windows would not fit
// an empty queue, so do its shapes with more than an equal share of it: their
// windows are read from the costs in LDS, the other shapes' fit.  (2^16 shapes of
// up to 96 candidates, all of them one tile repeated: 91 us, and 64 with only the
// first twentieth so; with such batches cut in half until they fit, 211 and 141.)
// A run per wave, cut where the LDS is full, takes short calls and long lists
// where fixed batches of eight shapes left waves idle or went without the queue:
// 1000 shapes of up to 96 candidates 16.1 -> 7.0 us, 2^14 of up to 384 87.4 -> 30.7.
// Bound: vector instructions and latency.  Over a launch of 2^16 shapes it issues
// 0.45 to 0.53 of them per CU-cycle: each wave has one batch, so that all load at
// their start and evaluate the queues at their end together.  The LDS of a wave
// leaves room for 24 waves per CU, so the kernel asks for 6 waves per SIMD (at most
// 80 VGPRs).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(6))) void k_select_tile(const TileArgs A)
{
    constexpr int W = BLOCK / 64;
    __shared__ TileQueue queues[W];
    __shared__ int queued[W];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    TileQueue& q = queues[wv];
    const int64_t wave = (int64_t)blockIdx.x * W + wv;
    const float finf = __builtin_huge_valf();
    int64_t s0 = wave * A.per;
    const int64_t end = s0 + A.per < A.n ? s0 + A.per : A.n;
    int ns = 0, qn = 0;
    for (;;) {
        const bool done = s0 >= end;
        const TileArgs& B = late_args();
        // lane k < kTileBatch holds shape s0 + k
        const int64_t si = s0 + lane;
        bool has = lane < kTileBatch && si < end;
        int32_t M = 0, N = 0, K = 0, t = 0;
        int64_t a = 0, b = 0;
        if (has) {
            M = B.sh.M[si];
            N = B.sh.N[si];
            K = B.sh.K[si];
            t = B.sh.dtype[si];
            a = B.off[si];
            b = B.off[si + 1];
            clamp_list(B.n_cand, a, b);
        }
        // list lengths, saturated
        const int32_t len = (int32_t)(b - a < kTileSpan + 1 ? b - a : kTileSpan + 1);
        const int32_t inc = sum_upto(len);
        const int nb = __popcll(__ballot(has && inc <= kTileSpan));   // shapes of this batch
        has = lane < nb;
        bool fin = false;
        int32_t rank = 0;   // among the batch's shapes with a finite minimum
        int32_t T = 0;
        int r = -1;         // among the batch's shapes that have candidates
        if (nb > 0) {
            T = __builtin_amdgcn_readlane(inc, nb - 1);
            const int32_t P = inc - len;             // first batch position of lane's shape
            const bool some = has && len > 0;
            r = (int)lanes_below(__ballot(some));
            r = some ? r : -1;
            wave_lds_sync();   // the previous batch's lanes are done reading
            if (lane < kTileSpan / 64) q.ends[lane] = 0;
            if (some) {
                q.bmin[r] = ~0u;
                TileShape z = tile_shape(B.S.cf, B.tk, M, N, K, t);
                // a <= n_cand < 2^31 and P < kTileSpan, so D fits 32 bits
                z.D = (int32_t)(a - P);
                q.bs[r] = z;
            }
            wave_lds_sync();
            if (some)
                __hip_atomic_fetch_or(&q.ends[(inc - 1) >> 6], 1ull << ((inc - 1) & 63), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WAVEFRONT);
            wave_lds_sync();
            // pass 1: float32 costs to LDS and the per-shape minimum
            int before = 0;
            for (int32_t v0 = 0; v0 < T; v0 += 64) {
                const int32_t v = v0 + lane;
                const int sl = lane_slot(q, v0 >> 6, before);
                if (v < T) {
                    const TileShape z = q.bs[sl];
                    const float c = tile_cost(A.S.st, A.S.cf, A.tk, z, A.code[(uint32_t)(v + z.D)]);
                    q.cost32[v] = c;
                    __hip_atomic_fetch_min(&q.bmin[sl], __float_as_uint(c), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WAVEFRONT);
                }
            }
            wave_lds_sync();
            // per shape: the window threshold, or the empty result
            float thr = -finf;
            if (some) {
                const float c32 = __uint_as_float(q.bmin[r]);
                fin = c32 < finf;
                if (fin) thr = c32 * (1.0f + kTileWindow);
            }
            if (has && !fin) {
                const TileArgs& L = late_args();
                L.best[si] = -1;
                L.best_cost[si] = __builtin_huge_val();
                L.near_tie[si] = 0;
            }
            rank = (int32_t)lanes_below(__ballot(fin));
            if (some) {
                q.bs[r].thr = thr;
                q.bs[r].rank = rank;
                q.bs[r].P = P;
            }
        }
        int nf = __popcll(__ballot(fin));
        // The one flush site.  The first pass flushes at the end, or when the
        // batch's shapes would not find queue slots; then the batch's window
        // is appended after entry qn (shapes taking slots from ns in batch
        // order), entries past the queue's end counted but not written.  If
        // the queue overflowed, the next pass evaluates what it held and appends
        // the window again to the empty queue; if it overflowed from empty, the
        // shapes with more than an equal share of it go without the queue, and
        // the others' windows fit.
        bool flush = done || ns + nf > kTileSlots;
        int cnt = 0;
        for (;;) {
            if (flush) {
                // Every queued candidate in float64 (codes and shapes are read
                // back from memory, one load per lane); then one lane per shape
                // scans that shape's entries (ascending candidate index) and
                // writes its result.  Each wave comes here once with `done`, so
                // the block's barriers match.
                int e = lane, step = 64, total = qn;
                if (done) {
                    if (lane == 0) queued[wv] = qn;
                    __syncthreads();
                    e = (int)threadIdx.x;
                    step = BLOCK;
                    total = 0;
                    for (int k = 0; k < W; ++k) total += queued[k];
                } else {
                    wave_lds_sync();
                }
                const TileArgs& L = late_args();
                for (; e < total; e += step) {
                    int k = wv, x = e;
                    if (done)
                        for (k = 0; k < W - 1 && x >= queued[k]; ++k) x -= queued[k];
                    TileQueue& p = queues[k];
                    const int64_t i = p.shape[p.key[x] >> 24];
                    p.cost[x] = exact_cost(L.S, L.sh.M[i], L.sh.N[i], L.sh.K[i], L.sh.dtype[i], L.code[p.cand[x]]);
                }
                if (done) __syncthreads();
                else wave_lds_sync();
                // every slot has its minimum's entry, and entries are in slot order
                for (int x = lane; x < qn; x += 64) {
                    const uint32_t sl = q.key[x] >> 24;
                    if (x == 0 || q.key[x - 1] >> 24 != sl) q.cand[sl] = (uint32_t)x;
                }
                wave_lds_sync();
                if (lane < ns) {
                    const int e1 = lane + 1 < ns ? (int)q.cand[lane + 1] : qn;
                    Best2 res{__builtin_huge_val(), __builtin_huge_val(), 0x7fffffff};
                    for (int x = (int)q.cand[lane]; x < e1; ++x)
                        res.add(q.cost[x], (int32_t)(q.key[x] & 0xffffffu));
                    write_best(res, q.shape[lane], L.best, L.best_cost, L.near_tie);
                }
                if (done) break;
                wave_lds_sync();   // the queue is refilled next
                ns = 0;
                qn = 0;
            }
            if (nb == 0) break;
            if (fin) q.shape[ns + rank] = si;
            wave_lds_sync();   // the shapes' thresholds and ranks
            cnt = 0;
            int before = 0;
            for (int32_t v0 = 0; v0 < T; v0 += 64) {
                // every lane takes part in the ballot
                const int32_t v = v0 + lane;
                const int sl = lane_slot(q, v0 >> 6, before);
                const TileShape& z = q.bs[v < T ? sl : 0];
                const bool w = v < T && q.cost32[v] <= z.thr;
                const uint64_t m = __ballot(w);
                const int e = qn + cnt + (int)lanes_below(m);
                if (w && e < kTileQueue) {
                    const int32_t jl = v - z.P;
                    q.key[e] = ((uint32_t)(ns + z.rank) << 24) | (uint32_t)jl;
                    q.cand[e] = (uint32_t)(v + z.D);
                }
                cnt += __popcll(m);
            }
            if (qn + cnt <= kTileQueue) break;
            flush = qn > 0;
            if (flush) continue;
            // the windows' sizes, in the minima's place
            if (lane < kTileBatch) q.bmin[lane] = 0u;
            wave_lds_sync();
            before = 0;
            for (int32_t v0 = 0; v0 < T; v0 += 64) {
                const int32_t v = v0 + lane;
                const int sl = lane_slot(q, v0 >> 6, before);
                if (v < T && q.cost32[v] <= q.bs[sl].thr)
                    __hip_atomic_fetch_add(&q.bmin[sl], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
            wave_lds_sync();
            const bool wide = fin && (int)q.bmin[fin ? r : 0] * nf > kTileQueue;
            for (uint64_t w = __ballot(wide); w; w &= w - 1) {
                const int k = __builtin_ctzll(w);
                wide_window(late_args(), q, q.bs[__builtin_amdgcn_readlane(r, k)], s0 + k, lane);
            }
            fin = fin && !wide;
            rank = (int32_t)lanes_below(__ballot(fin));
            nf = __popcll(__ballot(fin));
            wave_lds_sync();
            if (r >= 0) {
                q.bs[r].rank = rank;
                if (!fin) q.bs[r].thr = -finf;
            }
        }
        if (done) break;
        qn += cnt;
        ns += nf;
        const int alone = nb == 0 ? 1 : 0;   // a list too long for LDS
        const TileArgs& L = late_args();
        for (int k = 0; k < alone; ++k) direct_shape(L, s0, lane);
        s0 += nb + alone;
    }
}

template <int BLOCK>
static void select_t(const ShapePtrs& sh, const int32_t* off, const uint32_t* code, int64_t n,
                     int64_t n_cand, const Set& S, int32_t* best, double* best_cost,
                     uint8_t* near_tie, int grid_mult, hipStream_t stream)
{
    const int64_t wpb = BLOCK / 64;
    const int64_t waves = (int64_t)resident_blocks(reinterpret_cast<const void*>(&k_select_tile<BLOCK>), BLOCK) * wpb;
    const int64_t per = tile_run(n, n_cand, waves, grid_mult);
    const int64_t b = ((n + per - 1) / per + wpb - 1) / wpb;
    k_select_tile<BLOCK><<<(int)b, BLOCK, 0, stream>>>(
        TileArgs{sh, off, code, n, n_cand, per, best, best_cost, near_tie, tile_const(S.st), S});
}

// Every candidate's float32 cost (the selection's first pass): a wave per
// shape, its lanes over the shape's list; grid-stride over shapes.
__global__ __launch_bounds__(256) void k_tile_costs(ShapePtrs sh, const int32_t* __restrict__ off,
                                                     const uint32_t* __restrict__ code, int64_t n,
                                                     int64_t n_cand, Struct st, Const<float> c, TileConst tk,
                                                     float* __restrict__ cost)
{
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; i < n; i += nw) {
        int64_t a = off[i], b = off[i + 1];
        clamp_list(n_cand, a, b);
        const int32_t M = sh.M[i], N = sh.N[i], K = sh.K[i], t = sh.dtype[i];
        const TileShape z = tile_shape(c, tk, M, N, K, t);
        for (int64_t j = a + lane; j < b; j += 64) cost[j] = tile_cost(st, c, tk, z, code[j]);
    }
}

hipError_t launch_tile_costs(const ShapePtrs& sh, const int32_t* off, const uint32_t* code, int64_t n,
                             int64_t n_cand, const Set& S, float* cost, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t want = (n + 3) / 4;
    const int64_t cap = (int64_t)resident_blocks(reinterpret_cast<const void*>(&k_tile_costs), 256) * 4;
    const int64_t b = want < cap ? want : cap;
    k_tile_costs<<<(int)(b < 1 ? 1 : b), 256, 0, stream>>>(sh, off, code, n, n_cand, S.st, S.cf, tile_const(S.st), cost);
    return hipGetLastError();
}

hipError_t launch_select_tile(const ShapePtrs& sh, const int32_t* off, const uint32_t* code,
                              int64_t n, int64_t n_cand, const Set& S, int32_t* best,
                              double* best_cost, uint8_t* near_tie, const LaunchCfg& c,
                              hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    switch (c.block) {
    case 64: select_t<64>(sh, off, code, n, n_cand, S, best, best_cost, near_tie, c.grid_mult, stream); break;
    case 128: select_t<128>(sh, off, code, n, n_cand, S, best, best_cost, near_tie, c.grid_mult, stream); break;
    case 256: select_t<256>(sh, off, code, n, n_cand, S, best, best_cost, near_tie, c.grid_mult, stream); break;
    case 512: select_t<512>(sh, off, code, n, n_cand, S, best, best_cost, near_tie, c.grid_mult, stream); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace wm
