// Segment chains (FP32): the likelihood by forward vectors instead of segment
// products, verified on the device.
//
// A product of positive matrices forgets where it started: after some steps
// all rows of Gamma P(x_s) ... Gamma P(x_t) are parallel, so the forward
// vector at the start of a segment is fixed, up to a factor, by the last few
// observations before it.  Every segment b therefore starts from a flat vector
// `warm` steps before its first observation, holds s_b (its start vector) when
// it gets there and e_b (its end vector) after its last one, and
//     ln L = ln sum(delta) + sum_b ln( sum(e_b) / sum(s_b) )
// provided that s_b is parallel to e_{b-1}.  That is checked for every segment,
// entry by entry (relative difference eps_b <= kChainTol, i.e. the projective
// distance of the two vectors, which the remaining chain cannot increase); a
// segment that starts elsewhere is run again from e_{b-1}.  Where the check
// cannot be met the set's `fail` word is raised and the launches of the product
// path behind it, which otherwise return at once, compute ln L.
//
// ln L is off by at most sum_b eps_b.  What is left of a flat start has the
// same sign in every segment of a record without events, so a walker whose sum
// is more than rounding may come to (chain_budget) runs its segments once more,
// from their neighbours' ends: what the flat starts left shrinks by the rate of
// the first run, what rounding left does not, and stands.  (Two groups of
// states, K = 20, T = 20,000, no events: ln L off by 1.4e-6 relative without
// the second run, by 8e-8 with it; 36 -> 45 us.)
//
// Work: K^2 instead of K^3 multiply-adds per observation.  A step is a matrix
// product again: the start-state columns of the product path become the
// vectors of 16 consecutive segments.
#pragma once

#include "hmm_kernels.hpp"

namespace hmm {

constexpr int kChainCols = 16;     // segments per pair (columns of an MFMA tile)
constexpr int kChainStep = 4;      // steps per staged chunk: 16 x 4 observations = 64 lanes
constexpr int kChainRepairs = 3;   // reruns of segments from their neighbours' ends
constexpr float kChainTol = 0x1p-16f;
// The scale of a column lags one step behind, so a column's largest entry
// varies; below this a flushed entry could matter (see kChainMinGamma).
constexpr float kChainLow = 0x1p-40f;

// Sum over the four lanes that hold one column of a 16-wide tile.
template <typename F>
__device__ __forceinline__ F column_sum16(F x)
{
    x += __shfl_xor(x, 32);
    x += __shfl_xor(x, 16);
    return x;
}

// Row-wise shift by one lane within 16 lanes (lane 0 of a row receives 0).
__device__ __forceinline__ float from_left_column(float x) { return __uint_as_float(dpp_u<0x111>(__float_as_uint(x))); }

// Barrier of the workgroup ordering LDS accesses only: loads of observations
// ahead of their use stay in flight across it (__syncthreads waits for them).
__device__ __forceinline__ void chain_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A wave-uniform value the compiler cannot see to be one, as a scalar.
__device__ __forceinline__ int scalar(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t scalar(int64_t x)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)x);
    return (int64_t)(((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) | lo);
}

// What a walker's starts may differ by in sum without another run: obs
// observations, ln: its part of ln L.  FP32 rounds every entry at every
// observation, and where an observation recurs so does its rounding: ln L of a
// record without events is off by 0.1..5e-7 per observation (segment products
// and vectors alike, K = 20..80).
__device__ __forceinline__ float chain_budget(int64_t obs, double ln)
{
    return 0x1p-24f * ((float)obs + fabsf((float)ln));
}

// Relative difference of an entry s from its neighbour's r e; what lies below
// 2^-100 of the sum ss is not compared (it cannot contribute: a vector whose
// entries spread that far is refused, kChainLow and kChainMinGamma).
__device__ __forceinline__ float chain_diff(float s, float e, float ss, float r)
{
    const float d = fabsf(s - r * e) - 0x1p-100f * ss;
    return d > 0.f ? d / fmaxf(s, r * e) : 0.f;
}

// Whether reruns can still meet the tolerance.  The largest relative difference
// diff is left after `steps` steps of forgetting; at that rate the tolerance
// needs steps * ln(tol) / ln(diff) of them, and `left` more are available,
// times `grant` (the rate is an estimate).
__device__ __forceinline__ bool chain_hopeless(float diff, int steps, int left, float grant)
{
    if (!(diff < 1.f)) return true;
    return (float)steps * logf(kChainTol) < grant * (float)(steps + left) * logf(fmaxf(diff, kChainTol));
}

// Reruns of a walker most of whose starts differ: the chain forgets slowly
// everywhere, so the starts checked across walkers differ too and the second
// launch walks everything again.  After the first pass n reruns cost
// W + (2 n + 1) q steps; they are worth it while the segment products behind
// would take longer.
__device__ __forceinline__ int chain_slow_repairs(int W, int q, int product_steps)
{
    return min(max(0, (product_steps - W - q) / (2 * q)), kChainRepairs);
}

// s parallel to e: |s - r e| <= tol s with r = ss / es (ss, es the sums of
// the two vectors), with chain_diff's limit.  False for NaN and for a zero vector.
__device__ __forceinline__ bool chain_parallel(float s, float e, float ss, float r)
{
    return fabsf(s - r * e) <= kChainTol * s + 0x1p-100f * ss;
}

static_assert(sizeof(StateConst) == 64, "k_chain reads the constants as 8 doubles per state");

// Workgroup shapes of k_chain: NP walkers with NS stagers each.  A stager's
// VALU work and a walker's matrix work do not overlap on one SIMD (measured:
// they add up), so a wavefront per SIMD is the best use of a CU while the
// segments allow it, and fewer, longer segments repeat less warm-up.
//  K <= 32: the stager is the longer of the two.  Short sequences take one
//    walker with two stagers (the latency of a step decides), longer ones two
//    pairs.
//  K > 32: two pairs, and for long sequences four (two wavefronts per SIMD:
//    15 % more throughput at K = 80, where the walker is the longer one; MFMA
//    55 % and VALU issue 40 % of the SIMDs' time).
struct ChainShape {
    int NP, NS;
    int64_t segs() const { return 16 * (int64_t)NP; }
    int threads() const { return 64 * NP * (1 + NS); }
    // two buffers of 4 ceil(K / 4) x 64 staged emissions per walker (160 KiB
    // at K = 80 and four walkers); the words exchanged between passes reuse it
    size_t lds(int K) const { return (size_t)NP * 2 * ((K + 3) / 4 * 4) * 64 * 4; }
};

inline ChainShape chain_shape(int K, bool big)
{
    if (K <= 32) return big ? ChainShape{2, 1} : ChainShape{1, 2};
    return big ? ChainShape{4, 1} : ChainShape{2, 1};
}

// Larger of two numbers in one instruction (fmax also quiets NaNs, in two).
__device__ __forceinline__ double max_f64(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ float max_f32(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// mask ? a : b for a mask of all ones or zeros, without a branch (a ternary
// here is compiled to one, with the loads of the state's constants inside).
__device__ __forceinline__ double select_f64(int mask, double a, double b)
{
    const int lo = (__double2loint(a) & mask) | (__double2loint(b) & ~mask);
    const int hi = (__double2hiint(a) & mask) | (__double2hiint(b) & ~mask);
    return __hiloint2double(hi, lo);
}

// Pointers of a descriptor are known to be global memory only here: without
// the cast their loads are flat ones, which wait for LDS traffic too.
// Constants of the launch (uniform_ptr) are then read by scalar loads.
template <typename T>
using global_ptr = __attribute__((address_space(1))) T *;
template <typename T>
using uniform_ptr = const __attribute__((address_space(4))) T *;

// The observations of one pair's segments, addressed by 32-bit offsets from a
// wave-uniform base (the first observation its warm-up can reach): scalar base
// and one vector register per address.  Every load is unconditional and can
// stay in flight across chunks; flags, counts and values are clamped to the
// record (T >= 4).  Locations belong to the caller only where the flag is 1:
// they come through a buffer descriptor, and an observation without one asks
// for an offset outside it, which reads as zero and touches no memory.
struct RawObs {
    double x, y;
    int f;
};

// Most observations a window reaches over: a pair's segments (kChainCols of at
// most 2^22 observations), its warm-up and the chunks fetched ahead.
constexpr int kChainWindow = 1 << 27;

template <bool GEN>
struct ObsWindow {
    global_ptr<const char> flag, xy;   // flag / cnt and values at the base
    __amdgpu_buffer_rsrc_t loc;        // locations from the base on
    int kind;
    int hi;                            // last observation of the record, relative to the base

    __device__ __forceinline__ void init(const Obs &o, int64_t base, int64_t T)
    {
        kind = GEN ? o.kind : kEmisTremor;
        hi = scalar((int)min((int64_t)kChainWindow - 1, T - 1 - base));
        const char *f = nullptr, *v = nullptr;
        if (kind == kEmisPoisson) f = reinterpret_cast<const char *>(o.cnt + base);
        else if (kind == kEmisTremor) f = reinterpret_cast<const char *>(o.flag + base);
        if (GEN && kind == kEmisGauss1) v = reinterpret_cast<const char *>(o.xy + base);
        flag = (global_ptr<const char>)f;
        xy = (global_ptr<const char>)v;
        if constexpr (!GEN)
            loc = __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(o.xy + 2 * base), 0, (int)(16u * (hi + 1u)),
                                                    0x00020000);
    }
    // Observation o: tremor model, the location where its flag is 1; other
    // kinds, the count (to f) or the value.
    __device__ __forceinline__ RawObs value(int o, int f) const
    {
        RawObs r{0.0, 0.0, 1};
        if constexpr (!GEN) {
            // outside the record (o < 0, o > hi) the offset is outside the descriptor too
            const uint32_t at = f == 1 ? 16u * (uint32_t)o : 0xfffffff0u;
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            const u4 p = __builtin_amdgcn_raw_buffer_load_b128(loc, (int)at, 0, 0);
            r.x = __hiloint2double((int)p.y, (int)p.x);
            r.y = __hiloint2double((int)p.w, (int)p.z);
        } else {
            (void)f;
            const uint32_t i = (uint32_t)min(max(o, 0), hi);
            if (kind == kEmisPoisson) r.f = *(global_ptr<const int32_t>)(flag + 4u * i);
            else r.x = *(global_ptr<const double>)(xy + 8u * i);
        }
        return r;
    }
    // The flags of observations o .. o + 3 as they lie in memory (one
    // unaligned word, clamped into the record) and where they start in it.
    __device__ __forceinline__ int flag_word(int o) const
    {
        typedef int word_t __attribute__((aligned(1)));
        if constexpr (GEN) return 0;
        else return *(global_ptr<const word_t>)(flag + (uint32_t)min(max(o, 0), hi - 3));
    }
    // flag of observation o + u, from that word
    __device__ __forceinline__ int flag_of(int word, int o, int u) const
    {
        const unsigned at = 8u * (unsigned)(o - min(max(o, 0), hi - 3)) + 8u * u;   // 0..24 inside the record
        return (int)(((unsigned)word >> (at & 31u)) & 0xffu);
    }
};

// ---------------------------------------------------------------------------
// The emission stage of a pair: scaled emissions ê of the next four steps of
// its 16 segments, E[state][4 * segment + step].
//   ê = 2^(lam - sh), lam = log2 e in FP64 (the formula of
//   state_log2_emission / generic_log2_emission), sh = floor(max_k lam):
// the largest ê of a step lies in [1, 2).  lam - sh = n + f, f in [0, 1), with n
// from the low word of (lam - f) + (1.5 * 2^52 - sh); only f is rounded to
// FP32.  0 below 2^-200 and for steps without an observation.
//
// Two layouts, by how many state constants a lane can hold:
//  - up to kStagerSlots slots (K <= 32): lane (segment c, group g) evaluates
//    states 4 j + g of its segment at all four steps, the constants of its
//    states in registers for the whole launch; the shift's maximum crosses the
//    four lanes of a segment.
//  - above: lane (segment, step) evaluates every state, the constants read by
//    scalar loads, two states ahead of their use.  A group of two states keeps
//    the VALU busy for about as long as a scalar load takes; without the
//    prefetch K = 80 waited 300 cycles per state.
// ---------------------------------------------------------------------------
constexpr int kStagerSlots = 8;

// Fields of StateConst a kind uses: all but lx for the tremor model; mx, cxx,
// a1 and lx for the others (their second coordinate is 0).
template <bool GEN>
__device__ __forceinline__ double chain_log2_emission(const double (&c)[8], int mask, double x, double y)
{
    const double d0 = x - c[0];
    if constexpr (GEN) {
        (void)mask;
        (void)y;
        return fma(c[7], x, c[5]) + d0 * (c[2] * d0);
    } else {
        const double d1 = y - c[1];
        const double q = c[5] + d0 * (c[2] * d0 + c[3] * d1) + c[4] * (d1 * d1);
        return select_f64(mask, q, c[6]);
    }
}

// Validity of one observation; an invalid one is replaced by "no tremor" (its
// result is discarded).  mask: all ones where the density branch applies.
template <bool GEN>
__device__ __forceinline__ void chain_check_obs(int kind, bool live, RawObs &o, int &mask, int &bad)
{
    if constexpr (!GEN) {
        const bool fin = isfinite(o.x) & isfinite(o.y), one = o.f == 1;
        bad |= (int)(live & ((o.f > 1) | (one & !fin)));
        mask = (one & fin) ? -1 : 0;
        asm volatile("" : "+v"(mask));   // kept as a bit mask: v_bfi_b32 instead of moves and v_cndmask_b32
    } else if (kind == kEmisPoisson) {
        bad |= (int)(live & (o.f < 0));
        o.x = (double)max(o.f, 0);
    } else {
        const bool fin = isfinite(o.x);
        bad |= (int)(live & !fin);
        o.x = fin ? o.x : 0.0;
    }
}

// The shift floor(max lam), |shift| <= 5e8 (four of them add up in 32 bits); a
// step whose maximum is beyond that gets zero emissions, which fails the chain.
__device__ __forceinline__ int chain_shift(float m)
{
    return (int)floorf(__builtin_amdgcn_fmed3f(m, -5.0e8f, 5.0e8f));
}

// The fraction is taken in [0, 1), as the product path's emission stage takes
// it, so both round a step's emissions alike: steps without a location repeat
// the same K roundings, which move ln L by 1e-9 relative (a fraction in [-1/2,
// 1/2) rounds finer but differently, and moved it by up to 5e-9 against the
// product path; now 1e-11..3e-10.  K = 25, T = 105,000: 50.3 -> 54.5 us,
// T = 1e6: 92.4 -> 93.6 us).
__device__ __forceinline__ float chain_emission(double lam, double magic, double low)
{
    const double l = max_f64(lam, low);
    const double f = __builtin_amdgcn_fract(l);
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((float)f), __double2loint((l - f) + magic));
}

// Segment b of a set as a pair sees it: its first observation relative to the
// pair's window, and its live steps as (unsigned)(rel - lo) < n, rel = 0 at the
// first observation: from the start of the record (or of the warm-up) to the
// segment's end; n = 0 past the last segment.
__device__ __forceinline__ void chain_segment(const SetDesc &d, int64_t b, int64_t base, int W, int &off, int &lo,
                                              int &n)
{
    off = lo = n = 0;
    if (b < d.cnb) {
        const int64_t t0 = packed_seg_start(b, d.cq, d.cr);
        off = (int)(t0 - base);
        lo = -(int)min(t0, (int64_t)W);
        n = (int)d.cq + (b < d.cr ? 1 : 0) - lo;
    }
}

// NS stagers share a walker's chunk by its steps (the second layout: NS = 1).
template <int NSL, bool GEN, int NS, bool REGS = (NSL <= kStagerSlots)>
struct ChainStager;

template <int NSL, bool GEN, int NS>
struct ChainStager<NSL, GEN, NS, true> {
    static constexpr int NU = kChainStep / NS;   // steps of a chunk this stager evaluates

    // observations of the next D chunks, in flight: a chunk takes about
    // 0.3 us + 0.1 us per slot, a load from HBM 1 us or more
    static constexpr int D = NSL <= 4 ? 4 : 2;
    ObsWindow<GEN> win;
    int off, lo, n;          // segment's first observation in the window; live: (unsigned)(rel - lo) < n
    int c, g, u0, bad;
    long long ssum;          // shifts of the segment (the same on the four lanes of a segment)
    double cst[NSL][8];
    RawObs raw[D][NU];
    int words[D];            // their flags
    int ahead[D];            // the flags of the D chunks after those

    __device__ __forceinline__ void init(const SetDesc &d, int64_t b0, int64_t base, int W, int lane, int part)
    {
        win.init(d.obs, base, d.T);
        u0 = part * NU;
        c = lane & 15;
        g = lane >> 4;
        chain_segment(d, b0 + c, base, W, off, lo, n);
        bad = 0;
        const global_ptr<const double> sc = (global_ptr<const double>)(const double *)d.sc;
#pragma unroll
        for (int j = 0; j < NSL; ++j)
#pragma unroll
            for (int f = 0; f < 8; ++f) cst[j][f] = sc[8 * (4 * j + g) + f];
    }
    // (ahead[slot] holds the chunk's flags)
    __device__ __forceinline__ void fetch(int rel, int slot)
    {
        words[slot] = ahead[slot];
        ahead[slot] = win.flag_word(off + rel + D * kChainStep);
#pragma unroll
        for (int u = 0; u < NU; ++u)
            raw[slot][u] = win.value(off + rel + u0 + u, win.flag_of(words[slot], off + rel, u0 + u));
    }
    __device__ __forceinline__ bool counts() const { return g == 0; }
    // the first chunk of a pass starts at step rel
    __device__ __forceinline__ void start(int rel)
    {
        ssum = 0;
#pragma unroll
        for (int k = 0; k < D; ++k) ahead[k] = win.flag_word(off + rel + k * kChainStep);
#pragma unroll
        for (int k = 0; k < D; ++k) fetch(rel + k * kChainStep, k);
    }
    // stages the chunk at rel, held in slot, and fetches the chunk D later
    // there (the slots rotate by unrolling: moving a load in flight would
    // wait for it)
    __device__ __forceinline__ void stage(int rel, float *E, int slot)
    {
        RawObs now[NU];
        const int word = words[slot];
#pragma unroll
        for (int u = 0; u < NU; ++u) now[u] = raw[slot][u];
        fetch(rel + D * kChainStep, slot);
        float ev[NSL][NU];
        int part = 0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            int mask = -1;
            const bool live = (unsigned)(rel + u0 + u - lo) < (unsigned)n;
            if (!GEN) now[u].f = win.flag_of(word, off + rel, u0 + u);
            chain_check_obs<GEN>(win.kind, live, now[u], mask, bad);
            double lam[NSL];
            double m = -INFINITY;
#pragma unroll
            for (int j = 0; j < NSL; ++j) {
                lam[j] = chain_log2_emission<GEN>(cst[j], mask, now[u].x, now[u].y);
                m = max_f64(m, lam[j]);
            }
            // over the four lanes of the segment, in FP32 (any integer near the
            // maximum serves as the shift)
            float mf = (float)m;   // NaN only for discarded data
            auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mf), __float_as_uint(mf), false, false);
            mf = max_f32(__uint_as_float(r[0]), __uint_as_float(r[1]));
            r = __builtin_amdgcn_permlane16_swap(__float_as_uint(mf), __float_as_uint(mf), false, false);
            mf = max_f32(__uint_as_float(r[0]), __uint_as_float(r[1]));
            const int sh = chain_shift(mf);
            part += live ? sh : 0;
            const double dsh = (double)(live ? sh : 1000000);
            const double magic = 6755399441055744.0 - dsh, low = dsh - 200.0;
#pragma unroll
            for (int j = 0; j < NSL; ++j) ev[j][u] = chain_emission(lam[j], magic, low);
        }
        if (rel >= 0) ssum += part;
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
            float *dst = E + (4 * j + g) * 64 + 4 * c + u0;
            if constexpr (NU == 4) *reinterpret_cast<float4 *>(dst) = float4{ev[j][0], ev[j][1], ev[j][2], ev[j][3]};
            else *reinterpret_cast<float2 *>(dst) = float2{ev[j][0], ev[j][1]};
        }
    }
};

template <int NSL, bool GEN>
struct ChainStager<NSL, GEN, 1, false> {
    typedef double d8 __attribute__((ext_vector_type(8)));
    static constexpr int D = 2;
    ObsWindow<GEN> win;
    int off, lo, n;          // as above; off and lo of the lane's step (segment lane / 4, step lane % 4)
    int lane, bad;
    long long ssum;
    uniform_ptr<d8> sc;
    RawObs raw[D];
    int words[D], ahead[D];

    __device__ __forceinline__ void init(const SetDesc &d, int64_t b0, int64_t base, int W, int lane_, int)
    {
        win.init(d.obs, base, d.T);
        lane = lane_;
        chain_segment(d, b0 + (lane >> 2), base, W, off, lo, n);
        off += lane & 3;
        lo -= lane & 3;
        bad = 0;
        sc = (uniform_ptr<d8>)(const d8 *)d.sc;
    }
    __device__ __forceinline__ void fetch(int rel, int slot)
    {
        words[slot] = ahead[slot];
        ahead[slot] = win.flag_word(off + rel + D * kChainStep);
        raw[slot] = win.value(off + rel, win.flag_of(words[slot], off + rel, 0));
    }
    __device__ __forceinline__ bool counts() const { return true; }
    __device__ __forceinline__ void start(int rel)
    {
        ssum = 0;
#pragma unroll
        for (int k = 0; k < D; ++k) ahead[k] = win.flag_word(off + rel + k * kChainStep);
#pragma unroll
        for (int k = 0; k < D; ++k) fetch(rel + k * kChainStep, k);
    }
    __device__ __forceinline__ void stage(int rel, float *E, int slot)
    {
        RawObs now = raw[slot];
        if (!GEN) now.f = win.flag_of(words[slot], off + rel, 0);
        fetch(rel + D * kChainStep, slot);
        const bool live = (unsigned)(rel - lo) < (unsigned)n;
        int mask = -1;
        chain_check_obs<GEN>(win.kind, live, now, mask, bad);
        // the pointer is made new for every chunk: hoisted out of the chunk
        // loop the constants would not fit in the scalar registers
        uniform_ptr<d8> p = sc;
        asm volatile("" : "+s"(p));
        double lam[4 * NSL];
        double m = -INFINITY;
        d8 c0 = p[0], c1 = p[1];
#pragma unroll
        for (int k = 0; k < 4 * NSL; k += 2) {
            // wait for this group's constants, then start the next group's loads
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            d8 n0 = c0, n1 = c1;
            if (k + 2 < 4 * NSL) {
                n0 = p[k + 2];
                n1 = p[k + 3];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const d8 v = h == 0 ? c0 : c1;
                const double cc[8] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
                lam[k + h] = chain_log2_emission<GEN>(cc, mask, now.x, now.y);
                m = max_f64(m, lam[k + h]);
            }
            __builtin_amdgcn_sched_barrier(0);
            c0 = n0;
            c1 = n1;
        }
        const int sh = chain_shift((float)m);
        if (rel >= 0) ssum += live ? sh : 0;
        const double dsh = (double)(live ? sh : 1000000);
        const double magic = 6755399441055744.0 - dsh, low = dsh - 200.0;
#pragma unroll
        for (int k = 0; k < 4 * NSL; ++k) E[k * 64 + lane] = chain_emission(lam[k], magic, low);
    }
};

// ---------------------------------------------------------------------------
// Workgroup = NP walkers, then NP * NS stagers (ChainShape).  Walker p advances
// the vectors of 16 consecutive segments on the matrix cores; its stagers
// evaluate the emissions of the next four steps of those segments meanwhile,
// into the other half of an LDS double buffer.
//
// mode 0: every segment; writes s of each walker's first segment (vs), e of
//   its last (ve) and its sum of ln ratios (part).
// mode 1: verifies vs against the neighbouring walker's ve and returns unless
//   they differ; then reruns the workgroup's segments with those first
//   segments started from ve, requires that the ends stay the same, and
//   replaces part.
// ---------------------------------------------------------------------------
template <int MT, int NSL, bool GEN, int NP, int NS>
__device__ __forceinline__ void chain_body(const SetDesc &d, int64_t wg, int mode)
{
    typedef Tile<16>::acc_t acc_t;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    int *ism = reinterpret_cast<int *>(smem);                           // a verdict per walker
    long long *shifts = reinterpret_cast<long long *>(smem) + 8;        // a sum per stager
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool walker = wave < NP;
    const int pair = walker ? wave : (wave - NP) % NP, share = walker ? 0 : (wave - NP) / NP;
    const int K = d.K;
    const int64_t gw = scalar(wg * NP + pair);   // this walker among the set's
    const int64_t b0 = gw * kChainCols;            // its first segment
    const int64_t nb = d.cnb, q = d.cq, qr = d.cr;
    const bool pair_live = b0 < nb;

    auto verdicts = [&]() {   // of the workgroup's walkers, or'ed
        int v = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p) v |= ism[p];
        return v;
    };
    // one decision for the workgroup (the words may change while it runs)
    if (threadIdx.x == 0) ism[0] = (*d.fail != 0 || *d.status != 0) ? 1 : 0;
    chain_barrier();
    const bool skip = ism[0] != 0;
    chain_barrier();
    if (skip) return;
    bool redo = false;   // mode 1: this pair's first segment starts from ve
    if (mode == 1) {
        if (walker && pair_live && gw > 0) {
            const global_ptr<const float> sv = (global_ptr<const float>)(d.vs + gw * (16 * MT));
            const global_ptr<const float> ev = (global_ptr<const float>)(d.ve + (gw - 1) * (16 * MT));
            const bool hi = lane + 64 < K;
            const float s0 = lane < K ? sv[lane] : 0.f, e0 = lane < K ? ev[lane] : 0.f;
            const float s1 = hi ? sv[lane + 64] : 0.f, e1 = hi ? ev[lane + 64] : 0.f;
            float ss = s0 + s1, es = e0 + e1;
            for (int o = 32; o > 0; o >>= 1) {
                ss += __shfl_xor(ss, o);
                es += __shfl_xor(es, o);
            }
            const float r = ss / es;
            const bool ok = (lane >= K || chain_parallel(s0, e0, ss, r)) && (!hi || chain_parallel(s1, e1, ss, r));
            redo = !__all(ok);
        }
        if (walker && lane == 0) ism[pair] = redo ? 1 : 0;
        chain_barrier();
        const int any = verdicts();
        chain_barrier();
        if (!any) return;
    }

    // steps relative to a segment's first observation: the warm-up from -W, the
    // segment from 0 to rel_end (rounded up to chunks)
    const int W = scalar(*d.warm);
    const int rel_end = scalar((int)q + (qr > 0 ? 1 : 0));
    constexpr int BUF = 4 * NSL * 64;
    float *buf = smem + pair * (2 * BUF);          // two buffers of [4 NSL][64]

    if (!walker) {
        // ------------------------------------------------------------ stager
        ChainStager<NSL, GEN, NS> sg;
        constexpr int D = ChainStager<NSL, GEN, NS>::D;
        static_assert(D % 2 == 0, "chunk p of a run uses slot p % D and buffer p % 2");
        const int64_t t0 = pair_live ? packed_seg_start(b0, q, qr) : 0;
        sg.init(d, b0, scalar(t0 > W ? t0 - W : (int64_t)0), W, lane, share);
        for (int pass = 0;; ++pass) {
            const int rel0 = pass == 0 ? -W : 0;
            sg.start(rel0);
            sg.stage(rel0, buf, 0);
            chain_barrier();
            for (int rel = rel0; rel < rel_end; rel += D * kChainStep) {
#pragma unroll
                for (int p = 0; p < D; ++p) {
                    const int r = rel + p * kChainStep;
                    if (r >= rel_end) break;
                    if (r + kChainStep < rel_end)
                        sg.stage(r + kChainStep, buf + ((p + 1) % 2) * BUF, (p + 1) % D);
                    chain_barrier();
                }
            }
            // the buffers are free: the shifts of the pass for the walker's
            // part of ln L, then its verdict
            const long long ssum = wave_sum_i64(sg.counts() ? sg.ssum : 0);
            if (lane == 0) shifts[pair * NS + share] = ssum;
            chain_barrier();
            chain_barrier();
            const int any = verdicts();
            chain_barrier();
            if (any != 1) break;
        }
        if (__any(sg.bad) && lane == 0) atomicOr(d.status, kBadData);
        return;
    }

    // ---------------------------------------------------------------- walker
    const int c = lane & 15, g = lane >> 4;
    const int64_t b = b0 + c;
    const bool live = b < nb;
    int off, lo, n;
    chain_segment(d, b, 0, W, off, lo, n);
    const int last = pair_live ? (int)(nb - b0 < kChainCols ? nb - b0 : kChainCols) - 1 : 0;   // last live column
    // chunks with every live column active: from its first column's first
    // observation on, up to the length of its last (shortest) segment
    const int rel_lo = scalar(pair_live ? -(int)min(packed_seg_start(b0, q, qr), (int64_t)W) : 0);
    const int rel_hi = scalar(pair_live ? (int)q + (b0 + last < qr ? 1 : 0) : 0);
    constexpr int KP = 16 * MT;
    // Gamma^T in the slot-major order of the product kernels
    const global_ptr<const float> GF = (global_ptr<const float>)(d.GF);
    float A[MT][NSL];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NSL; ++j) A[m][j] = GF[(j * 4 + g) * KP + phys_state<16, MT>(16 * m + c)];
    const float *er = buf + g * 64 + 4 * c;   // staged emissions of state 4 j + g: + 256 j

    float y[NSL], s[NSL];
    // start: the exact delta (times a power of two) where the warm-up reaches
    // back to the first observation, else flat
    {
        const bool exact = live && packed_seg_start(b, q, qr) <= W;
        double dmax = 0.0;
        for (int k = lane; k < K; k += 64) dmax = fmax(dmax, d.delta[k]);
        for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
        int e0 = 0;
        if (dmax > 0.0 && isfinite(dmax)) frexp(dmax, &e0);
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
            const int k = 4 * j + g;
            y[j] = k < K ? (exact ? (float)ldexp(d.delta[k], -e0) : 1.f) : 0.f;
            s[j] = 0.f;
        }
    }
    float scale = 1.f, mlow = 0x1p+60f;
    int ep = 0, eacc = 0;
    long long E = 0;
    bool mism = false;

    auto run_chunk = [&](int rel, int o, auto masked) {
        constexpr bool MASK = decltype(masked)::value;
        // steps whose emissions are read at once (registers allow four up to 12 slots)
        constexpr int RD = NSL <= 12 ? 4 : 2;
        float ev[NSL][RD];
#pragma unroll
        for (int u = 0; u < kChainStep; ++u) {
            if (u % RD == 0) {
#pragma unroll
                for (int j = 0; j < NSL; ++j) {
                    const float *src = er + j * 256 + o + u;
                    if constexpr (RD == 4) {
                        const float4 v = *reinterpret_cast<const float4 *>(src);
                        ev[j][0] = v.x;
                        ev[j][1] = v.y;
                        ev[j][2] = v.z;
                        ev[j][3] = v.w;
                    } else {
                        const float2 v = *reinterpret_cast<const float2 *>(src);
                        ev[j][0] = v.x;
                        ev[j][1] = v.y;
                    }
                }
            }
            float mx = 0.f;
            float yn[NSL];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                acc_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < NSL; ++j) acc = mfma<16>(A[m][j], y[j], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = 4 * m + r;
                    if (j >= NSL) continue;
                    yn[j] = acc[r] * (ev[j][u % RD] * scale);
                    mx = umax_f(mx, yn[j]);
                }
            }
            mx = column_max<16>(mx);
            const bool act = !MASK || (unsigned)(rel + u - lo) < (unsigned)n;
#pragma unroll
            for (int j = 0; j < NSL; ++j) y[j] = act ? yn[j] : y[j];
            if (act) {
                eacc += ep;
                ep = fexp(mx);
                scale = __builtin_amdgcn_ldexpf(1.f, -ep);
                mlow = fminf(mlow, mx);
            }
        }
        E += eacc;
        eacc = 0;
    };
    auto column_total = [&](const float (&v)[NSL]) {
        float t = 0.f;
#pragma unroll
        for (int j = 0; j < NSL; ++j) t += v[j];
        return column_sum16(t);
    };

    float ss = 0.f, es = 0.f;
    double part = 0.0;
    bool settled = false;   // another run for the sum of the differences has been asked for
    float before = 0.f;     // that sum in the pass before
    for (int pass = 0;; ++pass) {
        const int rel0 = pass == 0 ? -W : 0;
        int o = 0;   // buffer of the chunk
        chain_barrier();
        for (int rel = rel0; rel < rel_end; rel += kChainStep) {
            if (rel == 0) {
                if (redo && pass == 0 && c == 0) {
                    const global_ptr<const float> ev = (global_ptr<const float>)(d.ve + (gw - 1) * KP);
#pragma unroll
                    for (int j = 0; j < NSL; ++j) y[j] = ev[4 * j + g];
                    scale = 1.f;
                    ep = 0;
                }
#pragma unroll
                for (int j = 0; j < NSL; ++j) s[j] = y[j];
                E = 0;
            }
            if (rel >= rel_lo && rel + kChainStep <= rel_hi) run_chunk(rel, o, std::integral_constant<bool, false>());
            else run_chunk(rel, o, std::integral_constant<bool, true>());
            o ^= BUF;
            chain_barrier();
        }
        ss = column_total(s);
        es = column_total(y);
        const float pes = from_left_column(es);
        const float r = ss / pes;
        const bool inner = live && c > 0;
        bool ok = true;
        float pv[NSL], diff = 0.f;
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
            pv[j] = from_left_column(y[j]);
            ok = ok && chain_parallel(s[j], pv[j], ss, r);
            diff = fmaxf(diff, chain_diff(s[j], pv[j], ss, r));
        }
        // largest difference of each segment's start, their sum and largest
        if (!inner) diff = 0.f;
        diff = fmaxf(diff, __shfl_xor(diff, 32));
        diff = fmaxf(diff, __shfl_xor(diff, 16));
        const int differ = __popcll(__ballot(g == 0 && diff > kChainTol));   // segments
        float sum = diff;
        for (int o2 = 8; o2 > 0; o2 >>= 1) {
            sum += __shfl_xor(sum, o2);
            diff = fmaxf(diff, __shfl_xor(diff, o2));
        }
        // this walker's part of ln L
        part = 0.0;
        if (live && g == 0) part = kLn2 * (double)E + log((double)es / (double)ss);
        part = wave_sum_f64(part);
        chain_barrier();   // the stagers' shifts are in LDS
        long long stot = 0;
#pragma unroll
        for (int k = 0; k < NS; ++k) stot += shifts[pair * NS + k];
        part += kLn2 * (double)stot;
        const bool sound = fabs(part) < __builtin_inf();   // not L = 0, nothing overflowed
        mism = __any(inner && !ok) || !sound;
        // bit 0: run again; bit 1: give the set back.  At most kChainRepairs runs
        // for differences above the tolerance, and one of each walker for their sum
        int verdict = 0;
        if (mism) {
            // most starts differ and the products cost little: strictly by the rate
            const int most = chain_slow_repairs(W, (int)q, d.product_steps);
            const bool strict = last >= kChainCols / 2 && 2 * differ > last && most < kChainRepairs;
            const int left = max(0, (strict ? most : kChainRepairs) - pass);
            const bool end = !sound || pass >= kChainRepairs || (strict && pass > 0 && sum > 0.5f * before) ||
                             chain_hopeless(diff, W + pass * rel_end, left * rel_end, strict ? 1.f : 1.5f);
            verdict = end ? 3 : 1;
        } else if (!settled && sum > chain_budget((int64_t)(last + 1) * q, part)) {
            verdict = 1;
            settled = true;
        }
        before = sum;
        if (lane == 0) ism[pair] = verdict;
        chain_barrier();
        const int any = verdicts();
        chain_barrier();
        if (any != 1) break;
        // again from the first observation, each segment from its neighbour's end
        const int sh = -fexp(pes);
#pragma unroll
        for (int j = 0; j < NSL; ++j) {
            y[j] = c > 0 ? __builtin_amdgcn_ldexpf(pv[j], sh) : s[j];
        }
        scale = 1.f;
        ep = 0;
    }
    bool fail = mism || __any(live && !(mlow >= kChainLow && ss > 0.f && es > 0.f && es < 0x1p+100f));
    if (!pair_live) return;
    const global_ptr<float> vep = (global_ptr<float>)(d.ve + gw * KP);
    if (mode == 0) {
        if (c == 0) {
            const global_ptr<float> vsp = (global_ptr<float>)(d.vs + gw * KP);
#pragma unroll
            for (int j = 0; j < NSL; ++j) vsp[4 * j + g] = s[j];
        }
        if (c == last) {
#pragma unroll
            for (int j = 0; j < NSL; ++j) vep[4 * j + g] = y[j];
        }
    } else {
        // the neighbour to the right was verified against the old end
        float o[NSL];
#pragma unroll
        for (int j = 0; j < NSL; ++j) o[j] = vep[4 * j + g];
        const float os = column_total(o);
        const float r = es / os;
        bool ok = true;
#pragma unroll
        for (int j = 0; j < NSL; ++j) ok = ok && chain_parallel(y[j], o[j], es, r);
        fail = fail || __any(c == last && !ok);
    }
    if (lane == 0) {
        d.part[gw] = part;
        if (fail) atomicOr(d.fail, 1);
    }
}

// Single set: workgroup = blockIdx.x.
template <int MT, int NSL, bool GEN, int NP, int NS>
__global__ __launch_bounds__(64 * NP * (1 + NS)) void k_chain(SetDesc d, int mode)
{
    chain_body<MT, NSL, GEN, NP, NS>(d, blockIdx.x, mode);
}

}  // namespace hmm
