// Viterbi by score vectors over segments, verified on the device: the max-plus
// counterpart of the segment chains (hmm_chain.hpp).
//
// Survivor paths of all states at one time soon share an ancestor, going back;
// from there on the score vector is fixed up to a constant by the observations
// alone, and the best path up to some time is fixed by a few observations after
// it.  Segment b therefore runs the plain recursion
//   d_t[j] = max_i (d_{t-1}[i] + log2 Gamma_ij) + log2 e_t,j   (largest entry 0)
// from a flat vector kVitWarm steps before its first observation (s_b: the
// vector it has got to there, e_b: the one after its last observation), carries
// on kVitAhead steps past its end, and backtracks from the best state there:
// its own part of the path is written.  This is the exact solution when
// s_b = e_{b-1} and the state in which segment b ends is the one before the
// first of segment b + 1, for every b; both are checked.  A segment that
// differs is run again from e_{b-1} to that state (and must then end as
// before); if that fails, or Gamma has entries below 2^-56, the max-plus
// product path behind it runs.
//
// The score is that of the returned path, added up as the product path rounds
// it.  Its segments' products are FP32 matrices kept near their largest entry;
// the row of the state in which the path enters a segment follows, bit by bit,
// the recursion along the path alone, given each step's largest entry over the
// matrix - and that is the largest entry of a vector started flat at the
// segment's first observation, since rounding is monotone and so commutes with
// the maximum over rows.  Wavefronts of the first launch write those (mx);
// k_vit_path_score follows the path through them.  (Summed up in another way
// the score is as exact - 1e-9 to 4e-9 either way, from rounding errors that
// recur at every observation without a location - but moves by that much.)
//
// Work: K^2 instead of K^3 additions and maxima per observation.  One wavefront
// holds 64 / HW segments, lane = state (K > 64: two states per lane); the
// column of log2 Gamma stays in registers, the vector goes round through LDS,
// the backpointers of a segment (bytes) stay in LDS.  What bounds it: VALU
// issue (K = 25: 100 instructions a step, 160 with the backpointers, of which
// 50 are the comparisons and selects of the argmax; 68 % of the SIMDs' time at
// T = 1e6), and a step's chain of LDS round trip, additions and row maxima, 0.37
// us, where a SIMD holds only one wavefront (K = 64, T = 105,000: 47 %).  K = 25, T = 1e6: 1.55 -> 0.34 ms for the call (0.28 without
// the score's flat vectors), K = 64, T = 105,000: 3.2 -> 0.23 ms.
#pragma once

#include "hmm_chain.hpp"

namespace hmm {

// Steps of warm-up and lookahead.  Tremor data, K = 8..80: of segments with 32
// / 48 / 64..72 steps of warm-up 0.6 / 0.1 / 0.05 % did not meet, with 80 none
// of 4,000; with 24 / 32 / 44 steps of lookahead 0.3 / 0.03 / 0.02 %, with 48
// none.  One segment that differs costs the call another pass over a segment
// (40 to 80 us); 72 and 44 steps did so at one T in three, at a gain of 8 us.
constexpr int kVitWarm = 96, kVitAhead = 64;
// Largest difference of two vectors (largest entry 0, log2) taken as rounding:
// a few 2^-24 of the entries' size per step; vectors whose survivors have not
// met differ by tenths.
__device__ __forceinline__ bool vit_same(float a, float b)
{
    return a == b || fabsf(a - b) <= 0x1p-12f + 0x1p-18f * fabsf(a);   // a == b: both -inf too
}

struct VitChain {
    const uint8_t *flag;
    const double *xy;
    const StateConst *sc;
    const float *lg;         // [KB][KB] log2 Gamma, -inf outside K
    const double *delta;
    int *status, *fail;
    float *sv, *ev;          // [nb][KR] vectors at the segments' starts and ends
    int32_t *endst, *pre;    // [nb] state at the segment's end, state before its start
    float *mx;               // [T] largest entry of the flat vectors' steps
    double *acc;             // [fnb] score of the path in a product segment (log2)
    int32_t *path;
    int64_t fnb, fL;         // segments of the product path, their length
    int64_t T, nb, q, r;     // segments of q or (the first r) q + 1 observations
    int K, KB;
    int rows;                // of backpointers of a segment: its length + kVitAhead
    int cblocks;             // workgroups of segments; the first launch's others walk flat vectors
};

__device__ __forceinline__ float max3_f32(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// arg <- the smallest of I .. I + 3 whose entry equals m, else as it was.  The
// four comparisons come first: a select reads its mask two wait states or more
// after the comparison.
template <int I>
__device__ __forceinline__ void vit_arg4(int &arg, float a, float b, float c, float e, float m)
{
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_eq_f32_e64 %4, %8, %9\n\t"
        "v_cmp_eq_f32_e64 %3, %7, %9\n\t"
        "v_cmp_eq_f32_e64 %2, %6, %9\n\t"
        "v_cmp_eq_f32_e64 %1, %5, %9\n\t"
        "v_cndmask_b32_e64 %0, %0, %13, %4\n\t"
        "v_cndmask_b32_e64 %0, %0, %12, %3\n\t"
        "v_cndmask_b32_e64 %0, %0, %11, %2\n\t"
        "v_cndmask_b32_e64 %0, %0, %10, %1"
        : "+v"(arg), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(a), "v"(b), "v"(c), "v"(e), "v"(m), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
}

// arg <- the smallest i in [LO, HI) with x[i] == m, counted from BASE.
template <int LO, int HI, int BASE, int N>
__device__ __forceinline__ void vit_arg(int &arg, const float (&x)[N], float m)
{
    if constexpr (HI - LO >= 4) {
        vit_arg4<HI - 4 - BASE>(arg, x[HI - 4], x[HI - 3], x[HI - 2], x[HI - 1], m);
        vit_arg<LO, HI - 4, BASE>(arg, x, m);
    } else if constexpr (HI > LO) {   // repeated entries of the first index change nothing
        constexpr int n = HI - LO;
        constexpr int i1 = n > 1 ? LO + 1 : LO, i2 = n > 2 ? LO + 2 : LO;
        arg = x[i2] == m ? i2 - BASE : arg;
        arg = x[i1] == m ? i1 - BASE : arg;
        arg = x[LO] == m ? LO - BASE : arg;
    }
}

// max(v, v moved within a row of 16 lanes); the move reads v two wait states
// after it was written.
#define HMM_VIT_ROW_MAX(v, move)                                                                          \
    asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 " move " row_mask:0xf bank_mask:0xf" : "=v"(v) : "v"(v))

// Maximum over the HW lanes of a segment, in every one of them.
template <int HW>
__device__ __forceinline__ float seg_max(float v)
{
    HMM_VIT_ROW_MAX(v, "quad_perm:[1,0,3,2]");
    HMM_VIT_ROW_MAX(v, "quad_perm:[2,3,0,1]");
    HMM_VIT_ROW_MAX(v, "row_half_mirror");
    HMM_VIT_ROW_MAX(v, "row_mirror");   // every lane holds its row's maximum
    if constexpr (HW >= 32) asm("s_nop 1" : "+v"(v));   // the swap reads it
    if constexpr (HW >= 32) {
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = max_f32(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    if constexpr (HW >= 64) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = max_f32(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

__device__ __forceinline__ void vit_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// States K padded to KR for the vector's 16-byte reads.
__host__ __device__ constexpr int vit_kr(int KK) { return (KK + 3) / 4 * 4; }

// LDS of one segment: the vector, one chunk of observations, and rows of
// backpointers (their number is the plan's).
template <int KR, int HW>
struct VitLds {
    static constexpr int vec = 4 * (KR > 64 ? 128 : HW);      // every lane writes
    static constexpr int obs = HW * 24;                       // x, y, flag
    static constexpr int fixed = (vec + obs + 15) / 16 * 16;
};
__host__ __device__ constexpr int vit_psi_bytes(int KR, int rows) { return (rows * KR + 128 + 15) / 16 * 16; }

// Whether at least three in four of 64 segments spread over the record start
// elsewhere than their neighbours end, by eight entries of the vectors: the
// record forgets too slowly, a rerun of nearly every segment would not meet its
// old end either.  Asked by wavefronts that have a segment to run again (K = 25,
// T = 10^6, Gamma_ii 0.95, no location information: 2,020 -> 1,890 us, products
// alone 1,550; K = 64, T = 105,000: 3,583 -> 3,465, 3,225).
__device__ __forceinline__ bool vit_most_differ(const VitChain &v, int kr, int lane)
{
    if (v.nb <= 64) return false;
    const int64_t s = 1 + lane * (v.nb - 1) / 64;
    const float *a = v.sv + s * kr, *e = v.ev + (s - 1) * kr;
    bool differ = false;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int j = i * v.K / 8;
        differ = differ || !vit_same(a[j], e[j]);
    }
    return __popcll(__ballot(differ)) >= 48;
}

// mode 0: every segment.  mode 1: the check, and the segments that differ.
// KK: states the loops run over (K itself for K <= 32).
template <int KK, int HW>
__global__ __launch_bounds__(64) void k_vit_chain(VitChain v, int mode)
{
    constexpr int KR = vit_kr(KK);
    constexpr int NS = KR > 64 ? 2 : 1;   // states per lane: j and j + 64
    typedef VitLds<KR, HW> Lds;
    extern __shared__ __attribute__((aligned(16))) unsigned char vsm[];
    const int lane = threadIdx.x & 63, h = lane / HW, l = lane % HW;
    const int K = v.K;
    // workgroups from cblocks on (first launch only): flat vectors
    const bool flat = (int)blockIdx.x >= v.cblocks;
    const int64_t b = (int64_t)((int)blockIdx.x - (flat ? v.cblocks : 0)) * (64 / HW) + h;
    const bool live = b < (flat ? v.fnb : v.nb);
    const int64_t bb = live ? b : 0;
    if (__builtin_amdgcn_readfirstlane(*v.fail) != 0 || __builtin_amdgcn_readfirstlane(*v.status) != 0) return;
    unsigned char *mine = vsm + h * (Lds::fixed + vit_psi_bytes(KR, v.rows));
    float *vec = reinterpret_cast<float *>(mine);
    double *obx = reinterpret_cast<double *>(mine + Lds::vec);   // [HW][3]: x, y, flag
    unsigned char *psi = mine + Lds::fixed;
    const int64_t t0 = flat ? bb * v.fL : bb * v.q + (bb < v.r ? bb : v.r);
    const int len = !live ? 0 : (flat ? (int)min(v.fL, v.T - t0) : (int)v.q + (bb < v.r ? 1 : 0));
    const bool inner = live && b > 0, last = b + 1 >= v.nb;

    bool redo = false;
    int want_end = -1;
    if (mode == 1) {
        // this segment's start against its neighbour's end, its end state
        // against the one its other neighbour came from
        bool bad = false;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int j = l + 64 * s;
            if (inner && j < K) bad = bad || !vit_same(v.sv[b * KR + j], v.ev[(b - 1) * KR + j]);
        }
        if (live && !last) {
            want_end = v.pre[b + 1];
            bad = bad || want_end != v.endst[b];
        }
        redo = seg_max<HW>(bad ? 1.f : 0.f) > 0.f;
        if (!__any(redo)) return;
        if (vit_most_differ(v, KR, lane)) {
            if (lane == 0) atomicOr(v.fail, 1);
            return;
        }
    }

    // constants of this lane's states, and their columns of log2 Gamma
    double mx_[NS], my_[NS], cxx[NS], cxy[NS], cyy[NS], a1[NS], a0[NS];
    float lg[NS][KK];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int j = l + 64 * s;
        const StateConst c = v.sc[j < K ? j : 0];
        mx_[s] = c.mx;
        my_[s] = c.my;
        cxx[s] = c.cxx;
        cxy[s] = c.cxy;
        cyy[s] = c.cyy;
        a1[s] = j < K ? c.a1 : -INFINITY;
        a0[s] = j < K ? c.a0 : -INFINITY;
#pragma unroll
        for (int i = 0; i < KK; ++i) lg[s][i] = j < v.KB ? v.lg[i * v.KB + j] : -INFINITY;
    }

    // start vector: the initial distribution where the warm-up reaches back to
    // the first observation, a neighbour's end in a rerun, else flat
    float d[NS];
    float po = 0.f;   // K > 32: what the vector's largest entry is, else 0
    const bool exact = t0 <= kVitWarm && !flat;
    {
        float top = -INFINITY;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int j = l + 64 * s;
            float x = -INFINITY;
            if (j < K) {
                if (mode == 1 && inner) x = v.ev[(b - 1) * KR + j];
                else x = exact ? (float)log2(v.delta[j]) : 0.f;
            }
            d[s] = x;
            top = fmaxf(top, x);
        }
        top = seg_max<HW>(top);
        const bool fin = top > -INFINITY;
#pragma unroll
        for (int s = 0; s < NS; ++s) d[s] = fin ? d[s] - top : d[s];
    }

    // observations of the next chunk, one per lane; the flag a chunk earlier:
    // where it is not 1 the location is not the caller's to read (a word of the
    // constants instead, never used)
    double ox, oy;
    int of, oflag, bad = 0;
    auto place = [&](int rel) {
        const int64_t t = t0 + rel + l;
        return t < 0 ? (int64_t)0 : (t < v.T ? t : v.T - 1);
    };
    auto fetch = [&](int rel) {
        of = oflag;
        const double2 p = *(of == 1 ? reinterpret_cast<const double2 *>(v.xy) + place(rel)
                                    : reinterpret_cast<const double2 *>(v.sc));
        ox = p.x;
        oy = p.y;
        oflag = v.flag[place(rel + HW)];
    };
    // steps that the segment takes: inside the record, to its lookahead's end
    const int ahead = mode == 1 || flat ? 0 : kVitAhead;   // a rerun knows its end state
    const int lo = t0 < kVitWarm ? -(int)t0 : -kVitWarm;   // not reached before 0 by flat vectors
    const int hi = !live ? -kVitWarm : (int)(v.T - t0 < len + ahead ? v.T - t0 : (int64_t)(len + ahead));
    const int rel_end = flat ? (int)v.fL : (int)v.q + (v.r > 0 ? 1 : 0) + ahead;
    float de[NS];   // the vector after the segment's last observation
#pragma unroll
    for (int s = 0; s < NS; ++s) de[s] = d[s];
    // steps [from, to).  KIND 1: with backpointers; 2: flat vectors, whose
    // largest entries take the observations' place in LDS.  The order of
    // operations is that of the product kernels, up to 32 states
    // ((d + log2 Gamma) + log2 e) - max, above with the maximum taken off the
    // next step's log2 e.  Rows past a segment's last
    // step are written too and never read; entries past KR spill into the next
    // row, which is written after.
    auto walk = [&](int from, int to, auto kind_) {
        constexpr int KIND = decltype(kind_)::value;
        constexpr bool MAIN = KIND == 1;
        oflag = v.flag[place(from)];
        fetch(from);
        for (int rc = from; rc < to; rc += HW) {
            {   // the chunk's observations to LDS, the next chunk's loads in flight
                const bool one = of == 1, finite = isfinite(ox) && isfinite(oy);
                if (MAIN && rc + l < len && (of > 1 || (one && !finite))) bad = 1;
                obx[3 * l] = one && finite ? ox : 0.0;
                obx[3 * l + 1] = one && finite ? oy : 0.0;
                reinterpret_cast<int64_t *>(obx)[3 * l + 2] = one && finite ? -1 : 0;   // select mask
                if (rc + HW < to) fetch(rc + HW);
            }
            const int n = min(HW, to - rc);
            for (int u = 0; u < n; ++u) {
                const int rel = rc + u;
#pragma unroll
                for (int s = 0; s < NS; ++s) vec[l + 64 * s] = d[s];
                vit_lds_sync();
                const double x = obx[3 * u], y = obx[3 * u + 1];
                const int64_t dens = reinterpret_cast<const int64_t *>(obx)[3 * u + 2];
                float nd[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    float x_[KR];
#pragma unroll
                    for (int i4 = 0; i4 < KR / 4; ++i4) {
                        const float4 q = reinterpret_cast<const float4 *>(vec)[i4];
                        x_[4 * i4] = q.x;
                        x_[4 * i4 + 1] = q.y;
                        x_[4 * i4 + 2] = q.z;
                        x_[4 * i4 + 3] = q.w;
                    }
#pragma unroll
                    for (int i = 0; i < KK; ++i) x_[i] += lg[s][i];
                    float m = x_[0];
#pragma unroll
                    for (int i = 1; i + 1 < KK; i += 2) m = max3_f32(m, x_[i], x_[i + 1]);
                    if constexpr (KK % 2 == 0) m = max_f32(m, x_[KK - 1]);
                    if constexpr (MAIN) {   // smallest index on ties
                        int arg = 0;
                        if constexpr (KK > 64) {
                            vit_arg<64, KK, 64>(arg, x_, m);
                            arg += 64;
                        }
                        vit_arg<0, (KK > 64 ? 64 : KK), 0>(arg, x_, m);
                        psi[rel * KR + l + 64 * s] = (unsigned char)arg;
                    }
                    const double d0 = x - mx_[s], d1 = y - my_[s];
                    const double qd = a1[s] + d0 * (cxx[s] * d0 + cxy[s] * d1) + cyy[s] * (d1 * d1);
                    const int64_t la = (__double_as_longlong(qd) & dens) | (__double_as_longlong(a0[s]) & ~dens);
                    const float le = (float)__longlong_as_double(la);
                    nd[s] = m + (KK > 32 ? le - po : le);
                }
                const float top = seg_max<HW>(NS == 2 ? max_f32(nd[0], nd[NS - 1]) : nd[0]);
                const float sub = top > -INFINITY ? top : 0.f;
                const bool act = rel >= lo && rel < hi;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    d[s] = act ? (KK > 32 ? nd[s] : nd[s] - sub) : d[s];
                    if constexpr (MAIN) de[s] = rel < len ? (KK > 32 ? d[s] - sub : d[s]) : de[s];
                }
                if constexpr (KK > 32) po = act ? sub : po;
                if constexpr (KIND == 2) reinterpret_cast<float *>(obx)[6 * u] = sub;
            }
            if constexpr (KIND == 2) {
                vit_lds_sync();
                if (l < n && rc + l < len) v.mx[t0 + rc + l] = reinterpret_cast<const float *>(obx)[6 * l];
                vit_lds_sync();   // the next chunk's observations (another type) come after these reads
            }
        }
    };
    if (flat) {
        walk(0, rel_end, std::integral_constant<int, 2>());
        return;
    }
    if (mode == 0) {
        walk(-kVitWarm, 0, std::integral_constant<int, 0>());
        if (inner) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (l + 64 * s < K) v.sv[b * KR + l + 64 * s] = d[s] - po;
        }
    }
    walk(0, rel_end, std::integral_constant<int, 1>());
    if (__any(bad) && lane == 0) atomicOr(v.status, kBadData);
    {
        bool same = true;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int j = l + 64 * s;
            if (!live || j >= K) continue;
            if (mode == 0) v.ev[b * KR + j] = de[s];
            else if (redo) same = same && vit_same(de[s], v.ev[b * KR + j]);
        }
        if (!same) atomicOr(v.fail, 1);   // the neighbour was checked against the old end
    }

    // best state at the end of the lookahead (smallest index on ties)
    int e;
    {
        float top = -INFINITY;
        int at = 0x7fffffff;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (l + 64 * s < K) top = fmaxf(top, d[s]);
        top = seg_max<HW>(top);
#pragma unroll
        for (int s = NS - 1; s >= 0; --s)
            if (l + 64 * s < K && d[s] == top) at = l + 64 * s;
        // smallest index over the lanes, as a maximum of -index (exact in FP32)
        const float neg = seg_max<HW>(at == 0x7fffffff ? -1.0e6f : -(float)at);
        e = neg <= -1.0e6f ? 0 : (int)-neg;
        if (!(top > -INFINITY) && live) atomicOr(v.fail, 1);   // no path: the product path reports it
        if (want_end >= 0) e = want_end;
    }
    vit_lds_sync();
    // backtracking; lane l collects steps l, l + HW, ... of the segment's part
    const bool write = live && (mode == 0 || redo);
    int keep = 0, e_own = 0;
    for (int rc = (rel_end - 1) / HW * HW; rc >= 0; rc -= HW) {
        for (int u = min(HW, rel_end - rc) - 1; u >= 0; --u) {
            const int rel = rc + u;
            e_own = rel == len - 1 ? e : e_own;
            keep = u == l ? e : keep;
            const int f = psi[rel * KR + e];
            e = rel < hi ? f : e;
        }
        if (write && rc + l < len) v.path[t0 + rc + l] = keep;
    }
    if (l == 0 && write) {
        if (mode == 0) {
            v.endst[b] = e_own;
            v.pre[b] = e;
        } else if (e != v.pre[b]) {
            atomicOr(v.fail, 1);   // the neighbour was checked against the old one
        }
    }
}

// Score of the path in the product segments, one wavefront each: lane = step
// for what does not depend on the sum, then the steps in order.  KD: the
// kernels above 32 states' order of operations.
template <bool KD>
__global__ __launch_bounds__(256) void k_vit_path_score(VitChain v)
{
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= v.fnb || *v.fail != 0 || *v.status != 0) return;
    const int64_t t0 = b * v.fL, t1 = min(v.T, t0 + v.fL);
    float r = 0.f, po = 0.f;
    double acc = 0.0;
    for (int64_t tc = t0; tc < t1; tc += 64) {
        const int n = (int)min((int64_t)64, t1 - tc);
        float a = 0.f, e = 0.f, m = 0.f;
        if (lane < n) {
            const int64_t t = tc + lane;
            const int j = v.path[t], i = t > 0 ? v.path[t - 1] : v.pre[0];
            const bool tremor = v.flag[t] == 1;
            double2 x{0.0, 0.0};
            if (tremor) x = reinterpret_cast<const double2 *>(v.xy)[t];
            a = v.lg[i * v.KB + j];
            e = (float)state_log2_emission(v.sc[j], tremor, x.x, x.y);
            m = v.mx[t];
        }
        acc += (double)m;
        if constexpr (KD) {
            const float before = __shfl_up(m, 1);
            e = lane < n ? e - (lane == 0 ? po : before) : 0.f;
            po = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m), n - 1));
        }
        // lanes past the end hold zeros, which leave r as it is: whole halves,
        // unrolled (28 -> 25 us at K = 25, T = 1e6 against a loop over n; the rest
        // is the FP64 emission and the gathers of 64 steps at a time)
        for (int u0 = 0; u0 < n; u0 += 32) {
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                r += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), u0 + u));
                r += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e), u0 + u));
                if constexpr (!KD) r -= __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m), u0 + u));
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) v.acc[b] = acc + (double)(r - po) + (b == 0 ? log2(v.delta[v.pre[0]]) : 0.0);
}

}  // namespace hmm
