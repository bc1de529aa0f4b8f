// Batched likelihood: many parameter sets (MCMC chains or proposals) with
// uneven K and T evaluated by one captured launch sequence, and the segment
// length autotuner.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <new>
#include <numeric>

#include "hmm_host.hpp"

namespace hmmh {

// Sets that share one kernel instantiation (operand precision, tile shape,
// live contraction slots) form a class: one segment launch and one fold
// launch per class.
struct BatchClass {
    KernelSet ks;          // blocked paths
    const void *serial = nullptr;  // plain-forward path: k_serial_batch<KP>
    int KP = 0;
    int *ids = nullptr;    // plain-forward path: the class's set ids (device)
    // batched segment kernel (k_blocked or, with G > 1 segments per
    // wavefront, k_blocked_packed), its wavefronts per workgroup and LDS
    const void *seg = nullptr;
    int G = 1, waves = 1;
    size_t seg_lds = 0;
    int W = 1, W2 = 1;     // segments per segment job, wavefronts of a fold workgroup
    int64_t L = 0;
    int grid = 0;          // workgroups of the persistent segment launch (0: one per job)
    int *queue = nullptr;  // its atomic job counter (device)
    double cost = 0.0;     // sum over jobs of observations * KP^3 (class order)
    size_t nprod = 0;      // product slots (segment products and pre-fold outputs)
    std::vector<int> sets;
    size_t job0 = 0, njobs = 0;   // WgJob table range
    size_t fjob0 = 0, nfjobs = 0; // FoldJob table range (one per set)
    size_t pjob0 = 0, npjobs = 0; // pre-fold FoldJob table range (sets with many products)
    float *M = nullptr;
    long long *E = nullptr, *S = nullptr;
};

struct BatchPlan {
    // what the plan was built for
    int n = 0, algo = 0;
    std::vector<int32_t> K;
    std::vector<int64_t> T, param_off, obs_off;
    const double *params = nullptr;
    const uint8_t *flag = nullptr;
    const double *xy = nullptr;
    double *out = nullptr;
    std::map<std::pair<int, int>, int64_t> tuned;
    std::map<std::pair<int, int>, int> tunedW;
    bool persistent = true;
    int packing = 1;
    bool chain = false;      // segment chains first (default tuning knobs, FP32)
    // device memory and the pinned host copy of the descriptor tables at its
    // start (sets and prep jobs first).  Another plan takes both over, once the
    // device has been synchronised; events, streams and graphs are a plan's own.
    // `copied` follows the last copy out of the pinned buffer.
    void *mem = nullptr;
    size_t mem_bytes = 0;
    char *host = nullptr;
    size_t host_bytes = 0;
    size_t o_prep = 0, pointer_bytes = 0, table_bytes = 0;   // offsets in the tables
    hipEvent_t copied = nullptr;
    SetDesc *sets = nullptr;
    PrepJob *prep = nullptr;
    WgJob *jobs = nullptr;
    FoldJob *fjobs = nullptr;
    FoldJob *pjobs = nullptr;
    // two words per class, zeroed at the start of every launch sequence: its
    // job counter, and whether a set of it is left to the product path
    int *queues = nullptr;
    ChainJob *cjobs = nullptr;   // workgroups of the segment chains
    size_t ncjobs = 0, chain_lds = 0;
    int *cls = nullptr;          // class of every set
    std::vector<BatchClass> classes;
    // captured launch sequence (classes forked onto parallel branches): from
    // the second call with the same descriptors on, the first one launches it
    // directly on the caller's stream (a capture costs more than the launches
    // it saves once).
    bool launched = false;
    static constexpr int kBranches = 4;
    hipStream_t cap = nullptr;
    hipStream_t aux[kBranches] = {};
    hipEvent_t fork = nullptr, join[kBranches] = {};
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

void batch_plan_free(BatchPlan *bp)
{
    if (!bp) return;
    if (bp->exec) (void)hipGraphExecDestroy(bp->exec);
    if (bp->graph) (void)hipGraphDestroy(bp->graph);
    if (bp->cap) (void)hipStreamDestroy(bp->cap);
    for (int i = 0; i < BatchPlan::kBranches; ++i) {
        if (bp->aux[i]) (void)hipStreamDestroy(bp->aux[i]);
        if (bp->join[i]) (void)hipEventDestroy(bp->join[i]);
    }
    if (bp->fork) (void)hipEventDestroy(bp->fork);
    if (bp->copied) (void)hipEventDestroy(bp->copied);
    if (bp->mem) (void)hipFree(bp->mem);
    if (bp->host) (void)hipHostFree(bp->host);
    delete bp;
}

namespace {

// Segment length of a class.  Workgroups run one per CU, in rounds of 256;
// a round costs about L steps plus a fixed per-workgroup part (emission
// setup, the in-workgroup tree) worth kWgOverhead steps.  The length
// minimises rounds(L) * (L + kWgOverhead) over kMinL..4096, so that the last
// round is not left mostly empty (and a set too short to fill the chip in one
// round at a longer length is cut finer).  A tuned value wins.
constexpr int kWgOverhead = 32;
constexpr int64_t kMinL = 16;   // shortest segment the cost model considers

// A set whose final fold would take more than kPrefoldF products per
// wavefront gets one more fold level first (a lone long set cut into short
// segments: its final workgroup would otherwise chain many products).
constexpr int kPrefoldF = 2;

int64_t class_L(const hmm_ctx *ctx, const BatchPlan &bp, const BatchClass &c, int algo, int W)
{
    for (int s : c.sets) {
        auto it = ctx->tuned_L.find({bp.K[s], algo});
        if (it != ctx->tuned_L.end() && it->second > 0) return it->second;
    }
    if (ctx->block_len > 0) return ctx->block_len;
    int64_t best = kMinL;
    double best_cost = -1.0;
    for (int64_t L = kMinL; L <= 4096; ++L) {
        if (best_cost >= 0.0 && (double)(L + kWgOverhead) >= best_cost) break;   // rounds >= 1: no better from here on
        int64_t wgs = 0;
        for (int s : c.sets) {
            const int64_t nseg = (bp.T[s] + L - 1) / L;
            wgs += (nseg + W - 1) / W;
        }
        const int64_t rounds = std::max<int64_t>(1, (wgs + 255) / 256);
        const double cost = (double)rounds * (double)(L + kWgOverhead);
        if (best_cost < 0.0 || cost < best_cost) {
            best_cost = cost;
            best = L;
        }
    }
    return best;
}

// Most wavefronts per workgroup of a class's segment kernel.
int max_waves(const BatchClass &c) { return c.G > 1 ? c.ks.packWaves : c.ks.seg_waves(); }

// Segment-kernel waves per workgroup of a class: a tuned value wins (w > 0:
// w waves, at most the kernel's maximum; w < 0: the maximum divided by -w,
// the autotuner's candidates), else the maximum.
int class_waves(const hmm_ctx *ctx, const BatchPlan &bp, const BatchClass &c, int algo)
{
    const int wmax = max_waves(c);
    for (int s : c.sets) {
        auto it = ctx->tuned_W.find({bp.K[s], algo});
        if (it == ctx->tuned_W.end() || it->second == 0) continue;
        return it->second > 0 ? std::min(it->second, wmax) : std::max(1, wmax / -it->second);
    }
    return wmax;
}

// The kernel that identifies a class: the batched segment kernel (the packed
// one where the packing mode gives one for K), or the plain-forward kernel.
const void *class_key(const KernelSet &ks, bool serial)
{
    if (serial) return ks.seg1;
    return ks.segPB ? ks.segPB : ks.segB;
}

// Fill kernel for the classes' words {job counter, left to the product path}
// (a kernel, not a memset node, so that the captured graph replays it reliably).
__global__ void k_init_words(int *p, int n, int left)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        p[2 * i] = 0;
        p[2 * i + 1] = left;
    }
}

// Segment chains of a batch: the plan of set s (empty: product path only) and
// the segment length all sets share.  One workgroup (32 segments) per CU, as
// many as are resident, but segments of at most kBatchChainLen: long ones leave
// few workgroups of very different cost (K = 8 and K = 64 in one launch), and
// at this length the warm-up is 8..20 % of the work.  A set takes part where the
// sets of its K bracket together are long enough (chain_min_T): in a batch the
// launches are shared.
constexpr int64_t kBatchChainLen = 512;

void plan_batch_chains(const BatchPlan &bp, std::vector<ChainPlan> *cps)
{
    cps->assign(bp.n, ChainPlan());
    int64_t total = 0, bracket[4] = {};
    auto bracket_of = [](int K) { return K <= 4 ? 0 : (K <= 16 ? 1 : (K <= 25 ? 2 : 3)); };
    for (int s = 0; s < bp.n; ++s) {
        total += bp.T[s];
        bracket[bracket_of(bp.K[s])] += bp.T[s];
    }
    const int64_t segs = 256 * ChainShape{2, 1}.segs();
    const int64_t L = std::max(kChainMinLen, std::min(kBatchChainLen, (total + segs - 1) / segs));
    for (int s = 0; s < bp.n; ++s)
        if (bracket[bracket_of(bp.K[s])] >= chain_min_T(bp.K[s]))
            (*cps)[s] = cut_chain(bp.T[s], L, ChainShape{2, 1});
}

// Cost of one chain step of 32 segments, in units of a matrix instruction:
// the longer of the walker's products and the stager's evaluations.
double chain_step_cost(int K)
{
    const int nsl = (K + 3) / 4, mt = (K + 15) / 16;
    return std::max(8.0 + mt * nsl, 8.0 + 2.9 * nsl);
}

const void *serial_kernel(int KP)
{
    switch (KP) {
    case 16: return reinterpret_cast<const void *>(&k_serial_batch<16>);
    case 32: return reinterpret_cast<const void *>(&k_serial_batch<32>);
    case 64: return reinterpret_cast<const void *>(&k_serial_batch<64>);
    case 96: return reinterpret_cast<const void *>(&k_serial_batch<96>);
    default: return reinterpret_cast<const void *>(&k_serial_batch<128>);
    }
}

// Ends the context's plan: its launches, copies and graph replays are over
// before anything it owns is given back or taken over.
int retire(hmm_ctx *ctx, BatchPlan &bp)
{
    BatchPlan *old = ctx->batch;
    if (!old) return HMM_OK;
    if (hipDeviceSynchronize() != hipSuccess) return HMM_E_DEVICE;
    std::swap(bp.mem, old->mem);
    std::swap(bp.mem_bytes, old->mem_bytes);
    std::swap(bp.host, old->host);
    std::swap(bp.host_bytes, old->host_bytes);
    batch_plan_free(old);
    ctx->batch = nullptr;
    return HMM_OK;
}

// Whether a buffer of `held` bytes serves a plan that needs `bytes`: large
// enough, and not so large that a small plan would hold on to a big one's.
bool serves(size_t held, size_t bytes) { return held >= bytes && held / 4 <= bytes + (size_t(4) << 20); }

// Device memory of a plan (the tables are a part of it) and their pinned copy:
// the ones taken over where they serve (nothing is queued that uses them),
// else new ones.  32 mixed sets with other descriptors on every call: 533 us;
// 690 where the job tables are made after the wait of retire and not before it,
// 1,188 with new memory each time as well.
int allocate(BatchPlan &bp, size_t bytes)
{
    if (!serves(bp.mem_bytes, bytes)) {
        if (bp.mem) (void)hipFree(bp.mem);
        bp.mem = nullptr;
        bp.mem_bytes = 0;
        if (hipMalloc(&bp.mem, bytes) != hipSuccess) {
            (void)hipGetLastError();
            bp.mem = nullptr;
            return HMM_E_NOMEM;
        }
        bp.mem_bytes = bytes;
    }
    if (!serves(bp.host_bytes, bp.table_bytes)) {
        if (bp.host) (void)hipHostFree(bp.host);
        bp.host = nullptr;
        bp.host_bytes = 0;
        if (hipHostMalloc(reinterpret_cast<void **>(&bp.host), bp.table_bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            bp.host = nullptr;
            return HMM_E_NOMEM;
        }
        bp.host_bytes = bp.table_bytes;
    }
    return hipEventCreateWithFlags(&bp.copied, hipEventDisableTiming) == hipSuccess ? HMM_OK : HMM_E_DEVICE;
}

// Copies the first `bytes` of the tables, ordered on st after the launches
// that still read the old ones.
int upload(BatchPlan &bp, size_t bytes, hipStream_t st)
{
    const bool sent = hipMemcpyAsync(bp.mem, bp.host, bytes, hipMemcpyHostToDevice, st) == hipSuccess;
    if (sent && hipEventRecord(bp.copied, st) == hipSuccess) return HMM_OK;
    (void)hipGetLastError();
    if (sent) (void)hipStreamSynchronize(st);   // no event says when the copy is over
    return HMM_E_DEVICE;
}

// New input and output buffers for a plan's descriptors: only the pointers in
// the tables change.  The plan has no buffers (no call matches it) until the
// copy is under way, so a call after a failed one copies again.
int set_pointers(BatchPlan &bp, const double *params, const uint8_t *flag, const double *xy, double *out,
                 hipStream_t st)
{
    if (hipEventSynchronize(bp.copied) != hipSuccess) return HMM_E_DEVICE;
    SetDesc *hs = reinterpret_cast<SetDesc *>(bp.host);
    PrepJob *hp = reinterpret_cast<PrepJob *>(bp.host + bp.o_prep);
    bp.out = nullptr;
    for (int s = 0; s < bp.n; ++s) {
        hs[s].obs = Obs{flag + bp.obs_off[s], xy + 2 * bp.obs_off[s], nullptr, kEmisTremor, 0};
        hs[s].delta = hp[s].params = params + bp.param_off[s];
        hs[s].out = out + s;
    }
    const int rc = upload(bp, bp.pointer_bytes, st);
    if (rc != HMM_OK) return rc;
    bp.params = params;
    bp.flag = flag;
    bp.xy = xy;
    bp.out = out;
    return HMM_OK;
}

// Workgroups of a kernel that a CU holds at once (asked once per launch shape).
int resident_groups(const void *fn, int threads, size_t lds)
{
    static std::mutex mu;
    static std::map<std::pair<const void *, std::pair<int, size_t>>, int> known;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_pair(fn, std::make_pair(threads, lds));
    auto it = known.find(key);
    if (it != known.end()) return it->second;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess || per_cu < 1) {
        (void)hipGetLastError();
        return 1;
    }
    known[key] = per_cu;
    return per_cu;
}

int build(hmm_ctx *ctx, BatchPlan &bp, hipStream_t st)
{
    const int n = bp.n;
    const bool serial = (bp.algo == HMM_SERIAL_F32);
    // classes: sets sharing one kernel instantiation
    std::vector<KernelSet> kss(n);
    std::vector<int> kp(n);
    for (int s = 0; s < n; ++s) {
        if (serial) {
            kp[s] = serial_kp(bp.K[s]);
            kss[s].seg1 = serial_kernel(kp[s]);
        } else {
            if (!select_kernels(bp.algo, bp.K[s], &kss[s], bp.packing, true)) return HMM_E_UNSUPPORTED;
            kp[s] = kss[s].KP();
        }
    }
    // packed kernels only for the K whose sets give at least one workgroup
    // per CU at the shortest segments (a few short sequences fill the chip
    // better with one segment per wavefront)
    if (!serial) {
        std::map<const void *, int64_t> jobs_min;   // packed kernel -> jobs at kMinL
        for (int s = 0; s < n; ++s) {
            if (!kss[s].segPB) continue;
            const int64_t W = (int64_t)kss[s].packWaves * kss[s].packG;
            const int64_t nb = (bp.T[s] + kMinL - 1) / kMinL;
            jobs_min[kss[s].segPB] += (nb + W - 1) / W;
        }
        for (int s = 0; s < n; ++s)
            if (kss[s].segPB && jobs_min[kss[s].segPB] < 256) choose_packing(0, bp.K[s], true, &kss[s]);
    }
    for (int s = 0; s < n; ++s) {
        const void *key = class_key(kss[s], serial);
        auto it = std::find_if(bp.classes.begin(), bp.classes.end(),
                               [&](const BatchClass &c) { return c.seg == key; });
        if (it == bp.classes.end()) {
            BatchClass c;
            c.ks = kss[s];
            c.KP = kp[s];
            c.seg = key;
            if (serial) c.serial = kss[s].seg1;
            c.G = (!serial && key == kss[s].segPB) ? kss[s].packG : 1;
            c.W = c.ks.seg_waves();
            c.W2 = group_waves(c.KP);
            bp.classes.push_back(c);
            it = bp.classes.end() - 1;
        }
        it->sets.push_back(s);
    }
    // job tables (host)
    std::vector<WgJob> jobs;
    std::vector<FoldJob> fjobs, pjobs;
    for (size_t ci = 0; ci < bp.classes.size(); ++ci) {
        BatchClass &c = bp.classes[ci];
        if (c.serial) continue;
        c.waves = class_waves(ctx, bp, c, bp.algo);
        c.W = c.waves * c.G;
        c.seg_lds = c.G > 1 ? (size_t)packed_region_bytes(c.ks.packNT, c.G) * c.waves
                            : c.ks.seg_region() * c.waves;
        c.L = class_L(ctx, bp, c, bp.algo, c.W);
        c.job0 = jobs.size();
        c.fjob0 = fjobs.size();
        c.pjob0 = pjobs.size();
        int64_t base = 0;
        for (int s : c.sets) {
            const int64_t nb = bp.T[s] > 0 ? (bp.T[s] + c.L - 1) / c.L : 0;
            const int64_t n1 = (nb + c.W - 1) / c.W;
            for (int64_t q = 0; q < n1; ++q) {
                WgJob j;
                j.seg0 = q * c.W;
                j.out = base + q;
                j.set = s;
                j.nseg = (int)std::min<int64_t>(c.W, nb - q * c.W);
                jobs.push_back(j);
            }
            FoldJob f;
            f.in0 = base;
            f.n_in = n1;
            f.out = 0;
            f.set = s;
            f.F = (int)std::max<int64_t>(1, (n1 + c.W2 - 1) / c.W2);
            f.final_ = 1;
            f.pad = 0;
            base += n1;
            if (f.F > kPrefoldF) {
                // a set with many products: one more fold level first, G = W2
                // products per workgroup, into slots after the segment products
                const int64_t npre = (n1 + c.W2 - 1) / c.W2;
                for (int64_t q = 0; q < npre; ++q) {
                    FoldJob g;
                    g.in0 = f.in0 + q * c.W2;
                    g.n_in = std::min<int64_t>(c.W2, n1 - q * c.W2);
                    g.out = base + q;
                    g.set = s;
                    g.F = 1;
                    g.final_ = 0;
                    g.pad = 0;
                    pjobs.push_back(g);
                }
                f.in0 = base;
                f.n_in = npre;
                f.F = (int)std::max<int64_t>(1, (npre + c.W2 - 1) / c.W2);
                base += npre;
            }
            fjobs.push_back(f);
        }
        c.njobs = jobs.size() - c.job0;
        c.nfjobs = fjobs.size() - c.fjob0;
        c.npjobs = pjobs.size() - c.pjob0;
        // queue order: decreasing work per job (observations of its
        // segments), so the longest jobs start first; slots stay as assigned
        auto job_obs = [&](const WgJob &j) {
            const int64_t T = bp.T[j.set];
            const int64_t a = j.seg0 * c.L, e = std::min<int64_t>(T, (j.seg0 + j.nseg) * c.L);
            return e - a;
        };
        std::stable_sort(jobs.begin() + c.job0, jobs.end(),
                         [&](const WgJob &x, const WgJob &y) { return job_obs(x) > job_obs(y); });
        for (size_t q = c.job0; q < jobs.size(); ++q)
            c.cost += (double)job_obs(jobs[q]) * c.KP * c.KP * c.KP;
        if (!grid_fits((int64_t)c.njobs, 64 * c.waves) || !grid_fits((int64_t)c.npjobs, 64 * c.W2))
            return HMM_E_UNSUPPORTED;
        c.nprod = (size_t)std::max<int64_t>(base, 1);
    }
    // the most expensive classes first (they start first on the branches)
    std::stable_sort(bp.classes.begin(), bp.classes.end(),
                     [](const BatchClass &x, const BatchClass &y) { return x.cost > y.cost; });
    // segment chains: plans and workgroups, the most expensive first
    std::vector<ChainPlan> cps(n);
    if (bp.chain) plan_batch_chains(bp, &cps);
    std::vector<ChainJob> cjobs;
    std::vector<double> ccost(n, 0.0);
    bp.chain_lds = 0;
    for (int s = 0; s < n; ++s) {
        for (int64_t w = 0; w < cps[s].wgs; ++w) cjobs.push_back(ChainJob{w, s, 0});
        if (cps[s].wgs > 0) {
            ccost[s] = chain_step_cost(bp.K[s]) * (double)(cps[s].q + 64);
            bp.chain_lds = std::max(bp.chain_lds, ChainShape{2, 1}.lds(bp.K[s]));
        }
    }
    std::stable_sort(cjobs.begin(), cjobs.end(),
                     [&](const ChainJob &x, const ChainJob &y) { return ccost[x.set] > ccost[y.set]; });
    bp.ncjobs = cjobs.size();
    if (!grid_fits((int64_t)bp.ncjobs, ChainShape{2, 1}.threads())) return HMM_E_UNSUPPORTED;
    // device memory: tables, per-set slots, per-class products
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    // the tables, copied from the host in one piece
    const size_t o_sets = take(sizeof(SetDesc) * n), o_prep = take(sizeof(PrepJob) * n);
    bp.o_prep = o_prep;
    bp.pointer_bytes = off;
    const size_t o_jobs = take(sizeof(WgJob) * std::max<size_t>(jobs.size(), 1));
    const size_t o_fjobs = take(sizeof(FoldJob) * std::max<size_t>(fjobs.size(), 1));
    const size_t o_pjobs = take(sizeof(FoldJob) * std::max<size_t>(pjobs.size(), 1));
    const size_t o_cjobs = take(sizeof(ChainJob) * std::max<size_t>(cjobs.size(), 1));
    const size_t o_ids = take(sizeof(int) * n);
    const size_t o_cls = take(sizeof(int) * n);
    bp.table_bytes = off;
    // what the kernels write
    const size_t o_status = take(sizeof(int) * n);
    const size_t o_queues = take(2 * sizeof(int) * std::max<size_t>(bp.classes.size(), 1));
    std::vector<size_t> o_chain(n), o_vs(n), o_ve(n), o_part(n);
    for (int s = 0; s < n; ++s) {
        if (cps[s].nb == 0) continue;
        o_chain[s] = take(sizeof(int) * kChainWords);
        o_vs[s] = take(sizeof(float) * kp[s] * cps[s].waves);
        o_ve[s] = take(sizeof(float) * kp[s] * cps[s].waves);
        o_part[s] = take(sizeof(double) * cps[s].waves);
    }
    std::vector<size_t> o_sc(n), o_gf(n);
    for (int s = 0; s < n; ++s) {
        const int KP = kp[s];
        o_sc[s] = take(sizeof(StateConst) * KP);
        o_gf[s] = take(sizeof(float) * KP * KP);
    }
    std::vector<size_t> o_m(bp.classes.size()), o_e(bp.classes.size()), o_s(bp.classes.size());
    for (size_t ci = 0; ci < bp.classes.size(); ++ci) {
        const int KP = bp.classes[ci].KP;
        if (bp.classes[ci].serial) continue;
        const size_t np = bp.classes[ci].nprod;
        o_m[ci] = take(sizeof(float) * KP * KP * np);
        o_e[ci] = take(sizeof(long long) * KP * np);
        o_s[ci] = take(sizeof(long long) * np);
    }
    // (the tables so far were made while the old plan may still be running)
    int rc = retire(ctx, bp);
    if (rc == HMM_OK) rc = allocate(bp, off);
    if (rc != HMM_OK) return rc;
    char *base = static_cast<char *>(bp.mem);
    bp.sets = reinterpret_cast<SetDesc *>(base + o_sets);
    bp.prep = reinterpret_cast<PrepJob *>(base + o_prep);
    bp.jobs = reinterpret_cast<WgJob *>(base + o_jobs);
    bp.fjobs = reinterpret_cast<FoldJob *>(base + o_fjobs);
    bp.pjobs = reinterpret_cast<FoldJob *>(base + o_pjobs);
    int *status = reinterpret_cast<int *>(base + o_status);
    bp.queues = reinterpret_cast<int *>(base + o_queues);
    bp.cjobs = reinterpret_cast<ChainJob *>(base + o_cjobs);
    bp.cls = reinterpret_cast<int *>(base + o_cls);
    int n_cu = 0;
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess ||
        n_cu < 1) {
        (void)hipGetLastError();
        n_cu = 256;
    }
    std::vector<int> ids;
    for (size_t ci = 0; ci < bp.classes.size(); ++ci) {
        BatchClass &c = bp.classes[ci];
        c.queue = bp.queues + 2 * ci;
        if (c.serial) {
            c.ids = reinterpret_cast<int *>(base + o_ids) + ids.size();
            ids.insert(ids.end(), c.sets.begin(), c.sets.end());
            continue;
        }
        c.M = reinterpret_cast<float *>(base + o_m[ci]);
        c.E = reinterpret_cast<long long *>(base + o_e[ci]);
        c.S = reinterpret_cast<long long *>(base + o_s[ci]);
    }
    const int64_t total = std::accumulate(bp.T.begin(), bp.T.end(), int64_t(0));
    std::vector<SetDesc> hs(n);
    std::vector<PrepJob> hp(n);
    std::vector<int> hc(n);
    for (int s = 0; s < n; ++s) {
        const BatchClass *c = nullptr;
        const void *key = class_key(kss[s], serial);
        for (const auto &cc : bp.classes)
            if (cc.seg == key) c = &cc;
        hc[s] = (int)(c - bp.classes.data());
        SetDesc &d = hs[s];
        d.obs = Obs{bp.flag + bp.obs_off[s], bp.xy + 2 * bp.obs_off[s], nullptr, kEmisTremor, 0};
        d.sc = reinterpret_cast<const StateConst *>(base + o_sc[s]);
        d.GF = reinterpret_cast<const float *>(base + o_gf[s]);
        d.delta = bp.params + bp.param_off[s];
        d.status = status + s;
        d.out = bp.out + s;
        d.T = bp.T[s];
        d.L = c->serial ? 0 : c->L;
        d.K = bp.K[s];
        PrepJob &pj = hp[s];
        pj.params = bp.params + bp.param_off[s];
        pj.sc = reinterpret_cast<StateConst *>(base + o_sc[s]);
        pj.GF = reinterpret_cast<float *>(base + o_gf[s]);
        pj.status = status + s;
        pj.chain = nullptr;
        if (cps[s].nb > 0) {
            Layout ly;
            ly.chain = o_chain[s];
            ly.vs = o_vs[s];
            ly.ve = o_ve[s];
            ly.part = o_part[s];
            set_chain(&d, base, ly, cps[s], total);
            pj.chain = d.fail;
        }
        pj.max_stay = chain_max_stay(cps[s].q);
        pj.pad = 0;
        pj.K = bp.K[s];
        pj.KP = kp[s];
    }
    auto put = [&](size_t o, const void *src, size_t bytes) {
        if (bytes > 0) std::memcpy(bp.host + o, src, bytes);
    };
    put(o_sets, hs.data(), sizeof(SetDesc) * n);
    put(o_prep, hp.data(), sizeof(PrepJob) * n);
    put(o_jobs, jobs.data(), sizeof(WgJob) * jobs.size());
    put(o_fjobs, fjobs.data(), sizeof(FoldJob) * fjobs.size());
    put(o_pjobs, pjobs.data(), sizeof(FoldJob) * pjobs.size());
    put(o_cjobs, cjobs.data(), sizeof(ChainJob) * cjobs.size());
    put(o_ids, ids.data(), sizeof(int) * ids.size());
    put(o_cls, hc.data(), sizeof(int) * n);
    rc = upload(bp, bp.table_bytes, st);
    if (rc != HMM_OK) return rc;
    if (bp.ncjobs > 0 && allow_lds(chain_kernel_batch(), bp.chain_lds) != HMM_OK) return HMM_E_DEVICE;
    for (auto &c : bp.classes) {
        if (c.serial) continue;
        const size_t rb = (size_t)region_bytes(c.ks.KP());
        if (allow_lds(c.seg, c.seg_lds) != HMM_OK || allow_lds(c.ks.foldB, rb * c.W2) != HMM_OK)
            return HMM_E_DEVICE;
        // persistent launch: as many workgroups as are resident at once
        c.grid = 0;
        if (bp.persistent) {
            const int per_cu = resident_groups(c.seg, 64 * c.waves, c.seg_lds);
            c.grid = (int)std::min<int64_t>((int64_t)c.njobs, (int64_t)per_cu * n_cu);
        }
    }
    return HMM_OK;
}

int enqueue_class(const BatchPlan &bp, const BatchClass &c, hipStream_t st)
{
    if (c.serial) {
        void *args[] = {(void *)&bp.sets, (void *)&c.ids};
        return hipLaunchKernel(c.serial, dim3((unsigned)c.sets.size()), dim3(64), args, 0, st) == hipSuccess
                   ? HMM_OK
                   : HMM_E_DEVICE;
    }
    SetDesc none{};
    const size_t rb = (size_t)region_bytes(c.ks.KP());
    if (c.njobs > 0 &&
        launch_seg(c.seg, (unsigned)(c.grid > 0 ? c.grid : (int64_t)c.njobs), c.waves, c.seg_lds, st, none, bp.sets,
                   bp.jobs + c.job0, (int64_t)c.njobs, c.M, c.E, c.S, c.grid > 0 ? c.queue : nullptr) != hipSuccess)
        return HMM_E_DEVICE;
    if (c.npjobs > 0 &&
        launch_fold(c.ks.foldB, (unsigned)c.npjobs, c.W2, rb * c.W2, st, none, bp.sets, bp.pjobs + c.pjob0, 0, 1, 0,
                    c.M, c.E, c.S, c.M, c.E, c.S) != hipSuccess)
        return HMM_E_DEVICE;
    if (launch_fold(c.ks.foldB, (unsigned)c.nfjobs, c.W2, rb * c.W2, st, none, bp.sets, bp.fjobs + c.fjob0, 0, 1,
                    1, c.M, c.E, c.S, nullptr, nullptr, nullptr) != hipSuccess)
        return HMM_E_DEVICE;
    return HMM_OK;
}

// The launch sequence of a plan: preparation, then every class.  With
// branches, class i runs on aux[i % kBranches] after the preparation and
// the main stream waits for all of them (parallel graph branches when
// captured), so that one class's tail overlaps the next class.
int enqueue(const BatchPlan &bp, hipStream_t st, const BatchClass *only = nullptr, bool branches = false)
{
    if (!only) hipLaunchKernelGGL(k_prepare_batch, dim3(bp.n), dim3(256), 0, st, bp.prep);
    // job counters of the persistent launches start at zero on every run; the
    // classes' second words at zero with segment chains (raised after them),
    // at one without
    if (!bp.classes.empty() && bp.queues)
        hipLaunchKernelGGL(k_init_words, dim3((unsigned)((bp.classes.size() + 255) / 256)), dim3(256), 0, st,
                           bp.queues, (int)bp.classes.size(), bp.ncjobs > 0 && !only ? 0 : 1);
    if (bp.ncjobs > 0 && !only) {
        for (int mode = 0; mode < 2; ++mode) {
            void *args[] = {(void *)&bp.sets, (void *)&bp.cjobs, &mode};
            if (hipLaunchKernel(chain_kernel_batch(), dim3((unsigned)bp.ncjobs), dim3(ChainShape{2, 1}.threads()), args,
                                bp.chain_lds, st) != hipSuccess)
                return HMM_E_DEVICE;
        }
        if (launch_chain_finish(bp.n, st, bp.sets, bp.cls, bp.queues) != hipSuccess) return HMM_E_DEVICE;
    }
    if (!branches) {
        for (const auto &c : bp.classes) {
            if (only && &c != only) continue;
            const int rc = enqueue_class(bp, c, st);
            if (rc != HMM_OK) return rc;
        }
        return HMM_OK;
    }
    if (hipEventRecord(bp.fork, st) != hipSuccess) return HMM_E_DEVICE;
    bool used[BatchPlan::kBranches] = {};
    for (size_t i = 0; i < bp.classes.size(); ++i) {
        const int b = (int)(i % BatchPlan::kBranches);
        if (!used[b] && hipStreamWaitEvent(bp.aux[b], bp.fork, 0) != hipSuccess) return HMM_E_DEVICE;
        used[b] = true;
        const int rc = enqueue_class(bp, bp.classes[i], bp.aux[b]);
        if (rc != HMM_OK) return rc;
    }
    for (int b = 0; b < BatchPlan::kBranches; ++b) {
        if (!used[b]) continue;
        if (hipEventRecord(bp.join[b], bp.aux[b]) != hipSuccess) return HMM_E_DEVICE;
        if (hipStreamWaitEvent(st, bp.join[b], 0) != hipSuccess) return HMM_E_DEVICE;
    }
    return HMM_OK;
}

// Streams and events of the branches, and the capture stream.
int make_branches(BatchPlan &bp)
{
    if (bp.fork) return HMM_OK;   // an earlier capture of this plan failed
    if (hipStreamCreateWithFlags(&bp.cap, hipStreamNonBlocking) != hipSuccess) return HMM_E_DEVICE;
    for (int b = 0; b < BatchPlan::kBranches; ++b) {
        if (hipStreamCreateWithFlags(&bp.aux[b], hipStreamNonBlocking) != hipSuccess) return HMM_E_DEVICE;
        if (hipEventCreateWithFlags(&bp.join[b], hipEventDisableTiming) != hipSuccess) return HMM_E_DEVICE;
    }
    if (hipEventCreateWithFlags(&bp.fork, hipEventDisableTiming) != hipSuccess) return HMM_E_DEVICE;
    return HMM_OK;
}

int capture(BatchPlan &bp)
{
    if (make_branches(bp) != HMM_OK) return HMM_E_DEVICE;
    if (hipStreamBeginCapture(bp.cap, hipStreamCaptureModeThreadLocal) != hipSuccess) return HMM_E_DEVICE;
    int rc = enqueue(bp, bp.cap, nullptr, bp.classes.size() > 1);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(bp.cap, &g);
    if (rc != HMM_OK || e != hipSuccess || !g) {
        if (g) (void)hipGraphDestroy(g);
        (void)hipGetLastError();
        return HMM_E_DEVICE;
    }
    bp.graph = g;
    if (hipGraphInstantiate(&bp.exec, bp.graph, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGetLastError();
        bp.exec = nullptr;
        return HMM_E_DEVICE;
    }
    return HMM_OK;
}

// The plan was built for these descriptors and options (any buffers).
bool same_plan(const BatchPlan &bp, const hmm_ctx *ctx, int n, const int32_t *K, const int64_t *T,
               const int64_t *param_off, const int64_t *obs_off, int algo)
{
    if (bp.n != n || bp.algo != algo) return false;
    if (bp.tuned != ctx->tuned_L || bp.tunedW != ctx->tuned_W || bp.persistent != ctx->batch_persistent ||
        bp.packing != ctx->packing || bp.chain != (algo == HMM_BLOCKED_F32 && ctx->default_plan()))
        return false;
    return std::equal(K, K + n, bp.K.begin()) && std::equal(T, T + n, bp.T.begin()) &&
           std::equal(param_off, param_off + n, bp.param_off.begin()) &&
           std::equal(obs_off, obs_off + n, bp.obs_off.begin());
}

bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &c) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return c != hipStreamCaptureStatusNone;
}

// The context's plan for these descriptors and buffers, its tables in place for
// what is enqueued on st next.  A stream that is being captured can use a plan
// that is there, but not change one.
int get_plan(hmm_ctx *ctx, int n, const int32_t *K, const int64_t *T, const int64_t *param_off,
             const double *params, const int64_t *obs_off, const uint8_t *flag, const double *xy, int algo,
             double *out, hipStream_t st, BatchPlan **res)
{
    BatchPlan *old = ctx->batch;
    if (old && same_plan(*old, ctx, n, K, T, param_off, obs_off, algo)) {
        *res = old;
        if (old->params == params && old->flag == flag && old->xy == xy && old->out == out) return HMM_OK;
        return capturing(st) ? HMM_E_DEVICE : set_pointers(*old, params, flag, xy, out, st);
    }
    if (capturing(st)) return HMM_E_DEVICE;
    BatchPlan *bp = new (std::nothrow) BatchPlan;
    if (!bp) return HMM_E_NOMEM;
    bp->n = n;
    bp->algo = algo;
    bp->K.assign(K, K + n);
    bp->T.assign(T, T + n);
    bp->param_off.assign(param_off, param_off + n);
    bp->obs_off.assign(obs_off, obs_off + n);
    bp->params = params;
    bp->flag = flag;
    bp->xy = xy;
    bp->out = out;
    bp->tuned = ctx->tuned_L;
    bp->tunedW = ctx->tuned_W;
    bp->persistent = ctx->batch_persistent;
    bp->packing = ctx->packing;
    bp->chain = algo == HMM_BLOCKED_F32 && ctx->default_plan();
    const int rc = build(ctx, *bp, st);
    if (rc != HMM_OK) {
        (void)hipDeviceSynchronize();   // a copy of the tables may be on its way
        batch_plan_free(bp);
        return rc;
    }
    ctx->batch = bp;
    *res = bp;
    return HMM_OK;
}

int check_batch(hmm_ctx *ctx, int32_t n, const int32_t *K, const int64_t *T, const int64_t *param_off,
                const double *params, int64_t params_len, const int64_t *obs_off, const uint8_t *flag,
                const double *xy, int64_t obs_len, int32_t algo, double *out)
{
    if (!ctx || n < 1 || !K || !T || !param_off || !params || !obs_off || !out) return HMM_E_INVALID_ARG;
    if (algo != HMM_SERIAL_F32 && algo != HMM_BLOCKED_F32 && algo != HMM_BLOCKED_BF16 && algo != HMM_BLOCKED_F16)
        return HMM_E_INVALID_ARG;
    const int kmax = (algo == HMM_SERIAL_F32) ? 128 : 80;
    bool any_obs = false;
    for (int s = 0; s < n; ++s) {
        if (K[s] < 1 || K[s] > kmax || T[s] < 0 || T[s] >= kMaxT || param_off[s] < 0 || obs_off[s] < 0)
            return HMM_E_INVALID_ARG;
        const int64_t blk = (int64_t)K[s] * (K[s] + 7);  // delta, Gamma, p, mu, Sigma
        if (param_off[s] > params_len - blk || obs_off[s] > obs_len - T[s]) return HMM_E_INVALID_ARG;
        any_obs |= T[s] > 0;
    }
    if (any_obs && (!flag || !xy)) return HMM_E_INVALID_ARG;
    if (any_obs && !xy_aligned(xy)) return HMM_E_INVALID_ARG;
    return HMM_OK;
}

int run_batch(hmm_ctx *ctx, int n, const int32_t *K, const int64_t *T, const int64_t *param_off,
              const double *params, const int64_t *obs_off, const uint8_t *flag, const double *xy, int algo,
              double *out, hipStream_t st)
{
    BatchPlan *bp = nullptr;
    int rc = get_plan(ctx, n, K, T, param_off, params, obs_off, flag, xy, algo, out, st, &bp);
    if (rc != HMM_OK) return rc;
    const bool user_capture = capturing(st);
    if (ctx->batch_graph && bp->launched && !bp->exec && !user_capture) {
        rc = capture(*bp);
        if (rc != HMM_OK) return rc;
    }
    if (bp->exec && !user_capture) return hipGraphLaunch(bp->exec, st) == hipSuccess ? HMM_OK : HMM_E_DEVICE;
    rc = enqueue(*bp, st);
    if (rc != HMM_OK) return rc;
    bp->launched = true;
    return hipGetLastError() == hipSuccess ? HMM_OK : HMM_E_DEVICE;
}

}  // namespace

}  // namespace hmmh

using namespace hmmh;

extern "C" {

int hmm_loglik_batched(hmm_ctx *ctx, int32_t n, const int32_t *K, const int64_t *T, const int64_t *param_off,
                       const double *params, int64_t params_len, const int64_t *obs_off, const uint8_t *flag,
                       const double *xy, int64_t obs_len, int32_t algo, void *stream, double *out)
{
    int rc = check_batch(ctx, n, K, T, param_off, params, params_len, obs_off, flag, xy, obs_len, algo, out);
    if (rc != HMM_OK) return rc;
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return HMM_E_DEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = run_batch(ctx, n, K, T, param_off, params, obs_off, flag, xy, algo, out, st);
    if (rc != HMM_OK) (void)hipGetLastError();   // reported here, not by the next call
    return rc;
}

int hmm_ctx_set_batch_graph(hmm_ctx *ctx, int32_t on)
{
    if (!ctx) return HMM_E_INVALID_ARG;
    ctx->batch_graph = on != 0;
    if (ctx->batch) {
        DeviceGuard dg(ctx->device);
        if (hipDeviceSynchronize() != hipSuccess) return HMM_E_DEVICE;
        batch_plan_free(ctx->batch);
        ctx->batch = nullptr;
    }
    return HMM_OK;
}

int hmm_ctx_set_batch_persistent(hmm_ctx *ctx, int32_t on)
{
    if (!ctx) return HMM_E_INVALID_ARG;
    ctx->batch_persistent = on != 0;
    if (ctx->batch) {
        DeviceGuard dg(ctx->device);
        if (hipDeviceSynchronize() != hipSuccess) return HMM_E_DEVICE;
        batch_plan_free(ctx->batch);
        ctx->batch = nullptr;
    }
    return HMM_OK;
}

int hmm_ctx_set_packing(hmm_ctx *ctx, int32_t mode)
{
    if (!ctx) return HMM_E_INVALID_ARG;
    if (mode != 0 && mode != 1 && mode != 2 && mode != 4 && mode != 5) return HMM_E_INVALID_ARG;
    ctx->packing = mode;
    if (ctx->batch) {
        DeviceGuard dg(ctx->device);
        if (hipDeviceSynchronize() != hipSuccess) return HMM_E_DEVICE;
        batch_plan_free(ctx->batch);
        ctx->batch = nullptr;
    }
    return HMM_OK;
}

int hmm_autotune_batched(hmm_ctx *ctx, int32_t n, const int32_t *K, const int64_t *T, const int64_t *param_off,
                         const double *params, int64_t params_len, const int64_t *obs_off, const uint8_t *flag,
                         const double *xy, int64_t obs_len, int32_t algo, double *out, int32_t reps,
                         int64_t *chosen_L)
{
    int rc = check_batch(ctx, n, K, T, param_off, params, params_len, obs_off, flag, xy, obs_len, algo, out);
    if (rc != HMM_OK) return rc;
    if (algo == HMM_SERIAL_F32) return HMM_E_UNSUPPORTED;
    if (reps < 1) reps = 3;
    DeviceGuard dg(ctx->device);
    if (!dg.ok) return HMM_E_DEVICE;
    // candidates: segment length x segment-kernel waves per workgroup (the
    // kernel's maximum, half of it); W = 0 stands for the maximum
    const int64_t candL[] = {256, 512, 1024, 2048, 4096};
    const int candW[] = {0, 2};   // 0: maximum; 2: half the maximum (divisor)
    // distinct K values of the batch, tuned one class at a time
    std::vector<int> ks(K, K + n);
    std::sort(ks.begin(), ks.end());
    ks.erase(std::unique(ks.begin(), ks.end()), ks.end());
    // the candidates run on a stream of their own
    if (hipDeviceSynchronize() != hipSuccess) return HMM_E_DEVICE;
    hipStream_t st = nullptr;
    if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) return HMM_E_DEVICE;
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    const bool graph_was = ctx->batch_graph;
    ctx->batch_graph = false;
    ctx->no_chain = true;   // the candidates are the product path's
    for (int k : ks) {
        ctx->tuned_L.erase({k, algo});
        ctx->tuned_W.erase({k, algo});
    }
    // classes are independent: time each class's launches under each candidate
    struct Best {
        double ms;
        int64_t L;
        int W;
    };
    std::map<const void *, Best> best;  // class segment kernel -> fastest (ms, L, waves)
    std::map<int, const void *> kseg;   // K -> its class's segment kernel
    for (int wdiv : candW) {
        for (int64_t L : candL) {
            for (int k : ks) {
                ctx->tuned_L[{k, algo}] = L;
                ctx->tuned_W[{k, algo}] = wdiv ? -wdiv : 0;
            }
            BatchPlan *bp = nullptr;
            rc = get_plan(ctx, n, K, T, param_off, params, obs_off, flag, xy, algo, out, st, &bp);
            if (rc != HMM_OK) break;
            hipLaunchKernelGGL(k_prepare_batch, dim3(bp->n), dim3(256), 0, st, bp->prep);
            for (const auto &c : bp->classes) {
                if (c.serial) continue;
                float tot = 0.f;
                for (int r = 0; r <= reps; ++r) {
                    (void)hipEventRecord(e0, st);
                    rc = enqueue(*bp, st, &c);
                    (void)hipEventRecord(e1, st);
                    if (rc != HMM_OK) break;
                    (void)hipEventSynchronize(e1);
                    float ms = 0.f;
                    (void)hipEventElapsedTime(&ms, e0, e1);
                    if (r > 0) tot += ms;  // first run warms up
                }
                const double avg = tot / reps;
                auto it = best.find(c.seg);
                if (it == best.end() || avg < it->second.ms) best[c.seg] = Best{avg, L, c.waves};
                for (int s : c.sets) kseg[bp->K[s]] = c.seg;
            }
            if (rc != HMM_OK) break;
        }
        if (rc != HMM_OK) break;
    }
    // record the winner for every K of each class
    if (rc == HMM_OK) {
        for (int k : ks) {
            auto ks_it = kseg.find(k);
            auto it = ks_it != kseg.end() ? best.find(ks_it->second) : best.end();
            ctx->tuned_L[{k, algo}] = (it != best.end()) ? it->second.L : 0;
            ctx->tuned_W[{k, algo}] = (it != best.end()) ? it->second.W : 0;
        }
        if (chosen_L)
            for (int s = 0; s < n; ++s) chosen_L[s] = ctx->tuned_L[{K[s], algo}];
    }
    ctx->batch_graph = graph_was;
    ctx->no_chain = false;
    (void)hipStreamSynchronize(st);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    (void)hipStreamDestroy(st);
    if (ctx->batch) {
        batch_plan_free(ctx->batch);
        ctx->batch = nullptr;
    }
    return rc;
}

}  // extern "C"
