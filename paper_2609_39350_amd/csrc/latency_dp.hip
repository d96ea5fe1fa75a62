// Least 1F1B iteration latency over every partition (Appendix B, Eq. 5, with
// the steady-state term of Eq. 4): for each candidate the partition, with the
// Section 3.4 prunings and per-stage recomputation, that minimises
//     T = sum_i c_i + sum_{i <= s} ceil(c_i / 3) + max(0, B - s - 1) * t,
// t = max_i c_i and s the first (1-based) stage whose cost is t (a stage's
// forward part is ceil(c / 3), its backward part the rest).  Ties: the least T,
// then the lower t, then the lexicographically smallest (b_{PP-1}, ..., b_1).
//
// Branch and bound over ranges of t.  For a range [lo, hi] one DP pass over
// (stage, end layer, z), z = 1 once the bottleneck stage is placed, relaxes
// "the bottleneck is the first largest stage" to "every stage costs at most hi
// and the bottleneck at least lo": before the bottleneck a stage weighs
// c + ceil(c / 3), the bottleneck c_s + ceil(c_s / 3) + max(0, B - s - 1) c_s,
// after it c.  The pass keeps the least (V, c_s) and, along that path, its
// largest stage m.  V is a lower bound of T for every t in the range.  If the
// path's bottleneck is its first largest stage, V is that partition's own
// latency, hence the least over the range (and c_s the least t reaching it);
// otherwise the range splits between c_s and m, which excludes the path from
// both halves.  A range is dropped once (V, lo) is not below an incumbent
// (T, t).  A single threshold (lo = hi) runs with c < t before the bottleneck
// and is exact.  The first ranges grow geometrically from t_bot, the least
// possible largest stage (one min-max pass).  Sweeping every distinct stage
// cost instead, as the definition does, took 190 passes a feasible 16- or
// 32-stage candidate of the 96-layer workload; the ranges take 10 to 20, in two
// to four rounds (a call at 96 layers, B = 32 and 64: 64.4 -> 2.8 ms; at 61 layers,
// B = 16, 32 and 64: 4.24 -> 0.84 ms).  The partition itself comes from one exact pass at
// the winning t: its back-trace keeps the set of (end layer, z) states on
// optimal paths and takes, stage by stage from the last, the smallest split
// point through which one continues optimally.
//
// Candidates of a key with B >= PP + 1 share a search: no steady-state count is
// clamped and every stage stores PP - s + 1 micro-batches, so the latency of a
// partition differs between two such B by (B - B') t.  A pass at B bounds a
// member B' by V + (B' - B) lo (B' >= B) or V - (B - B') hi, its valid path is
// an incumbent of every member, and a range stays open while any member may
// still gain there (evaluated next at the open member farthest from the last B).
//
// Mapping: one workgroup of two waves per (configuration, ordering) key,
// deepest first; the dispatcher hands the next key to whichever CU slot frees
// first.  The stage costs -- every (stage, end layer b in the stage's band,
// split point a in the window) with the memory test of its stored micro-batch
// count, recomputation and prunings 1 and 3, exactly as the threshold DP prices
// them -- are evaluated once a search into LDS, from layer prefix sums staged
// there.  A round runs up to eight ranges side by side: a slot of two DP rows
// each, 16 to 64 lanes a slot over the end layers (the bands of deep pipelines
// are narrow), so a wave's slots need no barrier inside a pass; what bounds a
// pass is its chain of PP dependent stage steps (61 layers: 13 waves a CU, VALU
// instructions in 61 % of the issue slots, 55 % of the wave cycles waiting).  Wave
// 0 keeps the list of open ranges, one a lane, and lane j holds the incumbent of
// the key's j-th candidate.  Integer min-plus work: no MFMA.
#include <algorithm>

#include "internal.h"

namespace hapmoe {
namespace {

constexpr int64_t kLBig = int64_t(1) << 62;   // "no path" inside the DP, far from overflow
constexpr int kLatWaves = 2;
constexpr int kLatThreads = 64 * kLatWaves;
constexpr int kLatSlots = 8;    // ranges a round may run side by side
constexpr int kLatNodes = 24;   // open ranges a search keeps; with more than kLatNodes - 2 slots of
                                // them one range is swept threshold by threshold instead of splitting
// Launches in tiers of LDS a workgroup: every key with the size that the host
// expects the deepest pipelines to take (at least 20 KB: at 128 VGPRs no more
// than the eight workgroups of that size run on a CU), then the keys that did
// not fit with 40, 80 and 160 KB.  One size that holds them all matters: with
// the 32-stage keys of the 96-layer workload left to a second launch, both
// launches end with a tail (5.8 against 2.8 ms).
constexpr int kLatTiers = 4;
constexpr int kLatLdsTiers[kLatTiers] = {20 * 1024, 40 * 1024, 80 * 1024, 160 * 1024};
constexpr int64_t kLatMaxGrid = int64_t(1) << 30;   // workgroups a launch (keys beyond: grid-stride)
constexpr int kLatTableLimit = 162048;   // documented: 9 bytes a stage cost, 16 bytes a DP state
constexpr int32_t kStatusRetry = 3;      // between the launches only: the key needs more LDS

struct LatHead {
    uint64_t cmax;       // largest finite stage cost (as a weight)
    uint64_t ctop;       // upper bound of every stage cost of the key
    int64_t tbot;        // least possible largest stage (as a weight)
    int32_t nt, relax;   // ranges of this round (0: done); statistics
    int64_t slo[kLatSlots], shi[kLatSlots];               // the round's ranges (weights)
    int64_t rV[kLatSlots], rT[kLatSlots], rM[kLatSlots];   // their results
    int32_t sB[kLatSlots];
    int64_t nlo[kLatNodes], nhi[kLatNodes], nV[kLatNodes];   // open ranges: bounds, V of the pass they came from
    int32_t nB[kLatNodes], nE[kLatNodes];                    // that pass's B, the B to evaluate at next
};
constexpr int kLatHeadBytes = ((int)sizeof(LatHead) + 15) & ~15;
// the largest documented table and its working space always fit the last tier:
// 8 n + 2 nv for costs and split ranges, then the larger of the staged prefix
// sums (at most 16 * 128 * 7 + 28 * 128), 16 nv of final states and one slot's
// rows (80 * 127), under 9 n + 16 nv <= 162,048 and n <= 127 nv <= 127 * 4,064
static_assert(kLatHeadBytes <= 3200, "working space beside the largest table");

__device__ inline int64_t ceil3(int64_t c) { return (c + 2) / 3; }

// The cost table holds each stage cost c as w = c + ceil(c / 3), the weight of a
// stage before the bottleneck (kLBig: no such stage).  w is strictly increasing
// in c, so ranges, largest stages and thresholds are kept as weights, and c
// comes back without a division: c = 3m, 3m + 1, 3m + 2 give w = 4m, 4m + 2,
// 4m + 3, so c = 3 (w >> 2) + ((w & 3) + 1) / 2 (for a w between two weights
// the larger c).  Stage costs stay below 2^60, so 2 w + 1 stays below 2^63.
__device__ inline int64_t cost_weight(int64_t c) { return c >= kLBig ? kLBig : c + ceil3(c); }
__device__ inline int64_t weight_cost(int64_t w) { return 3 * (w >> 2) + (((w & 3) + 1) >> 1); }

__device__ inline int lat_rl(int v, int src) { return __builtin_amdgcn_readlane(v, src); }

__device__ inline int64_t lat_rl64(int64_t v, int src)
{
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, src);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), src);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ inline int64_t lat_shfl64(int64_t v, int src)
{
    const int lo = __shfl((int)(uint32_t)(uint64_t)v, src, 64);
    const int hi = __shfl((int)(uint32_t)((uint64_t)v >> 32), src, 64);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ inline int lat_scan(int x, int lane)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Wave-wide minimum (every lane active, every lane gets the result): each
// 16-lane row by DPP row rotations, then the four rows from lanes 0, 16, 32, 48.
__device__ inline int64_t lat_min(int64_t v)
{
#define LAT_ROT_MIN(CTRL)                                                                              \
    do {                                                                                               \
        const int lo_ = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(uint64_t)v, CTRL, 0xf, 0xf, false); \
        const int hi_ = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), CTRL, 0xf, 0xf, false); \
        const int64_t o_ = (int64_t)(((uint64_t)(uint32_t)hi_ << 32) | (uint32_t)lo_);                \
        v = o_ < v ? o_ : v;                                                                           \
    } while (0)
    LAT_ROT_MIN(0x128);   // row_ror 8
    LAT_ROT_MIN(0x124);   // row_ror 4
    LAT_ROT_MIN(0x122);   // row_ror 2
    LAT_ROT_MIN(0x121);   // row_ror 1
#undef LAT_ROT_MIN
    int64_t m = kLBig + kLBig / 2;   // above every value
#pragma unroll
    for (int r = 0; r < 64; r += 16) {
        const int64_t o = lat_rl64(v, r);
        m = o < m ? o : m;
    }
    return m;
}

__device__ inline int lat_sum32(int v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// LDS operations of a wave are processed in order: a compiler fence is enough
// between the steps of one wave.
__device__ inline void lat_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct LatI2 {
    int64_t x, y;
};

// Type of a cost weight in LDS: 32 bits where every stage cost of the key has a
// weight below 2^31 (costs below 1.6 s: all but the shallowest pipelines of the
// larger models), which halves the table, the slot rows and the instructions on
// weights, else 64.  Sums are 64-bit in both.
template <typename WT> struct LatW;
template <> struct LatW<uint32_t> {
    static constexpr uint32_t none = 0xffffffffu;   // no such stage
    static __device__ inline uint32_t cost(uint32_t w) { return 3 * (w >> 2) + (((w & 3) + 1) >> 1); }
};
template <> struct LatW<int64_t> {
    static constexpr int64_t none = kLBig;
    static __device__ inline int64_t cost(int64_t w) { return weight_cost(w); }
};

__device__ inline void lat_write(hapmoe_dp_result *out, int status, int64_t obj, int64_t sum, int64_t tmax,
                                 uint32_t rmask, const uint32_t (&lw)[kMaxStages / 4])
{
    uint4 *dst = reinterpret_cast<uint4 *>(out);
    dst[0] = uint4{(uint32_t)(uint64_t)obj, (uint32_t)((uint64_t)obj >> 32), (uint32_t)(uint64_t)sum,
                   (uint32_t)((uint64_t)sum >> 32)};
    dst[1] = uint4{(uint32_t)(uint64_t)tmax, (uint32_t)((uint64_t)tmax >> 32), (uint32_t)status, rmask};
    dst[2] = uint4{lw[0], lw[1], lw[2], lw[3]};
    dst[3] = uint4{lw[4], lw[5], lw[6], lw[7]};
}

// lds_bytes: the workgroup's LDS; retry: process only the keys whose candidates
// an earlier launch marked kStatusRetry (the last launch marks none)
template <bool STATS>
__global__ __launch_bounds__(kLatThreads, 4) void k_latency_dp(const unsigned char *__restrict__ img,
                                                            const hapmoe_candidate *__restrict__ cand,
                                                            const unsigned char *__restrict__ tab, TablesLayout L,
                                                            int64_t first, int64_t count, hapmoe_dp_result *res,
                                                            int32_t *stats, int lds_bytes, int retry, int last)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const ImageHeader &H = *reinterpret_cast<const ImageHeader *>(img);
    LatHead &D = *reinterpret_cast<LatHead *>(smem);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = H.n_layers, W = N + 1, nB = H.n_micro;
    const int64_t np = L.np;
    const uint32_t zero_words[kMaxStages / 4] = {};
    // the (configuration, ordering) keys holding candidates [first, first + count)
    const int64_t key_lo = first / nB, n_keys = (first + count - 1) / nB - key_lo + 1;

    auto do_key = [&](int64_t kq) {
        // keys are PP-ascending: the deepest pipelines (the most work) go first
        const int64_t key = key_lo + n_keys - 1 - kq, cfg = key / H.n_orders;
        const int PP = __builtin_amdgcn_readfirstlane(cand[key * nB].pp);
        const PiInfo *pi = reinterpret_cast<const PiInfo *>(tab + L.off_pi) + cfg;
        const KeyInfo *ki = reinterpret_cast<const KeyInfo *>(tab + L.off_key) + key;
        const int64_t *mem = reinterpret_cast<const int64_t *>(tab + L.off_mem) + cfg * 4 * np;
        const int64_t *time = reinterpret_cast<const int64_t *>(tab + L.off_time) + cfg * L.n_masks * 3 * np;
        // stage s in lane s of every wave (the arrays hold kMaxStages entries)
        int mask = 0, lo = 0, hi = 0, bp = 0;
        if (lane < kMaxStages) {
            mask = ki->mask[lane];
            lo = ki->lo[lane];
            hi = ki->hi[lane];
            bp = ki->bpair[lane];
        }
        // lane j holds the key's j-th candidate (B = micro[j])
        const int64_t inst = key * nB + lane;
        const bool inr = lane < nB && inst >= first && inst < first + count;
        const int Bj = lane < nB ? H.micro[lane] : 1;
        hapmoe_dp_result *out = res + (inst - first);   // dereferenced only where inr
        int32_t *st_out = STATS ? stats + 4 * (inst - first) : nullptr;
        auto finish_if = [&](bool mine, int status) {   // a result without a partition
            if (mine && wave == 0) {
                lat_write(out, status, kInf, kInf, kInf, 0, zero_words);
                if (STATS) st_out[0] = st_out[1] = st_out[2] = st_out[3] = 0;
            }
        };
        if (pi->status != HAPMOE_STATUS_OK) {
            finish_if(inr, HAPMOE_STATUS_OVERFLOW);
            return;
        }
        if (lane >= PP) mask = lo = hi = bp = 0;

        // ---- stage layout: bands of end layers under the pruning-1 windows ----
        const int cumlo = lat_scan(lo, lane), cumhi = lat_scan(hi, lane);
        const int totlo = lat_rl(cumlo, 63), tothi = lat_rl(cumhi, 63);
        int blo = N - (tothi - cumhi), bhi = N - (totlo - cumlo);
        blo = blo > cumlo ? blo : cumlo;
        bhi = bhi < cumhi ? bhi : cumhi;
        const int wd = lane < PP && bhi >= blo ? bhi - blo + 1 : 0;
        const int win = lane < PP ? hi - lo + 1 : 0;
        if (totlo > N || tothi < N || __any(lane < PP && wd == 0)) {
            finish_if(inr, HAPMOE_STATUS_INFEASIBLE);
            return;
        }
        const int csum = lat_scan(wd * win, lane), vsum = lat_scan(wd, lane);
        const int ncost = lat_rl(csum, 63), nv = lat_rl(vsum, 63);
        if (ncost * 8 + ((ncost + 15) & ~15) + nv * 16 > kLatTableLimit) {
            finish_if(inr, HAPMOE_STATUS_OVERFLOW);
            return;
        }
        int maxwd = wd;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const int o = __shfl_xor(maxwd, d, 64);
            maxwd = o > maxwd ? o : maxwd;
        }
        maxwd = __builtin_amdgcn_readfirstlane(maxwd);
        // the device-type sets in use, each stage's rank among them
        uint32_t used = 0;
        for (int m = 1; m <= kMaxMasks; ++m) used |= __any(mask == m) ? 1u << m : 0u;
        const int nset = __popc(used), set = __popc(used & ((1u << mask) - 1u));
        // packed stage fields, one readlane each: blo, wd, lo, win (all < 128), and
        // the offsets into the cost table and the (stage, end layer) rows
        const int pk1 = blo | (wd << 8) | (lo << 16) | (win << 24);
        const int pk2 = (csum - wd * win) | ((vsum - wd) << 16);
        const int voff = vsum - wd;
        int64_t cap = kInf;
        for (int h = 0; h < H.n_types; ++h)
            if ((mask >> h) & 1) cap = H.mem_bytes[h] < cap ? H.mem_bytes[h] : cap;
        const bool inner = lane < PP - 1;
        const int64_t p2p = inner ? pi->p2p[(bp >> 2) * kMaxTypes + (bp & 3)] : 0;
        const int bdiff = inner && ((bp >> 2) != (bp & 3)), mixed = __popc((uint32_t)mask) > 1;
        const int pk3 = mask | (set << 8) | (mixed << 16) | (bdiff << 17);
        const int64_t X = pi->x_bytes, eta_tbar = (int64_t)H.eta_prune * pi->tbar;
        const bool prune_het = H.prune_hetero != 0, recomp = H.allow_recompute != 0;

        // ---- layer prefix sums staged at the end of the LDS ----
        const int staged = nset * W * 16 + 3 * W * 8 + W * 4, off_stage = (lds_bytes - staged) & ~15;
        LatI2 *const TM = reinterpret_cast<LatI2 *>(smem + off_stage);
        int64_t *const MW = reinterpret_cast<int64_t *>(smem + off_stage + nset * W * 16), *const MA0 = MW + W,
                       *const MA1 = MA0 + W;
        int32_t *const MOE = reinterpret_cast<int32_t *>(MA1 + W);
        auto stage_sums = [&]() {
            for (int b = threadIdx.x; b < W; b += kLatThreads) {
                MW[b] = mem[b];
                MA0[b] = mem[np + b];
                MA1[b] = mem[2 * np + b];
                MOE[b] = (int32_t)mem[3 * np + b];
            }
            uint32_t rest = used;
            for (int k = 0; k < nset; ++k) {   // uniform
                const int64_t *src = time + (int64_t)(__ffs(rest) - 2) * 3 * np;   // set m at row m - 1
                rest &= rest - 1;
                for (int b = threadIdx.x; b < W; b += kLatThreads) TM[k * W + b] = LatI2{src[b], src[np + b]};
            }
        };
        // row r (a stage and an end layer) with its stage's fields (reads other
        // lanes: call with every lane active)
        struct Row {
            int st, b, plo, phi, atop, wn, ci, mask, set;
            bool act, mixed, bdiff;
            int64_t cap, p2p;
        };
        auto row_of = [&](int r) {
            Row R;
            R.act = r < nv;
            const int rr = R.act ? r : 0;
            int st = 0;
#pragma unroll
            for (int step = 16; step >= 1; step >>= 1) {
                const int c = st + step;
                const int vo = __shfl(voff, c < 64 ? c : 63, 64);
                if (c < PP && vo <= rr) st = c;
            }
            const int q1 = __shfl(pk1, st, 64), q2 = __shfl(pk2, st, 64), q3 = __shfl(pk3, st, 64);
            const int p1 = __shfl(pk1, st > 0 ? st - 1 : 0, 64);
            const int k = rr - (q2 >> 16);
            R.st = st;
            R.cap = lat_shfl64(cap, st);
            R.p2p = lat_shfl64(p2p, st);
            R.plo = st ? p1 & 0xff : 0;
            R.phi = st ? R.plo + ((p1 >> 8) & 0xff) - 1 : 0;
            R.b = (q1 & 0xff) + k;
            R.wn = q1 >> 24;
            R.atop = R.b - ((q1 >> 16) & 0xff);
            R.ci = (q2 & 0xffff) + k * R.wn;
            R.mask = q3 & 0xff;
            R.set = (q3 >> 8) & 0xff;
            R.mixed = (q3 >> 16) & 1;
            R.bdiff = (q3 >> 17) & 1;
            return R;
        };
        auto block_max = [&](uint64_t v, uint64_t &into) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                const uint64_t o = (uint64_t)lat_shfl64((int64_t)v, lane ^ d);
                v = o > v ? o : v;
            }
            if (lane == 0) atomicMax(reinterpret_cast<unsigned long long *>(&into), (unsigned long long)v);
        };
        if (off_stage < kLatHeadBytes) {
            finish_if(inr, kStatusRetry);   // the layout does not depend on B: the whole key
            return;
        }
        __syncthreads();   // the previous key is done with the LDS
        if (threadIdx.x == 0) D.ctop = 0;
        stage_sums();
        __syncthreads();
        {   // an upper bound of every stage cost: the longest segment of each row, recomputed
            uint64_t top = 0;
            for (int r0 = wave * 64; r0 < nv; r0 += kLatThreads) {
                const Row R = row_of(r0 + lane);
                const int a = R.atop - R.wn + 1 > R.plo ? R.atop - R.wn + 1 : R.plo;
                if (R.act && a <= R.b) {
                    const uint64_t c = (uint64_t)(TM[R.set * W + R.b].y - TM[R.set * W + a].y + R.p2p);
                    top = c > top ? c : top;
                }
            }
            block_max(top, D.ctop);
        }
        __syncthreads();
        const bool narrow = (int64_t)D.ctop < 3 * ((int64_t(1) << 31) / 4) - 8;   // uniform

        auto search = [&](auto tag) {
            using WT = decltype(tag);
            constexpr WT kNoW = LatW<WT>::none;
            // LDS after the header: stage costs [ncost] | usable split ranges [nv] u16 | a
            // region holding in turn the staged prefix sums (at its end), the slots' rows
            // and the final states
            const int off_jr = kLatHeadBytes + ((ncost * (int)sizeof(WT) + 15) & ~15),
                      off_reg = off_jr + ((nv * 2 + 15) & ~15);
            const int row_bytes = (2 * (16 + 3 * (int)sizeof(WT)) * maxwd + 15) & ~15;   // a slot: two rows
            // lanes a slot: as many as a band roughly holds, so that a wave runs several slots
            int lps = maxwd <= 24 ? 16 : (maxwd <= 48 ? 32 : 64);
            int nslot = kLatWaves * (64 / lps);
            const int want = last ? 1 : (nslot > 1 ? nslot / 2 : 1);   // fewer: a later launch
            while (nslot > 1 && off_reg + nslot * row_bytes > lds_bytes) {
                nslot >>= 1;
                lps = nslot < kLatWaves ? 64 : 2 * lps;
            }
            if (off_reg > off_stage || off_reg + nv * 16 > lds_bytes || off_reg + nslot * row_bytes > lds_bytes ||
                nslot < want) {
                finish_if(inr, kStatusRetry);
                return;
            }
            WT *const Cst = reinterpret_cast<WT *>(smem + kLatHeadBytes);
            // [first, last + 1) usable split point of a row
            uint16_t *const JR = reinterpret_cast<uint16_t *>(smem + off_jr);
            int64_t *const FS = reinterpret_cast<int64_t *>(smem + off_reg);   // final states
            bool fresh = true;   // the sums staged above are still there
            // Groups of the key's candidates that share one search: all those with
            // B >= PP + 1, then each one with B <= PP alone.
            const uint64_t shared = __ballot(inr && Bj >= PP + 1);
            uint64_t pending = __ballot(inr);
            while (pending) {
                const uint64_t grp = (pending & shared) ? (pending & shared)
                                                        : (uint64_t(1) << (__ffsll((unsigned long long)pending) - 1));
                pending &= ~grp;
                const bool member = (grp >> lane) & 1;
                const int lead = __ffsll((unsigned long long)grp) - 1;
                const int Bgrp = lat_rl(Bj, lead);   // any member: min(PP - s, B) is the same for all
                const bool many = (grp & (grp - 1)) != 0;

                // ---- every stage cost of the group, from the staged prefix sums ----
                if (!fresh) {
                    __syncthreads();   // the previous search is done with the region
                    stage_sums();
                }
                fresh = false;
                if (threadIdx.x == 0) {
                    D.cmax = 0;
                    D.relax = 0;
                }
                __syncthreads();
                {
                    uint64_t wmax = 0;
                    for (int r0 = wave * 64; r0 < nv; r0 += kLatThreads) {
                        const Row R = row_of(r0 + lane);
                        if (!R.act) continue;
                        const LatI2 *T = TM + R.set * W;
                        const int64_t *CM = R.mixed ? time + ((int64_t)(R.mask - 1) * 3 + 2) * np : nullptr;
                        const int64_t hc = (R.bdiff ? R.p2p : 0) + (CM ? CM[R.b] : 0);
                        const int64_t ms = (PP - R.st) < Bgrp ? (PP - R.st) : Bgrp;   // stored micro-batches
                        const LatI2 tb = T[R.b];
                        const int64_t wb = MW[R.b], a0b = MA0[R.b], a1b = MA1[R.b];
                        const int mb = MOE[R.b];
                        // memory, recomputation and pruning 3 only get worse as the split point
                        // falls: the usable split points of a row are one range
                        int j0 = 0, j1 = 0;
                        for (int j = 0; j < R.wn; ++j) {
                            const int a = R.atop - j;
                            int64_t c = kLBig;
                            if (a >= R.plo && a <= R.phi) {
                                const int64_t need = wb - MW[a] + ((mb - MOE[a]) > 0 ? X : 0);
                                const LatI2 ta = T[a];
                                if (!prune_het || hc - (CM ? CM[a] : 0) <= eta_tbar) {
                                    if (need + ms * (a0b - MA0[a]) <= R.cap)
                                        c = tb.x - ta.x + R.p2p;
                                    else if (recomp && need + ms * (a1b - MA1[a]) <= R.cap)
                                        c = tb.y - ta.y + R.p2p;
                                }
                            }
                            const int64_t w = cost_weight(c);
                            Cst[R.ci + j] = w < kLBig ? (WT)w : kNoW;
                            if (w < kLBig) {
                                j0 = j1 ? j0 : j;
                                j1 = j + 1;
                                wmax = (uint64_t)w > wmax ? (uint64_t)w : wmax;
                            }
                        }
                        JR[r0 + lane] = (uint16_t)(j0 | (j1 << 8));
                    }
                    block_max(wmax, D.cmax);
                    __syncthreads();
                }

                // ---- t_bot: the least possible largest stage (wave 0, in weights) ----
                if (wave == 0) {
                    WT *const MR = reinterpret_cast<WT *>(smem + off_reg);   // two rows
                    if (lane == 0) MR[0] = 0;   // layer 0 reached
                    lat_fence();
                    int pblo = 0;
                    for (int s = 0; s < PP; ++s) {
                        const int q1 = lat_rl(pk1, s), q2 = lat_rl(pk2, s);
                        const WT *Pr = MR + (s & 1) * maxwd;
                        WT *Cr = MR + ((s + 1) & 1) * maxwd;
                        for (int k = lane; k < ((q1 >> 8) & 0xff); k += 64) {
                            const int jr = JR[(q2 >> 16) + k], j1 = jr >> 8;
                            const WT *Wp = Cst + (q2 & 0xffff) + k * (q1 >> 24);
                            const int q0 = (q1 & 0xff) + k - ((q1 >> 16) & 0xff) - pblo;
                            WT best = kNoW;
                            for (int j = jr & 0xff; j < j1; ++j) {
                                const WT w = Wp[j], v = Pr[q0 - j];
                                const WT m = v > w ? v : w;
                                best = m < best ? m : best;
                            }
                            Cr[k] = best;
                        }
                        pblo = q1 & 0xff;
                        lat_fence();
                    }
                    if (lane == 0) {
                        const WT t = MR[(PP & 1) * maxwd];   // the last band is {N}
                        D.tbot = t == kNoW ? kLBig : (int64_t)t;
                    }
                }
                __syncthreads();
                const int64_t tbot = D.tbot;
                if (tbot >= kLBig) {   // uniform
                    finish_if(member, HAPMOE_STATUS_INFEASIBLE);
                    continue;
                }

                // this lane's incumbent (wave 0, members only): latency and largest stage (weight)
                int64_t best = kLBig, tbest = kLBig;
                int n_open = 0, swept = 0;
                bool scan = false;        // sweeping the first range threshold by threshold
                int64_t scan_lo = 0;      // ... the last one taken
                int e_cnt = 0, n_rest = 0;   // ranges the round evaluates, open ones it leaves
                int64_t my_lo = 0, my_hi = 0;   // lane i: the i-th slot's range and B
                int my_B = 1;
                if (wave == 0) {
                    // first ranges: [t_bot, t_bot], then up to t_bot (1 + 2^-7), 2^-6, ... 2^-2, and the rest
                    if (lane < 8) {
                        const int64_t top = (int64_t)D.cmax;
                        const int64_t a = lane == 0 ? tbot : tbot + (lane == 1 ? 0 : (tbot >> (9 - lane))) + 1;
                        int64_t z = lane == 0 ? tbot : (lane == 7 ? top : tbot + (tbot >> (8 - lane)));
                        z = z < top ? z : top;
                        D.nlo[lane] = a;
                        D.nhi[lane] = z;
                        D.nV[lane] = a <= z ? 0 : kLBig;   // empty: never below an incumbent
                        D.nB[lane] = Bgrp;
                    }
                    lat_fence();
                    n_open = 8;
                }
                for (;;) {
                    if (wave == 0) {
                        bool run = false;
                        while (!run) {
                            if (scan) {
                                // the next distinct stage costs of range 0, as many as there are slots.
                                // To its end: of 116,000 modelled searches 233 came here, and leaving
                                // when no member can gain any more would have saved two passes in one
                                int nt = 0;
                                const int64_t top = D.nhi[0];
                                for (; nt < nslot; ++nt) {
                                    int64_t wn = kLBig;
                                    for (int e = lane; e < ncost; e += 64) {
                                        const WT c = Cst[e];
                                        const int64_t w = c == kNoW ? kLBig : (int64_t)c;
                                        if (w > scan_lo && w < wn) wn = w;
                                    }
                                    wn = lat_min(wn);
                                    if (wn > top) break;
                                    if (lane == nt) my_lo = my_hi = wn;
                                    scan_lo = wn;
                                }
                                my_B = D.nE[0];
                                if (nt) {
                                    if (lane < nt) {
                                        D.slo[lane] = D.shi[lane] = my_lo;
                                        D.sB[lane] = my_B;
                                    }
                                    if (lane == 0) D.nt = nt;
                                    run = true;
                                } else {   // drop range 0
                                    scan = false;
                                    const int i = lane + 1 < n_open ? lane + 1 : 0;
                                    const int64_t l = D.nlo[i], h = D.nhi[i], v = D.nV[i];
                                    const int bb = D.nB[i];
                                    lat_fence();
                                    if (lane + 1 < n_open) {
                                        D.nlo[lane] = l;
                                        D.nhi[lane] = h;
                                        D.nV[lane] = v;
                                        D.nB[lane] = bb;
                                    }
                                    lat_fence();
                                    --n_open;
                                }
                                continue;
                            }
                            // which open ranges some member may still gain in, and the B to run them at
                            const int i = lane < n_open ? lane : 0;
                            const int64_t l = D.nlo[i], h = D.nhi[i], v = D.nV[i];
                            const int bb = D.nB[i];
                            const int64_t cl = weight_cost(l), ch = weight_cost(h);
                            bool open = false;
                            int be = Bgrp;
                            for (uint64_t g = grp; g; g &= g - 1) {
                                const int j = __ffsll((unsigned long long)g) - 1;
                                const int Bu = lat_rl(Bj, j);
                                const int64_t bu = lat_rl64(best, j), tu = lat_rl64(tbest, j);
                                const int d = Bu - bb;
                                const int64_t lb = v + (int64_t)d * (d >= 0 ? cl : ch);
                                const bool may = v < kLBig && (lb < bu || (lb == bu && l < tu));
                                if (may && (!open || (v > 0 && abs(d) > abs(be - bb)))) be = Bu;
                                open = open || may;
                            }
                            open = open && lane < n_open;
                            const uint64_t om = __ballot(open);
                            n_open = __popcll(om);
                            const int pos = __popcll(om & ((uint64_t(1) << lane) - 1));
                            lat_fence();
                            if (open) {
                                D.nlo[pos] = l;
                                D.nhi[pos] = h;
                                D.nV[pos] = v;
                                D.nB[pos] = bb;
                                D.nE[pos] = be;
                            }
                            lat_fence();
                            if (n_open == 0) {
                                if (lane == 0) D.nt = 0;
                                break;
                            }
                            if (n_open > kLatNodes - 2 * nslot) {   // the list could outgrow its space
                                scan = true;
                                scan_lo = D.nlo[0] - 1;
                                continue;
                            }
                            // one slot a range; with slots to spare every range runs in 2^lg pieces
                            e_cnt = n_open < nslot ? n_open : nslot;
                            n_rest = n_open - e_cnt;
                            int lg = 0;
                            while ((e_cnt << (lg + 1)) <= nslot) ++lg;
                            const int nt = e_cnt << lg;
                            if (lane < nt) {
                                const int k = lane >> lg, piece = lane & ((1 << lg) - 1);
                                const int64_t a = D.nlo[k], z = D.nhi[k];
                                const int64_t step = ((z - a) >> lg) + 1;
                                my_lo = a + piece * step;
                                my_hi = my_lo + step - 1 < z ? my_lo + step - 1 : z;   // below my_lo: empty
                                my_B = D.nE[k];
                                D.slo[lane] = my_lo;
                                D.shi[lane] = my_hi;
                                D.sB[lane] = my_B;
                            }
                            if (lane == 0) D.nt = nt;
                            run = true;
                        }
                    }
                    __syncthreads();
                    const int nt = D.nt;
                    if (nt == 0) break;   // uniform: every range is closed

                    // ---- one pass of every slot: two rows of (V0, V1 | M0, c_s, M1) a slot ----
                    {
                        const int sub = lane / lps, ll = lane - sub * lps;
                        const int slot = nslot < kLatWaves ? wave : wave * (64 / lps) + sub;
                        const bool on = slot < nt;
                        const int sl = on ? slot : 0;
                        const WT wlo = (WT)D.slo[sl], whi = (WT)D.shi[sl];
                        const WT wex = wlo == whi ? whi : kNoW;   // a single threshold: strictly below it
                        const int Bs = D.sB[sl];
                        // each [2 rows][maxwd]
                        int64_t *const V0 = reinterpret_cast<int64_t *>(smem + off_reg + sl * row_bytes);
                        int64_t *const V1 = V0 + 2 * maxwd;
                        WT *const M0 = reinterpret_cast<WT *>(V1 + 2 * maxwd);
                        WT *const T1 = M0 + 2 * maxwd, *const M1 = T1 + 2 * maxwd;
                        if (on && ll == 0) {   // layer 0 reached at cost 0
                            V0[0] = 0;
                            V1[0] = kLBig;
                            M0[0] = T1[0] = M1[0] = 0;
                        }
                        lat_fence();
                        int nrel = 0, pblo = 0;
                        for (int s = 0; s < PP; ++s) {
                            const int q1 = lat_rl(pk1, s), q2 = lat_rl(pk2, s);
                            const int wds = (q1 >> 8) & 0xff, wn = q1 >> 24;
                            const int steady = Bs - s - 2 > 0 ? Bs - s - 2 : 0;   // stage s + 1 (1-based) as bottleneck
                            const int pr = (s & 1) * maxwd, cr = maxwd - pr;
                            for (int k = ll; on && k < wds; k += lps) {
                                const int jr = JR[(q2 >> 16) + k], j1 = jr >> 8;
                                const WT *Wp = Cst + (q2 & 0xffff) + k * wn;
                                const int q0 = pr + (q1 & 0xff) + k - ((q1 >> 16) & 0xff) - pblo;
                                int64_t b0 = kLBig, b1 = kLBig;
                                WT m0 = 0, t1 = 0, m1 = 0;
                                // the stage cost only grows with j: done past hi
                                for (int j = jr & 0xff; j < j1; ++j) {
                                    const WT w = Wp[j];
                                    const int64_t v0 = V0[q0 - j], v1 = V1[q0 - j];
                                    const WT n0 = M0[q0 - j], u1 = T1[q0 - j], n1 = M1[q0 - j];
                                    if (w > whi) break;
                                    if (STATS) nrel += 2;
                                    const WT c = LatW<WT>::cost(w);
                                    const int64_t x0 = v0 + (int64_t)w;   // at least kLBig without a path
                                    const WT mm = n0 > w ? n0 : w;
                                    const bool k0 = w != wex && (x0 < b0 || (x0 == b0 && mm < m0));
                                    b0 = k0 ? x0 : b0;
                                    m0 = k0 ? mm : m0;
                                    // M1 = 2 m, plus 1 if an earlier stage cost as much: the bottleneck is
                                    // the first largest stage iff M1 == 2 c_s at the end
                                    const uint64_t st = (uint64_t)(uint32_t)steady * (uint64_t)c;
                                    const int64_t x1 = (int64_t)((uint64_t)x0 + st);
                                    const bool k1 = w >= wlo && v0 < kLBig && (x1 < b1 || (x1 == b1 && w < t1));
                                    b1 = k1 ? x1 : b1;
                                    t1 = k1 ? w : t1;
                                    m1 = k1 ? 2 * mm + (n0 >= w ? 1 : 0) : m1;
                                    const int64_t y = v1 + (int64_t)c;   // at least kLBig without a path
                                    const bool k2 = y < b1 || (y == b1 && u1 < t1 && v1 < kLBig);
                                    b1 = k2 ? y : b1;
                                    t1 = k2 ? u1 : t1;
                                    m1 = k2 ? (n1 > 2 * w ? n1 : 2 * w) : m1;
                                }
                                V0[cr + k] = b0;
                                V1[cr + k] = b1;
                                M0[cr + k] = m0;
                                T1[cr + k] = t1;
                                M1[cr + k] = m1;
                            }
                            pblo = q1 & 0xff;
                            lat_fence();
                        }
                        if (on && ll == 0) {   // the last band is {N}
                            const int fr = (PP & 1) * maxwd;
                            D.rV[slot] = V1[fr];
                            D.rT[slot] = (int64_t)T1[fr];
                            D.rM[slot] = (int64_t)M1[fr];
                        }
                        if (STATS) {
                            nrel = lat_sum32(nrel);
                            if (lane == 0) atomicAdd(&D.relax, nrel);
                        }
                    }
                    __syncthreads();
                    if (wave == 0) {
                        swept += nt;
                        const int i = lane < nt ? lane : 0;
                        const int64_t V = lane < nt ? D.rV[i] : kLBig, tau = D.rT[i], M = D.rM[i];
                        const bool hit = V < kLBig, valid = hit && M == 2 * tau;
                        for (uint64_t g = __ballot(valid); g; g &= g - 1) {   // partitions: incumbents of every member
                            const int j = __ffsll((unsigned long long)g) - 1;
                            const int64_t tw = lat_rl64(tau, j);
                            const int64_t T = lat_rl64(V, j) + (int64_t)(Bj - lat_rl(my_B, j)) * weight_cost(tw);
                            if (member && (T < best || (T == best && tw < tbest))) {
                                best = T;
                                tbest = tw;
                            }
                        }
                        if (scan) continue;   // single thresholds are exact: nothing to split
                        // the ranges that replace the evaluated ones, then the open ones left over
                        const int64_t m = M >> 1;
                        int64_t l0 = 1, h0 = 0, v0 = V, l1 = 1, h1 = 0, l2 = 1, h2 = 0;   // empty
                        if (valid) {
                            if (many) {   // other members: below c_s (no path there is as good), above it
                                l0 = my_lo;
                                h0 = tau - 1;
                                v0 = V + 1;
                                l1 = tau + 1;
                                h1 = my_hi;
                            }
                        } else if (hit && m > tau) {
                            const int64_t mid = tau + ((m - 1 - tau) >> 1);
                            l0 = my_lo;
                            h0 = mid;
                            l1 = mid + 1;
                            h1 = my_hi;
                        } else if (hit) {   // an earlier stage costs as much: c_s alone is exact
                            l0 = my_lo;
                            h0 = tau - 1;
                            v0 = V + 1;
                            l1 = tau;
                            h1 = tau;
                            l2 = tau + 1;
                            h2 = my_hi;
                        }
                        const bool c0 = lane < nt && l0 <= h0, c1 = lane < nt && l1 <= h1, c2 = lane < nt && l2 <= h2;
                        const uint64_t below = (uint64_t(1) << lane) - 1;
                        const uint64_t g0 = __ballot(c0), g1 = __ballot(c1), g2 = __ballot(c2);
                        int at = __popcll(g0 & below) + __popcll(g1 & below) + __popcll(g2 & below);
                        const int nc = __popcll(g0) + __popcll(g1) + __popcll(g2);
                        const int ri = lane < n_rest ? e_cnt + lane : 0;
                        const int64_t rl = D.nlo[ri], rh = D.nhi[ri], rv = D.nV[ri];
                        const int rb = D.nB[ri];
                        lat_fence();
                        auto push = [&](bool on, int64_t l, int64_t h, int64_t v) {
                            if (!on) return;
                            D.nlo[at] = l;
                            D.nhi[at] = h;
                            D.nV[at] = v;
                            D.nB[at] = my_B;
                            ++at;
                        };
                        push(c0, l0, h0, v0);
                        push(c1, l1, h1, V);
                        push(c2, l2, h2, V);
                        if (lane < n_rest) {
                            D.nlo[nc + lane] = rl;
                            D.nhi[nc + lane] = rh;
                            D.nV[nc + lane] = rv;
                            D.nB[nc + lane] = rb;
                        }
                        lat_fence();
                        n_open = nc + n_rest;
                    }
                }

                // ---- one exact pass and its back-trace for every winning t (wave 0) ----
                if (wave == 0) {
                    uint64_t left = grp;
                    while (left) {
                        const int j = __ffsll((unsigned long long)left) - 1;
                        const int64_t wt = lat_rl64(tbest, j), t = weight_cost(wt);
                        const int B = lat_rl(Bj, j);
                        const bool mine = member && ((left >> lane) & 1) && tbest == wt;
                        left &= ~__ballot(mine);
                        int pblo = 0, poff = 0;
                        for (int s = 0; s < PP; ++s) {
                            const int q1 = lat_rl(pk1, s), q2 = lat_rl(pk2, s);
                            const int voff_s = q2 >> 16;
                            const int64_t wb = wt + (B - s - 2 > 0 ? B - s - 2 : 0) * t;
                            for (int k = lane; k < ((q1 >> 8) & 0xff); k += 64) {
                                const int jr = JR[voff_s + k], j1 = jr >> 8;
                                const WT *Wp = Cst + (q2 & 0xffff) + k * (q1 >> 24);
                                const int q0 = (q1 & 0xff) + k - ((q1 >> 16) & 0xff) - pblo;
                                int64_t b0 = kLBig, b1 = kLBig;
                                for (int jj = jr & 0xff; jj < j1; ++jj) {
                                    const int64_t w = (int64_t)Wp[jj];
                                    int64_t v0 = 0, v1 = kLBig;
                                    if (s) {   // uniform
                                        v0 = FS[2 * (poff + q0 - jj)];
                                        v1 = FS[2 * (poff + q0 - jj) + 1];
                                    }
                                    if (w > wt) break;
                                    const int64_t x = v0 + w, y = v1 + weight_cost(w);
                                    const int64_t z = v0 < kLBig ? (int64_t)((uint64_t)v0 + (uint64_t)wb) : kLBig;
                                    b0 = w < wt && x < b0 ? x : b0;
                                    b1 = w == wt && z < b1 ? z : b1;
                                    b1 = y < b1 ? y : b1;
                                }
                                FS[2 * (voff_s + k)] = b0;
                                FS[2 * (voff_s + k) + 1] = b1;
                            }
                            pblo = q1 & 0xff;
                            poff = voff_s;
                            lat_fence();
                        }
                        // the smallest split point through which a live state continues optimally
                        int b = N, my_a = 0, my_b = 0;   // lane s: stage s's split points
                        bool live0 = false, live1 = true;
                        int64_t sum = 0;
                        for (int s = PP - 1; s >= 0; --s) {
                            const int q1 = lat_rl(pk1, s), q2 = lat_rl(pk2, s), p1 = s ? lat_rl(pk1, s - 1) : 0;
                            const int po = s ? lat_rl(pk2, s - 1) >> 16 : 0;
                            const int64_t steady = B - s - 2 > 0 ? B - s - 2 : 0;
                            const int k = b - (q1 & 0xff), row = (q2 >> 16) + k;
                            const int64_t tg0 = FS[2 * row], tg1 = FS[2 * row + 1];
                            const int jr = JR[row], a0 = b - ((q1 >> 16) & 0xff);
                            int a = -1;
                            // a falls as the lane rises: the highest lane of the highest chunk wins
                            for (int jb = (jr >> 8) > 64 ? 64 : 0; jb >= 0 && a < 0; jb -= 64) {   // uniform
                                const int jj = jb + lane;
                                bool f0 = false, f1 = false;
                                int64_t w = 0;
                                if (jj >= (jr & 0xff) && jj < (jr >> 8)) {
                                    w = (int64_t)Cst[(q2 & 0xffff) + k * (q1 >> 24) + jj];
                                    int64_t v0 = 0, v1 = kLBig;
                                    if (s) {
                                        v0 = FS[2 * (po + a0 - jj - (p1 & 0xff))];
                                        v1 = FS[2 * (po + a0 - jj - (p1 & 0xff)) + 1];
                                    }
                                    f0 = v0 < kLBig && ((live0 && w < wt && v0 + w == tg0) ||
                                                        (live1 && w == wt && v0 + w + steady * t == tg1));
                                    f1 = v1 < kLBig && live1 && w <= wt && v1 + weight_cost(w) == tg1;
                                }
                                const uint64_t m0 = __ballot(f0), m1 = __ballot(f1);
                                if (m0 | m1) {
                                    const int top = 63 - __clzll((long long)(m0 | m1));
                                    a = a0 - jb - top;
                                    live0 = (m0 >> top) & 1;
                                    live1 = (m1 >> top) & 1;
                                    sum += weight_cost(lat_rl64(w, top));
                                }
                            }
                            if (a < 0) break;   // cannot happen on an optimal path
                            my_a = lane == s ? a : my_a;
                            my_b = lane == s ? b : my_b;
                            b = a;
                        }
                        // recomputation where the stage does not fit without it
                        bool rc = false;
                        if (lane < PP) {
                            const int64_t ms = (PP - lane) < B ? (PP - lane) : B;
                            const int64_t need =
                                mem[my_b] - mem[my_a] + ((mem[3 * np + my_b] - mem[3 * np + my_a]) > 0 ? X : 0);
                            rc = need + ms * (mem[np + my_b] - mem[np + my_a]) > cap;
                        }
                        const uint32_t rmask = (uint32_t)__ballot(rc);
                        uint32_t lw[kMaxStages / 4];
                        const int len = lane < PP ? my_b - my_a : 0;
#pragma unroll
                        for (int w = 0; w < kMaxStages / 4; ++w) {
                            lw[w] = 0;
#pragma unroll
                            for (int q = 0; q < 4; ++q) lw[w] |= (uint32_t)(lat_rl(len, 4 * w + q) & 0xff) << (8 * q);
                        }
                        if (mine) lat_write(out, HAPMOE_STATUS_OK, best + ki->dp_const, sum, t, rmask, lw);
                        lat_fence();
                    }
                    if (STATS && member) {   // the group's passes; its relaxations on its first candidate
                        st_out[0] = swept;
                        st_out[1] = lane == lead ? D.relax : 0;
                        st_out[2] = st_out[3] = 0;
                    }
                }
            }
        };
        if (narrow)
            search(uint32_t(0));
        else
            search(int64_t(0));
    };

    // a workgroup a key; in a later launch lane i looks at the i-th of the
    // workgroup's next 64 keys
    const int64_t stride = (int64_t)(retry ? 64 : 1) * gridDim.x;
    for (int64_t q0 = blockIdx.x; q0 < n_keys; q0 += stride) {
        uint64_t todo = 1;
        if (retry) {
            const int64_t kq = q0 + (int64_t)lane * gridDim.x;
            bool again = false;
            if (kq < n_keys) {
                const int64_t at = (key_lo + n_keys - 1 - kq) * nB;   // the key's first candidate in range
                again = res[(at > first ? at : first) - first].status == kStatusRetry;
            }
            todo = __ballot(again);
            __syncthreads();   // every wave has read the marks before a result replaces one
        }
        for (; todo; todo &= todo - 1)
            do_key(q0 + (int64_t)(__ffsll((unsigned long long)todo) - 1) * gridDim.x);
    }
}

}  // namespace

// LDS that a key of each depth in `depths` is expected to take, the largest of
// them: its layout for the types listed in order (other orderings differ by a
// few percent), 32-bit costs.  An estimate: what it misses goes to the next tier.
int latency_dp_lds(const hapmoe_problem &p, const std::vector<int32_t> &depths)
{
    const int N = p.model.n_layers, W = N + 1, T = p.cluster.n_types;
    int G = 0, need = 0;
    for (int h = 0; h < T; ++h) G += p.cluster.count[h];
    for (const int PP : depths) {
        const int g = G / PP;
        int lo[kMaxStages], hi[kMaxStages], type = 0, end = p.cluster.count[0];
        int64_t speed[kMaxStages], sum = 0;
        for (int s = 0; s < PP; ++s) {   // the type of the stage's middle device
            while (type + 1 < T && s * g + g / 2 >= end) end += p.cluster.count[++type];
            sum += speed[s] = p.cluster.speed[type];
        }
        int tlo = 0, thi = 0;
        for (int s = 0; s < PP; ++s) {
            int64_t l = 1, u = N;
            if (p.params.prune_window == 2) {
                l = N / PP;
                u = (N + PP - 1) / PP;
            } else if (p.params.prune_window) {
                const int64_t dn = p.params.delta_num, den = (int64_t)p.params.delta_den * sum;
                l = (p.params.delta_den - dn) * speed[s] * N / den;
                u = ((p.params.delta_den + dn) * speed[s] * N + den - 1) / den;
            }
            lo[s] = (int)(l < 1 ? 1 : l);
            hi[s] = (int)(u > N ? N : u);
            tlo += lo[s];
            thi += hi[s];
        }
        int clo = 0, chi = 0, ncost = 0, nv = 0, maxwd = 0;
        for (int s = 0; s < PP; ++s) {
            clo += lo[s];
            chi += hi[s];
            const int blo = std::max(clo, N - (thi - chi)), bhi = std::min(chi, N - (tlo - clo));
            const int wd = std::max(0, bhi - blo + 1);
            ncost += wd * (hi[s] - lo[s] + 1);
            nv += wd;
            maxwd = std::max(maxwd, wd);
        }
        const int slots = maxwd <= 24 ? 8 : (maxwd <= 48 ? 4 : 2);
        const int region = std::max(std::max(std::min(PP, T) * W * 16 + W * 28, nv * 16), slots * 56 * maxwd);
        need = std::max(need, kLatHeadBytes + ncost * 4 + nv * 2 + region);
    }
    return need + need / 32;
}

hipError_t launch_latency_dp(const void *d_image, const hapmoe_candidate *d_cand, int n_micro,
                             const TablesLayout &L, const void *d_tables, int64_t first, int64_t count,
                             hapmoe_dp_result *d_res, int32_t *d_stats, int lds_hint, hipStream_t stream)
{
    if (count == 0) return hipSuccess;
    const int64_t n_keys = (first + count - 1) / n_micro - first / n_micro + 1;
    const auto *img = static_cast<const unsigned char *>(d_image);
    const auto *tab = static_cast<const unsigned char *>(d_tables);
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return hipErrorUnknown;
    auto go = [&](auto kern) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLatLdsTiers[kLatTiers - 1]);
        if (e != hipSuccess) return e;
        const int lds0 = std::min(std::max((lds_hint + 1023) & ~1023, kLatLdsTiers[0]), kLatLdsTiers[1]);
        for (int tier = 0; tier < kLatTiers; ++tier) {
            // one workgroup a key: the dispatcher hands the next key to whichever
            // CU slot frees first, which balances keys of very different work; the
            // later launches mostly find nothing to do and get a chip's worth
            const int lds = tier == 0 ? lds0 : kLatLdsTiers[tier];
            if (tier == 1 && lds == lds0) continue;
            const int64_t most = tier == 0 ? kLatMaxGrid : (int64_t)ncu * (kLatLdsTiers[kLatTiers - 1] / lds);
            const int64_t grid = n_keys < most ? n_keys : most;
            hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kLatThreads), lds, stream, img, d_cand, tab, L, first,
                               count, d_res, d_stats, lds, tier > 0 ? 1 : 0, tier == kLatTiers - 1 ? 1 : 0);
        }
        return hipGetLastError();
    };
    return d_stats ? go(k_latency_dp<true>) : go(k_latency_dp<false>);
}

}  // namespace hapmoe
