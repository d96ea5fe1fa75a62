// Per-stage data-parallel widths (stage_types = 3): the non-uniform PP/DP
// partitioning of the paper's contributions -- stage-wise parallelism knobs
// chosen jointly with the layer assignment (Section 1, the ablation of the
// evaluation) -- on the block device layout.  The devices are listed type by
// type in the candidate's ordering; stage i takes the next w_i half-groups of
// g/2 devices (g = G/PP), w_i in {1, 2, 3}, sum w_i = 2 PP, and runs DP_i =
// w_i DP / 2 replicas.  Every stage processes the same global micro-batch, so a
// replica holds r = 2 / w_i of the nominal tokens: the Section 3.2 terms are
// evaluated at that token count, the ZeRO-1 optimizer state over DP_i, the
// activations and MoE buffers at r; the boundary transfer is the sender's
// per-rank activation; the pruning-1 window follows the stage's share w_i P_i
// (g/2) / sum_h m_h P_h of the cluster's compute; pruning 3 and T_dp-sync +
// T_opt keep their nominal values.
//
// Kernel W1 (k_width_tables, one workgroup per configuration) writes layer
// prefix sums of the stage time without / with recomputation and of its
// communication for every device-type set at each width, and of the memory
// terms at each width.  Kernel W2 (k_width_dp, persistent workgroups over the
// candidates) runs, per candidate, the threshold DP over (stage, end layer,
// half-groups used): F_t[i][b][u] = min over (a, w) of F_t[i-1][a][u-w] +
// c_{i-1}(u-w, w; a, b) over stage costs <= t, ties to the smallest a, then the
// smallest w.  A pass at t gives a partition whose largest stage m keeps F constant
// on [m, t].  The sweep first passes at t_bot, the least possible largest stage (one
// min-max pass), then at infinity, then descends: the next threshold is min(m - 1,
// the largest that can still beat the incumbent), and the sweep ends at t_bot.  The
// incumbent of t_bot is close to the optimum for B well above 1, so few thresholds
// are left (61 layers, 16 stages, B = 16 to 64: 32 passes a feasible key when the
// sweep descended from infinity alone, 13 now).  The incumbent is replaced by a lower
// sum + (B-1) max, or an equal one with a lower max, so the result is the least
// objective, the least threshold reaching it and the back-trace there.
//
// Plain int64 min-plus work, bound by the instructions of a relaxation round and the
// latency of its LDS reads.  Only states whose end layer lies in the band that the
// windows leave between start and end are listed (half of the full rectangle and
// less); a first pass stores the feasible split points of every (state, width) as
// an interval, so that later passes read no memory terms; stage times, F of two
// levels, intervals, lists and back-trace pointers stay in LDS (61 layers, 16 stages:
// about 60 KB, two workgroups of eight waves a CU).  A key that needs more than tier 1
// is given is left to a last tier of one workgroup a CU, with lists, intervals and
// pointers in the workgroup's slice of the workspace.  61 layers, 31,296 keys, PP <=
// 16: the kernel 32.9 -> 2.36 ms (one state a lane over the full rectangle, costs from
// global memory and a one-lane back-trace before); VALU instructions take 46 % of the
// issue slots and 70 % of the wave cycles wait, for LDS and at the barrier of a level.
// Running a window's split points from the highest and leaving at the first above the
// threshold measured 4 % slower.
#include "internal.h"

namespace hapmoe {
namespace {

constexpr int kThreads = 256;     // of a width-table workgroup
// of a DP workgroup: LDS holds two a CU, and eight waves each hide more of the reads'
// latency than four (61 layers, PP <= 16: 2.66 against 3.03 ms a call)
constexpr int kDpThreads = 512;
constexpr int kLayerSlots = 128;   // >= kMaxLayers + 1
constexpr int kMemEntries = (3 * kLayerSlots + kDpThreads - 1) / kDpThreads;   // (width, layer) pairs a thread

__device__ inline int lg2i(int v) { return 31 - __clz(v); }

__device__ inline int64_t qterm(double x, unsigned *flag)
{
    if (!(x < (double)kTermLimit)) {
        atomicOr(flag, 1u);
        return kTermLimit;
    }
    return (int64_t)ceil(x);
}

// slowest link inside a device-type set (largest latency, smallest bandwidth)
__device__ inline void set_link(const ImageHeader &H, int mask, double &alpha, double &bw)
{
    bool first = true;
    alpha = 0.0;
    bw = 0.0;
    for (int h = 0; h < H.n_types; ++h) {
        if (!((mask >> h) & 1)) continue;
        for (int g = 0; g < H.n_types; ++g) {
            if (!((mask >> g) & 1)) continue;
            const double a = H.alpha[h * kMaxTypes + g], b = H.bw[h * kMaxTypes + g];
            if (first || a > alpha) alpha = a;
            if (first || b < bw) bw = b;
            first = false;
        }
    }
}

__device__ inline double ring_ar(double bytes, int w, double alpha, double bw)
{
    if (w == 1) return 0.0;
    const double steps = (double)(2 * (w - 1));
    return steps * alpha + ((steps * bytes) / (double)w) / bw;
}

// token share of one replica of a width-w stage
__device__ inline double ratio(int w) { return 2.0 / (double)w; }

// ---- kernel W1: width tables, one 256-thread workgroup per configuration ----
__global__ __launch_bounds__(kThreads) void k_width_tables(const unsigned char *__restrict__ img,
                                                           const hapmoe_candidate *__restrict__ cand,
                                                           int64_t per_config, int64_t cfg_lo, TablesLayout L,
                                                           unsigned char *__restrict__ tab)
{
    const ImageHeader &H = *reinterpret_cast<const ImageHeader *>(img);
    const uint8_t *is_moe = img + H.off_is_moe;
    const int64_t *pdense = reinterpret_cast<const int64_t *>(img + H.off_pdense);
    const int64_t *pexp = reinterpret_cast<const int64_t *>(img + H.off_pexp);
    const int64_t *act = reinterpret_cast<const int64_t *>(img + H.off_act);
    const int64_t *tdense = reinterpret_cast<const int64_t *>(img + H.off_tdense);
    const int64_t *tffn = reinterpret_cast<const int64_t *>(img + H.off_tffn);
    const double *skew = reinterpret_cast<const double *>(tab + L.off_layer);

    const int64_t cfg = cfg_lo + blockIdx.x;
    const int tid = threadIdx.x;
    const hapmoe_candidate c = cand[cfg * per_config];
    const int N = H.n_layers, T = H.n_types;
    const int64_t np = L.np;
    const int nm = (int)L.n_masks;

    __shared__ int64_t s_qce[3][kMaxTypes][kLayerSlots];   // q(comp) + q(expert) per width, type, layer
    __shared__ int64_t s_val[3][3][kLayerSlots];            // per width: w, a0, a1 of each layer
    __shared__ unsigned s_flag;
    if (tid == 0) s_flag = 0;
    __syncthreads();

    const double tok0 = (double)((int64_t)H.seq_len * H.mbs / c.cp);
    // per-layer terms at each width
    for (int i = tid; i < 3 * N; i += kThreads) {
        const int wi = i / N, l = i - wi * N, w = wi + 1;
        const double r = ratio(w);
        const double tok = tok0 * r;
        const bool moe = is_moe[l] != 0;
        for (int h = 0; h < T; ++h) {
            const int64_t off = (((int64_t)h * 4 + lg2i(c.tp)) * 4 + lg2i(c.cp)) * N + l;
            const double td = (double)tdense[off], tf = (double)tffn[off];
            double comp, expert;
            if (!moe) {
                comp = td * r;
                expert = 0.0;
            } else {
                const double route = H.route_coef[h] * (tok * (double)H.hidden);
                comp = (td - tf) * r + route;
                const double xexp = (H.moe_ffn_mult * (tf * r)) / ((H.eff[h] * (double)c.ep) * (double)c.tpe);
                expert = skew[l] * xexp;
            }
            s_qce[wi][h][l] = qterm(comp, &s_flag) + qterm(expert, &s_flag);
        }
        const int dp_i = c.dp * w / 2;
        const double beta_opt = 6.0 + 12.0 / (double)dp_i;
        const double wt = ((double)pdense[l] / (double)c.tp + (double)pexp[l] / (double)(c.ep * c.tpe)) * beta_opt;
        const double a0 = ((double)act[l] * r) / (double)(c.tp * c.cp);
        const int64_t qa0 = qterm(a0, &s_flag);
        s_val[wi][0][l] = qterm(wt, &s_flag);
        s_val[wi][1][l] = qa0;
        s_val[wi][2][l] = qterm(H.rc_act * (double)qa0, &s_flag);
    }
    __syncthreads();

    // memory prefix sums, then the stage times of every device-type set at every width:
    // a wave a row, layers 2 lane and 2 lane + 1 a lane, so that the per-layer terms of a
    // row are evaluated side by side (one thread a row before: 160 us, now 85, for
    // 1,304 configurations of 61 layers and 45 rows)
    int64_t *wmem = reinterpret_cast<int64_t *>(tab + L.off_wmem) + cfg * 3 * 4 * np;
    const int lane = tid & 63, wave = tid >> 6, l0 = 2 * lane;
    auto put_row = [&](int64_t *row, int64_t v0, int64_t v1) {   // all lanes of the wave
        int64_t sum = v0 + v1;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t y = __shfl_up(sum, d);
            if (lane >= d) sum += y;
        }
        if (lane == 0) row[0] = 0;
        if (l0 < N) row[l0 + 1] = sum - v1;
        if (l0 + 1 < N) row[l0 + 2] = sum;
    };
    for (int r = wave; r < 12; r += kThreads / 64) {
        const int wi = r / 4, f = r % 4;
        int64_t v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            v[q] = l0 + q >= N ? 0 : f < 3 ? s_val[wi][f][l0 + q] : (int64_t)(is_moe[l0 + q] != 0);
        put_row(wmem + (wi * 4 + f) * np, v[0], v[1]);
    }
    int64_t *wtime = reinterpret_cast<int64_t *>(tab + L.off_wtime) + cfg * nm * 3 * 3 * np;
    // a stage of at most three half-groups holds three types or more only if the
    // devices of a type fit strictly inside it: no such set is read otherwise.  The set
    // of all types is evaluated all the same: its latency, bandwidth and compute bound
    // those of every other set, so it marks an overflow whenever any set would.
    int least = H.count[0];
    for (int h = 1; h < T; ++h) least = H.count[h] < least ? H.count[h] : least;
    const int most_types = 3 * (H.total_devices / c.pp / 2) >= least + 2 ? T : 2;
    for (int i = wave; i < nm * 3; i += kThreads / 64) {
        const int m = i / 3 + 1, wi = i % 3;
        if (__popc(m) > most_types && m != nm) continue;
        const double r = ratio(wi + 1);
        double alpha, bw;
        set_link(H, m, alpha, bw);
        const double D = ((tok0 * r) * (double)H.hidden) * (double)H.elem_bytes;
        int64_t t0[2] = {0, 0}, t1[2] = {0, 0}, cm[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int l = l0 + q;
            if (l >= N) continue;
            double a2a, tp;
            if (!is_moe[l]) {
                a2a = 0.0;
                tp = 4.0 * ring_ar(D, c.tp, alpha, bw);
            } else {
                const double sk = skew[l];
                const double dm = (D * (double)H.top_k) * (1.0 - 1.0 / (double)c.ep);
                const double f_a2a = (double)(c.ep - 1) * alpha + dm / bw;
                const double f_ag = (double)(c.ep - 1) * alpha + (D * (double)(c.ep - 1)) / bw;
                a2a = sk * (4.0 * (f_ag < f_a2a ? f_ag : f_a2a));
                tp = 2.0 * ring_ar(D, c.tp, alpha, bw) + 2.0 * ring_ar(D, c.tpe, alpha, bw);
            }
            const double cpt =
                c.cp == 1 ? 0.0 : 3.0 * ((double)(c.cp - 1) * (alpha + ((2.0 * D) / (double)c.tp) / bw));
            cm[q] = qterm(a2a, &s_flag) + qterm(tp, &s_flag) + qterm(cpt, &s_flag);
            int64_t ce = -1;
            for (int h = 0; h < T; ++h)
                if ((m >> h) & 1) ce = s_qce[wi][h][l] > ce ? s_qce[wi][h][l] : ce;
            t0[q] = ce + cm[q];
            t1[q] = qterm(H.rc_time * (double)t0[q], &s_flag);
        }
        int64_t *P0 = wtime + ((int64_t)(m - 1) * 3 + wi) * 3 * np;
        put_row(P0, t0[0], t0[1]);
        put_row(P0 + np, t1[0], t1[1]);
        put_row(P0 + 2 * np, cm[0], cm[1]);
    }
    if (tid >= 64 && tid < 67) {   // MoE buffers of each width
        const int wi = tid - 64;
        const double r = ratio(wi + 1);
        const double tok = tok0 * r;
        const double D = (tok * (double)H.hidden) * (double)H.elem_bytes;
        const double dm = (D * (double)H.top_k) * (1.0 - 1.0 / (double)c.ep);
        reinterpret_cast<int64_t *>(tab + L.off_wx)[cfg * 4 + wi] =
            qterm(((8.0 * tok) * (double)H.top_k) + 2.0 * dm, &s_flag);
    }
    __syncthreads();
    if (tid == 0 && s_flag) reinterpret_cast<PiInfo *>(tab + L.off_pi)[cfg].status = HAPMOE_STATUS_OVERFLOW;
}

// ---- kernel W2: the DP, one (configuration, ordering) key per workgroup pass of the queue ----
struct WStage {     // stage on half-groups [u, u + w)
    int64_t cap, p2p;
    uint8_t mask, lo, hi, flags;   // flags: 1 mixed, 2 next stage starts on another type; mask 0: no stage
    uint16_t row, am;              // first entry of its stage-time row; its row of pruning-3 limits (mixed)
};

// the predecessors that one width gives the states of a (level, half-groups used) row:
// split point a is state fofs + a of the level before, at most min(b - lo, last)
struct WDesc {
    int64_t p2p;
    int16_t fofs;
    uint16_t row;
    uint8_t lo, last;
    uint16_t pad;
};

struct WLevel {
    int32_t first, n;   // states of levels 1 .. i - 1; of level i
    int32_t rows, ul;   // rows of levels 1 .. i - 1; half-groups used in the level's first row
};

constexpr int64_t kFar = int64_t(1) << 62;   // no path; above every stage sum
constexpr int kMaxRows = 45;                  // (device-type set, width) pairs
constexpr int kWidthLastLds = 160 * 1024 - 2048;   // dynamic LDS of the last tier
// what the last tier keeps in LDS at most (32 stages, 127 layers, ten contiguous type
// sets): stages, bands, levels, stage times, memory terms and F of two levels (33 rows
// of 96 end layers)
static_assert(65 * 3 * sizeof(WStage) + 33 * 65 * 4 + kLayerSlots + 33 * sizeof(WLevel) + 64 +
                      10 * 3 * kLayerSlots * 16 + 2 * 33 * 96 * 8 + 6 * kLayerSlots * 16 <= kWidthLastLds,
              "last tier");

// states of level i lie in half-groups used [units_lo, units_hi]
__host__ __device__ inline int units_lo(int i, int PP) { return i > 3 * i - PP ? i : 3 * i - PP; }
__host__ __device__ inline int units_hi(int i, int PP) { return 3 * i < PP + i ? 3 * i : PP + i; }
__host__ __device__ inline int level_rows(int i, int PP) { return units_hi(i, PP) - units_lo(i, PP) + 1; }

// floor(x / d) for d > 0 where only its sign matters below zero (-1)
__device__ inline int64_t floor_div(int64_t x, int64_t d) { return x < 0 ? -1 : x / d; }

template <int CTRL>
__device__ inline int64_t quad_swap(int64_t x)
{
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)x, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xf, 0xf, true);
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

__device__ inline int64_t wave_max(int64_t x)
{
#pragma unroll
    for (int d = 32; d; d >>= 1) {
        const int64_t y = __shfl_xor(x, d);
        x = y > x ? y : x;
    }
    return x;
}

// LAST: the tier of the keys whose regions exceed tier 1's LDS; state lists, intervals,
// back-trace pointers, descriptors and pruning-3 limits in the workgroup's slice
template <bool STATS, bool LAST>
__global__ __launch_bounds__(kDpThreads, 4) void k_width_dp(const unsigned char *__restrict__ img,
                                                       const hapmoe_candidate *__restrict__ cand, TablesLayout L,
                                                       const unsigned char *__restrict__ tab, int64_t first,
                                                       int64_t count, int lds_bytes,
                                                       unsigned char *__restrict__ slots, int64_t slot_bytes,
                                                       hapmoe_dp_result *__restrict__ res,
                                                       uint8_t *__restrict__ types_out,
                                                       uint8_t *__restrict__ widths_out, int32_t *__restrict__ stats,
                                                       uint32_t *__restrict__ queue, uint32_t *__restrict__ spill)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t s_t, s_x[3];
    __shared__ uint32_t s_qi, s_mixed, s_relax;
    __shared__ int32_t s_n_rows;
    __shared__ uint8_t s_on[kMaxRows + 3], s_src[kMaxRows + 3], s_id[kMaxRows + 3];   // rows in use: flag, pair, row
    __shared__ uint8_t s_mix[3 * (2 * kMaxStages + 1) + 1];                           // mixed stages, u * 3 + w - 1

    const ImageHeader &H = *reinterpret_cast<const ImageHeader *>(img);
    const uint8_t *is_moe = img + H.off_is_moe;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool lead = tid < 64;   // wave 0 back-traces and keeps the incumbents, lane j candidate j's
    const int N = H.n_layers, W = N + 1, T = H.n_types, nB = H.n_micro;
    const int64_t np = L.np;
    const bool prune_het = H.prune_hetero != 0, recomp = H.allow_recompute != 0;
    const int64_t key_lo = first / nB;
    // tier 1 takes the keys of candidates [first, first + count), the deepest first
    const int64_t n_keys = LAST ? (int64_t)queue[1] : (first + count - 1) / nB - key_lo + 1;
    uint32_t *const next_key = queue + (LAST ? 2 : 0);
    for (;;) {
        __syncthreads();   // the previous key is done with LDS
        if (tid == 0) {
            s_qi = atomicAdd(next_key, 1u);
            s_mixed = 0;
            if (STATS) s_relax = 0;
        }
        if (tid < kMaxRows) s_on[tid] = 0;
        __syncthreads();
        const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_qi);
        if ((int64_t)k >= n_keys) break;   // every workgroup exits once the queue is drained
        const int64_t key = LAST ? (int64_t)spill[k] : key_lo + n_keys - 1 - k;
        const hapmoe_candidate c = cand[key * nB];
        const int64_t cfg = key / H.n_orders;
        const int o = (int)(key - cfg * H.n_orders);
        const int PP = __builtin_amdgcn_readfirstlane(c.pp), U = 2 * PP, UP = U + 1;
        const PiInfo *pi = reinterpret_cast<const PiInfo *>(tab + L.off_pi) + cfg;
        const KeyInfo *ki = reinterpret_cast<const KeyInfo *>(tab + L.off_key) + key;
        const int64_t eta_tbar = (int64_t)H.eta_prune * pi->tbar;
        const int status = pi->status;
        const bool status_ok = status == HAPMOE_STATUS_OK;
        const int64_t *wtime = reinterpret_cast<const int64_t *>(tab + L.off_wtime) + cfg * L.n_masks * 3 * 3 * np;
        const int64_t *wmem = reinterpret_cast<const int64_t *>(tab + L.off_wmem) + cfg * 3 * 4 * np;

        // regions of LDS; the rest follows once the bands are known
        const int o_rs = UP * 3 * (int)sizeof(WStage), o_lev = (o_rs + (PP + 1) * UP * 2 + 15) & ~15;
        const int o_blo = o_lev + (PP + 1) * (int)sizeof(WLevel), o_bwd = o_blo + (PP + 1) * UP;
        const int o_lm = o_bwd + (PP + 1) * UP, o_tim = (o_lm + W + 15) & ~15;
        WStage *const st = reinterpret_cast<WStage *>(smem);
        uint16_t *const rs = reinterpret_cast<uint16_t *>(smem + o_rs);   // [level][units]: the row's first state
        WLevel *const lev = reinterpret_cast<WLevel *>(smem + o_lev);
        uint8_t *const blo = smem + o_blo, *const bwd = smem + o_bwd, *const lm = smem + o_lm;   // [level][units]

        // memory terms of kMemEntries (width, layer) pairs a thread, in registers
        int64_t mw[kMemEntries] = {}, ma0[kMemEntries] = {}, ma1[kMemEntries] = {};
        if (status_ok) {
#pragma unroll
            for (int q = 0; q < kMemEntries; ++q) {
                const int e = tid + q * kDpThreads, wi = e / W, b = e - wi * W;
                if (e < 3 * W) {
                    mw[q] = wmem[(wi * 4 + 0) * np + b];
                    ma0[q] = wmem[(wi * 4 + 1) * np + b];
                    ma1[q] = wmem[(wi * 4 + 2) * np + b];
                }
            }
        }
        if (tid < 3) s_x[tid] = reinterpret_cast<const int64_t *>(tab + L.off_wx)[cfg * 4 + tid];
        // ---- the stage on half-groups [u, u + w) of this ordering ----
        if (status_ok) {
            const int G = H.total_devices, half = G / PP / 2;
            int pos_type[kMaxTypes], pos_end[kMaxTypes];
            int acc = 0;
            int64_t total_speed = 0;
            for (int j = 0; j < T; ++j) {
                pos_type[j] = H.perm[o][j];
                acc += H.count[pos_type[j]];
                pos_end[j] = acc;
                total_speed += (int64_t)H.count[j] * H.speed[j];
            }
            auto type_of = [&](int d) {
                int t = pos_type[T - 1];
                for (int j = T - 1; j >= 0; --j)
                    if (d < pos_end[j]) t = pos_type[j];
                return t;
            };
            for (int i = tid; i < UP * 3; i += kDpThreads) {
                const int u = i / 3, w = i % 3 + 1;
                WStage x = {0, 0, 0, 0, 0, 0, 0, 0};
                if (u + w <= U) {
                    const int d0 = u * half, d1 = (u + w) * half;
                    int mask = 0;
                    for (int j = 0; j < T; ++j)
                        if (pos_end[j] - H.count[pos_type[j]] < d1 && pos_end[j] > d0) mask |= 1 << pos_type[j];
                    int64_t cap = -1;
                    int sp = 0;
                    for (int h = 0; h < T; ++h) {
                        if (!((mask >> h) & 1)) continue;
                        if (cap < 0 || H.mem_bytes[h] < cap) cap = H.mem_bytes[h];
                        if (sp == 0 || H.speed[h] < sp) sp = H.speed[h];
                    }
                    const int last = type_of(d1 - 1);
                    int flags = __popc(mask) > 1 ? 1 : 0;
                    int64_t p2p = 0;
                    if (u + w < U) {
                        const int nt = type_of(d1);
                        if (nt != last) flags |= 2;
                        const double a = H.alpha[last * kMaxTypes + nt], b = H.bw[last * kMaxTypes + nt];
                        const double r = ratio(w);
                        const double D = (((double)((int64_t)H.seq_len * H.mbs / c.cp) * r) * (double)H.hidden) *
                                         (double)H.elem_bytes;
                        p2p = (int64_t)ceil(2.0 * (a + (D / (double)c.tp) / b));
                    }
                    int64_t lo = 1, hi = N;
                    if (H.prune_window == 1) {
                        const int64_t dn = H.delta_num, dd = H.delta_den;
                        const int64_t num = (int64_t)w * sp * half * N, den = dd * total_speed;
                        lo = ((dd - dn) * num) / den;
                        hi = ((dd + dn) * num + den - 1) / den;
                        lo = lo < 1 ? 1 : lo;
                        hi = hi > N ? N : hi;
                    } else if (H.prune_window == 2) {
                        lo = N / PP;
                        hi = (N + PP - 1) / PP;
                    }
                    x.cap = cap;
                    x.p2p = p2p;
                    x.lo = (uint8_t)lo;
                    x.hi = (uint8_t)hi;
                    x.flags = (uint8_t)flags;
                    // a pure stage whose transfer alone fails pruning 3 is none at all
                    if (!(prune_het && flags == 2 && p2p > eta_tbar) && lo <= hi) {
                        x.mask = (uint8_t)mask;
                        s_on[(mask - 1) * 3 + w - 1] = 1;
                        if (prune_het && (flags & 1)) {
                            x.am = (uint16_t)atomicAdd(&s_mixed, 1u);
                            s_mix[x.am] = (uint8_t)i;
                        }
                    }
                }
                st[i] = x;
            }
        }
        for (int b = tid; b < W; b += kDpThreads) {   // [a, b) holds an MoE layer iff a < lm[b]
            int l = b;
            while (l > 0 && !is_moe[l - 1]) --l;
            lm[b] = (uint8_t)l;
        }
        __syncthreads();
        if (lead) {   // rows of the (device-type set, width) pairs in use
            const bool on = lane < kMaxRows && s_on[lane];
            const uint64_t m = __ballot(on);
            if (on) {
                const int r = __popcll(m & ((uint64_t(1) << lane) - 1));
                s_id[lane] = (uint8_t)r;
                s_src[r] = (uint8_t)lane;
            }
            if (lane == 0) s_n_rows = __popcll(m);
        }

        // ---- the end layers each (level, half-groups used) can have: reached from the
        // start and able to reach the end, as the windows allow ----
        {
            // reach[level][units] from the start (0, 1) and to the end (2, 3): least and most layers
            uint8_t *reach = smem + o_tim;
            const int plane = (PP + 1) * UP;
            const bool ok = status_ok;
            for (int i = 0; ok && i <= PP; ++i) {
                const int side = (tid >> 7) & 1, u = tid >= 256 ? 127 : tid & 127;   // side 1 walks backwards from the end
                const int lev = side ? PP - i : i;
                if (u < UP) {
                    int lo = 255, hi = 0;
                    if (i == 0) {
                        if (u == (side ? U : 0)) lo = 0;
                    } else {
                        for (int w = 1; w <= 3; ++w) {
                            const int u0 = side ? u : u - w, from = side ? u + w : u - w;
                            if (from < 0 || from > U) continue;
                            const WStage &x = st[u0 * 3 + w - 1];
                            const int at = (side ? lev + 1 : lev - 1) * UP + from;
                            const int l0 = reach[(2 * side) * plane + at];
                            if (x.mask == 0 || l0 == 255) continue;
                            const int nl = l0 + x.lo, nh = min(reach[(2 * side + 1) * plane + at] + x.hi, N);
                            if (nl > N) continue;
                            lo = min(lo, nl);
                            hi = max(hi, nh);
                        }
                    }
                    reach[(2 * side) * plane + lev * UP + u] = (uint8_t)lo;
                    reach[(2 * side + 1) * plane + lev * UP + u] = (uint8_t)hi;
                }
                __syncthreads();
            }
            for (int x = tid; ok && x < plane; x += kDpThreads) {
                int lo = 0, wd = 0;
                if (reach[x] != 255 && reach[2 * plane + x] != 255) {
                    lo = max((int)reach[x], N - (int)reach[3 * plane + x]);
                    wd = min((int)reach[plane + x], N - (int)reach[2 * plane + x]) - lo + 1;
                    wd = wd < 0 ? 0 : wd;
                }
                blo[x] = (uint8_t)lo;
                bwd[x] = (uint8_t)wd;
            }
            __syncthreads();
        }
        // the states of a level, row after row: one wave a level
        if (status_ok)
            for (int i = wave; i <= PP; i += kDpThreads / 64) {
                const int ul = units_lo(i, PP), nu = level_rows(i, PP);   // at most 33 rows
                const int wd = lane < nu ? bwd[i * UP + ul + lane] : 0;
                int sum = wd;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int y = __shfl_up(sum, d);
                    if (lane >= d) sum += y;
                }
                if (lane < nu) rs[i * UP + ul + lane] = (uint16_t)(sum - wd);
                if (lane == 63) {
                    lev[i].n = sum;
                    lev[i].ul = ul;
                }
            }
        __syncthreads();
        if (status_ok && lead) {
            const int n = lane <= PP ? lev[lane].n : 0, nr = lane >= 1 && lane <= PP ? level_rows(lane, PP) : 0;
            int fs = lane ? n : 0, fr = nr;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(fs, d), z = __shfl_up(fr, d);
                if (lane >= d) {
                    fs += y;
                    fr += z;
                }
            }
            if (lane <= PP) {
                lev[lane].first = fs - (lane ? n : 0);
                lev[lane].rows = fr - nr;
            }
        }
        __syncthreads();

        // ---- sizes of the remaining regions; a key that needs more goes to the last tier ----
        int fsz = 1, n_states = 0, n_desc = 0;
        bool shape_ok = status_ok;
        if (status_ok) {
            for (int i = 0; i <= PP; ++i) {
                const int n = lev[i].n;
                shape_ok = shape_ok && n > 0;
                fsz = max(fsz, n);
            }
            n_states = lev[PP].first + lev[PP].n;
            n_desc = lev[PP].rows + level_rows(PP, PP);
        }
        shape_ok = __builtin_amdgcn_readfirstlane(shape_ok);
        fsz = __builtin_amdgcn_readfirstlane(fsz);
        n_states = __builtin_amdgcn_readfirstlane(n_states);
        const int n_rows = __builtin_amdgcn_readfirstlane(s_n_rows);
        const int n_mixed = __builtin_amdgcn_readfirstlane((int)s_mixed);
        const int o_f = o_tim + n_rows * W * 16, o_val = o_f + 2 * fsz * 8, val_bytes = 2 * 3 * W * 16;
        // the memory terms serve the first pass only, the back-trace pointers the others
        const int o_iv = o_val + (LAST || n_states * 2 <= val_bytes ? val_bytes : (n_states * 2 + 15) & ~15);
        const int b_iv = n_states * 3 * 2, b_desc = n_desc * 3 * (int)sizeof(WDesc);
        const int o_desc = (o_iv + b_iv + 15) & ~15, o_list = o_desc + b_desc, o_am = o_list + n_states * 2;
        if (!LAST && shape_ok && o_am + n_mixed * W > lds_bytes) {
            if (tid == 0) spill[atomicAdd(queue + 1, 1u)] = (uint32_t)key;
            continue;
        }
        unsigned char *const slice = slots + (int64_t)blockIdx.x * slot_bytes;
        longlong2 *const tim = reinterpret_cast<longlong2 *>(smem + o_tim);   // {T0, T1} [row][b]
        int64_t *const F = reinterpret_cast<int64_t *>(smem + o_f);           // [level & 1][state]
        longlong2 *const val = reinterpret_cast<longlong2 *>(smem + o_val);   // [level & 1][width][b]
        // feasible split points of each (state, width): the least (low byte; 255: none) and
        // the least without recomputation (high byte)
        unsigned char *const big = LAST ? slice - o_desc : smem;   // where the regions from o_desc on lie
        WDesc *const desc = reinterpret_cast<WDesc *>(big + o_desc);
        uint16_t *const list = reinterpret_cast<uint16_t *>(big + o_list);    // row << 7 | b of each state
        uint8_t *const am = big + o_am;                                       // [mixed stage][b]: least split point
        const int o_tail = (o_am + n_mixed * W + 15) & ~15;
        uint16_t *const iv = LAST ? reinterpret_cast<uint16_t *>(big + o_tail) : reinterpret_cast<uint16_t *>(smem + o_iv);
        uint16_t *const arg = LAST ? iv + 3 * n_states : reinterpret_cast<uint16_t *>(smem + o_val);

        if (shape_ok) {
            // stage times: a wave a row
#pragma unroll 2
            for (int r = wave; r < n_rows; r += kDpThreads / 64) {
                const int64_t *P = wtime + (int64_t)s_src[r] * 3 * np;
                const int b0 = lane < W ? lane : 0, b1 = lane + 64 < W ? lane + 64 : 0;
                const longlong2 x = make_longlong2(P[b0], P[np + b0]), y = make_longlong2(P[b1], P[np + b1]);
                if (lane < W) tim[r * W + lane] = x;
                if (lane + 64 < W) tim[r * W + lane + 64] = y;
            }
            // communication only grows with the layers, so pruning 3 is a least split point
            for (int m = wave; m < n_mixed; m += kDpThreads / 64) {
                const WStage &x = st[s_mix[m]];
                const int64_t *P2 = wtime + ((int64_t)(x.mask - 1) * 9 + (s_mix[m] % 3) * 3 + 2) * np;
                const int64_t room = eta_tbar - ((x.flags & 2) ? x.p2p : 0);
                for (int b = lane; b < W; b += 64) {
                    int a = max(b - (int)x.hi, 0);
                    const int64_t pb = P2[b];
                    while (a < b && pb - P2[a] > room) ++a;
                    am[m * W + b] = (uint8_t)a;
                }
            }
            for (int i = tid; i < UP * 3; i += kDpThreads) {
                const int m = st[i].mask;
                if (m) st[i].row = (uint16_t)(s_id[(m - 1) * 3 + i % 3] * W);
            }
            // state lists
            for (int x = tid; x < PP * UP; x += kDpThreads) {
                const int i = x / UP + 1, u = x - (i - 1) * UP, r = u - units_lo(i, PP);
                const int wd = bwd[i * UP + u];
                if (!wd) continue;
                uint16_t *at = list + lev[i].first + rs[i * UP + u];
                const int b = blo[i * UP + u];
                for (int j = 0; j < wd; ++j) at[j] = (uint16_t)(r << 7 | (b + j));
            }
        }
        __syncthreads();
        if (shape_ok)
            for (int x = tid; x < PP * UP * 3; x += kDpThreads) {
                const int i = x / (UP * 3) + 1, y = x - (i - 1) * UP * 3, u = y / 3, wi = y - u * 3;
                const int ul = units_lo(i, PP), u0 = u - wi - 1;
                if (u < ul || u > units_hi(i, PP)) continue;
                WDesc d = {0, 0, 0, 255, 0, 0};   // none: no split point is at most 0 - 255
                if (u0 >= 0 && u0 >= units_lo(i - 1, PP) && u0 <= units_hi(i - 1, PP)) {
                    const WStage &z = st[u0 * 3 + wi];
                    const int at = (i - 1) * UP + u0;
                    if (z.mask && bwd[at]) {
                        d.p2p = z.p2p;
                        d.fofs = (int16_t)((int)rs[at] - (int)blo[at]);
                        d.row = z.row;
                        d.lo = z.lo;
                        d.last = (uint8_t)(blo[at] + bwd[at] - 1);
                    }
                }
                desc[(lev[i].rows + u - ul) * 3 + wi] = d;
            }
        __syncthreads();

        int64_t B = 1;   // the group's min(B, PP): every stage's stored micro-batches at most
        // weights + stored activations of stage i - 1 (prefix sums), without and with recomputation
        auto put_val = [&](int i) {
            const int64_t ms = (int64_t)(PP - i + 1) < B ? (int64_t)(PP - i + 1) : B;
#pragma unroll
            for (int q = 0; q < kMemEntries; ++q) {
                const int e = tid + q * kDpThreads;
                if (e < 3 * W)
                    val[(i & 1) * 3 * W + e] = make_longlong2(mw[q] + ms * ma0[q], mw[q] + ms * ma1[q]);
            }
        };
        uint32_t relax = 0;
        // A state is relaxed by the four lanes of a quad: widths 1 and 2 a lane each, width
        // 3 (the longest window) on two, its split points alternating.

        // first pass of a group: the least possible largest stage, and every state's
        // feasible split points (suffixes of the window: memory falls as a rises)
        auto first_pass = [&]() -> int64_t {
            if (tid == 0) F[0] = 0;   // level 0: (b, u) = (0, 0)
            put_val(1);
            __syncthreads();
            for (int i = 1; i <= PP; ++i) {
                const int64_t *Fp = F + ((i - 1) & 1) * fsz;
                int64_t *Fc = F + (i & 1) * fsz;
                const longlong2 *vl = val + (i & 1) * 3 * W;
                const WLevel lv = lev[i];
                const int ofs = __builtin_amdgcn_readfirstlane(lv.first), items = __builtin_amdgcn_readfirstlane(lv.n) * 4;
                const int dofs = __builtin_amdgcn_readfirstlane(lv.rows), ul = __builtin_amdgcn_readfirstlane(lv.ul);
                if (i < PP) put_val(i + 1);
                for (int e = tid; e < items; e += kDpThreads) {
                    const int q = e & 3, s = e >> 2, wi = q == 3 ? 2 : q;
                    const int x = list[ofs + s], b = x & 127, r = x >> 7;
                    const WDesc d = desc[(dofs + r) * 3 + wi];
                    int64_t best = kFar;
                    int amin = 255, a0 = 255;
                    const int ahi = min(b - (int)d.lo, (int)d.last);
                    if (ahi >= 0) {
                        const WStage z = st[(ul + r - wi - 1) * 3 + wi];
                        int a = max(b - (int)z.hi, 0);
                        const longlong2 *tr = tim + d.row, *vr = vl + wi * W;
                        const longlong2 tb = tr[b], vb = vr[b];
                        const int64_t p0 = tb.x + d.p2p, p1 = tb.y + d.p2p;
                        const int64_t k0 = vb.x - z.cap, k1 = vb.y - z.cap, xw = s_x[wi];
                        const int l = lm[b], bl = blo[(i - 1) * UP + ul + r - wi - 1];
                        a = max(a, bl);
                        if (prune_het && (z.flags & 1)) a = max(a, (int)am[z.am * W + b]);
                        const int step = wi == 2 ? 2 : 1;
                        for (a += q == 3 ? 1 : 0; a <= ahi; a += step) {
                            const int64_t prev = Fp[d.fofs + a];
                            const longlong2 va = vr[a], ta = tr[a];
                            const int64_t ex = a < l ? xw : 0;
                            const bool fit0 = va.x - ex >= k0;
                            const bool fit = fit0 || (recomp && va.y - ex >= k1);
                            const int64_t cst = fit0 ? p0 - ta.x : p1 - ta.y;
                            const int64_t v = prev > cst ? prev : cst;
                            if (STATS && fit && prev < kFar) ++relax;
                            if (fit) {
                                amin = min(amin, a);
                                if (fit0) a0 = min(a0, a);
                                best = v < best ? v : best;
                            }
                        }
                    }
                    {
                        const int64_t v = quad_swap<0xB1>(best);
                        best = v < best ? v : best;
                    }
                    {
                        const int64_t v = quad_swap<0x4E>(best);
                        best = v < best ? v : best;
                    }
                    const int am2 = __builtin_amdgcn_mov_dpp(amin, 0xB1, 0xf, 0xf, true);
                    const int a02 = __builtin_amdgcn_mov_dpp(a0, 0xB1, 0xf, 0xf, true);
                    if (q == 2) {
                        amin = min(amin, am2);
                        a0 = min(a0, a02);
                    }
                    if (q < 3) iv[(ofs + s) * 3 + q] = (uint16_t)(amin | a0 << 8);
                    if (q == 0) Fc[s] = best;
                }
                __syncthreads();
            }
            const int64_t f = F[(PP & 1) * fsz];   // the one state of the last level
            __syncthreads();
            return f;
        };
        // one pass at threshold t: the least stage sum with stages <= t, back-trace pointers
        auto pass = [&](int64_t t) -> int64_t {
            if (tid == 0) F[0] = 0;
            __syncthreads();
            for (int i = 1; i <= PP; ++i) {
                const int64_t *Fp = F + ((i - 1) & 1) * fsz;
                int64_t *Fc = F + (i & 1) * fsz;
                const WLevel lv = lev[i];
                const int ofs = __builtin_amdgcn_readfirstlane(lv.first), items = __builtin_amdgcn_readfirstlane(lv.n) * 4;
                const int dofs = __builtin_amdgcn_readfirstlane(lv.rows);
                for (int e = tid; e < items; e += kDpThreads) {
                    const int q = e & 3, s = e >> 2, wi = q == 3 ? 2 : q;
                    const int x = list[ofs + s], f = iv[(ofs + s) * 3 + wi];
                    const int b = x & 127, r = x >> 7;
                    const WDesc d = desc[(dofs + r) * 3 + wi];
                    int64_t best = kFar;
                    int bk = 0xffff;
                    int a = (f & 255) + (q == 3 ? 1 : 0);
                    const int a0 = f >> 8, ahi = min(b - (int)d.lo, (int)d.last);
                    if (a <= ahi) {
                        const longlong2 *tr = tim + d.row;
                        const longlong2 tb = tr[b];
                        const int64_t p0 = tb.x + d.p2p, p1 = tb.y + d.p2p;
                        const int64_t *fr = Fp + d.fofs;
                        const int step = wi == 2 ? 2 : 1;
                        for (; a <= ahi; a += step) {
                            const bool rc = a < a0;
                            const int64_t prev = fr[a];
                            const int64_t ta = reinterpret_cast<const int64_t *>(tr + a)[rc ? 1 : 0];
                            const int64_t cst = (rc ? p1 : p0) - ta;
                            const int64_t v = prev + cst;
                            if (STATS && prev < kFar && cst <= t) ++relax;
                            if (cst <= t && v < best) {
                                best = v;
                                bk = (a << 3) | (rc ? 1 : 0);
                            }
                        }
                        bk |= (wi + 1) << 1;
                    }
                    // the quad's best; ties to the smallest split point, then the smallest width
                    {
                        const int64_t v = quad_swap<0xB1>(best);
                        const int vk = __builtin_amdgcn_mov_dpp(bk, 0xB1, 0xf, 0xf, true);
                        if (v < best || (v == best && vk < bk)) { best = v; bk = vk; }
                    }
                    {
                        const int64_t v = quad_swap<0x4E>(best);
                        const int vk = __builtin_amdgcn_mov_dpp(bk, 0x4E, 0xf, 0xf, true);
                        if (v < best || (v == best && vk < bk)) { best = v; bk = vk; }
                    }
                    if (q == 0) {
                        Fc[s] = best;
                        arg[ofs + s] = (uint16_t)bk;
                    }
                }
                __syncthreads();
            }
            const int64_t f = F[(PP & 1) * fsz];
            __syncthreads();
            return f;
        };
        // wave 0: the pass's path, stage i in lane i; its largest stage
        int p_len = 0, p_w = 0, p_mask = 0;
        uint32_t p_rm = 0;
        auto trace = [&]() -> int64_t {
            int b = N, u = U, ma = 0, mb = 0, mu0 = 0, mrf = 0;
            for (int i = PP; i >= 1; --i) {
                const int x = arg[lev[i].first + rs[i * UP + u] + b - blo[i * UP + u]];
                const int a = x >> 3, w = (x >> 1) & 3;
                if (lane == i - 1) {
                    ma = a;
                    mb = b;
                    mu0 = u - w;
                    p_w = w;
                    mrf = x & 1;
                }
                b = a;
                u -= w;
            }
            int64_t cst = 0;
            if (lane < PP) {
                const WStage &x = st[mu0 * 3 + p_w - 1];
                const longlong2 tb = tim[x.row + mb], ta = tim[x.row + ma];
                cst = (mrf ? tb.y - ta.y : tb.x - ta.x) + x.p2p;
                p_len = mb - ma;
                p_mask = x.mask;
            }
            p_rm = (uint32_t)__ballot(mrf);
            return wave_max(cst);
        };

        // ---- one sweep per group of the key's candidates with equal min(B, PP) (their
        // stored micro-batch counts, hence every DP pass, are the same); lane j of wave 0
        // keeps the incumbent of candidate j, replaced by a lower sum + (B-1) max or an
        // equal one with a lower max.  The sweep starts at the least possible largest
        // stage, whose objective bounds the thresholds that can still win from above. ----
        const int64_t Bj = lane < nB ? H.micro[lane] : 0;
        const int vj = Bj < PP ? (int)Bj : PP;
        const int64_t idx = key * nB + lane;
        const bool mine = lane < nB && idx >= first && idx < first + count;
        for (int v_prev = 0;;) {
            int v = 1 << 30;   // the next value of min(B, PP) among candidates in range
            for (int j = 0; j < nB; ++j) {
                const int x = H.micro[j] < PP ? H.micro[j] : PP;
                const int64_t at = key * nB + j;
                if (x > v_prev && x < v && at >= first && at < first + count) v = x;
            }
            if (v == 1 << 30) break;
            v_prev = v;
            B = v;
            const bool member = lead && mine && vj == v;
            hapmoe_dp_result *const out = res + (idx - first);
            int64_t best = kInf, bestM = kInf, bestF = kInf;
            uint32_t brm = 0;
            int passes = 0;
            if (STATS) relax = 0;
            // wave 0 takes a pass's path (sum f) and returns the largest threshold a member still needs
            auto take = [&](int64_t f) -> int64_t {
                const int64_t mx = trace();
                const int64_t obj = f + (Bj - 1) * mx;
                const bool better = member && (obj < best || (obj == best && mx < bestM));
                if (better) {
                    best = obj;
                    bestM = mx;
                    bestF = f;
                    brm = p_rm;
                }
                for (uint64_t m = __ballot(better); m; m &= m - 1) {
                    const int64_t r = key * nB + __ffsll((unsigned long long)m) - 1 - first;
                    if (lane < kMaxStages) {
                        const bool on = lane < PP;
                        res[r].layers[lane] = on ? (uint8_t)p_len : 0;
                        types_out[r * kMaxStages + lane] = on ? (uint8_t)p_mask : 0;
                        widths_out[r * kMaxStages + lane] = on ? (uint8_t)p_w : 0;
                    }
                }
                // a lower threshold t' gives a sum >= f: it can win only if
                // f + (B-1) t' <= best (equal objectives go to the lower max)
                int64_t next = -1;
                if (member) {
                    next = mx - 1;
                    if (Bj > 1) {
                        const int64_t lim = floor_div(best - f, Bj - 1);
                        next = lim < next ? lim : next;
                    } else if (f > best) {
                        next = -1;
                    }
                }
                return wave_max(next);
            };
            int64_t t_bot = kFar;
            if (shape_ok) {
                t_bot = first_pass();
                ++passes;
            }
            if (t_bot < kFar) {
                // t_bot first: its incumbents bound the sweep; then from the top down
                for (int64_t t = t_bot;;) {
                    const int64_t f = pass(t);
                    ++passes;
                    if (lead) {
                        const int64_t next = take(f);
                        if (lane == 0) s_t = next;
                    }
                    __syncthreads();
                    const int64_t next = s_t;
                    __syncthreads();
                    if (passes == 2) {
                        t = kInf;
                    } else {
                        if (next <= t_bot) break;
                        t = next;
                    }
                }
            }
            if (STATS) {
                if (relax) atomicAdd(&s_relax, relax);
                __syncthreads();
            }
            if (member) {
                const bool ok = best != kInf;
                out->objective = ok ? best + ki->dp_const : kInf;
                out->stage_sum = bestF;
                out->t_max = bestM;
                out->status = status != HAPMOE_STATUS_OK ? HAPMOE_STATUS_OVERFLOW
                              : ok                        ? HAPMOE_STATUS_OK
                                                          : HAPMOE_STATUS_INFEASIBLE;
                out->recompute_mask = brm;
                if (STATS) {   // the shared sweep's relaxations on its first candidate
                    const uint64_t all = __ballot(member);
                    int32_t *so = stats + 4 * (idx - first);
                    so[0] = status == HAPMOE_STATUS_OK ? passes : 0;
                    so[1] = lane == __ffsll((unsigned long long)all) - 1 ? (int32_t)s_relax : 0;
                    so[2] = so[3] = 0;
                }
            }
            if (lead)
                for (uint64_t m = __ballot(member && best == kInf); m; m &= m - 1) {
                    const int64_t r = key * nB + __ffsll((unsigned long long)m) - 1 - first;
                    if (lane < kMaxStages)
                        res[r].layers[lane] = types_out[r * kMaxStages + lane] = widths_out[r * kMaxStages + lane] = 0;
                }
            if (STATS) {
                __syncthreads();
                if (tid == 0) s_relax = 0;
                __syncthreads();
            }
        }
    }
}

}  // namespace

hipError_t launch_width_tables(const void *d_image, const hapmoe_candidate *d_cand, int64_t per_config,
                               const TablesLayout &L, int64_t cfg_lo, int64_t n_cfg, void *d_tables, hipStream_t s)
{
    if (n_cfg <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_width_tables, dim3((unsigned)n_cfg), dim3(kThreads), 0, s,
                       static_cast<const unsigned char *>(d_image), d_cand, per_config, cfg_lo, L,
                       static_cast<unsigned char *>(d_tables));
    return hipGetLastError();
}

// states of a pipeline of PP stages at most: (level, half-groups used) rows times end layers
int64_t width_rows(int PP)
{
    int64_t rows = 0;
    for (int i = 1; i <= PP; ++i) rows += level_rows(i, PP);
    return rows;
}

// one workgroup's slice of the last tier: descriptors, pruning-3 limits, and a list
// entry, three intervals and a back-trace pointer (two bytes each) a state
int64_t width_dp_slot_bytes(int n_layers, int ppmax)
{
    int64_t most = 0;
    for (int PP = 1; PP <= ppmax && PP <= n_layers; ++PP) {
        const int64_t rows = width_rows(PP), states = rows * (n_layers - PP + 1);
        const int64_t b = rows * 3 * (int64_t)sizeof(WDesc) + states * 10 + 3 * (2 * PP + 1) * (n_layers + 1) + 64;
        most = b > most ? b : most;
    }
    return align256(most);
}

// queue counters, the keys of the last tier (at most one a candidate), its slices
int64_t width_dp_ws_bytes(int n_layers, int ppmax, int64_t n_cand)
{
    const int64_t n = n_cand > 0 ? n_cand : 1;
    const int64_t slots = n < kWidthDpMaxSlots ? n : kWidthDpMaxSlots;
    return 256 + align256(4 * n) + slots * width_dp_slot_bytes(n_layers, ppmax);
}

// LDS a workgroup of tier 1 is given: the regions of k_width_dp for a pipeline of
// ppmax stages, with end-layer bands of the width the windows leave half way,
// narrowing towards both ends, and type sets that are pure or pairs of neighbours
int width_dp_lds_bytes(const hapmoe_problem &p, int ppmax)
{
    const int N = p.model.n_layers, W = N + 1, T = p.cluster.n_types;
    const hapmoe_params &q = p.params;
    int most = 0;
    for (int PP = ppmax; PP >= 1; PP /= 2) {
        const int UP = 2 * PP + 1;
        int wm = N - PP + 1;
        if (q.prune_window == 1) {
            const int x = (int)((int64_t)q.delta_num * N / q.delta_den) + PP / 2 + 2;
            wm = x < wm ? x : wm;
        } else if (q.prune_window == 2) {
            wm = PP / 2 + 1 < wm ? PP / 2 + 1 : wm;
        }
        int states = 0, fsz = 1;
        for (int i = 1; i <= PP; ++i) {
            int w = q.prune_window == 1 ? 3 * (i < PP - i ? i : PP - i) + 1 : wm;
            w = w < wm ? w : wm;
            const int n = level_rows(i, PP) * w;
            states += n;
            fsz = n > fsz ? n : fsz;
        }
        const int head = 3 * UP * (int)sizeof(WStage) + 4 * (PP + 1) * UP + (PP + 1) * (int)sizeof(WLevel) + W + 64;
        const int reach = 4 * (PP + 1) * UP;   // the band search, before the rest is there
        const int val = 6 * W * 16 > 2 * states ? 6 * W * 16 : 2 * states;
        const int rest = (6 * T - 4) * W * 16 + 2 * fsz * 8 + val + 8 * states +
                         (int)width_rows(PP) * 3 * (int)sizeof(WDesc) + 3 * (T - 1) * W;
        const int bytes = head + (rest > reach ? rest : reach);
        most = bytes > most ? bytes : most;
    }
    return most < kWidthLastLds ? (most + 255) & ~255 : kWidthLastLds;
}

__global__ void k_width_reset(uint32_t *q) { q[threadIdx.x] = 0; }

hipError_t launch_width_dp(const hapmoe_problem &p, const void *d_image, const hapmoe_candidate *d_cand, int ppmax,
                           const TablesLayout &L, const void *d_tables, int64_t first, int64_t count,
                           hapmoe_dp_result *d_res, uint8_t *d_types, uint8_t *d_widths, int32_t *d_stats, void *d_ws,
                           hipStream_t s)
{
    if (count == 0) return hipSuccess;
    const int64_t slot = width_dp_slot_bytes(p.model.n_layers, ppmax);
    const int64_t nB = p.space.n_micro, n_keys = (first + count - 1) / nB - first / nB + 1;
    auto *queue = static_cast<uint32_t *>(d_ws);   // tier 1's next key, keys of the last tier, its next key
    auto *spill = reinterpret_cast<uint32_t *>(static_cast<unsigned char *>(d_ws) + 256);
    auto *slots = static_cast<unsigned char *>(d_ws) + 256 + align256(4 * count);
    hipLaunchKernelGGL(k_width_reset, dim3(1), dim3(4), 0, s, queue);
    const auto *img = static_cast<const unsigned char *>(d_image);
    const auto *tab = static_cast<const unsigned char *>(d_tables);
    auto go = [&](auto kern, int lds, int64_t grid) -> hipError_t {
        if (lds > 65536) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kDpThreads), lds, s, img, d_cand, L, tab, first, count,
                           lds, slots, slot, d_res, d_types, d_widths, d_stats, queue, spill);
        return hipGetLastError();
    };
    const int lds = width_dp_lds_bytes(p, ppmax);
    int per_cu = 160 * 1024 / (lds + 1024);   // 4 workgroups of 8 waves fill a CU
    per_cu = per_cu < 1 ? 1 : per_cu > 4 ? 4 : per_cu;
    const int64_t g1 = n_keys < 256 * per_cu ? n_keys : 256 * per_cu;
    const int64_t g2 = n_keys < kWidthDpMaxSlots ? n_keys : kWidthDpMaxSlots;
    if (const hipError_t e = d_stats ? go(k_width_dp<true, false>, lds, g1) : go(k_width_dp<false, false>, lds, g1))
        return e;
    return d_stats ? go(k_width_dp<true, true>, kWidthLastLds, g2) : go(k_width_dp<false, true>, kWidthLastLds, g2);
}

}  // namespace hapmoe
