// The iterations of a small LP in one workgroup.  The matrix stays in
// registers, in both orders, y and xbar in LDS, and every thread keeps or
// finds in LDS its columns' and rows' other operands, so an iteration costs
// two workgroup barriers instead of two kernel launches.
//
// A launched half of a 200 x 500 LP takes about 3 us whatever it computes:
// dispatch, then a chain of dependent loads (row pointers, indices, gathered
// vector) from beyond the L2.  Here a half is a chain through LDS, and what
// bounds it is the instructions one CU can issue, which is why the indices
// are premultiplied, the rows padded to one static pattern with groups of
// loads in flight, and why LPs past some ten thousand entries take the
// launched kernels (they would not fit the registers either).  Measured, us
// per iteration with the checks, launched -> resident, float64 / mixed: 200 x
// 500 with 2,500 entries 6.3 -> 1.0 / 6.8 -> 1.1; 400 x 1,000 with 5,000 6.4 ->
// 1.7 / 7.0 -> 2.0; 800 x 2,000 with 10,000 (mixed only) 7.0 -> 3.8 where no row
// passes variant 3's 24 entries (four of ten such LPs; the others are launched);
// transportation 40 x 100 with 8,000 entries 7.0 -> 2.6 / 6.7 -> 3.1.  A step of
// the power iteration 13 us in six launches -> about 1 us.
//
// A launch runs whole cycles, iterations and check: the check's products come
// from the same registers, its sums are formed as the check kernels form them
// (blocks of 256 elements, then the blocks), and the restart is applied in
// place.  The power iteration of the step size runs in one launch likewise.
//
// Every sum is formed in the order of the launched kernels: there G threads
// share a row, thread l adding entries l, l + G, ..., and a tree joins them.
// Here h = G / A threads share it with A <= 4 accumulators each: thread l' adds
// positions l', l' + h, ... into accumulators 0, 1, ... in turn, and joins
// first its own, then the threads', in the tree's order.  The updates are the
// same functions, so a handle may take either path for any part of a phase
// with the same bits.
#include "pdhg_device.hpp"
#include "pdhg_internal.hpp"
#include "pdhg_kernels.hpp"

namespace pdhg {

constexpr int kResThreads = 512;
constexpr int kResTable = 64;       // Halpern weights per refill
constexpr int kResMaxIters = 1024;  // iterations per launch without checks
constexpr int kResColWaves = 64;    // waves of 64 columns, of 64 rows
constexpr int kResRowWaves = 16;
constexpr int kResLds = 160 * 1024; // LDS of a CU

// The dual half's rounds: round q gives rows row0.. to 2^hs threads each.
// A segment of rows starts a round of its own.
constexpr int kResRounds = 2;
struct ResRounds {
    int count;
    int row0[kResRounds], row1[kResRounds], hs[kResRounds];
    int acc[kResRounds];   // accumulators per thread
    int slots[kResRounds]; // entries per thread
};

template <typename V>
struct ResMatrix { // the model's matrix
    int m, n;
    const int *rp, *ci, *tp, *ti;
    const V *av, *atv;
    ResRounds dual;
    int ep; // longest column
};

template <typename V>
struct ResArgs {
    ResMatrix<V> mat;
    double *ch, *bh; // what the iterations read (mixed mode: anchored, rewritten at a restart)
    const V *lh, *uh;
    const int8_t *sense;
    V *x;
    double *xa, *ya, *xp, *y, *yp;
    DevState *st;
    int i0, first, store; // iterations before the launch and in its first cycle; keep the candidate
    // cycles with checks (0: `first` iterations, no check): later cycles of
    // `len` iterations, check mode, and what only a check reads
    int cycles, len, mode, orig;
    const double *chk_ch, *chk_bh, *dr, *dc, *c0, *l0, *u0;
    const float *aerr, *aerr_t;
    double *ety;
};

// Where the columns' operands stay: in registers; all in LDS; or chat, lhat
// and uhat in LDS and x and x_a in registers (where all of them would not fit
// the LDS).
enum ResOps { OPS_REGS, OPS_LDS, OPS_SPLIT };

// The LDS arrays, in this order (n columns, m rows; the gathered ones end in
// a zero that padding entries read).
template <typename V>
struct ResLds {
    double *y, *yp, *ax, *w, *wa, *colp, *rowp, *ch, *xa, *xc;
    DevState *st;
    V *x, *lh, *uh, *xb;
};

template <typename V>
__host__ __device__ __forceinline__ size_t res_carve(char *base, int m, int n, int ops, ResLds<V> &l)
{
    size_t at = 0;
    auto take = [&](size_t bytes) {
        char *q = base + at;
        at += (bytes + 7) / 8 * 8;
        return q;
    };
    const size_t M = (size_t)m, N = (size_t)n, vb = sizeof(V);
    const size_t cd = ops != OPS_REGS ? 8 * N : 0, cv = ops != OPS_REGS ? vb * N : 0;
    l.y = (double *)take(8 * (M + 1));
    l.yp = (double *)take(8 * (M + 1));
    l.ax = (double *)take(8 * M);
    l.w = (double *)take(8 * kResTable);
    l.wa = (double *)take(8 * kResTable);
    l.colp = (double *)take(8 * 7 * kResColWaves);
    l.rowp = (double *)take(8 * 6 * kResRowWaves);
    l.st = (DevState *)take(sizeof(DevState));
    l.ch = (double *)take(cd);
    l.xa = (double *)take(ops == OPS_LDS ? 8 * N : 0);
    l.x = (V *)take(ops == OPS_LDS ? vb * N : 0);
    l.lh = (V *)take(cv);
    l.uh = (V *)take(cv);
    l.xb = (V *)take(vb * (N + 1));
    // the candidate for the check's product: xbar's place in float64 (dead by then)
    l.xc = vb == 8 ? (double *)l.xb : (double *)take(8 * (N + 1));
    return at;
}

static size_t res_lds(int m, int n, bool fp32, int ops)
{
    ResLds<float> f;
    ResLds<double> d;
    return fp32 ? res_carve<float>(nullptr, m, n, ops, f) : res_carve<double>(nullptr, m, n, ops, d);
}

// One thread's share of a row: entries val[0..], gathered at byte offsets
// MUL off[0..] of `vec`, position s into accumulator s % A, in groups of `step`
// whose loads go out together (count: positions in use, uniform; the padding
// past a row's own entries adds 0 x 0).  FUSED: fused multiply-adds, else
// products rounded before they are added.
template <int A, bool FUSED, int step, bool KEEP, int MUL, int N, typename V, typename VX>
__device__ __forceinline__ double res_dot(V (&val)[N], const int (&off)[N], const VX *vec, int count)
{
    const char *base = (const char *)vec;
    double acc[A] = {};
#pragma unroll
    for (int s0 = 0; s0 < N; s0 += step) {
        if (s0 < count) {
            double g[step];
#pragma unroll
            for (int u = 0; u < step; u++) g[u] = (double)*(const VX *)(base + MUL * off[s0 + u]);
#pragma unroll
            for (int u = 0; u < step; u++) {
                if (KEEP) asm("" : "+v"(val[s0 + u]));
                const double v = (double)val[s0 + u];
                if (FUSED) {
                    acc[u % A] = __builtin_fma(v, g[u], acc[u % A]);
                } else {
#pragma clang fp contract(off)
                    const double t = v * g[u];
                    acc[u % A] = acc[u % A] + t;
                }
            }
        }
    }
    if constexpr (A == 4) return (acc[0] + acc[2]) + (acc[1] + acc[3]);
    else if constexpr (A == 2) return acc[0] + acc[1];
    else return acc[0];
}

// The matrix in a thread's registers.  Columns j = tid + p kResThreads, R of
// them with at most EP entries each; row q of the thread's group in round q
// (-1: none, or another thread of the group updates it), at most ED entries
// each.  Offsets in bytes: pa into a vector of doubles, da into one of V;
// padding entries have value 0 and the zero slot's offset.
template <typename V, int EP, int R, int Q, int ED>
struct ResRegs {
    V pv[R][EP], dv[Q][ED];
    int pa[R][EP], da[Q][ED], row[Q];
};

template <typename V, int EP, int R, int Q, int ED>
__device__ __forceinline__ void res_load(ResRegs<V, EP, R, Q, ED> &k, const ResMatrix<V> &a, int tid)
{
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int j = tid + p * kResThreads;
        const int beg = j < a.n ? a.tp[j] : 0, end = j < a.n ? a.tp[j + 1] : 0;
#pragma unroll
        for (int e = 0; e < EP; e++) {
            const bool have = beg + e < end;
            k.pv[p][e] = have ? a.atv[beg + e] : (V)0;
            k.pa[p][e] = 8 * (have ? a.ti[beg + e] : a.m);
        }
    }
#pragma unroll
    for (int q = 0; q < Q; q++) {
        k.row[q] = -1;
        if (q < a.dual.count) {
            const int hs = a.dual.hs[q], h = 1 << hs, sub = tid & (h - 1);
            const int r = a.dual.row0[q] + (tid >> hs);
            const bool mine = r < a.dual.row1[q];
            const int beg = mine ? a.rp[r] : 0, end = mine ? a.rp[r + 1] : 0;
#pragma unroll
            for (int s = 0; s < ED; s++) {
                const int e = beg + sub + h * s;
                const bool have = e < end;
                k.dv[q][s] = have ? a.av[e] : (V)0;
                k.da[q][s] = (int)sizeof(V) * (have ? a.ci[e] : a.n);
            }
            if (mine && sub == 0) k.row[q] = r;
        }
    }
}

// the same values with another matrix of the same pattern (the float matrix's
// rounding error at a check), one column or round at a time
template <typename V, int EP>
__device__ __forceinline__ void res_reload_column(float (&v)[EP], const ResMatrix<V> &a, const float *val, unsigned j)
{
    const unsigned beg = (int)j < a.n ? a.tp[j] : 0, end = (int)j < a.n ? a.tp[j + 1] : 0;
#pragma unroll
    for (int e = 0; e < EP; e++) v[e] = beg + e < end ? val[beg + e] : 0.0f;
}

template <typename V, int ED>
__device__ __forceinline__ void res_reload_round(float (&v)[ED], const ResMatrix<V> &a, const float *val, int q,
                                                 unsigned tid)
{
    const unsigned hs = a.dual.hs[q], h = 1 << hs, sub = tid & (h - 1);
    const unsigned r = a.dual.row0[q] + (tid >> hs);
    const bool mine = (int)r < a.dual.row1[q];
    const unsigned beg = mine ? a.rp[r] : 0, end = mine ? a.rp[r + 1] : 0;
#pragma unroll
    for (int s = 0; s < ED; s++) {
        const unsigned e = beg + sub + h * s;
        v[s] = e < end ? val[e] : 0.0f;
    }
}

// round q's row sums with vec (byte offsets MUL da), in the group's first thread
template <bool FMA, bool KEEP, int MUL, int ED, typename V, typename W, typename VX>
__device__ __forceinline__ double res_round(V (&dv)[ED], const int (&da)[ED], const ResMatrix<W> &a, int q, const VX *vec)
{
    const int cnt = a.dual.slots[q], hs = a.dual.hs[q];
    double h;
    if (a.dual.acc[q] == 4) h = res_dot<4, FMA, 8, KEEP, MUL>(dv, da, vec, cnt);
    else if (a.dual.acc[q] == 2) h = res_dot<2, FMA, 8, KEEP, MUL>(dv, da, vec, cnt);
    else h = res_dot<1, FMA, 8, KEEP, MUL>(dv, da, vec, cnt);
    if (hs > 3) h += lane_up<8>(h);
    if (hs > 2) h += lane_up<4>(h);
    if (hs > 1) h += lane_up<2>(h);
    if (hs > 0) h += lane_up<1>(h);
    return h;
}

// does round q hold a row for the wave of threads wave0.. (uniform)
template <typename V>
__device__ __forceinline__ bool res_wave_in(const ResMatrix<V> &a, int q, int wave0)
{
    return q < a.dual.count && a.dual.row0[q] + (wave0 >> a.dual.hs[q]) < a.dual.row1[q];
}

// One quantity from its waves' partials, as blocks of 256 elements (4 waves)
// and a finishing workgroup form it: lane b adds block b's waves in order, and
// a tree joins the blocks.  Lane 0 of the calling wave gets it.
__device__ __forceinline__ double res_fold(const double *part, int blocks, bool is_max, int lane)
{
    double v = 0.0;
    if (lane < blocks) {
        const double *w = part + 4 * lane;
        double b = w[0];
        for (int k = 1; k < 4; k++) b = is_max ? fmax(b, w[k]) : b + w[k];
        v = is_max ? fmax(0.0, b) : 0.0 + b;
    }
    return is_max ? wave_max(v) : wave_sum(v);
}

template <int NQ>
__device__ __forceinline__ void res_wave_partials(double (&t)[NQ], unsigned max_mask, double *part, int waves, int wave,
                                                  int lane)
{
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        const double v = (max_mask >> q) & 1u ? wave_max(t[q]) : wave_sum(t[q]);
        if (lane == 0) part[q * waves + wave] = v;
    }
}

// Columns: R per thread, at most EP entries each, A accumulators.  Rows: Q
// rounds of at most ED entries per thread; FMA: the lane groups' fused
// products, else the tiles' rounded ones.
template <typename V, int A, int EP, int R, int Q, int ED, bool FMA, int OPS>
__global__ __launch_bounds__(kResThreads) void k_resident(ResArgs<V> a)
{
    extern __shared__ __align__(16) char res_lds_base[];
    if (a.st->done) return;
    const int tid = threadIdx.x, m = a.mat.m, n = a.mat.n;
    const int wave0 = __builtin_amdgcn_readfirstlane(tid); // the wave's first thread
    constexpr bool delta = sizeof(V) == sizeof(float);
    constexpr int MUL = 8 / sizeof(V); // byte offsets into a vector of doubles
    constexpr int CSTEP = EP < 4 ? EP : 4;
    ResLds<V> l;
    (void)res_carve<V>(res_lds_base, m, n, OPS, l);
    constexpr bool LC = OPS != OPS_REGS, LX = OPS == OPS_LDS; // chat, lhat, uhat; x, x_a in LDS
    constexpr int RC = LC ? 1 : R, RX = LX ? 1 : R;
    // larger variants hold their float entries only as floats: converted once
    // before the loop (what the compiler does by itself) they would spill
    constexpr bool KEEP = delta && R * EP + Q * ED > 48;

    for (int k = tid; k < m; k += kResThreads) l.y[k] = a.y[k];
    if (tid == 0) {
        l.y[m] = l.yp[m] = 0.0; // what the padding entries gather
        l.xb[n] = (V)0;
        l.xc[n] = 0.0;
    }
    for (int k = tid; k < (int)(sizeof(DevState) / 8); k += kResThreads) ((double *)l.st)[k] = ((const double *)a.st)[k];
    ResRegs<V, EP, R, Q, ED> k;
    res_load(k, a.mat, tid);
    V xv[RX], lo[RC], hi[RC];
    double xan[RX], cj[RC];
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int j = tid + p * kResThreads;
        if (j < n) {
            if (LX) {
                l.x[j] = a.x[j];
                l.xa[j] = a.xa[j];
            } else {
                xv[p % RX] = a.x[j];
                xan[p % RX] = a.xa[j];
            }
            if (LC) {
                l.ch[j] = a.ch[j];
                l.lh[j] = a.lh[j];
                l.uh[j] = a.uh[j];
            } else {
                cj[p % RC] = a.ch[j];
                lo[p % RC] = a.lh[j];
                hi[p % RC] = a.uh[j];
            }
        }
    }
    double yan[Q], br[Q];
    int8_t sn[Q];
#pragma unroll
    for (int q = 0; q < Q; q++)
        if (k.row[q] >= 0) {
            yan[q] = a.ya[k.row[q]];
            br[q] = a.bh[k.row[q]];
            sn[q] = a.sense[k.row[q]];
        }
    __syncthreads(); // the state
    for (int cyc = 0; cyc == 0 || cyc < a.cycles; cyc++) {
        const int len = cyc == 0 ? a.first : a.len;
        StepScalars sc = step_scalars(l.st, 0);
        for (int i = 0; i < len; i++) {
            // Halpern weights of the next iterations, one pair of divisions per
            // thread (everyone read the last ones two barriers ago)
            if (i % kResTable == 0 && tid < kResTable) {
                const StepScalars q = step_scalars(l.st, a.i0 + i + tid);
                l.w[tid] = q.w;
                l.wa[tid] = q.wa;
            }
            const bool store = a.store && i == len - 1;
            __syncthreads(); // y in place
            sc.w = l.w[i % kResTable];
            sc.wa = l.wa[i % kResTable];
#pragma unroll
            for (int p = 0; p < R; p++) {
                if (p * kResThreads + wave0 < n) { // uniform over the wave
                    const double g = res_dot<A, false, CSTEP, KEEP, 1>(k.pv[p], k.pa[p], l.y, a.mat.ep);
                    const int j = tid + p * kResThreads;
                    if (j < n) {
                        const double aj = LX ? l.xa[j] : xan[p % RX];
                        const V xs = LX ? l.x[j] : xv[p % RX];
                        const PrimalStep<V> u = primal_step<V>(
                            g, iterate_value<V>(xs, aj), LC ? l.ch[j] : cj[p % RC],
                            (double)(LC ? l.lh[j] : lo[p % RC]), (double)(LC ? l.uh[j] : hi[p % RC]), aj, sc);
                        l.xb[j] = u.xbar;
                        if (LX) l.x[j] = u.x;
                        else xv[p % RX] = u.x;
                        if (store) a.xp[(unsigned)j] = u.cand;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < Q; q++) {
                if (res_wave_in(a.mat, q, wave0)) {
                    const double h = res_round<FMA, KEEP, 1>(k.dv[q], k.da[q], a.mat, q, l.xb);
                    const int r = k.row[q];
                    if (r >= 0) {
                        double cand;
                        l.y[r] = dual_step(h, l.y[r], br[q], yan[q], sn[q], sc, cand);
                        if (store) {
                            a.yp[(unsigned)r] = cand;
                            l.yp[r] = cand;
                        }
                    }
                }
            }
        }
        if (a.cycles == 0) break;
        // ---- the check of the candidate (xp, yp); its thread number is opaque, so
        // that no address of the check stays in registers over the iterations
        unsigned ct = tid;
        asm volatile("" : "+v"(ct));
        __syncthreads(); // xbar read, yp complete
#pragma unroll
        for (int p = 0; p < R; p++) {
            const unsigned j = ct + p * kResThreads;
            if ((int)j < n) l.xc[j] = a.xp[j]; // this thread's own store
        }
        if (!delta && tid == 0) l.xc[n] = 0.0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (res_wave_in(a.mat, q, wave0)) {
                double h = res_round<FMA, KEEP, MUL>(k.dv[q], k.da[q], a.mat, q, l.xc);
                if (delta && a.aerr) {
                    float ev[ED];
                    res_reload_round<V, ED>(ev, a.mat, a.aerr, q, ct);
                    h += res_round<FMA, false, MUL>(ev, k.da[q], a.mat, q, l.xc);
                }
                if (k.row[q] >= 0) l.ax[k.row[q]] = h;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int wave = ct >> 6, lane = ct & 63;
        const int bn = (n + kBlock - 1) / kBlock, bm = (m + kBlock - 1) / kBlock;
#pragma unroll
        for (int p = 0; p < R; p++) {
            const unsigned j = ct + p * kResThreads;
            if (p * kResThreads + wave0 < bn * kBlock) { // every wave of the columns' blocks (uniform)
                double g = res_dot<A, false, CSTEP, KEEP, 1>(k.pv[p], k.pa[p], l.yp, a.mat.ep);
                if (delta && a.aerr) {
                    float ev[EP];
                    res_reload_column<V, EP>(ev, a.mat, a.aerr_t, j);
                    const double e = res_dot<A, false, CSTEP, false, 1>(ev, k.pa[p], l.yp, a.mat.ep);
                    g += e;
                    if ((int)j < n) a.ety[j] = e;
                }
                double t[7] = {0, 0, 0, 0, 0, 0, 0}; // DH2, D2, DINF, CTX, BND, DX2, NAN
                if ((int)j < n) {
                    double c, lj, uj;
                    check_model<V>(a.orig != 0, j, a.chk_ch, a.lh, a.uh, a.c0, a.l0, a.u0, a.dc, c, lj, uj);
                    const double lam = c - g;
                    const double zp = (!is_inf_lo(lj) && lam > 0.0) ? lam : 0.0;
                    const double zm = (!is_inf_up(uj) && lam < 0.0) ? -lam : 0.0;
                    const double rd = lam - (zp - zm);
                    const double rdu = rd / a.dc[j];
                    const double xj = l.xc[j];
                    const double dx = xj - (LX ? l.xa[j] : xan[p % RX]);
                    t[0] = rd * rd;
                    t[1] = rdu * rdu;
                    t[2] = fabs(rdu);
                    t[3] = c * xj;
                    if (zp > 0.0) t[4] = lj * zp;
                    if (zm > 0.0) t[4] = -(uj * zm);
                    t[5] = dx * dx;
                    t[6] = isfinite(xj) ? 0.0 : 1.0;
                }
                res_wave_partials(t, 1u << 2, l.colp, kResColWaves, p * (kResThreads / 64) + wave, lane);
            }
            __builtin_amdgcn_sched_barrier(0); // one column's loads at a time: the registers hold the matrix
        }
        __syncthreads(); // ax complete
#pragma unroll
        for (int p = 0; p < kResRounds; p++) {
            const unsigned r = ct + p * kResThreads;
            if (p * kResThreads + wave0 < bm * kBlock) {
                double t[6] = {0, 0, 0, 0, 0, 0}; // PH2, P2, PINF, BTY, DY2, NAN
                if ((int)r < m) {
                    const double b = a.chk_bh[r];
                    double d = b - l.ax[r];
                    const int8_t s = a.sense[r];
                    if (s == '<') d = d < 0.0 ? d : 0.0;
                    else if (s == '>') d = d > 0.0 ? d : 0.0;
                    else if (s == 'N') d = 0.0; // dropped by the dual push
                    const double ru = d / a.dr[r];
                    const double yi = l.yp[r];
                    const double dy = yi - a.ya[r];
                    t[0] = d * d;
                    t[1] = ru * ru;
                    t[2] = fabs(ru);
                    t[3] = b * yi;
                    t[4] = dy * dy;
                    t[5] = isfinite(yi) ? 0.0 : 1.0;
                }
                res_wave_partials(t, 1u << 2, l.rowp, kResRowWaves, p * (kResThreads / 64) + wave, lane);
            }
        }
        __syncthreads();
        if (wave == 0) {
            double v[Q_COUNT + 1];
            const int rq[6] = {Q_PH2, Q_P2, Q_PINF, Q_BTY, Q_DY2, Q_NAN};
            const int cq[7] = {Q_DH2, Q_D2, Q_DINF, Q_CTX, Q_BND, Q_DX2, Q_COUNT};
#pragma unroll
            for (int q = 0; q < 6; q++) v[rq[q]] = res_fold(l.rowp + q * kResRowWaves, bm, q == 2, lane);
#pragma unroll
            for (int q = 0; q < 7; q++) v[cq[q]] = res_fold(l.colp + q * kResColWaves, bn, q == 2, lane);
            if (lane == 0) check_decide(l.st, v, a.mode, len);
        }
        __syncthreads();
        if (l.st->done) break;
        if (l.st->restart_flag) { // x = x_a = x+, y = y_a = y+, and in the mixed mode the anchored data
#pragma unroll
            for (int p = 0; p < R; p++) {
                const unsigned j = ct + p * kResThreads;
                if ((int)j < n) {
                    const double v = l.xc[j];
                    a.xa[j] = v;
                    if (LX) {
                        l.x[j] = delta ? (V)0 : (V)v;
                        l.xa[j] = v;
                    } else {
                        xv[p % RX] = delta ? (V)0 : (V)v;
                        xan[p % RX] = v;
                    }
                    if (delta && a.aerr) {
                        const double c = a.chk_ch[j] - a.ety[j]; // this thread's own store
                        a.ch[j] = c;
                        if (LC) l.ch[j] = c;
                        else cj[p % RC] = c;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < Q; q++) {
                const int r = k.row[q];
                if (r >= 0) {
                    const double v = l.yp[r];
                    l.y[r] = v;
                    a.ya[r] = v;
                    yan[q] = v;
                    if (delta && a.aerr) {
                        br[q] = a.chk_bh[r] - l.ax[r];
                        a.bh[r] = br[q];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int j = tid + p * kResThreads;
        if (j < n) a.x[j] = LX ? l.x[j] : xv[p % RX];
    }
#pragma unroll
    for (int q = 0; q < Q; q++)
        if (k.row[q] >= 0) a.y[k.row[q]] = l.y[k.row[q]];
    if (a.cycles > 0)
        for (int q = tid; q < (int)(sizeof(DevState) / 8); q += kResThreads) ((double *)a.st)[q] = ((const double *)l.st)[q];
}

// The power iteration on Ahat'Ahat (pdhg_setup.hip) in one launch: at most
// `steps` steps from v = (1 + U) / ||1 + U||; pw = {lambda, done, steps, ||1 + U||}.
template <typename V, int A, int EP, int R, int Q, int ED, bool FMA>
__global__ __launch_bounds__(kResThreads) void k_resident_power(ResMatrix<V> a, int steps, double tol,
                                                               double *__restrict__ pw)
{
    extern __shared__ __align__(16) char res_lds_base[];
    const int tid = threadIdx.x, m = a.m, n = a.n, wave = tid >> 6, lane = tid & 63;
    const int wave0 = __builtin_amdgcn_readfirstlane(tid);
    constexpr int MUL = 8 / sizeof(V);
    constexpr int CSTEP = EP < 4 ? EP : 4;
    constexpr bool KEEP = sizeof(V) == sizeof(float) && R * EP + Q * ED > 48;
    double *s_u = (double *)res_lds_base, *s_v = s_u + m + 1, *s_cp = s_v + n + 1, *s_rp = s_cp + kResColWaves,
           *s_r = s_rp + kResRowWaves; // two folded sums
    const int bn = (n + kBlock - 1) / kBlock, bm = (m + kBlock - 1) / kBlock;
    ResRegs<V, EP, R, Q, ED> k;
    res_load(k, a, tid);
    if (tid == 0) {
        s_u[m] = 0.0;
        s_v[n] = 0.0;
    }
    // part[wave] of the squares of one value per column
    auto column_squares = [&](const double (&v)[R]) {
#pragma unroll
        for (int p = 0; p < R; p++)
            if (p * kResThreads + wave0 < bn * kBlock) {
                double t[1] = {tid + p * kResThreads < n ? v[p] * v[p] : 0.0};
                res_wave_partials(t, 0u, s_cp, kResColWaves, p * (kResThreads / 64) + wave, lane);
            }
    };
    double w[R];
#pragma unroll
    for (int p = 0; p < R; p++) w[p] = power_start(tid + p * kResThreads);
    column_squares(w);
    __syncthreads();
    if (wave == 0) {
        const double s = res_fold(s_cp, bn, false, lane);
        if (lane == 0) s_r[0] = sqrt(s);
    }
    __syncthreads();
    const double norm = s_r[0];
    double lam = 0.0, taken = 0.0;
    bool done = false;
#pragma unroll
    for (int p = 0; p < R; p++)
        if (tid + p * kResThreads < n) s_v[tid + p * kResThreads] = w[p] / norm;
    for (int it = 0; it < steps && !done; it++) {
        __syncthreads(); // v in place, the sums read
#pragma unroll
        for (int q = 0; q < Q; q++)
            if (res_wave_in(a, q, wave0)) {
                const double h = res_round<FMA, KEEP, MUL>(k.dv[q], k.da[q], a, q, s_v);
                if (k.row[q] >= 0) s_u[k.row[q]] = h;
            }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < R; p++)
            if (p * kResThreads + wave0 < n) w[p] = res_dot<A, false, CSTEP, KEEP, 1>(k.pv[p], k.pa[p], s_u, a.ep);
        column_squares(w);
#pragma unroll
        for (int p = 0; p < kResRounds; p++)
            if (p * kResThreads + wave0 < bm * kBlock) {
                const int r = tid + p * kResThreads;
                const double u = r < m ? s_u[r] : 0.0;
                double t[1] = {u * u};
                res_wave_partials(t, 0u, s_rp, kResRowWaves, p * (kResThreads / 64) + wave, lane);
            }
        __syncthreads();
        if (wave < 2) {
            const double s = wave == 0 ? res_fold(s_rp, bm, false, lane) : res_fold(s_cp, bn, false, lane);
            if (lane == 0) s_r[wave] = s;
        }
        __syncthreads();
        const double rho = s_r[0], ww = s_r[1];
        lam = sqrt(ww);
        taken += 1.0;
        done = power_stops(rho, ww, lam, tol);
        if (!done) {
#pragma unroll
            for (int p = 0; p < R; p++)
                if (tid + p * kResThreads < n) s_v[tid + p * kResThreads] = w[p] / lam;
        }
    }
    if (tid == 0) {
        pw[0] = lam;
        pw[1] = done ? 1.0 : 0.0;
        pw[2] = taken;
        pw[3] = norm;
    }
}

// ------------------------------------------------------------------- plan ---
// out[k] = longest row of segment k
__global__ __launch_bounds__(kBlock) void k_longest(RowSegs sg, const int *__restrict__ rp, int *__restrict__ out)
{
    const int k = blockIdx.x;
    double v[1] = {0.0};
    for (int r = sg.row0[k] + threadIdx.x; r < sg.row0[k + 1]; r += kBlock) v[0] = fmax(v[0], (double)(rp[r + 1] - rp[r]));
    block_reduce<1>(v, 1u);
    if (threadIdx.x == 0) out[k] = (int)v[0];
}

// The kernel variants, smallest first: A, EP, R, Q, ED, OPS, and the precision
// (4 or 8 bytes per entry; 0: both).
#define PDHG_RES_VARIANTS(X) \
    X(4, 8, 1, 1, 32, OPS_REGS, 0) \
    X(4, 8, 4, 1, 32, OPS_LDS, 0) \
    X(4, 8, 4, 2, 24, OPS_LDS, 4) \
    X(1, 4, 2, 1, 32, OPS_REGS, 0) \
    X(1, 2, 8, 2, 16, OPS_SPLIT, 0)

// Rules: the library's own kernel choice (a caller who named kernels with
// lanes_* or autotune gets those); columns in tiles of 64 rows of at most 8
// entries or of 256 rows of at most 4 (whose tiles then never pass one chunk
// of entries, so the order is that of one chunk); rows in tiles of 256, 64 or
// 32 rows, of at most one chunk of 2,048 entries, or in lane groups; and a
// variant that holds the LP.  So one column of more than 8 entries, or a row past
// a variant's entries a thread, sends an LP to the launched kernels.
hipError_t resident_plan(pdhg_solver *s)
{
    s->res = pdhg_solver::Resident{};
    const pdhg_params &p = s->p;
    if (!s->lone || s->m <= 0 || s->n <= 0 || s->nnz <= 0 || s->m > kResRounds * kResThreads || s->n > 8 * kResThreads ||
        s->nnz > kResMaxNnz || p.lanes_at || p.lanes_a || p.autotune)
        return hipSuccess;
    const int A = s->kern_at == -64 ? 4 : s->kern_at == -256 ? 1 : 0;
    const bool segs = s->kern_a == kRowSegs;
    if (A == 0 || !(segs || s->kern_a == -64 || s->kern_a == -32 || s->kern_a == -256)) return hipSuccess;
    RowSegs sg = s->segs;
    if (!segs) {
        sg = RowSegs{};
        sg.count = 1;
        sg.row0[1] = s->m;
        sg.lanes[0] = 256 / -s->kern_a; // threads per row of the tiles
    }
    ResRounds rd{};
    for (int k = 0; k < sg.count; k++) {
        const int acc = sg.lanes[k] < 4 ? sg.lanes[k] : 4, hs = __builtin_ctz((unsigned)(sg.lanes[k] / acc));
        const int per = kResThreads >> hs;
        for (int r = sg.row0[k]; r < sg.row0[k + 1]; r += per) {
            if (rd.count == kResRounds) return hipSuccess;
            const int q = rd.count++;
            rd.row0[q] = r;
            rd.row1[q] = r + per < sg.row0[k + 1] ? r + per : sg.row0[k + 1];
            rd.hs[q] = hs;
            rd.acc[q] = acc;
            rd.slots[q] = k; // the segment, until its longest row is known
        }
    }
    int longest[1 + kMaxSegs] = {s->longest_col, s->longest_row};
    if (segs) { // per segment
        int *out = (int *)s->redout; // small scratch of the handle, free outside a check
        hipLaunchKernelGGL(k_longest, dim3(sg.count), dim3(kBlock), 0, s->stream, sg, s->rp, out);
        hipError_t e = hipMemcpyAsync(longest + 1, out, sizeof(int) * (size_t)sg.count, hipMemcpyDeviceToHost, s->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
        if (e != hipSuccess) return e;
    }
    int slots = 0;
    for (int q = 0; q < rd.count; q++) {
        rd.slots[q] = (longest[1 + rd.slots[q]] + (1 << rd.hs[q]) - 1) >> rd.hs[q];
        slots = rd.slots[q] > slots ? rd.slots[q] : slots;
    }
    if (!segs && -s->kern_a * longest[1] > kTileU * 256) return hipSuccess;
    const int cols = (s->n + kResThreads - 1) / kResThreads;
    int which = 0, k = 0;
#define PDHG_RES_FITS(AA, EEP, RR, QQ, EED, OOPS, VB)                                                              \
    k++;                                                                                                            \
    if (!which && A == AA && longest[0] <= EEP && cols <= RR && rd.count <= QQ && slots <= EED && (!VB || s->fp32 == (VB == 4)) && \
        res_lds(s->m, s->n, s->fp32, OOPS) <= kResLds)                                                       \
        which = k;
    PDHG_RES_VARIANTS(PDHG_RES_FITS)
#undef PDHG_RES_FITS
    s->res.variant = which;
    s->res.fma = segs;
    s->res.ep = longest[0];
    s->res.rounds = rd.count;
    for (int q = 0; q < rd.count; q++) {
        s->res.row0[q] = rd.row0[q];
        s->res.row1[q] = rd.row1[q];
        s->res.hs[q] = rd.hs[q];
        s->res.acc[q] = rd.acc[q];
        s->res.slots[q] = rd.slots[q];
    }
    return hipSuccess;
}

template <typename K>
static hipError_t res_allow_lds(K *kernel)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kResLds);
}

// one launch of the plan's variant: the cycle kernel on `a`, or with `pw` the power iteration
template <typename V, int A, int EP, int R, int Q, int ED, bool FMA, int OPS>
static hipError_t res_launch(pdhg_solver *s, const ResArgs<V> &a, double *pw)
{
    hipError_t e;
    if (pw) {
        auto *kernel = &k_resident_power<V, A, EP, R, Q, ED, FMA>;
        const size_t lds = sizeof(double) * ((size_t)a.mat.m + a.mat.n + 4 + kResColWaves + kResRowWaves);
        if ((e = res_allow_lds(kernel)) != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kResThreads), lds, s->stream, a.mat, s->p.power_iters, s->p.power_tol, pw);
    } else {
        auto *kernel = &k_resident<V, A, EP, R, Q, ED, FMA, OPS>;
        if ((e = res_allow_lds(kernel)) != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kResThreads), res_lds(a.mat.m, a.mat.n, s->fp32, OPS), s->stream, a);
    }
    return hipGetLastError();
}

template <typename V>
static hipError_t res_dispatch(pdhg_solver *s, const ResArgs<V> &a, double *pw)
{
    int k = 0;
    hipError_t e = hipErrorInvalidValue;
#define PDHG_RES_LAUNCH(AA, EEP, RR, QQ, EED, OOPS, VB)                                              \
    k++;                                                                                             \
    if constexpr (!VB || sizeof(V) == VB) {                                                          \
        if (s->res.variant == k)                                                                     \
            e = s->res.fma ? res_launch<V, AA, EEP, RR, QQ, EED, true, OOPS>(s, a, pw)               \
                           : res_launch<V, AA, EEP, RR, QQ, EED, false, OOPS>(s, a, pw);             \
    }
    PDHG_RES_VARIANTS(PDHG_RES_LAUNCH)
#undef PDHG_RES_LAUNCH
    return e;
}

template <typename V>
static ResArgs<V> res_args(pdhg_solver *s)
{
    ResArgs<V> a{};
    a.mat.m = s->m;
    a.mat.n = s->n;
    a.mat.rp = s->rp;
    a.mat.ci = s->ci;
    a.mat.tp = s->tp;
    a.mat.ti = s->ti;
    a.mat.av = (const V *)s->ahat;
    a.mat.atv = (const V *)s->ahat_t;
    a.mat.ep = s->res.ep;
    a.mat.dual.count = s->res.rounds;
    for (int q = 0; q < s->res.rounds; q++) {
        a.mat.dual.row0[q] = s->res.row0[q];
        a.mat.dual.row1[q] = s->res.row1[q];
        a.mat.dual.hs[q] = s->res.hs[q];
        a.mat.dual.acc[q] = s->res.acc[q];
        a.mat.dual.slots[q] = s->res.slots[q];
    }
    a.ch = s->chc;
    a.bh = s->bhc;
    a.lh = (const V *)s->lh;
    a.uh = (const V *)s->uh;
    a.sense = s->sense;
    a.x = (V *)s->x;
    a.xa = (double *)s->xa;
    a.ya = (double *)s->ya;
    a.xp = (double *)s->xp;
    a.y = (double *)s->y;
    a.yp = (double *)s->yp;
    a.st = s->st;
    a.orig = s->model_original ? 1 : 0;
    a.chk_ch = s->ch;
    a.chk_bh = (const double *)s->bh;
    a.dr = s->dr;
    a.dc = s->dc;
    a.c0 = s->c;
    a.l0 = s->l;
    a.u0 = s->u;
    a.aerr = (const float *)s->aerr;
    a.aerr_t = (const float *)s->aerr_t;
    a.ety = s->ety;
    return a;
}

template <typename V>
static hipError_t res_iterations(pdhg_solver *s, int count, bool store)
{
    ResArgs<V> a = res_args<V>(s);
    hipError_t e = hipSuccess;
    for (int i0 = 0; i0 < count && e == hipSuccess; i0 += kResMaxIters) {
        a.i0 = i0;
        a.first = count - i0 < kResMaxIters ? count - i0 : kResMaxIters;
        a.store = store && i0 + a.first == count;
        e = res_dispatch<V>(s, a, nullptr);
    }
    return e;
}

hipError_t resident_iterations(pdhg_solver *s, int count, bool store)
{
    return s->fp32 ? res_iterations<float>(s, count, store) : res_iterations<double>(s, count, store);
}

// The restart history and the undo of learned fixes belong to the launched check.
int resident_cycles_max(const pdhg_solver *s, int mode, int first)
{
    if (s->res.variant == 0 || (mode == 1 && s->hx) || (mode == 2 && s->learned_active)) return 0;
    const int K = s->p.check_every;
    if (first > kResMaxIters || K > kResMaxIters) return 0;
    return 1 + (kResMaxIters - first) / K;
}

template <typename V>
static hipError_t res_cycles(pdhg_solver *s, int first, int cycles, int mode)
{
    ResArgs<V> a = res_args<V>(s);
    a.first = first;
    a.store = 1;
    a.cycles = cycles;
    a.len = s->p.check_every;
    a.mode = mode;
    return res_dispatch<V>(s, a, nullptr);
}

hipError_t resident_cycles(pdhg_solver *s, int first, int cycles, int mode)
{
    return s->fp32 ? res_cycles<float>(s, first, cycles, mode) : res_cycles<double>(s, first, cycles, mode);
}

hipError_t resident_power(pdhg_solver *s, double *pw)
{
    return s->fp32 ? res_dispatch<float>(s, res_args<float>(s), pw) : res_dispatch<double>(s, res_args<double>(s), pw);
}

} // namespace pdhg
