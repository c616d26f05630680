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
// 500 with 2,500 entries 6.3 -> 1.4 / 6.9 -> 1.5; 400 x 1,000 with 5,000 6.4 ->
// 1.9 / 7.0 -> 2.1; 800 x 2,000 with 10,000 (mixed only) 7.0 -> 3.7;
// transportation 40 x 100 with 8,000 entries 7.1 -> 2.7 / 6.7 -> 3.3.
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
constexpr int kResMaxIters = 1024;  // iterations per launch
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
struct ResArgs {
    int m, n;
    const int *rp, *ci, *tp, *ti;
    const V *av, *atv;
    const double *ch, *bh;
    const V *lh, *uh;
    const int8_t *sense;
    V *x;
    const double *xa, *ya;
    double *xp, *y, *yp;
    const DevState *st;
    ResRounds dual;
    int ep; // longest column
    int i0, len, store;
};

// Where the columns' operands stay: in registers; all in LDS; or chat, lhat
// and uhat in LDS and x and x_a in registers (float64, where all of them
// would not fit the LDS).
enum ResOps { OPS_REGS, OPS_LDS, OPS_SPLIT };

// LDS: y (m) and a zero, Halpern weights, xbar (n) and a zero, and the
// columns' operands that stay there (n each)
static size_t res_lds(int m, int n, size_t vb, int ops)
{
    const size_t M = (size_t)m, N = (size_t)n;
    return 8 * (M + 1) + 16 * kResTable + vb * (N + 1) + 16 +
           (ops == OPS_LDS ? 16 * N + 3 * vb * N : ops == OPS_SPLIT ? 8 * N + 2 * vb * N : 0);
}

// One thread's share of a row: entries val[0..], gathered at byte offsets
// off[0..] of `vec`, position s into accumulator s % A, in groups of `step`
// whose loads go out together (count: positions in use, uniform; the padding
// past a row's own entries adds 0 x 0).  FUSED: fused multiply-adds, else
// products rounded before they are added.
template <int A, bool FUSED, int step, int N, bool KEEP, typename V, typename VX>
__device__ __forceinline__ double res_dot(V (&val)[N], const int (&off)[N], const VX *vec, int count)
{
    const char *base = (const char *)vec;
    double acc[A] = {};
#pragma unroll
    for (int s0 = 0; s0 < N; s0 += step) {
        if (s0 < count) {
            double g[step];
#pragma unroll
            for (int u = 0; u < step; u++) g[u] = (double)*(const VX *)(base + off[s0 + u]);
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

// Columns: R per thread, at most EP entries each, A accumulators.  Rows: Q
// rounds of at most ED entries per thread; FMA: the lane
// groups' fused products, else the tiles' rounded ones.
template <typename V, int A, int EP, int R, int Q, int ED, bool FMA, int OPS>
__global__ __launch_bounds__(kResThreads) void k_resident(ResArgs<V> a)
{
    extern __shared__ __align__(16) char res_lds_base[];
    const DevState *st = a.st;
    if (st->done) return;
    const int tid = threadIdx.x, m = a.m, n = a.n;
    double *s_y = (double *)res_lds_base;
    double *s_w = s_y + m + 1, *s_wa = s_w + kResTable;
    constexpr bool LC = OPS != OPS_REGS, LX = OPS == OPS_LDS; // chat, lhat, uhat; x, x_a in LDS
    double *s_ch = s_wa + kResTable, *s_xa = s_ch + (LC ? n : 0);
    V *s_x = (V *)(s_xa + (LX ? n : 0)), *s_lh = s_x + (LX ? n : 0), *s_uh = s_lh + (LC ? n : 0);
    V *s_xb = s_uh + (LC ? n : 0);
    const int wave0 = __builtin_amdgcn_readfirstlane(tid); // the wave's first thread

    for (int k = tid; k < m; k += kResThreads) s_y[k] = a.y[k];
    if (tid == 0) {
        s_y[m] = 0.0; // what the padding entries gather
        s_xb[n] = (V)0;
    }
    // columns j = tid + p kResThreads: entries (padding: value 0, the zero slot) and operands
    V pv[R][EP];
    int pa[R][EP];
    constexpr int RC = LC ? 1 : R, RX = LX ? 1 : R;
    // the largest variants hold their float entries only as floats: converted
    // once before the loop (what the compiler does by itself) they would spill
    constexpr bool KEEP = sizeof(V) == sizeof(float) && 2 * (R * EP + Q * ED) > 128;
    V xv[RX], lo[RC], hi[RC];
    double xan[RX], cj[RC];
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int j = tid + p * kResThreads;
        const int beg = j < n ? a.tp[j] : 0, end = j < n ? a.tp[j + 1] : 0;
#pragma unroll
        for (int e = 0; e < EP; e++) {
            const bool have = beg + e < end;
            pv[p][e] = have ? a.atv[beg + e] : (V)0;
            pa[p][e] = 8 * (have ? a.ti[beg + e] : m);
        }
        if (j < n) {
            if (LX) {
                s_x[j] = a.x[j];
                s_xa[j] = a.xa[j];
            } else {
                xv[p % RX] = a.x[j];
                xan[p % RX] = a.xa[j];
            }
            if (LC) {
                s_ch[j] = a.ch[j];
                s_lh[j] = a.lh[j];
                s_uh[j] = a.uh[j];
            } else {
                cj[p % RC] = a.ch[j];
                lo[p % RC] = a.lh[j];
                hi[p % RC] = a.uh[j];
            }
        }
    }
    // rows: round q's row of this thread's group (-1: none), its entries and operands
    V dv[Q][ED];
    int da[Q][ED], row[Q];
    double yan[Q], br[Q];
    int8_t sn[Q];
#pragma unroll
    for (int q = 0; q < Q; q++) {
        row[q] = -1;
        if (q < a.dual.count) {
            const int hs = a.dual.hs[q], h = 1 << hs, sub = tid & (h - 1);
            const int r = a.dual.row0[q] + (tid >> hs);
            const bool mine = r < a.dual.row1[q];
            const int beg = mine ? a.rp[r] : 0, end = mine ? a.rp[r + 1] : 0;
#pragma unroll
            for (int s = 0; s < ED; s++) {
                const int e = beg + sub + h * s;
                const bool have = e < end;
                dv[q][s] = have ? a.av[e] : (V)0;
                da[q][s] = (int)sizeof(V) * (have ? a.ci[e] : n);
            }
            if (mine && sub == 0) {
                row[q] = r;
                yan[q] = a.ya[r];
                br[q] = a.bh[r];
                sn[q] = a.sense[r];
            }
        }
    }
    StepScalars sc = step_scalars(st, 0);
    for (int i = 0; i < a.len; i++) {
        // Halpern weights of the next iterations, one pair of divisions per
        // thread (everyone read the last ones two barriers ago)
        if (i % kResTable == 0 && tid < kResTable) {
            const StepScalars q = step_scalars(st, a.i0 + i + tid);
            s_w[tid] = q.w;
            s_wa[tid] = q.wa;
        }
        const bool store = a.store && i == a.len - 1;
        __syncthreads(); // y in place
        sc.w = s_w[i % kResTable];
        sc.wa = s_wa[i % kResTable];
#pragma unroll
        for (int p = 0; p < R; p++) {
            if (p * kResThreads + wave0 < n) { // uniform over the wave
                const double g = res_dot<A, false, EP < 4 ? EP : 4, EP, KEEP>(pv[p], pa[p], s_y, a.ep);
                const int j = tid + p * kResThreads;
                if (j < n) {
                    const double aj = LX ? s_xa[j] : xan[p % RX];
                    const V xs = LX ? s_x[j] : xv[p % RX];
                    const PrimalStep<V> u = primal_step<V>(
                        g, iterate_value<V>(xs, aj), LC ? s_ch[j] : cj[p % RC], (double)(LC ? s_lh[j] : lo[p % RC]),
                        (double)(LC ? s_uh[j] : hi[p % RC]), aj, sc);
                    s_xb[j] = u.xbar;
                    if (LX) s_x[j] = u.x;
                    else xv[p % RX] = u.x;
                    if (store) a.xp[j] = u.cand;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (q < a.dual.count && a.dual.row0[q] + (wave0 >> a.dual.hs[q]) < a.dual.row1[q]) { // uniform over the wave
                const int hs = a.dual.hs[q], cnt = a.dual.slots[q];
                double h;
                if (a.dual.acc[q] == 4) h = res_dot<4, FMA, 8, ED, KEEP>(dv[q], da[q], s_xb, cnt);
                else if (a.dual.acc[q] == 2) h = res_dot<2, FMA, 8, ED, KEEP>(dv[q], da[q], s_xb, cnt);
                else h = res_dot<1, FMA, 8, ED, KEEP>(dv[q], da[q], s_xb, cnt);
                if (hs > 3) h += lane_up<8>(h);
                if (hs > 2) h += lane_up<4>(h);
                if (hs > 1) h += lane_up<2>(h);
                if (hs > 0) h += lane_up<1>(h);
                const int r = row[q];
                if (r >= 0) {
                    double cand;
                    s_y[r] = dual_step(h, s_y[r], br[q], yan[q], sn[q], sc, cand);
                    if (store) a.yp[r] = cand;
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < R; p++) {
        const int j = tid + p * kResThreads;
        if (j < n) a.x[j] = LX ? s_x[j] : xv[p % RX];
    }
#pragma unroll
    for (int q = 0; q < Q; q++)
        if (row[q] >= 0) a.y[row[q]] = s_y[row[q]];
}

// ------------------------------------------------------------------- plan ---
// out[0] = longest column, out[1 + k] = longest row of segment k
__global__ __launch_bounds__(kBlock) void k_longest(int n, const int *__restrict__ tp, RowSegs sg,
                                                   const int *__restrict__ rp, int *__restrict__ out)
{
    const int k = blockIdx.x; // 0: the columns, else segment k - 1
    const int r0 = k == 0 ? 0 : sg.row0[k - 1], r1 = k == 0 ? n : sg.row0[k];
    const int *ptr = k == 0 ? tp : rp;
    double v[1] = {0.0};
    for (int r = r0 + threadIdx.x; r < r1; r += kBlock) v[0] = fmax(v[0], (double)(ptr[r + 1] - ptr[r]));
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
    X(1, 2, 8, 2, 16, OPS_LDS, 4) \
    X(1, 2, 8, 2, 16, OPS_SPLIT, 8)

// Rules: the library's own kernel choice (a caller who named kernels with
// lanes_* or autotune gets those); columns in tiles of 64 rows of at most 8
// entries or of 256 rows of at most 4 (whose tiles then never pass one chunk
// of entries, so the order is that of one chunk); rows in tiles of 256, 64 or
// 32 rows, of at most one chunk of 2,048 entries, or in lane groups; and a
// variant that holds the LP.
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
    int *out = (int *)s->redout, longest[1 + kMaxSegs] = {}; // small scratch of the handle, free outside a check
    hipLaunchKernelGGL(k_longest, dim3(1 + sg.count), dim3(kBlock), 0, s->stream, s->n, s->tp, sg, s->rp, out);
    hipError_t e = hipMemcpyAsync(longest, out, sizeof(int) * (1 + (size_t)sg.count), hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return e;
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
        res_lds(s->m, s->n, s->fp32 ? 4 : 8, OOPS) <= kResLds)                                                       \
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

template <typename V, int A, int EP, int R, int Q, int ED, bool FMA, int OPS>
static hipError_t res_launch(pdhg_solver *s, const ResArgs<V> &a)
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_resident<V, A, EP, R, Q, ED, FMA, OPS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kResLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_resident<V, A, EP, R, Q, ED, FMA, OPS>), dim3(1), dim3(kResThreads),
                       res_lds(a.m, a.n, sizeof(V), OPS), s->stream, a);
    return hipGetLastError();
}

template <typename V>
static hipError_t res_iterations(pdhg_solver *s, int count, bool store)
{
    ResArgs<V> a{};
    a.m = s->m;
    a.n = s->n;
    a.rp = s->rp;
    a.ci = s->ci;
    a.tp = s->tp;
    a.ti = s->ti;
    a.av = (const V *)s->ahat;
    a.atv = (const V *)s->ahat_t;
    a.ch = s->chc;
    a.bh = s->bhc;
    a.lh = (const V *)s->lh;
    a.uh = (const V *)s->uh;
    a.sense = s->sense;
    a.x = (V *)s->x;
    a.xa = (const double *)s->xa;
    a.ya = (const double *)s->ya;
    a.xp = (double *)s->xp;
    a.y = (double *)s->y;
    a.yp = (double *)s->yp;
    a.st = s->st;
    a.ep = s->res.ep;
    a.dual.count = s->res.rounds;
    for (int q = 0; q < s->res.rounds; q++) {
        a.dual.row0[q] = s->res.row0[q];
        a.dual.row1[q] = s->res.row1[q];
        a.dual.hs[q] = s->res.hs[q];
        a.dual.acc[q] = s->res.acc[q];
        a.dual.slots[q] = s->res.slots[q];
    }
    hipError_t e = hipSuccess;
    for (int i0 = 0; i0 < count && e == hipSuccess; i0 += kResMaxIters) {
        a.i0 = i0;
        a.len = count - i0 < kResMaxIters ? count - i0 : kResMaxIters;
        a.store = store && i0 + a.len == count;
        int k = 0;
        e = hipErrorInvalidValue;
#define PDHG_RES_LAUNCH(AA, EEP, RR, QQ, EED, OOPS, VB)                                             \
    k++;                                                                                             \
    if constexpr (!VB || sizeof(V) == VB) {                                                            \
        if (s->res.variant == k)                                                                     \
            e = s->res.fma ? res_launch<V, AA, EEP, RR, QQ, EED, true, OOPS>(s, a)                   \
                           : res_launch<V, AA, EEP, RR, QQ, EED, false, OOPS>(s, a);                 \
    }
        PDHG_RES_VARIANTS(PDHG_RES_LAUNCH)
#undef PDHG_RES_LAUNCH
    }
    return e;
}

hipError_t resident_iterations(pdhg_solver *s, int count, bool store)
{
    return s->fp32 ? res_iterations<float>(s, count, store) : res_iterations<double>(s, count, store);
}

} // namespace pdhg
