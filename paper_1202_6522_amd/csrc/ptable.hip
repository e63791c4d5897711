// Stored-P Legendre stage (Sec. 3.1, precomputed P_n^m; the runtime choice
// between the two algorithms is the tuning of Sec. 3.2).
//
// The table holds P_n^m(x_i) for every order m, degree n and northern
// latitude pair i, as doubles, split by the parity of j = n - m (the mirror
// fold of Sec. 3.1 pairs even j with F_N + F_S and odd j with F_N - F_S).
// Per (m, parity q) the degrees j = 2 jq + q form rows jq, the pairs form
// columns; both are padded to multiples of 16 with zeros and cut into 16 x 16
// blocks (2 KB), laid out block row by block row.  Inside a block, entry
// (jl, pl) sits at
//     (jl / 4) 64 + (pl / 4) 16 + (jl % 4) 4 + pl % 4,
// so that the 4 degrees x 16 pairs the synthesis feeds one matrix
// instruction, and the 16 degrees x 4 pairs the analysis feeds one, are each
// four whole 128-byte lines.
//
// With several fields of the same shape the Legendre stage is then a dense
// contraction per order: synthesis F[pair][col] = sum_j P[j][pair] Q[j][col],
// analysis Q[j][col] = sum_pair P[j][pair] G[pair][col], where a column is
// (field, re/im).  Both run on the FP64 matrix cores
// (v_mfma_f64_16x16x4_f64: D[16x16] += A[16x4] B[4x16]).  The table is built
// on the device from the plan's own recurrence tables (lane starts, segment
// shifts), so an entry is 0 exactly where the on-the-fly kernels drop the
// term (the polar cut), and equals gamma_n u_n elsewhere.
#include <hip/hip_runtime.h>

#include "shtn_internal.h"

namespace shtn {

typedef double d4 __attribute__((ext_vector_type(4)));

// m-major index of (n = m, m): the first coefficient of order m.
__device__ __forceinline__ long order_base(int L, int m) { return (long)m * (2 * L + 1 - m) / 2 + m; }

// A workgroup of the two passes is kSpWaves waves of one order: they share the
// order's inputs, which the workgroup puts in LDS.
constexpr int kSpWaves = 4;
constexpr int kXcdCus = 32;

// XCD-aware placement: workgroup b of a launch runs on XCD b % kXcds, and an
// XCD's workgroups go to its CUs in turn.  The nu workgroups of order m all go
// to XCD m % kXcds, one after another in that XCD's share of the launch
// (orders ascending, longest first); every second run of 32 is taken
// backwards, so that a CU gets long and short ones.  False past the last
// order.
__device__ __forceinline__ int xcd_slot()
{
    const int slot = blockIdx.x / kXcds;
    const int lo = slot & ~(kXcdCus - 1), n = gridDim.x / kXcds;
    return (slot & kXcdCus) && lo + kXcdCus <= n ? 2 * lo + kXcdCus - 1 - slot : slot;
}
__device__ __forceinline__ bool xcd_unit(int nu, int M, int& u, int& m)
{
    const int slot = xcd_slot();
    const int k = slot / nu;
    u = slot - k * nu;
    m = blockIdx.x % kXcds + kXcds * k;
    return m <= M;
}

// Workgroup p of XCD x's queue where order m = x + 8 k has ceil((L+1-m) / w)
// of them (w degrees each): the orders with n are consecutive, so the search
// takes one step per n.  False past the last.
__device__ __forceinline__ bool xcd_unit_of(int p, int w, int L, int M, int& u, int& m)
{
    const int x = blockIdx.x % kXcds;
    int k0 = 0;
    const int all = x <= M ? (M - x) / kXcds + 1 : 0;  // orders of this XCD
    for (int n = (L + w - x) / w; n > 0 && k0 < all; n--) {
        // orders with n or more
        const int k1 = min(all, (L + 1 - x - w * (n - 1) + kXcds - 1) / kXcds);
        const int c = (k1 - k0) * n;
        if (p < c) {
            const int k = p / n;
            u = p - k * n;
            m = x + kXcds * (k0 + k);
            return true;
        }
        p -= c;
        k0 = k1;
    }
    return false;
}

// One 16 x 16 tile of inputs per parity and column tile in LDS, one row per
// contraction index; two of each, one read while the other is written.  Rows
// 144 bytes apart: the complex values written by the lanes of a column fall in
// different banks, and so (but for one of 16 columns) do the four rows read at
// once.
constexpr int kBRow = 18;
template <int CT>
using BTiles = double[2][2][CT][16 * kBRow];

// The workgroup's LDS writes are seen after this; loads from global memory
// stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ int ptab_in_block(int jl, int pl)
{
    return (jl >> 2) * 64 + (pl >> 2) * 16 + (jl & 3) * 4 + (pl & 3);
}

// ---------------------------------------------------------------------------
// Builder: one thread per (order, pair column, padded to whole blocks).  The
// recurrence is the synthesis kernel's (same steps, same segment shifts, same
// lane starts), so a lane is 0 before its start step.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_ptable_build(const DevPlan* plan, const long* boff, double* tab, int npt)
{
    const DevPlan& P = *plan;
    const int m = blockIdx.y;
    const int pair = blockIdx.x * 64 + threadIdx.x;
    if (pair >= npt * 16) return;
    const int L = P.L, npair = P.npair;
    const int nj = L - m + 1;
    const long base = order_base(L, m);
    const bool act = pair < npair;
    const size_t q = (size_t)m * npair + (act ? pair : 0);
    const int jst = act ? P.inj_j[q] : nj;
    const double2 y = act ? *(const double2*)(P.inj_y + 2 * q) : make_double2(0.0, 0.0);
    const double x = act ? P.xp[pair] : 0.0;
    const int* segexp = P.segexp + P.segoff[m];
    const int pt = pair >> 4, pl = pair & 15;
    double* t0 = tab + boff[2 * m] * 256;
    double* t1 = tab + boff[2 * m + 1] * 256;
    auto at = [&](double* t, int jq) -> double& {
        return t[((long)(jq >> 4) * npt + pt) * 256 + ptab_in_block(jq & 15, pl)];
    };
    double ua = 0.0, ub = 0.0;
    for (int j = 0; j < nj; j += 2) {
        if (j > 0 && j % kSegLen == 0) {
            const int d = segexp[j / kSegLen];
            ua = ldexp(ua, d);
            ub = ldexp(ub, d);
        }
        if (j == jst) {  // start steps are multiples of kInject, hence even
            ua = y.x;
            ub = y.y;
        }
        ua = fma(x, ub, P.beta[base + j] * ua);
        at(t0, j >> 1) = j >= jst ? P.gamma[base + j] * ua : 0.0;
        if (j + 1 < nj) {
            ub = fma(x, ua, P.beta[base + j + 1] * ub);
            at(t1, j >> 1) = j + 1 >= jst ? P.gamma[base + j + 1] * ub : 0.0;
        }
    }
    // zero rows up to the end of the last block row of each parity
    const int c0 = (nj + 1) >> 1, c1 = nj >> 1;
    for (int jq = c0; jq < ((c0 + 15) & ~15); jq++) at(t0, jq) = 0.0;
    for (int jq = c1; jq < ((c1 + 15) & ~15); jq++) at(t1, jq) = 0.0;
}

// ---------------------------------------------------------------------------
// Synthesis (or the adjoint of the analysis): one workgroup per (order, group
// of kSpWaves RT pair tiles, group of CT column tiles), RT pair tiles per wave.
// Lane l feeds A[pair l%16][degree l/16] and B[degree l/16][column l%16] and
// holds D[pair l/16 + 4 r][column l%16], r < 4.  Even and odd degrees accumulate
// apart; the fold north = E + O, south = E - O is then lane-local.
//
// Bound by the table's bytes, read once per 32 fields: 268 MB at lmax 511, 50
// us at the rate of a plain read of as much.  The order's coefficients go
// through LDS once per workgroup instead of through L2 once per wave, and the
// table past the caches, which it would sweep clear of them.  16 fields at lmax
// 511: 71.5 us (waves that read their own coefficients and waited for
// each block's operands: 104.9).
// ---------------------------------------------------------------------------
template <int RT, int CT>
__global__ void __launch_bounds__(64 * kSpWaves, 2) k_sp_synth(PtabArgs a)
{
    __shared__ __attribute__((aligned(16))) BTiles<CT> bt;
    const DevPlan& P = *a.plan;
    const int npg = (a.npt + RT - 1) / RT;
    int pg, m;
    if (!xcd_unit((npg + kSpWaves - 1) / kSpWaves, P.M, pg, m)) return;
    const int tid = threadIdx.x;
    pg = pg * kSpWaves + __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = P.L, nlat = P.nlat, npair = P.npair;
    const int npt = a.npt;
    const int nj = L - m + 1;
    const long base = order_base(L, m);
    const int lane = tid & 63;
    const int col = lane & 15, kk = lane >> 4;
    const int comp = col & 1;

    // Every address, plan value and weight the epilogue needs is read here,
    // before the first store: the output may alias them for all the compiler
    // knows, so reads placed between the stores would each wait on memory.
    const long ts = P.f_ts;
    double* fo[CT];
    bool fv[CT];
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int f = (blockIdx.y * CT + c) * 8 + (col >> 1);
        fv[c] = f < a.nfields;
        const int fc = fv[c] ? f : 0;
        fo[c] = a.out + (a.f_off ? a.f_off[fc] : (long)fc * 2 * P.f_size) + comp;
    }
    // the coefficients this thread puts in LDS: degree 32 br + lj of one field
    // per column tile
    const int lj = tid & 31, lf = tid >> 5;
    const double2* qs[CT];
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int f = (blockIdx.y * CT + c) * 8 + lf;
        const int fc = f < a.nfields ? f : 0;
        qs[c] = (const double2*)(a.in + (a.q_off ? a.q_off[fc] : (long)fc * 2 * P.nlm)) + base;
    }
    // pair tiles past the last one read tile pg RT (or, in a wave past the
    // last, the last group's): their output rows are never stored
    const int pgc = min(pg, npg - 1);
    int tr[RT];
#pragma unroll
    for (int r = 0; r < RT; r++) tr[r] = pgc * RT + r < npt ? r : 0;
    const int a_off = ptab_in_block(kk, lane & 15);  // + 64 s for step s of a block

    d4 acc[2][RT][CT];
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int r = 0; r < RT; r++)
#pragma unroll
            for (int c = 0; c < CT; c++) acc[q][r][c] = d4{0.0, 0.0, 0.0, 0.0};

    // A block row (32 degrees) is two steps, one per parity (the odd parity has
    // as many rows as the even one, or one fewer: its missing row reloads the
    // even row).  The table's operands of a step are loaded while the matrix
    // instructions of the step before run, past the caches (each is used
    // once), every load unconditional from a valid address.  Degrees past the
    // order's last (among them the whole missing odd row) have coefficient 0.
    // Operands of pair rows past the last and of field columns past
    // the last are left as loaded: they only reach outputs that are never
    // stored.
    const int nbr0 = (((nj + 1) >> 1) + 15) >> 4, nbr1 = ((nj >> 1) + 15) >> 4;
    const double* t0 = a.tab + a.boff[2 * m] * 256 + (long)pgc * RT * 256 + a_off;
    const double* t1 = a.tab + a.boff[2 * m + 1] * 256 + (long)pgc * RT * 256 + a_off;
    struct Ops {
        double a[4][RT];
    };
    auto load = [&](Ops& o, int br, int q) {
        const double* tb = (q && br < nbr1 ? t1 : t0) + (long)br * npt * 256;
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int r = 0; r < RT; r++) o.a[s][r] = __builtin_nontemporal_load(tb + tr[r] * 256 + s * 64);
        // (the loads stay ahead of the matrix instructions that follow)
        __builtin_amdgcn_sched_barrier(0);
    };
    double2 qv[CT];
    auto load_q = [&](int br) {
        const int j = min(32 * br + lj, nj - 1);
#pragma unroll
        for (int c = 0; c < CT; c++) qv[c] = qs[c][j];
        __builtin_amdgcn_sched_barrier(0);
    };
    auto put_q = [&](int br) {
        const bool in = 32 * br + lj < nj;
#pragma unroll
        for (int c = 0; c < CT; c++)
            *(double2*)&bt[br & 1][lj & 1][c][(lj >> 1) * kBRow + 2 * lf] =
                make_double2(in ? qv[c].x : 0.0, in ? qv[c].y : 0.0);
    };
    auto run = [&](const Ops& o, int br, int q) {
#pragma unroll
        for (int s = 0; s < 4; s++) {
            double bv[CT];
#pragma unroll
            for (int c = 0; c < CT; c++) bv[c] = bt[br & 1][q][c][(4 * s + kk) * kBRow + col];
#pragma unroll
            for (int r = 0; r < RT; r++)
#pragma unroll
                for (int c = 0; c < CT; c++)
                    acc[q][r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[s][r], bv[c], acc[q][r][c], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    Ops even, odd;
    load_q(0);
    load(even, 0, 0);
    put_q(0);
    lds_barrier();
    for (int br = 0; br < nbr0 - 1; br++) {
        load_q(br + 1);
        load(odd, br, 1);
        run(even, br, 0);
        load(even, br + 1, 0);
        run(odd, br, 1);
        put_q(br + 1);
        lds_barrier();
    }
    load(odd, nbr0 - 1, 1);
    run(even, nbr0 - 1, 0);
    run(odd, nbr0 - 1, 1);
    if (pg >= npg) return;

    // For the adjoint of the analysis the output carries (2 pi/nphi) w_i / c_m.
    const double cm = a.adjoint ? (2.0 * M_PI / P.nphi) * (m == 0 ? 1.0 : 0.5) : 1.0;
    double sc[RT][4];
#pragma unroll
    for (int r = 0; r < RT; r++)
#pragma unroll
        for (int i = 0; i < 4; i++)
            sc[r][i] = a.adjoint ? cm * P.wfull[min((pg * RT + r) * 16 + kk + 4 * i, npair - 1)] : 1.0;
#pragma unroll
    for (int r = 0; r < RT; r++) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int pair = (pg * RT + r) * 16 + kk + 4 * i;
            if (pair >= npair) continue;
            const int is = nlat - 1 - pair;
#pragma unroll
            for (int c = 0; c < CT; c++) {
                if (!fv[c]) continue;
                const double e = acc[0][r][c][i], o = acc[1][r][c][i];
                fo[c][2 * f_index(ts, m, pair)] = sc[r][i] * (e + o);
                if (is != pair) fo[c][2 * f_index(ts, m, is)] = sc[r][i] * (e - o);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Analysis (or the adjoint of the synthesis): one workgroup per (order, group
// of kSpWaves JT block rows of each parity, group of CT column tiles), JT block
// rows per wave; the contraction runs over all pairs, 4 per matrix
// instruction.  Lane l feeds A[degree l%16][pair l/16] and B[pair l/16][column
// l%16] = the folded, weighted longitude coefficients, and holds D[degree l/16
// + 4 r][column l%16].
//
// Bound as the synthesis is; the longitude coefficients are folded once per
// workgroup.  16 fields at lmax 511: 84.6 us (waves on their own: 123.2; with
// two buffers of operands 110, and the more waves of different orders ran side
// by side the slower, 131: their inputs then no longer fit the caches).
// ---------------------------------------------------------------------------
template <int JT, int CT>
__global__ void __launch_bounds__(64 * kSpWaves, 2) k_sp_analys(PtabArgs a)
{
    __shared__ __attribute__((aligned(16))) BTiles<CT> bt;
    const DevPlan& P = *a.plan;
    int g, m;
    if (!xcd_unit_of(xcd_slot(), 32 * JT * kSpWaves, P.L, P.M, g, m)) return;
    const int tid = threadIdx.x;
    g = g * kSpWaves + __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = P.L, nlat = P.nlat, npair = P.npair;
    const int npt = a.npt;
    const int nj = L - m + 1;
    const int nbr0 = (((nj + 1) >> 1) + 15) >> 4, nbr1 = ((nj >> 1) + 15) >> 4;
    const long base = order_base(L, m);
    const int lane = tid & 63;
    const int col = lane & 15, kk = lane >> 4;
    const int comp = col & 1;

    // Output bases are read here, before the first store (which, for all the
    // compiler knows, may alias them).
    double* qo[CT];
    bool fv[CT];
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int f = (blockIdx.y * CT + c) * 8 + (col >> 1);
        fv[c] = f < a.nfields;
        const int fc = fv[c] ? f : 0;
        qo[c] = a.out + (a.q_off ? a.q_off[fc] : (long)fc * 2 * P.nlm) + 2 * base + comp;
    }
    bool rv[2][JT];
    const double* tq[2][JT];
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int t = 0; t < JT; t++) {
            const int br = g * JT + t;
            rv[q][t] = br < (q ? nbr1 : nbr0);
            // a block row past the last of its parity (the odd parity of
            // order lmax has none) reads the first even one: its accumulator
            // rows are degrees past the order's last, never stored
            const long blk = rv[q][t] ? a.boff[2 * m + q] + (long)br * npt : a.boff[2 * m];
            tq[q][t] = a.tab + blk * 256 + ptab_in_block(lane & 15, kk);  // + 256 pt + 16 (step % 4)
        }
    // the coefficients this thread puts in LDS, folded and weighted: pair
    // 16 pt + lp of field lf (8 CT fields: with an odd CT half of the workgroup
    // has one less)
    const int lp = tid & 15, lf = tid >> 4;
    constexpr int NL = (CT + 1) / 2;  // fields per thread, 16 apart
    const double2* fp[NL];
#pragma unroll
    for (int i = 0; i < NL; i++) {
        const int f = blockIdx.y * CT * 8 + lf + 16 * i;
        const int fc = f < a.nfields && lf + 16 * i < 8 * CT ? f : 0;
        fp[i] = (const double2*)(a.in + (a.f_off ? a.f_off[fc] : (long)fc * 2 * P.f_size));
    }

    d4 acc[2][JT][CT];
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int t = 0; t < JT; t++)
#pragma unroll
            for (int c = 0; c < CT; c++) acc[q][t][c] = d4{0.0, 0.0, 0.0, 0.0};

    // A pair tile is two steps of 2 x 4 pairs.  The table's operands of a step
    // are loaded while the matrix instructions of the step before run, past
    // the caches (each is used once), unconditionally from
    // valid addresses (pairs past the last read the last pair with weight 0).
    struct Ops {
        double pa[2][2][JT];
    };
    auto load = [&](Ops& o, int pt, int hf) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int t = 0; t < JT; t++)
                    o.pa[i][q][t] = __builtin_nontemporal_load(tq[q][t] + pt * 256 + (2 * hf + i) * 16);
        // (the loads stay ahead of the matrix instructions that follow)
        __builtin_amdgcn_sched_barrier(0);
    };
    double2 vn[NL], vs[NL];
    double wv;
    auto load_f = [&](int pt) {
        const int pc = min(pt * 16 + lp, npair - 1);
        wv = P.wq[pc];
#pragma unroll
        for (int i = 0; i < NL; i++) {
            vn[i] = fp[i][f_index(P.f_ts, m, pc)];
            vs[i] = fp[i][f_index(P.f_ts, m, nlat - 1 - pc)];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto put_f = [&](int pt) {
        const int pair = pt * 16 + lp;
        const bool middle = (nlat & 1) && pair == npair - 1;
        const double wt = pair >= npair ? 0.0 : (a.adjoint ? (middle ? 0.5 : 1.0) : wv);
        const int o = lp * kBRow + 2 * (lf & 7);
#pragma unroll
        for (int i = 0; i < NL; i++) {
            if (lf + 16 * i >= 8 * CT) continue;
            const int c = (lf >> 3) + 2 * i;
            *(double2*)&bt[pt & 1][0][c][o] = make_double2(wt * (vn[i].x + vs[i].x), wt * (vn[i].y + vs[i].y));
            *(double2*)&bt[pt & 1][1][c][o] = make_double2(wt * (vn[i].x - vs[i].x), wt * (vn[i].y - vs[i].y));
        }
    };
    auto run = [&](const Ops& o, int pt, int hf) {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            double bv[2][CT];
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int c = 0; c < CT; c++) bv[q][c] = bt[pt & 1][q][c][(4 * (2 * hf + i) + kk) * kBRow + col];
#pragma unroll
            for (int t = 0; t < JT; t++)
#pragma unroll
                for (int c = 0; c < CT; c++) {
                    acc[0][t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.pa[i][0][t], bv[0][c], acc[0][t][c], 0, 0, 0);
                    acc[1][t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.pa[i][1][t], bv[1][c], acc[1][t][c], 0, 0, 0);
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const bool any = g * JT < nbr0;  // else this wave only helps with the inputs
    Ops lo, hi;
    load_f(0);
    load(lo, 0, 0);
    put_f(0);
    lds_barrier();
    for (int pt = 0; pt < npt - 1; pt++) {
        load_f(pt + 1);
        if (any) {
            load(hi, pt, 1);
            run(lo, pt, 0);
            load(lo, pt + 1, 0);
            run(hi, pt, 1);
        }
        put_f(pt + 1);
        lds_barrier();
    }
    if (!any) return;
    load(hi, npt - 1, 1);
    run(lo, npt - 1, 0);
    run(hi, npt - 1, 1);

    const double cm = (m == 0 || !a.adjoint) ? 1.0 : 2.0;
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int t = 0; t < JT; t++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int j = 2 * ((g * JT + t) * 16 + kk + 4 * i) + q;
                if (j >= nj) continue;
#pragma unroll
                for (int c = 0; c < CT; c++) {
                    if (!fv[c]) continue;
                    const double v = (m == 0 && comp == 1) ? 0.0 : cm * acc[q][t][c][i];
                    qo[c][2 * j] = v;
                }
            }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int launch_ptable_build(const DevPlan* plan, const long* boff, double* tab, int npt, int M, void* stream)
{
    hipLaunchKernelGGL(k_ptable_build, dim3((npt * 16 + 63) / 64, M + 1), dim3(64), 0, (hipStream_t)stream,
                       plan, boff, tab, npt);
    return (int)hipGetLastError();
}

template <int RT, int CT>
static int launch_sp_synth_t(const PtabArgs& a, int M, void* stream)
{
    const int npg = (a.npt + RT - 1) / RT;
    const int nfg = (a.nfields + 8 * CT - 1) / (8 * CT);
    const int nx = kXcds * ((M + kXcds) / kXcds) * ((npg + kSpWaves - 1) / kSpWaves);
    hipLaunchKernelGGL((k_sp_synth<RT, CT>), dim3(nx, nfg), dim3(64 * kSpWaves), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

template <int JT, int CT>
static int launch_sp_analys_t(const PtabArgs& a, int L, int M, void* stream)
{
    const int nfg = (a.nfields + 8 * CT - 1) / (8 * CT);
    int units = 0;  // workgroups of XCD 0, which has the most (see xcd_unit_of)
    for (int m = 0; m <= M; m += kXcds) units += (L - m + 32 * JT * kSpWaves) / (32 * JT * kSpWaves);
    hipLaunchKernelGGL((k_sp_analys<JT, CT>), dim3(kXcds * units, nfg), dim3(64 * kSpWaves), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// Column tiles of a launch, and pair tiles (block rows) per wave.  ct > 0: as
// set; a call of at most 8 fields fills one column tile, a second would only
// add columns that are never stored.  ct = 0: one pair tile, and column tiles
// for all fields up to 32, then as even as can be, so that the table is read as
// few times as can be (24 fields at lmax 511, synthesis and analysis in us:
// three column tiles 90.4 and 108.8, two and two 133.9 and 148.1).
static int column_tiles(int nfields, int ct)
{
    const int all = (nfields + 7) / 8;
    if (ct > 0) return all == 1 ? 1 : ct;
    const int groups = (all + 3) / 4;
    return (all + groups - 1) / groups;
}

int launch_sp_synth(const PtabArgs& a, int M, int rt, int ct, void* stream)
{
    ct = column_tiles(a.nfields, ct);
#define SHTN_SP(RV, CV) \
    if (rt == RV && ct == CV) return launch_sp_synth_t<RV, CV>(a, M, stream);
    SHTN_SP(1, 1) SHTN_SP(2, 1) SHTN_SP(4, 1) SHTN_SP(1, 2) SHTN_SP(2, 2) SHTN_SP(4, 2)
    SHTN_SP(1, 3) SHTN_SP(1, 4)
#undef SHTN_SP
    return (int)hipErrorInvalidValue;
}

int launch_sp_analys(const PtabArgs& a, int L, int M, int jt, int ct, void* stream)
{
    ct = column_tiles(a.nfields, ct);
#define SHTN_SP(JV, CV) \
    if (jt == JV && ct == CV) return launch_sp_analys_t<JV, CV>(a, L, M, stream);
    SHTN_SP(1, 1) SHTN_SP(2, 1) SHTN_SP(4, 1) SHTN_SP(1, 2) SHTN_SP(2, 2) SHTN_SP(4, 2)
    SHTN_SP(1, 3) SHTN_SP(1, 4)
#undef SHTN_SP
    return (int)hipErrorInvalidValue;
}

}  // namespace shtn
