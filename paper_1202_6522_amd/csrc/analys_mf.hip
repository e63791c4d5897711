// Legendre analysis of several fields at once on gfx950: P_n^m on the fly
// (FP64 vector ALUs), the sums over latitudes on the FP64 matrix cores.
//
// Q_n^m = gamma_n sum_pairs u_n G, with G = w (F_N +- F_S) the folded, weighted
// longitude coefficients (the plus sign for even n - m).  With several fields
// the sum is a contraction: rows are degrees, columns the real and imaginary
// parts of the fields, and it runs on v_mfma_f64_4x4x4: four independent
// products D[4 x 4] += A[4 x 4] B[4 x 4].  Lane l = 16 k + 4 b + i feeds A_b[i][k]
// and B_b[k][i] and holds D_b[k][i]: rows are four degrees of one parity,
// columns two fields, and k and b run over sixteen latitude pairs.
//
// The recurrence needs a lane per latitude pair and gives one degree at a
// time; A needs four degrees side by side in the lanes of a quad.  The values
// of an octet of degrees therefore pass through LDS: one row of 64 pairs per
// degree is written, and A is read back with the quad's lanes on four rows.
// (LDS instructions of one wave run in order, so no barrier is needed, and
// they take no vector-ALU issue; moving the values between lanes by DPP would
// take four vector instructions per degree.)
//
// Bound by the FP64 pipe, which matrix and vector instructions share: per 64
// pairs and octet 16 (four fields) or 32 (eight) matrix instructions of 17
// cycles and 16 vector ones of 4.6, next to 32 LDS accesses of 4.4 (a CU's
// four SIMDs share its LDS, so at four fields it is nearly as busy).  Against
// the vector kernel (legendre.hip) the reduction over lanes goes, 5
// instructions per degree and field, and the recurrence is shared.  Measured
// (library events, us, vector kernel and this one): lmax 511, 16 fields, 123
// and 84; lmax 1023, 4 fields, 178 and 152, 8 fields, 348 and 267; lmax 2047, 4
// fields, 1295 and 987.  Tried and not kept: v_mfma_f64_16x16x4 for eight fields
// in passes of 32 degrees (lmax 511, 16 fields: 108), two scalar fields (slower than
// the vector kernel at lmax 511 and 1023).
#include <algorithm>

#include "legendre_dev.h"

namespace shtn {

constexpr int kOct = 8;          // degrees per pass: one start checkpoint to the next
// Row strides in LDS (doubles), free of bank conflicts: the four degree rows a
// quad reads start one double apart, the rows of partial sums four.
constexpr int kMfStride = 65, kSumStride = 68;
static_assert(kOct == kInject, "one start checkpoint per pass");

// One pass over the slots PF .. LP-1 (the slots below belong to latitude
// blocks that have not started): d[q][c] += the octet's products of parity q
// with column group c (fields 2 c and 2 c + 1).
// XT: with x P in place of P, whose parity is the other one.
template <int LP, int CG, int PF, bool XT = false>
__device__ __forceinline__ void mf_octet(const double (&x)[LP], double (&ua)[LP], double (&ub)[LP],
                                         const double (&b)[kOct], const double (&g)[LP][4][2][CG],
                                         double (*rows)[kMfStride], double (&d)[2][CG])
{
    const int lane = threadIdx.x & 63;
    const int rd = (lane & 60);  // 16 k + 4 b
    const int ri = lane & 3;     // degree row of a quad's lane
    double a[2][2][4];           // A operands of this slot and the one before: [slot][parity][s]
#pragma unroll
    for (int p = PF; p <= LP; p++) {
        if (p < LP) {
            // eight steps of the recurrence; row q 4 + t holds degree 2 t + q
            double v[kOct];
#pragma unroll
            for (int t = 0; t < kOct; t += 2) {
                ua[p] = fma(x[p], ub[p], b[t] * ua[p]);
                ub[p] = fma(x[p], ua[p], b[t + 1] * ub[p]);
                v[t] = ua[p];
                v[t + 1] = ub[p];
            }
#pragma unroll
            for (int t = 0; t < kOct; t++) rows[(t & 1) * 4 + (t >> 1)][lane] = XT ? x[p] * v[t] : v[t];
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int s = 0; s < 4; s++) a[p & 1][q][s] = rows[q * 4 + ri][rd + s];
        }
        if (p > PF) {
            const int o = p - 1;
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int q = 0; q < 2; q++)
#pragma unroll
                    for (int c = 0; c < CG; c++)
                        d[q][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[o & 1][q][s], g[o][s][XT ? 1 - q : q][c], d[q][c], 0, 0, 0);
        }
    }
}

// One workgroup per unit (degrees [j0, j1) of one order), 2 CG fields; W waves
// cover 64 LP latitude pairs each.  CG = 2 or 4 column groups: four or eight
// fields; with CG = 1 the four columns are the parts of two.  VEC: the fields
// are the components of tangent vectors (vector.hip): inputs are divided by
// sin(theta), and the unit with the order's last degree, L, also gives the sum
// with x P_L in place of P_L (a.top).
template <int LP, int CG, int W, bool VEC>
__global__ void __launch_bounds__(64 * W, 2) k_legendre_analys_mf(LegArgs a)
{
    constexpr int NF = 2 * CG;
    constexpr int NV = CG > 1 ? CG / 2 : 1;  // outputs of an octet per lane
    constexpr int kMfChunk = 128 / NV;  // degrees whose sums several waves exchange at once
    __shared__ double rows_w[W][kOct][kMfStride];
    // sums of a chunk per wave: one octet is NV values per lane
    __shared__ double acc[W][W > 1 ? kMfChunk / kOct * 64 * NV : 1];

    __builtin_amdgcn_s_setprio(3);
    // every unit runs once per field group, one after another on its XCD
    const int slot = blockIdx.x / kXcds / a.groups;
    const int unit = slot * kXcds + blockIdx.x % kXcds;
    const int group = a.group0 + blockIdx.x / kXcds - slot * a.groups;
    cip U = (cip)a.units + (size_t)unit * kUnitInts;
    const int m = U[U_M];
    if (m < 0) return;
    const int field0 = group * NF;
    const int nf = min(NF, a.nfields - field0);
    cplan P = (cplan)a.plans + U[U_PLAN];
    const int L = P->L, nlat = P->nlat, npair = P->npair;
    const long fts = P->f_ts;
    const long nlm = P->nlm;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // which latitudes a wave takes turns with the unit (see legendre.hip)
    const int wid = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int wv = W > 1 ? (wid + slot) & (W - 1) : 0;
    const int pb = wv * 64 * LP;
    const int wb = wv * LP;
    const int j0 = U[U_PB], j1 = U[U_J1], js0 = U[U_JS], jwin = U[U_JW], rst = U[U_RST];
    const long base = (long)m * (2 * L + 1 - m) / 2 + m;
    cdp bet = (cdp)P->beta + base;
    cip segexp = (cip)P->segexp + ((cip)P->segoff)[m];
    cip ckm = (cip)P->ck_mask + (size_t)m * P->nck * 2;
    double (*rows)[kMfStride] = rows_w[wid];

    // degrees before the first started lane: every term is dropped
    for (int e = tid; e < (js0 - j0) * 2; e += 64 * W)
        for (int f = 0; f < nf; f++) a.out[(long)(field0 + f) * 2 * nlm + 2 * (base + j0) + e] = 0.0;
    const bool last = VEC && j1 == L - m + 1;
    if (js0 >= j1) {
        if (last && tid < 2 * nf) a.top[2 * ((long)(field0 + (tid >> 1)) * (P->M + 1) + m) + (tid & 1)] = 0.0;
        return;
    }

    // Columns: group 0 holds the real parts of fields 0 to 3, 1 their
    // imaginary parts (2 and 3 those of fields 4 to 7), so lane n of a quad
    // loads whole complex values of field n (and n + 4).  (Fields past the
    // last repeat it and are not stored.)  A single group holds field n / 2,
    // real part at even n, imaginary part at odd n.
    double x[LP], ua[LP], ub[LP];
    double g[LP][4][2][CG];
    const bool from_rst = rst >= 0 && js0 == j0;
    // every load of the set-up is issued before any is used
    {
        double w[LP][4], xs[LP][4];
        double2 r[LP];
        // byte offsets from the first field (at most eight fields of 268 MB)
        gcp F = (gcp)(a.in + (long)field0 * 2 * P->f_size + 2 * m * kFTile);
        unsigned fo[NV];
#pragma unroll
        for (int v = 0; v < NV; v++)
            fo[v] = CG > 1 ? (unsigned)min(4 * v + (lane & 3), nf - 1) * (unsigned)(P->f_size * 16)
                           : (unsigned)min((lane >> 1) & 1, nf - 1) * (unsigned)(P->f_size * 16) + 8 * (lane & 1);
        const unsigned ts16 = (unsigned)fts * 16;
        gcp xp = (gcp)P->xp, wq = (gcp)P->wq;
        // (past the last pair the first one's values, with weight 0, as in the
        // vector kernel: seen only when they are infinite or not a number)
        auto pair_of = [&](int i) { return (unsigned)(i < npair ? i : 0); };
        auto lat_off = [&](int i) { return (unsigned)(i >> kFTileLg) * ts16 + (unsigned)(i & (kFTile - 1)) * 16; };
#pragma unroll
        for (int p = 0; p < LP; p++) {
            x[p] = ld1(xp, 8 * pair_of(pb + p * 64 + lane));
#pragma unroll
            for (int s = 0; s < 4; s++) {
                // B rows: the pairs whose values sit in lanes 16 k + 4 b + s
                const unsigned pair = pair_of(pb + p * 64 + (lane & 60) + s);
                w[p][s] = ld1(wq, 8 * pair);
                if constexpr (VEC) xs[p][s] = ld1(xp, 8 * pair);
                const unsigned on = lat_off((int)pair), os = lat_off(nlat - 1 - (int)pair);
#pragma unroll
                for (int v = 0; v < NV; v++) {
                    if constexpr (CG > 1) {
                        const double2 vn = ld2(F, fo[v] + on), vs = ld2(F, fo[v] + os);
                        g[p][s][0][2 * v] = vn.x;
                        g[p][s][0][2 * v + 1] = vn.y;
                        g[p][s][1][2 * v] = vs.x;
                        g[p][s][1][2 * v + 1] = vs.y;
                    } else {
                        g[p][s][0][0] = ld1(F, fo[v] + on);
                        g[p][s][1][0] = ld1(F, fo[v] + os);
                    }
                }
            }
        }
        if (from_rst) {
            gcp ry = (gcp)(P->rst_y + 2 * ((size_t)rst * npair));
#pragma unroll
            for (int p = 0; p < LP; p++) r[p] = ld2(ry, 16 * pair_of(pb + p * 64 + lane));
        } else {
#pragma unroll
            for (int p = 0; p < LP; p++) r[p] = make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const bool act = pb + p * 64 + lane < npair;
            if (!act) x[p] = 0.0;
            ua[p] = act ? r[p].x : 0.0;
            ub[p] = act ? r[p].y : 0.0;
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const int pair = pb + p * 64 + (lane & 60) + s;
                const bool middle = (nlat & 1) && pair == npair - 1;
                double wt = pair >= npair ? 0.0 : (a.adjoint ? (middle ? 0.5 : 1.0) : w[p][s]);
                if constexpr (VEC) wt = wt / sqrt((1.0 - xs[p][s]) * (1.0 + xs[p][s]));
#pragma unroll
                for (int c = 0; c < CG; c++) {
                    const double vn = g[p][s][0][c], vs = g[p][s][1][c];
                    g[p][s][0][c] = wt * (vn + vs);
                    g[p][s][1][c] = wt * (vn - vs);
                }
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);

    // this lane's outputs of an octet, after the sum over b: b = lane / 4 % 4
    // picks parity q = b % 2 and column group b / 2 (+ 2 v) of row i = lane / 16
    const int oq = (lane >> 2) & 1, oc = (lane >> 3) & 1;
    const int oj = 2 * (lane >> 4) + oq;
    const int of = CG > 1 ? lane & 3 : (lane >> 1) & 1;  // + 4 v
    const int comp = CG > 1 ? oc : lane & 1;
    const bool mine = CG > 1 || oc == 0;  // (a single group: lane groups 2 and 3 repeat 0 and 1)
    double* out = a.out + (long)(field0 + of) * 2 * nlm + 2 * base + comp;
    gcp gam = (gcp)(P->gamma + base);
    const double cm = (m == 0 || !a.adjoint) ? 1.0 : 2.0;

    DBlk<kOct> bn;
    load_blk(bn, bet + js0);
    DBlk2u<2> mkw;
    load_u32(mkw, ckm + 2 * (js0 / kOct));
    int shn = 0;  // js0 is a segment start (the plan rounds it down)
    for (int c = js0; c < j1; c += kOct) {
        const int sh = shn;
        // this octet's scalars have arrived before the next ones are asked for
        // (scalar loads return out of order: a wait is for all of them)
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        double b[kOct];
#pragma unroll
        for (int t = 0; t < kOct; t++) b[t] = bn.v[t];
        const unsigned mk = (mkw.v[0] >> wb) & ((1u << LP) - 1u);
        const unsigned lv = (mkw.v[1] >> wb) & ((1u << LP) - 1u);
        const int cn = c + kOct;
        load_blk(bn, bet + cn);
        load_u32(mkw, ckm + 2 * (cn / kOct));
        shn = (cn < j1 && cn % kSegLen == 0) ? segexp[cn / kSegLen] : 0;
        const double gl = ld1(gam, 8 * (unsigned)min(c + oj, j1 - 1));
        __builtin_amdgcn_sched_barrier(0);
        if (sh != 0) rescale(ua, ub, sh);
        if (mk != 0u && c <= jwin) start_slots(ua, ub, P, m, pb, mk, c);
        double d[2][CG];
        auto clear = [&] {
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int k = 0; k < CG; k++) d[q][k] = 0.0;
        };
        clear();
        // the states before the order's last degrees, which then run again with x P
        double va[LP], vb[LP];
        const bool again = last && cn >= j1;
        if (VEC && again) {
#pragma unroll
            for (int p = 0; p < LP; p++) {
                va[p] = ua[p];
                vb[p] = ub[p];
            }
        }
        switch (lv ? __builtin_ctz(lv) : LP) {
        case 0: mf_octet<LP, CG, 0>(x, ua, ub, b, g, rows, d); break;
        case 1: mf_octet<LP, CG, (1 < LP ? 1 : LP)>(x, ua, ub, b, g, rows, d); break;
        case 2: mf_octet<LP, CG, (2 < LP ? 2 : LP)>(x, ua, ub, b, g, rows, d); break;
        case 3: mf_octet<LP, CG, (3 < LP ? 3 : LP)>(x, ua, ub, b, g, rows, d); break;
        default: break;  // no slot live
        }
        // sum over b (lanes 4 apart in a row of 16), through LDS: lane group b
        // adds up parity b % 2 of column group b / 2
        double val[NV];
        double* sums = &rows[0][0];
        auto sum_b = [&] {
#pragma unroll
            for (int v = 0; v < NV; v++) {
#pragma unroll
                for (int k = 0; k < (CG > 1 ? 2 : 1); k++)
#pragma unroll
                    for (int q = 0; q < 2; q++) sums[(2 * k + q) * kSumStride + lane] = d[q][2 * v + k];
                const double* br = sums + ((lane >> 2) & (CG > 1 ? 3 : 1)) * kSumStride + (lane & 51);
                val[v] = (br[0] + br[4]) + (br[8] + br[12]);
            }
        };
        sum_b();
        auto store = [&](double s, int j, double gm, int v) {
            if (mine && of + 4 * v < nf && j < j1)
                out[(long)(4 * v) * 2 * nlm + 2 * j] = m == 0 && comp == 1 ? 0.0 : cm * gm * s;
        };
        if constexpr (W == 1) {
#pragma unroll
            for (int v = 0; v < NV; v++) store(val[v], c + oj, gl, v);
        } else {
            const int jc = (c - js0) & ~(kMfChunk - 1);  // first degree of the chunk, from js0
#pragma unroll
            for (int v = 0; v < NV; v++) acc[wv][((c - js0 - jc) / kOct * NV + v) * 64 + lane] = val[v];
            if (cn >= j1 || (cn - js0) % kMfChunk == 0) {
                // add up the waves' sums, wave by wave an octet each
                __syncthreads();
                const int no = (min(kMfChunk, j1 - js0 - jc) + kOct - 1) / kOct;
                for (int e = wid; e < no; e += W) {
                    const int j = js0 + jc + e * kOct + oj;
                    const double gm = ld1(gam, 8 * (unsigned)min(j, j1 - 1));
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        double s = acc[0][(e * NV + v) * 64 + lane];
#pragma unroll
                        for (int k = 1; k < W; k++) s += acc[k][(e * NV + v) * 64 + lane];
                        store(s, j, gm, v);
                    }
                }
                __syncthreads();
            }
        }
        if constexpr (VEC) {
            if (again) {
                clear();
                switch (lv ? __builtin_ctz(lv) : LP) {
                case 0: mf_octet<LP, CG, 0, true>(x, va, vb, b, g, rows, d); break;
                case 1: mf_octet<LP, CG, (1 < LP ? 1 : LP), true>(x, va, vb, b, g, rows, d); break;
                case 2: mf_octet<LP, CG, (2 < LP ? 2 : LP), true>(x, va, vb, b, g, rows, d); break;
                case 3: mf_octet<LP, CG, (3 < LP ? 3 : LP), true>(x, va, vb, b, g, rows, d); break;
                default: break;
                }
                sum_b();
                if constexpr (W > 1) {
                    // (the workgroup is past its last chunk's sums)
#pragma unroll
                    for (int v = 0; v < NV; v++) acc[wv][v * 64 + lane] = val[v];
                    __syncthreads();
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        val[v] = acc[0][v * 64 + lane];
#pragma unroll
                        for (int k = 1; k < W; k++) val[v] += acc[k][v * 64 + lane];
                    }
                }
                if (wid == 0 && mine && c + oj == j1 - 1) {
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        if (of + 4 * v < nf)
                            a.top[2 * ((long)(field0 + of + 4 * v) * (P->M + 1) + m) + comp] =
                                m == 0 && comp == 1 ? 0.0 : cm * gl * val[v];
                }
            }
        }
    }
}

template <int W, class K>
static int launch_mf_t(K kernel, int fields, const LegLaunch& l, void* stream)
{
    const int groups = (l.nfields + fields - 1) / fields;
    // (a launch's threads are counted in 32 bits: one launch unless the call
    // has far more fields than the card holds)
    const int most = std::max(1, (1 << 25) / (l.nunits * W));
    for (int g0 = 0; g0 < groups; g0 += most) {
        const int ng = std::min(most, groups - g0);
        LegArgs a{l.plans, l.units, l.q_off, l.f_off, l.in, l.out, l.nfields, l.adjoint, l.nunits, ng, g0, W, l.top};
        hipLaunchKernelGGL(kernel, dim3((unsigned)l.nunits * ng), dim3(64 * W), 0, (hipStream_t)stream, a);
    }
    return (int)hipGetLastError();
}

int launch_legendre_analys_mf(const LegLaunch& l, int npair, int nf, void* stream)
{
    if (l.nunits <= 0) return 0;
    const int w = mf_waves(npair, nf);
    const int lp = npair <= 64 ? 1 : (npair <= 128 || nf == 8 ? 2 : 4);
#define SHTN_M(LPV, CV, WV) \
    if (nf == 2 * CV && lp == LPV && w == WV)                                                        \
        return l.top ? launch_mf_t<WV>(k_legendre_analys_mf<LPV, CV, WV, true>, 2 * CV, l, stream)   \
                     : launch_mf_t<WV>(k_legendre_analys_mf<LPV, CV, WV, false>, 2 * CV, l, stream);
    SHTN_M(1, 2, 1) SHTN_M(2, 2, 1) SHTN_M(4, 2, 1) SHTN_M(4, 2, 2) SHTN_M(4, 2, 4) SHTN_M(4, 2, 8)
    SHTN_M(1, 4, 1) SHTN_M(2, 4, 1) SHTN_M(2, 4, 2) SHTN_M(2, 4, 4) SHTN_M(2, 4, 8)
#undef SHTN_M
    // one vector field
#define SHTN_V(LPV, WV)                          \
    if (nf == 2 && lp == LPV && w == WV && l.top) \
        return launch_mf_t<WV>(k_legendre_analys_mf<LPV, 1, WV, true>, 2, l, stream);
    SHTN_V(1, 1) SHTN_V(2, 1) SHTN_V(4, 1) SHTN_V(4, 2) SHTN_V(4, 4) SHTN_V(4, 8)
#undef SHTN_V
    return (int)hipErrorInvalidValue;
}

}  // namespace shtn
