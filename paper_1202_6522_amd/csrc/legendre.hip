// Legendre stage of the Gauss-Legendre SHT on gfx950: FP64 vector ALUs.
//
// Synthesis (Sec. 2.2, eq. synth_direct) and analysis (Sec. 2.3, eq. gauss)
// with P_n^m generated on the fly by the three-term recurrence of Sec. 3.2
// (eq. rec), the equatorial mirror symmetry of Sec. 3.1 folded in (one lane
// carries the pair of latitudes x and -x: even degrees n-m add, odd degrees
// subtract), and the underflow guard of Sec. 3.5 with the polar threshold of
// Sec. 3.1 resolved at plan time: every lane starts at the step where its
// |P_n^m| first matters, from a state stored by the plan, and a wave skips
// the steps in which none of its lanes has started.
//
// The recurrence runs in the rescaled form u_n = x u_{n-1} + beta_n u_{n-2}
// (two FP64 operations per step: one multiply by an SGPR coefficient and one
// FMA), with P_n^m = gamma_n u_n; gamma is folded into the spectrum as the
// synthesis loads it and applied after the reduction in the analysis.
// Recurrence coefficients are wave-uniform and are read with scalar loads into
// SGPRs, in blocks of several degrees; their table is padded past its last
// entry so a block load at the end of an order stays in bounds.
//
// One synthesis unit = one wave of 64 lanes, LP latitude pairs per lane and FW
// fields that share the plan.
#include <hip/hip_runtime.h>

#include "legendre_dev.h"

namespace shtn {

// ---------------------------------------------------------------------------
// Synthesis: F_m(theta) for one order, LP pairs per lane, FW fields.
//
// Bound by the FP64 VALU, whose clock the chip's power holds to about 2.0-2.2
// GHz under this load: 2 + 2 FW instructions per degree and pair.  What kept
// the kernel from that rate was the feeding of the coefficients (as scalar
// loads they shared a small cache, so eight waves of one order had to run in
// one workgroup, and several fields per wave gained nothing) and the uneven
// sum of the waves a SIMD was dealt.  Here the 16 lanes of every row of a wave
// hold the coefficients of 16 degrees, loaded as one vector, and each FMA
// picks its degree by a row broadcast of its operand.  A wave then depends on
// no other, and units can be placed freely (synth_unit).  Measured (library
// events, us, before and after): lmax 1023, one field, 49.7 -> 41.6 (and the
// launch that multiplied the spectrum by gamma, 5.7, is gone), four fields
// 167.9 -> 90.2; lmax 2047 276.5 -> 235.5; lmax 511, 16 fields, 103.8 -> 55.6;
// lmax 255 12.5 -> 10.2.
// ---------------------------------------------------------------------------
template <int LP, int FW>
struct SynthState {
    double x[LP], ua[LP], ub[LP];
    double er[LP][FW], ei[LP][FW], orr[LP][FW], oi[LP][FW];
};

// Degrees per group of coefficients: the 16 lanes of each row of a wave hold
// the coefficients of 16 consecutive degrees.
constexpr int kGroup = 16;

// acc += c(lane T of the reader's row of 16 lanes) * u: the coefficient is
// broadcast by the operand's own lane select (DPP row_newbcast), which the
// compiler does not form by itself for FP64.  c must have been written by a
// load or at least two instructions earlier (ready_for_dpp).
template <int T>
__device__ __forceinline__ void fmac_row(double& acc, double c, double u)
{
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(c), "v"(u), "n"(T));
}

// Two wait states between the instructions that wrote these registers and
// their first use as a broadcast operand.
template <int FW>
__device__ __forceinline__ void ready_for_dpp(double2 (&q)[FW])
{
    if constexpr (FW == 1)
        asm volatile("s_nop 1" : "+v"(q[0].x), "+v"(q[0].y));
    else if constexpr (FW == 2)
        asm volatile("s_nop 1" : "+v"(q[0].x), "+v"(q[0].y), "+v"(q[1].x), "+v"(q[1].y));
    else
        asm volatile("s_nop 1"
                     : "+v"(q[0].x), "+v"(q[0].y), "+v"(q[1].x), "+v"(q[1].y), "+v"(q[2].x), "+v"(q[2].y),
                       "+v"(q[3].x), "+v"(q[3].y));
}

// Keeps a uniform branch a branch (the compiler would turn a short body into
// selects that run on every pass).
__device__ __forceinline__ void keep_branch() { asm volatile(""); }

// Step T of a group (degree offset 16 g + T).  Even T advance ua and feed the
// even (E) sums, odd T advance ub and feed the odd (O) sums.
template <int LP, int FW, int T>
__device__ __forceinline__ void synth_step(SynthState<LP, FW>& s, double b, const double2 (&q)[FW])
{
    if constexpr (T % 2 == 0) {
#pragma unroll
        for (int p = 0; p < LP; p++) s.ua[p] = fma(s.x[p], s.ub[p], b * s.ua[p]);
#pragma unroll
        for (int f = 0; f < FW; f++) {
#pragma unroll
            for (int p = 0; p < LP; p++) {
                fmac_row<T>(s.er[p][f], q[f].x, s.ua[p]);
                fmac_row<T>(s.ei[p][f], q[f].y, s.ua[p]);
            }
        }
    } else {
#pragma unroll
        for (int p = 0; p < LP; p++) s.ub[p] = fma(s.x[p], s.ua[p], b * s.ub[p]);
#pragma unroll
        for (int f = 0; f < FW; f++) {
#pragma unroll
            for (int p = 0; p < LP; p++) {
                fmac_row<T>(s.orr[p][f], q[f].x, s.ub[p]);
                fmac_row<T>(s.oi[p][f], q[f].y, s.ub[p]);
            }
        }
    }
}

// Steps T .. TE-1 of a group.
template <int LP, int FW, int T, int TE>
__device__ __forceinline__ void synth_steps(SynthState<LP, FW>& s, const double (&b)[kGroup], const double2 (&q)[FW])
{
    if constexpr (T < TE) {
        synth_step<LP, FW, T>(s, b[T], q);
        synth_steps<LP, FW, T + 1, TE>(s, b, q);
    }
}

// Steps T .. TE-1 of a group, n of them (wave-uniform): the state stays that
// of the order's last degree.
template <int LP, int FW, int T, int TE>
__device__ __forceinline__ void synth_tail(SynthState<LP, FW>& s, const double (&b)[kGroup], const double2 (&q)[FW], int n)
{
    if constexpr (T < TE) {
        if (n > 0) {
            keep_branch();
            synth_step<LP, FW, T>(s, b[T], q);
            synth_tail<LP, FW, T + 1, TE>(s, b, q, n - 1);
        }
    }
}

// Unit and field group of a synthesis wave.  The unit list is eight queues,
// one per XCD (entry 8 s + x is entry s of XCD x's queue), each longest first;
// every unit runs once per field group, the groups of a unit one after
// another.  A workgroup takes `waves` consecutive entries of its queue.
// Small launches take one wave per workgroup, which spreads them over the
// whole chip.  Larger ones take four: waves of nearly the same length on the
// four SIMDs of a CU.  An XCD's workgroups go to its 32 CUs in turn, and a CU
// holds about six of them: nearly all of a one-field call is resident at once,
// so what a CU is dealt decides when it ends.  Every second run of 32
// workgroups is therefore taken backwards, so that a CU gets long and short
// units in turn.  (At lmax 1023 the work of the SIMDs then spreads by 1.2%;
// taken forwards throughout by 16%, and the kernel ended with the busiest,
// 45.8 us against 37.3.)  Orders are dealt to the queues in turn, so those of a
// plan with few orders differ much in length; its field groups then go from
// queue to queue, each XCD taking every order for some of the fields.  (256
// fields at lmax 4000, synthesis with its FFT: of one order 1,440 -> 470
// us, of nine 2,953 -> 2,080; the recurrence tables of 64 orders still lie in
// each XCD's L2.)
constexpr int kSynthWaves = 4;
constexpr int kXcdCus = 32;

__device__ __forceinline__ bool synth_unit(const LegArgs& a, int wave, int& unit, int& group)
{
    const int x = blockIdx.x % kXcds, n = gridDim.x / kXcds;
    int w = blockIdx.x / kXcds;
    const int lo = w & ~(kXcdCus - 1);
    if (a.waves > 1 && (w & kXcdCus) && lo + kXcdCus <= n) w = 2 * lo + kXcdCus - 1 - w;
    const int p = w * a.waves + wave;
    const int s = p / a.groups;
    group = a.group0 + p - s * a.groups;
    unit = s * kXcds + (a.rotate ? (x + group) % kXcds : x);
    return unit < a.nunits;
}

// Waves a SIMD should hold: with two pairs and four fields per lane the
// registers are kept to 128, four waves (left alone the compiler takes 133).
template <int LP, int FW>
constexpr int synth_waves() { return LP * FW == 8 ? 4 : 1; }

// VEC: the fields are the components of tangent vectors (vector.hip): the sums
// get a term top x P_L(x), whose P_L is the state after the order's last
// degree, and are divided by sin(theta).
template <int LP, int FW, bool VEC>
__global__ void __launch_bounds__(64 * kSynthWaves, (synth_waves<LP, FW>())) k_legendre_synth(LegArgs a)
{
    // wave-uniform for the compiler, so unit data and beta stay in SGPRs
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int unit, group;
    // the memory round trips of the set-up go ahead of the steps of the waves
    // that are under way (a late wave would wait behind all of them)
    __builtin_amdgcn_s_setprio(3);
    if (!synth_unit(a, wave, unit, group)) return;
    cip U = (cip)a.units + (size_t)unit * kUnitInts;
    const int m = U[U_M];
    if (m < 0) return;
    const int field0 = U[U_FIELD] + group * FW;
    if (field0 >= a.nfields) return;
    const int nf = min(U[U_NF], a.nfields - field0);
    cplan P = (cplan)a.plans + U[U_PLAN];
    const int L = P->L, nlat = P->nlat, npair = P->npair;
    const long fts = P->f_ts;
    const long nlm = P->nlm;
    const int pb = U[U_PB];
    long qoff[FW];
    long foff[FW];
#pragma unroll
    for (int f = 0; f < FW; f++) {
        const int ff = field0 + min(f, nf - 1);
        qoff[f] = field_q_off(a, ff, nlm);
        foff[f] = field_f_off(a, ff, P->f_size);
    }

    if (U[U_ZERO]) {
        // no latitude of the block reaches the polar threshold: F_m = 0 there
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const int pair = pb + p * 64 + lane;
            if (pair >= npair) continue;
            const int is = nlat - 1 - pair;
#pragma unroll
            for (int f = 0; f < FW; f++) {
                if (f >= nf) continue;
                double* F = a.out + foff[f];
                *(double2*)(F + 2 * f_index(fts, m, pair)) = make_double2(0.0, 0.0);
                *(double2*)(F + 2 * f_index(fts, m, is)) = make_double2(0.0, 0.0);
            }
        }
        return;
    }
    const int jstart = U[U_JS], jwin = U[U_JW];
    const long base = (long)m * (2 * L + 1 - m) / 2 + m;
    const int nj = L - m + 1;
    cdp bet = (cdp)P->beta + base;
    cip segexp = (cip)P->segexp + ((cip)P->segoff)[m];
    // this lane's coefficient of a group: degree offset 16 g + lane % 16
    const int lj = lane & (kGroup - 1);
    gcp gam = (gcp)(P->gamma + base);
    gcp qs[FW];
#pragma unroll
    for (int f = 0; f < FW; f++) qs[f] = (gcp)(a.in + qoff[f] + 2 * base);

    // Group operands: raw coefficients and gamma of this lane's degree
    // (clamped to the order's last), beta of the 16 degrees in SGPRs.
    double2 qa[FW], qb[FW];
    double ga, gb;
    auto load_q = [&](double2 (&q)[FW], double& g, int j0) {
        const unsigned j = (unsigned)min(j0 + lj, nj - 1);
        g = ld1(gam, 8 * j);
#pragma unroll
        for (int f = 0; f < FW; f++) q[f] = ld2(qs[f], 16 * j);
    };
    // gamma folded in; degrees past the order's last contribute exactly 0
    auto scale_q = [&](double2 (&q)[FW], double g, int j0) {
#pragma unroll
        for (int f = 0; f < FW; f++) q[f] = make_double2(g * q[f].x, g * q[f].y);
        if (j0 + kGroup > nj) {
            keep_branch();
            const bool in = j0 + lj < nj;
#pragma unroll
            for (int f = 0; f < FW; f++) q[f] = make_double2(in ? q[f].x : 0.0, in ? q[f].y : 0.0);
        }
        ready_for_dpp(q);
    };
    double ba[kGroup], bb[kGroup];
    auto load_b = [&](double (&b)[kGroup], int j0) {
        typedef const __attribute__((address_space(4))) DN<kGroup>* cbp;
        cbp pb16 = (cbp)(bet + j0);
#pragma unroll
        for (int i = 0; i < kGroup; i++) b[i] = pb16->v[i];
    };

    // The order runs in segments of 32 degrees: an even and an odd group.
    // Coefficients are loaded one segment ahead, beta one group ahead (the
    // table is padded, and no group past the order's last is loaded).
    const int js0 = jstart & ~(kSegLen - 1);
    load_q(qa, ga, js0);
    load_q(qb, gb, js0 + kGroup);
    // Lane starts: nearly every lane of a block starts at the block's first
    // start, from the state loaded here; the few that join later (4% of the
    // blocks at lmax 1023) load theirs when their step comes.
    SynthState<LP, FW> s;
    int sj[LP];
    gcp inj_y = (gcp)(P->inj_y + 2 * ((size_t)m * npair));
    {
        double2 y[LP];
        gcp inj_j = (gcp)(P->inj_j + (size_t)m * npair);
        gcp xp = (gcp)P->xp;
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const int pair = pb + p * 64 + lane;
            const unsigned pc = (unsigned)min(pair, npair - 1);
            y[p] = ld2(inj_y, 16 * pc);
            sj[p] = *(const __attribute__((address_space(1))) int*)(inj_j + 4 * pc);
            s.x[p] = ld1(xp, 8 * pc);
        }
        load_b(ba, js0);
#pragma unroll
        for (int p = 0; p < LP; p++) {
            if (pb + p * 64 + lane >= npair) sj[p] = nj;
            s.ua[p] = sj[p] == jstart ? y[p].x : 0.0;
            s.ub[p] = sj[p] == jstart ? y[p].y : 0.0;
#pragma unroll
            for (int f = 0; f < FW; f++) s.er[p][f] = s.ei[p][f] = s.orr[p][f] = s.oi[p][f] = 0.0;
        }
    }
    int shn = segexp[js0 / kSegLen];
    auto join = [&](int j) {
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const bool go = sj[p] == j;
            if (__any(go)) {
                const double2 y = ld2(inj_y, 16 * (unsigned)min(pb + p * 64 + lane, npair - 1));
                s.ua[p] = go ? y.x : s.ua[p];
                s.ub[p] = go ? y.y : s.ub[p];
                // (used here, so that the wait for the load stays in this branch)
                asm volatile("" : "+v"(s.ua[p]), "+v"(s.ub[p]));
            }
        }
    };

    // Half a group: kInject = 8 steps, from the first start on and while the
    // order has degrees; up to the last start, lanes join at its checkpoint.
    static_assert(kInject == 8 && kGroup == 16, "two start checkpoints per group");
#define SHTN_SYNTH_HALF(JH, T0, B, Q)                            \
    if ((JH) >= jstart && (JH) < nj) {                           \
        if ((JH) > jstart && (JH) <= jwin) {                     \
            keep_branch();                                       \
            join(JH);                                            \
        }                                                        \
        if (VEC && (JH) + 8 > nj)                                \
            synth_tail<LP, FW, T0, T0 + 8>(s, B, Q, nj - (JH));  \
        else                                                     \
            synth_steps<LP, FW, T0, T0 + 8>(s, B, Q);            \
    }
    __builtin_amdgcn_s_setprio(0);
    for (int js = js0; js < nj; js += kSegLen) {
        const int jn = js + kSegLen < nj ? js + kSegLen : js;  // next segment (or this one again: not used)
        const int jo = js + kGroup < nj ? js + kGroup : js;    // odd group (likewise)
        const int sh = js > jstart ? shn : 0;
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): ba and the shift
        __builtin_amdgcn_sched_barrier(0);
        load_b(bb, jo);
        shn = segexp[jn / kSegLen];
        __builtin_amdgcn_sched_barrier(0);
        rescale(s.ua, s.ub, sh);
        scale_q(qa, ga, js);
        SHTN_SYNTH_HALF(js, 0, ba, qa)
        SHTN_SYNTH_HALF(js + 8, 8, ba, qa)
        load_q(qa, ga, jn);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): bb
        __builtin_amdgcn_sched_barrier(0);
        load_b(ba, jn);
        __builtin_amdgcn_sched_barrier(0);
        scale_q(qb, gb, js + kGroup);
        SHTN_SYNTH_HALF(js + 16, 0, bb, qb)
        SHTN_SYNTH_HALF(js + 24, 8, bb, qb)
        load_q(qb, gb, jn + kGroup);
    }
#undef SHTN_SYNTH_HALF
    __builtin_amdgcn_s_setprio(3);

    // Mirror fold: north = E + O, south = E - O.  For the adjoint of the
    // analysis the output carries (2 pi/nphi) w_i / c_m.
    const double cm = a.adjoint ? (2.0 * M_PI / P->nphi) * (m == 0 ? 1.0 : 0.5) : 1.0;
    if constexpr (VEC) {
        // x P_L is odd about the equator where P_L is even
        const double gl = ((cdp)P->gamma)[base + nj - 1];
        double2 t[FW];
#pragma unroll
        for (int f = 0; f < FW; f++) {
            cdp tp = (cdp)a.top + 2 * ((long)(field0 + min(f, nf - 1)) * (P->M + 1) + m);
            t[f] = make_double2(tp[0], tp[1]);
        }
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const double xp = s.x[p] * (gl * ((nj & 1) ? s.ua[p] : s.ub[p]));
#pragma unroll
            for (int f = 0; f < FW; f++) {
                if (nj & 1) {
                    s.orr[p][f] = fma(xp, t[f].x, s.orr[p][f]);
                    s.oi[p][f] = fma(xp, t[f].y, s.oi[p][f]);
                } else {
                    s.er[p][f] = fma(xp, t[f].x, s.er[p][f]);
                    s.ei[p][f] = fma(xp, t[f].y, s.ei[p][f]);
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < LP; p++) {
        const int pair = pb + p * 64 + lane;
        if (pair >= npair) continue;
        double sc = a.adjoint ? cm * P->wfull[pair] : 1.0;
        if constexpr (VEC) sc = sc / sqrt((1.0 - s.x[p]) * (1.0 + s.x[p]));
        const int is = nlat - 1 - pair;
#pragma unroll
        for (int f = 0; f < FW; f++) {
            if (f >= nf) continue;
            double* F = a.out + foff[f];
            *(double2*)(F + 2 * f_index(fts, m, pair)) =
                make_double2(sc * (s.er[p][f] + s.orr[p][f]), sc * (s.ei[p][f] + s.oi[p][f]));
            if (is != pair)
                *(double2*)(F + 2 * f_index(fts, m, is)) = make_double2(sc * (s.er[p][f] - s.orr[p][f]),
                                                                        sc * (s.ei[p][f] - s.oi[p][f]));
        }
    }
}

// ---------------------------------------------------------------------------
// Analysis: Q_n^m = gamma_n sum_pairs u_n (w (F_N +- F_S)), one wave covers all
// latitude pairs of one order (64 LP >= npair) for a range of degrees.
// ---------------------------------------------------------------------------
template <int LP, int FW>
struct AState {
    double x[LP], ua[LP], ub[LP];
    // folded, weighted inputs: even-degree (w (F_N + F_S)) and odd-degree
    // (w (F_N - F_S)) parts, the component this lane keeps (k) and the one it
    // hands to its neighbour lane (s): even lanes keep the real part, odd
    // lanes the imaginary part
    double ek[LP][FW], es[LP][FW], ok[LP][FW], os[LP][FW];
};

// v of the neighbouring lane (lanes 2i and 2i+1 swap; DPP quad_perm [1,0,3,2]).
__device__ __forceinline__ double swap_lane_pair(double v)
{
    const long long b = __double_as_longlong(v);
    // every lane is active here, so the "old" operand is never used; passing
    // the source itself saves the moves that would initialise it
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, 0xB1, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), 0xB1, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Two recurrence steps, an even one (ua and the even inputs) and the odd one
// after it (ub and the odd inputs), on the pair slots PF..LP-1; the slots
// below PF belong to latitude blocks none of whose lanes has started, hold 0
// and would add exactly 0.  Both steps advance the recurrence first, then
// their four sums (kept and handed-over component of each step) are
// accumulated side by side over the slots, so four independent chains of
// fused multiply-adds share the latency.  Returns per field and step the
// lane pair's partial sum over its pairs of the kept component: real part on
// even lanes, imaginary part on odd lanes.
template <int LP, int FW, int PF>
__device__ __forceinline__ void analys_step_pair(AState<LP, FW>& s, double b0, double b1, double (&out0)[FW],
                                                 double (&out1)[FW])
{
#pragma unroll
    for (int p = PF; p < LP; p++) s.ua[p] = fma(s.x[p], s.ub[p], b0 * s.ua[p]);
#pragma unroll
    for (int p = PF; p < LP; p++) s.ub[p] = fma(s.x[p], s.ua[p], b1 * s.ub[p]);
    double sk0[FW], ss0[FW], sk1[FW], ss1[FW];
#pragma unroll
    for (int f = 0; f < FW; f++) sk0[f] = ss0[f] = sk1[f] = ss1[f] = 0.0;
#pragma unroll
    for (int p = PF; p < LP; p++) {
#pragma unroll
        for (int f = 0; f < FW; f++) {
            sk0[f] = fma(s.ek[p][f], s.ua[p], sk0[f]);
            ss0[f] = fma(s.es[p][f], s.ua[p], ss0[f]);
            sk1[f] = fma(s.ok[p][f], s.ub[p], sk1[f]);
            ss1[f] = fma(s.os[p][f], s.ub[p], ss1[f]);
        }
    }
#pragma unroll
    for (int f = 0; f < FW; f++) {
        out0[f] = sk0[f] + swap_lane_pair(ss0[f]);
        out1[f] = sk1[f] + swap_lane_pair(ss1[f]);
    }
}

// kInject steps (one start checkpoint to the next) on slots PF..LP-1, the
// rows of steps t0 .. t0 + kInject - 1 of the pass written to LDS (PF = LP:
// no slot live, zero rows).  t0 is even, so a step's parity is that of t.
template <int LP, int FW, int PF, int RS>
__device__ __forceinline__ void analys_half(AState<LP, FW>& s, const double (&b)[kInject], double* rows, int t0)
{
#pragma unroll
    for (int t = 0; t < kInject; t += 2) {
        double v0[FW], v1[FW];
        if (PF < LP) {
            analys_step_pair<LP, FW, PF>(s, b[t], b[t + 1], v0, v1);
        } else {
#pragma unroll
            for (int f = 0; f < FW; f++) v0[f] = v1[f] = 0.0;
        }
#pragma unroll
        for (int f = 0; f < FW; f++) {
            rows[((t0 + t) * FW + f) * RS] = v0[f];
            rows[((t0 + t + 1) * FW + f) * RS] = v1[f];
        }
    }
}

// The half for the first live slot pf (wave-uniform).
template <int LP, int FW, int RS>
__device__ __forceinline__ void analys_half_from(int pf, AState<LP, FW>& s, const double (&b)[kInject],
                                                 double* rows, int t0)
{
    // (pf <= LP; a case k >= LP is the no-live-slot variant: zero rows)
    switch (pf) {
    case 0: analys_half<LP, FW, 0, RS>(s, b, rows, t0); break;
    case 1: analys_half<LP, FW, (1 < LP ? 1 : LP), RS>(s, b, rows, t0); break;
    case 2: analys_half<LP, FW, (2 < LP ? 2 : LP), RS>(s, b, rows, t0); break;
    case 3: analys_half<LP, FW, (3 < LP ? 3 : LP), RS>(s, b, rows, t0); break;
    case 4: analys_half<LP, FW, (4 < LP ? 4 : LP), RS>(s, b, rows, t0); break;
    case 5: analys_half<LP, FW, (5 < LP ? 5 : LP), RS>(s, b, rows, t0); break;
    case 6: analys_half<LP, FW, (6 < LP ? 6 : LP), RS>(s, b, rows, t0); break;
    case 7: analys_half<LP, FW, (7 < LP ? 7 : LP), RS>(s, b, rows, t0); break;
    default: analys_half<LP, FW, LP, RS>(s, b, rows, t0); break;
    }
}

// The degrees of a unit run in passes of SC = kChunk / FW degrees.  In a pass
// each lane pair's partial sums (one row per degree and field, one column
// per thread: real parts in even columns, imaginary parts in odd ones) go to
// LDS, while the sums of the previous pass are read back, added over the
// columns (two lanes per output, padded rows) and stored.  The rows are the
// wave's own and lie in one buffer: one wave executes its LDS operations in
// order, so the reads of the previous pass, issued before this pass's writes,
// need no barrier.
// A workgroup of W waves covers 64 LP W latitude pairs, 64 LP consecutive ones
// per wave, pair slot p of a wave's lanes being one 64-pair block.  A pass
// runs as halves of kInject steps; each half first injects the start states of
// the blocks with lanes starting at its checkpoint, then runs only the slots
// from the first one whose block has started (the polar optimisation of Sec.
// 3.1 at the granularity of 64 latitudes).
// With W > 1 the waves run apart for chunks of kWideChunk degrees: each puts
// its sums in LDS, and at the end of a chunk the workgroup adds them up and
// stores the outputs.  (With the waves in step for every pass, as before, all
// of them took as long as the one at the equator, and the SIMD it ran on set
// the time: lmax 4095 2,747 -> 2,407 us, lmax 2047 337 -> 323.)
constexpr int kWideChunk = 256;

template <int LP, int FW, int W>
struct AnalysGeom {
    static constexpr int SC = kChunk / FW;  // degrees per pass
    static constexpr int NR = SC * FW;      // rows per pass
    static constexpr int NT = 64;           // columns
    static constexpr int PR = 2;            // lanes per output (row, component)
    static constexpr int NK = NT / 2 / PR;  // columns each of them adds
    // row stride NT + 2 PR doubles: a lane's PR-wide column groups of
    // consecutive rows start 4 PR banks apart, so the 32 lanes of a half-wave
    // read distinct banks
    static constexpr int RS = NT + 2 * PR;
    static constexpr int NH = SC / kInject;  // halves per pass
    // sums of a chunk: one per wave, degree, field and component
    static constexpr int NA = W > 1 ? kWideChunk * FW * 2 : 1;
};

// One unit: degrees [j0, j1) of one order for all latitude pairs (the
// workgroup's W waves), the outputs stored; uniform over the workgroup.
template <int LP, int FW, int W>
__device__ __forceinline__ void analys_unit(
    const LegArgs& a, int ui,
    double (&red_w)[W][AnalysGeom<LP, FW, W>::NR][AnalysGeom<LP, FW, W>::RS],
    double (&acc)[W][AnalysGeom<LP, FW, W>::NA])
{
    using G = AnalysGeom<LP, FW, W>;
    constexpr int SC = G::SC, NR = G::NR, NT = G::NT, PR = G::PR, NK = G::NK, RS = G::RS, NH = G::NH;
    static_assert(2 * NR * PR == NT, "the lanes cover the outputs");
    static_assert(kSegLen % SC == 0, "passes tile a segment");
    static_assert(SC % kInject == 0, "passes are whole halves");
    static_assert(kInject % 2 == 0, "halves keep the step parity");
    static_assert(LP <= 8 && LP * W <= kMaxMaskBlocks, "one mask word covers the unit's blocks");

    __builtin_amdgcn_s_setprio(3);
    cip U = (cip)a.units + (size_t)ui * kUnitInts;
    const int m = U[U_M];
    if (m < 0) return;
    const int field0 = U[U_FIELD] + blockIdx.y * FW;
    if (field0 >= a.nfields) return;
    const int nf = min(U[U_NF], a.nfields - field0);
    cplan P = (cplan)a.plans + U[U_PLAN];
    const int L = P->L, nlat = P->nlat, npair = P->npair;
    const long fts = P->f_ts;
    const long nlm = P->nlm;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // which part of the latitudes a wave takes turns with the unit: the waves
    // near the pole have less to do, and a workgroup's waves go to the SIMDs
    // in a fixed order
    const int wid = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int wv = W > 1 ? (wid + ui / kXcds) & (W - 1) : 0;
    const int pb = wv * 64 * LP;  // first latitude pair of this wave
    const int wb = wv * LP;       // its first 64-pair block
    const int j0 = U[U_PB], j1 = U[U_J1], js0 = U[U_JS], jwin = U[U_JW], rst = U[U_RST];
    const long base = (long)m * (2 * L + 1 - m) / 2 + m;
    const int nj = L - m + 1;
    cdp bet = (cdp)P->beta + base;
    cip segexp = (cip)P->segexp + ((cip)P->segoff)[m];
    // per checkpoint: blocks with lanes starting there, blocks started
    cip ckm = (cip)P->ck_mask + (size_t)m * P->nck * 2;
    double (&red)[NR][RS] = red_w[wid];

    long qoff[FW];
    long foff[FW];
#pragma unroll
    for (int f = 0; f < FW; f++) {
        const int ff = field0 + min(f, nf - 1);
        qoff[f] = field_q_off(a, ff, nlm);
        foff[f] = field_f_off(a, ff, P->f_size);
    }

    // degrees before the first started lane: every term is dropped
    for (int j = j0 + (tid >> 1); j < js0; j += 32 * W) {
#pragma unroll
        for (int f = 0; f < FW; f++)
            if (f < nf) a.out[qoff[f] + 2 * (base + j) + (tid & 1)] = 0.0;
    }
    if (js0 >= j1) return;

    // Unit setup.  Every global load is issued before any of them is used
    // (indices clamped to valid entries, inactive lanes masked afterwards),
    // so the setup costs one memory round trip.
    AState<LP, FW> s;
    const bool from_rst = rst >= 0 && js0 == j0;
    {
        const bool odd = lane & 1;
        int pc[LP];
        bool act[LP];
        double xv[LP], wl[LP];
        double2 r[LP], fn[LP][FW], fsth[LP][FW];
#pragma unroll
        for (int p = 0; p < LP; p++) {
            const int pair = pb + p * 64 + lane;
            act[p] = pair < npair;
            pc[p] = act[p] ? pair : 0;
            xv[p] = P->xp[pc[p]];
            wl[p] = P->wq[pc[p]];
#pragma unroll
            for (int f = 0; f < FW; f++) {
                const double* F = a.in + foff[f];
                fn[p][f] = *(const double2*)(F + 2 * f_index(fts, m, pc[p]));
                fsth[p][f] = *(const double2*)(F + 2 * f_index(fts, m, nlat - 1 - pc[p]));
            }
        }
        if (from_rst) {
#pragma unroll
            for (int p = 0; p < LP; p++)
                r[p] = *(const double2*)(P->rst_y + 2 * ((size_t)rst * npair + pc[p]));
        } else {
#pragma unroll
            for (int p = 0; p < LP; p++) r[p] = make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int p = 0; p < LP; p++) {
            s.x[p] = act[p] ? xv[p] : 0.0;
            s.ua[p] = act[p] ? r[p].x : 0.0;
            s.ub[p] = act[p] ? r[p].y : 0.0;
            // folded, weighted inputs; a lane that has not started holds a
            // zero state, so it adds exactly 0 whatever its inputs
            const bool middle = (nlat & 1) && pc[p] == npair - 1;
            const double wt = !act[p] ? 0.0 : (a.adjoint ? (middle ? 0.5 : 1.0) : wl[p]);
#pragma unroll
            for (int f = 0; f < FW; f++) {
                const double2 vn = fn[p][f], vs = fsth[p][f];
                const double er = wt * (vn.x + vs.x), ei = wt * (vn.y + vs.y);
                const double orr = wt * (vn.x - vs.x), oi = wt * (vn.y - vs.y);
                s.ek[p][f] = odd ? ei : er;
                s.es[p][f] = odd ? er : ei;
                s.ok[p][f] = odd ? oi : orr;
                s.os[p][f] = odd ? orr : oi;
            }
        }
    }

    // Warm L2 with the beta entries of this unit (one word per 64-byte line
    // per lane, consumed at the end).
    __builtin_amdgcn_sched_barrier(0);
    unsigned pf_sink;
    {
        const int nbytes = (j1 - js0 + 2 * SC) * 8;
        const int off = lane * 64;
        pf_sink = *(const unsigned*)((const char*)(P->beta + base + js0) + (off < nbytes ? off : 0));
    }
    __builtin_amdgcn_s_setprio(0);
    const double cm = (m == 0 || !a.adjoint) ? 1.0 : 2.0;
    const int o = lane / PR;       // output of this lane: (row, component)
    const int h = lane % PR;       // its part of the columns
    const int row = o >> 1, comp = o & 1;
    const int t_out = row / FW;
    const int f_out = row % FW;
    cdp gam_tab = (cdp)P->gamma + base;

    // beta is loaded one half ahead (the second half's while the first
    // runs, the next pass's first half's after an explicit wait for the
    // second), the segment shift and the start masks one pass ahead; the
    // tables are padded past the last order.  Each explicit lgkmcnt(0) wait
    // comes before the next scalar load is issued, so no wait drains a load
    // just issued (scalar loads return out of order: a wait is always for
    // all of them).  A partial last pass runs all SC steps: the extra
    // degrees belong to no output and are not stored.
    static_assert(NH == 1 || NH == 2, "one or two halves per pass");
    DBlk<kInject> bh0, bh1;
    load_blk(bh0, bet + js0);
    DBlk2u<2 * NH> mkw;
    load_u32(mkw, ckm + 2 * (js0 / kInject));
    int shn = 0;        // js0 is a segment start (the plan rounds it down)
    for (int c = js0; c < j1 + SC; c += SC) {
        const bool compute = c < j1;
        const int sh = shn;
        // The scalar loads above have arrived before the LDS reads of the
        // previous pass's sums are issued (one counter covers both kinds), so
        // the steps below wait on neither and the reads complete under them.
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        // this wave's slots: starting at each checkpoint, started by it
        unsigned mk[NH], lv[NH];
#pragma unroll
        for (int hh = 0; hh < NH; hh++) {
            mk[hh] = (mkw.v[2 * hh] >> wb) & ((1u << LP) - 1u);
            lv[hh] = (mkw.v[2 * hh + 1] >> wb) & ((1u << LP) - 1u);
        }
        double part[NK];
#pragma unroll
        for (int k = 0; k < NK; k++) part[k] = red[row][2 * (k * PR + h) + comp];
        // gamma of this lane's output in that pass, needed after the steps
        const double gl = W > 1 ? 0.0 : gam_tab[min(max(c - SC, js0) + t_out, j1 - 1)];
        if (compute) {
            const int cn = c + SC;
            // two halves: the second half's beta; one half: the next pass's
            load_blk(bh1, bet + c + kInject);
            load_u32(mkw, ckm + 2 * (cn / kInject));
            shn = (cn < j1 && cn % kSegLen == 0) ? segexp[cn / kSegLen] : 0;
            __builtin_amdgcn_sched_barrier(0);
            if (sh != 0) rescale(s.ua, s.ub, sh);
            if (mk[0] != 0u && c <= jwin) start_slots(s.ua, s.ub, P, m, pb, mk[0], c);
            analys_half_from<LP, FW, RS>(lv[0] ? __builtin_ctz(lv[0]) : LP, s, bh0.v, &red[0][lane], 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NH == 2) {
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): bh1, the masks, the shift
                __builtin_amdgcn_sched_barrier(0);
                load_blk(bh0, bet + cn);
                __builtin_amdgcn_sched_barrier(0);
                const int c1 = c + kInject;
                if (mk[1] != 0u && c1 <= jwin) start_slots(s.ua, s.ub, P, m, pb, mk[1], c1);
                analys_half_from<LP, FW, RS>(lv[1] ? __builtin_ctz(lv[1]) : LP, s, bh1.v, &red[0][lane], kInject);
            } else {
                bh0 = bh1;
            }
        }
        if (c > js0) {
            double s0 = part[0], s1 = part[1], s2 = part[2], s3 = part[3];
#pragma unroll
            for (int k = 4; k < NK; k += 4) {
                s0 += part[k];
                s1 += part[k + 1];
                s2 += part[k + 2];
                s3 += part[k + 3];
            }
            double sum = (s0 + s1) + (s2 + s3);
#pragma unroll
            for (int q = 1; q < PR; q <<= 1) sum += __shfl_xor(sum, q);
            const int j_out = c - SC + t_out;
            if constexpr (W == 1) {
                if (h == 0 && j_out < j1 && f_out < nf) {
                    double val = cm * gl * sum;
                    if (m == 0 && comp == 1) val = 0.0;
                    a.out[qoff[f_out] + 2 * (base + j_out) + comp] = val;
                }
            } else {
                const int jc = (c - SC - js0) & ~(kWideChunk - 1);  // first degree of the chunk, from js0
                // (by latitudes: the order of the sum is the same for every unit)
                if (h == 0) acc[wv][((j_out - js0 - jc) * FW + f_out) * 2 + comp] = sum;
                if (c >= j1 || (c - js0) % kWideChunk == 0) {
                    // the chunk's last pass is in: add up the waves' sums
                    __syncthreads();
                    const int n = min(kWideChunk, j1 - js0 - jc) * FW * 2;
                    for (int e = tid; e < n; e += 64 * W) {
                        double v = acc[0][e];
#pragma unroll
                        for (int w = 1; w < W; w++) v += acc[w][e];
                        const int f = (e >> 1) % FW, j = js0 + jc + (e >> 1) / FW;
                        if (f < nf) {
                            v *= cm * P->gamma[base + j];
                            if (m == 0 && (e & 1)) v = 0.0;
                            a.out[qoff[f] + 2 * (base + j) + (e & 1)] = v;
                        }
                    }
                    __syncthreads();
                }
            }
        }
    }
    // keeps the prefetch load alive; nfields is never negative
    if (a.nfields < 0) a.out[lane] = (double)pf_sink;
}

// One workgroup per unit.
template <int LP, int FW, int W>
__global__ void __launch_bounds__(64 * W) k_legendre_analys(LegArgs a)
{
    using G = AnalysGeom<LP, FW, W>;
    __shared__ double red[W][G::NR][G::RS];
    __shared__ double acc[W][G::NA];
    analys_unit<LP, FW, W>(a, blockIdx.x, red, acc);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int LP, int FW, bool VEC>
static int launch_synth_t(const LegLaunch& l, void* stream)
{
    // (a launch's threads are counted in 32 bits: one launch unless the call
    // has far more fields than the card holds)
    const int most = std::max(1, (1 << 25) / l.nunits);
    for (int g0 = 0; g0 < l.grid_y; g0 += most) {
        const int ng = std::min(most, l.grid_y - g0);
        // two waves per SIMD or fewer: one per workgroup (lmax 255, one
        // field: 10.2 us, with four 11.2; lmax 511: 16.2, with four 17.9)
        const int waves = (long)l.nunits * ng > 2048 ? kSynthWaves : 1;
        LegArgs a{l.plans, l.units, l.q_off, l.f_off, l.in, l.out, l.nfields, l.adjoint, l.nunits, ng, g0, waves, l.top,
                  l.rotate};
        const int per_xcd = (l.nunits / kXcds * ng + waves - 1) / waves;
        hipLaunchKernelGGL((k_legendre_synth<LP, FW, VEC>), dim3(kXcds * per_xcd), dim3(64 * waves), 0,
                           (hipStream_t)stream, a);
    }
    return (int)hipGetLastError();
}

template <int LP, int FW, int W>
static int launch_analys_t(const LegLaunch& l, void* stream)
{
    LegArgs a{l.plans, l.units, l.q_off, l.f_off, l.in, l.out, l.nfields, l.adjoint, l.nunits, 1, 0, W};
    hipLaunchKernelGGL((k_legendre_analys<LP, FW, W>), dim3(l.nunits, l.grid_y), dim3(64 * W), 0,
                       (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_legendre_synth(const LegLaunch& l, void* stream)
{
    if (l.nunits <= 0) return 0;
#define SHTN_S(LPV, FWV) \
    if (l.lp == LPV && l.fw == FWV && !l.top) return launch_synth_t<LPV, FWV, false>(l, stream);
    SHTN_S(1, 1) SHTN_S(2, 1) SHTN_S(4, 1)
    SHTN_S(1, 2) SHTN_S(2, 2) SHTN_S(4, 2)
    SHTN_S(1, 4) SHTN_S(2, 4)
#undef SHTN_S
    // (vector transforms: the combinations an automatic tiling takes; two pairs
    // and four fields per lane would need more registers than four waves per
    // SIMD have)
#define SHTN_V(LPV, FWV) \
    if (l.lp == LPV && l.fw == FWV && l.top) return launch_synth_t<LPV, FWV, true>(l, stream);
    SHTN_V(1, 1) SHTN_V(2, 1) SHTN_V(1, 2) SHTN_V(2, 2) SHTN_V(1, 4)
#undef SHTN_V
    return (int)hipErrorInvalidValue;
}

int launch_legendre_analys(const LegLaunch& l, void* stream)
{
    if (l.nunits <= 0) return 0;
#define SHTN_A(LPV, FWV, WV) \
    if (l.lp == LPV && l.fw == FWV && l.waves == WV) return launch_analys_t<LPV, FWV, WV>(l, stream);
    SHTN_A(1, 1, 1) SHTN_A(2, 1, 1) SHTN_A(4, 1, 1) SHTN_A(8, 1, 1)
    SHTN_A(1, 2, 1) SHTN_A(2, 2, 1) SHTN_A(4, 2, 1)
    SHTN_A(2, 1, 2) SHTN_A(4, 1, 2) SHTN_A(8, 1, 2)
    SHTN_A(2, 2, 2) SHTN_A(4, 2, 2)
    SHTN_A(4, 1, 4) SHTN_A(8, 1, 4)
#undef SHTN_A
    return (int)hipErrorInvalidValue;
}

}  // namespace shtn
