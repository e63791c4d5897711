// Device helpers shared by the on-the-fly Legendre kernels (legendre.hip,
// analys_mf.hip): scalar and vector loads, launch arguments, recurrence states.
#pragma once

#include <hip/hip_runtime.h>

#include "shtn_internal.h"

namespace shtn {

typedef const __attribute__((address_space(4))) double* cdp;
typedef const __attribute__((address_space(4))) int* cip;
typedef const __attribute__((address_space(4))) long* clp;
typedef const __attribute__((address_space(4))) DevPlan* cplan;
typedef const __attribute__((address_space(1))) char* gcp;

// Loads at a 32-bit byte offset from a wave-uniform base.
__device__ __forceinline__ double ld1(gcp base, unsigned off)
{
    return *(const __attribute__((address_space(1))) double*)(base + off);
}
__device__ __forceinline__ double2 ld2(gcp base, unsigned off)
{
    const __attribute__((address_space(1))) double* p = (const __attribute__((address_space(1))) double*)(base + off);
    return make_double2(p[0], p[1]);
}

// A block of wave-uniform scalar operands.
template <int N>
struct DN {
    double v[N];
};

struct LegArgs {
    const DevPlan* plans;
    const int* units;
    const long* q_off;  // per field: spectrum offset in doubles (null: f * 2 nlm)
    const long* f_off;  // per field: F offset in doubles (null: f * 2 f_size)
    const double* in;
    double* out;
    int nfields;
    int adjoint;
    int nunits;
    // synthesis: field groups (of FW fields) of this launch, and the first one
    int groups, group0;
    int waves;  // synthesis: waves per workgroup
    // vector transforms: per (field, order) the coefficient of x P_L (synthesis),
    // or the sum with x P_L (analysis), at 2 (f (M+1) + m)
    double* top = nullptr;
    int rotate = 0;  // synthesis: a unit's field groups go to the XCDs in turn (see synth_unit)
};

__device__ __forceinline__ long field_q_off(const LegArgs& a, int f, long nlm)
{
    return a.q_off ? ((clp)a.q_off)[f] : (long)f * 2 * nlm;
}

__device__ __forceinline__ long field_f_off(const LegArgs& a, int f, long fsize)
{
    return a.f_off ? ((clp)a.f_off)[f] : (long)f * 2 * fsize;
}

// Segment shift of the recurrence states.
template <int LP>
__device__ __forceinline__ void rescale(double (&ua)[LP], double (&ub)[LP], int sh)
{
#pragma unroll
    for (int p = 0; p < LP; p++) {
        ua[p] = __builtin_amdgcn_ldexp(ua[p], sh);
        ub[p] = __builtin_amdgcn_ldexp(ub[p], sh);
    }
}

template <int N>
struct DBlk {
    double v[N];
};

template <int N>
struct DBlk2u {
    unsigned v[N];
};

// A block of N wave-uniform 32-bit words through the scalar cache.
template <int N>
__device__ __forceinline__ void load_u32(DBlk2u<N>& d, cip src)
{
    typedef const __attribute__((address_space(4))) DBlk2u<N>* cbp;
    cbp p = (cbp)src;
#pragma unroll
    for (int i = 0; i < N; i++) d.v[i] = p->v[i];
}

// A block of N wave-uniform doubles through the scalar cache.
template <int N>
__device__ __forceinline__ void load_blk(DBlk<N>& d, cdp src)
{
    typedef const __attribute__((address_space(4))) DBlk<N>* cbp;
    cbp p = (cbp)src;
#pragma unroll
    for (int i = 0; i < N; i++) d.v[i] = p->v[i];
}

// Start checkpoint cc: in the slots whose block has a lane starting there
// (bits of mk, wave-uniform), the lanes whose start step is cc take their
// stored state, loaded here: few units start lanes (two or three blocks per
// unit at lmax 1023), and the states of the others are never read.
// (one slot, whose first latitude pair is pb)
__device__ __forceinline__ void start_slot(double& ua, double& ub, cplan P, int m, int pb, int cc)
{
    const int npair = P->npair;
    const int pair = pb + (threadIdx.x & 63);
    const unsigned pc = (unsigned)min(pair, npair - 1);
    const int sj = *(const __attribute__((address_space(1))) int*)((gcp)(P->inj_j + (size_t)m * npair) + 4 * pc);
    const double2 y = ld2((gcp)(P->inj_y + 2 * ((size_t)m * npair)), 16 * pc);
    const bool go = pair < npair && sj == cc;
    ua = go ? y.x : ua;
    ub = go ? y.y : ub;
    // (used here, so that the wait for the loads stays in the caller's branch)
    asm volatile("" : "+v"(ua), "+v"(ub));
}

template <int LP>
__device__ __forceinline__ void start_slots(double (&ua)[LP], double (&ub)[LP], cplan P, int m, int pb, unsigned mk,
                                            int cc)
{
#pragma unroll
    for (int p = 0; p < LP; p++)
        if (mk & (1u << p)) start_slot(ua[p], ub[p], P, m, pb + p * 64, cc);
}

}  // namespace shtn
