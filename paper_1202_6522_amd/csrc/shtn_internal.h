// Internal structures shared by the host plan code, the C-ABI layer and the
// HIP kernels.  Not part of the public interface (include/shtn.h).
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace shtn {

// Rescaled recurrence (Sec. 3.2, eq. rec, divided through by
// alpha_n = prod_{j=m+1}^{n} a_j^m):
//   y_n = x y_{n-1} + beta_n y_{n-2},  beta_n = -((n-1)^2 - m^2)/((2n-1)(2n-3)),
//   P_n^m(x) = alpha_n y_n.
// The kernels carry u_n = y_n 2^{E_s} where E_s is constant over a segment of
// kSegLen consecutive degrees, so u stays within the range of P; at a segment
// start both recurrence states are multiplied by 2^{E_s - E_{s-1}} (exact).
// gamma_n = alpha_n 2^{-E_s} maps u back to P.
constexpr int kSegLen = 32;
// Underflow guard (Sec. 3.5), run at plan time: the host follows every
// (order, latitude pair) recurrence from n = m in a scaled form
// u = w 2^{-kGuardUnit k} (every kGuardEvery steps a value with k > 0 and
// |w| >= 1 is multiplied by 2^{-kGuardUnit} and k decremented), so values far
// below the double range are tracked exactly.
constexpr int kGuardUnit = 256;
constexpr int kGuardEvery = 4;
// Polar threshold (Sec. 3.1, polar optimisation): contributions with
// |P_n^m| < 2^kPolarLog2 are dropped (the default; a plan may raise the
// threshold, trading accuracy for work, see Plan::polar_log2).  A lane starts at the first checkpoint
// (a multiple of kInject steps) of the block of kInject steps in which its
// |P_n^m| first reaches 2^kPolarLog2 -- or earlier, at the first start of
// its 64-pair block, when its state there is a normal double (see
// lane_starts); before its start the lane holds 0, so it adds exactly 0 and
// the kernels carry no exponent.  The host stores the state (u_{j-2},
// u_{j-1}) entering that step as plain doubles.  A block none of whose
// latitudes reaches the threshold for an order never starts.
constexpr int kPolarLog2 = -200;
constexpr int kInject = 8;
// Analysis accumulates kChunk consecutive degrees per lane before a
// cross-lane reduction.
constexpr int kChunk = 16;
// Entries of zero padding after the table that the kernels read in blocks
// (beta): a block starting at an order's last degree
// stays in bounds.
constexpr int kTablePad = 32;
// Pairs per lane and waves of an analysis unit covering npair latitude pairs
// (the smallest power-of-two coverage, up to 8 pairs per lane first).
inline void analys_shape(int npair, int& lp, int& waves)
{
    lp = 1;
    waves = 1;
    while (64 * lp * waves < npair) {
        if (lp < 8) lp *= 2;
        else waves *= 2;
    }
}
// Largest latitude-pair count one analysis unit covers (4 waves x 64 lanes x
// 8 pairs).
constexpr int kMaxAnalysPairs = 2048;

// One work unit of a Legendre kernel = one wave (kUnitInts ints).  Steps j
// count degrees from the order: n = m + j.
enum UnitField {
    U_FIELD = 0,  // first field of the unit (relative; plus blockIdx.y * fw for plan calls)
    U_NF = 1,     // number of fields in the unit (<= fw)
    U_PLAN = 2,   // plan index (batch) or 0
    U_M = 3,      // order m, or -1 for a unit without work
    U_JS = 4,     // first step executed (lanes start there or later)
    U_JW = 5,     // last step at which a lane of the unit starts (injection window; analysis: -1 if none)
    U_PB = 6,     // synthesis: first latitude pair of the block; analysis: first output step j0
    U_J1 = 7,     // analysis: one past the last output step
    U_RST = 8,    // analysis: restart slot of j0 or -1 (j0 = 0)
    U_ZERO = 9,   // synthesis: 1 if no lane of the block ever starts (F written as 0)
};
constexpr int kUnitInts = 12;

// A synthesis unit and its work (steps from the first start on; 0 for a unit
// that only writes zeros).
struct SynthUnit {
    int u[kUnitInts];
    long cost;
};

// Tables of a plan's device buffer, in buffer order (Plan::table_off).
enum DevTable {
    TB_XP = 0,
    TB_WQ,
    TB_WFULL,
    TB_BETA,
    TB_GAMMA,
    TB_INJ_J,
    TB_INJ_Y,
    TB_SEGEXP,
    TB_SEGOFF,
    TB_RST_Y,
    TB_TW,
    TB_RTW,
    TB_SYNTH_UNITS,
    TB_ANALYS_UNITS,
    TB_CK_MASK,
    TB_MF_UNITS,  // kMfLists - 1 tables (list 0 is TB_ANALYS_UNITS)
    TB_SHORT_UNITS = TB_MF_UNITS + 2,
    TB_COUNT
};
// Unit lists of the several-field analysis: pieces of 1, 2 and 4 times the
// plan's split.
constexpr int kMfLists = 3;
static_assert(TB_SHORT_UNITS == TB_MF_UNITS + kMfLists - 1, "one table per further list");
// Waves of an analysis with pieces of 64 degrees up to which pieces of 32 are
// the faster: there are SIMDs to spare, and a wave's time is its steps
// (one field, us: lmax 127 8.1 and 7.2, 255 9.9 and 8.0, 400, of 1470 waves, 13.0
// and 11.8; 450, of 1860, 13.5 and 14.0; two fields at lmax 340, of 2160, 13.9 and
// 14.9).
constexpr long kShortUnits = 1600;

// Lane-start summaries per block of 64 latitude pairs (the pair slot of a
// wave lane: pairs [64 b, 64 b + 64) form block b).  blk_first[m][b]: the
// first start step of the block's lanes of order m (nj if none starts; host
// only).  ck_mask[m][2 k]: bit b set iff some lane of block b starts at the
// checkpoint j = kInject k; ck_mask[m][2 k + 1]: bit b set iff some lane of
// block b has started at or before it.  A kernel skips the slots whose block
// has not started and injects start states only into the blocks whose bit is
// set.
constexpr int kBlkPairs = 64;
constexpr int kMaxMaskBlocks = 32;  // blocks one 32-bit mask covers (2048 pairs)

// Device-resident view of a plan (stored at the start of its device buffer).
struct DevPlan {
    const double* xp;      // [npair] x = cos(theta) of the northern node of each pair
    const double* wq;      // [npair] analysis weight per pair (middle node of odd nlat halved)
    const double* wfull;   // [npair] Gauss weight per pair
    const double* beta;    // [nlm] rescaled recurrence coefficient, m-major
    const double* gamma;   // [nlm] output scale gamma_n
    const int* inj_j;      // [(M+1) * npair] step at which the lane starts (n = m + j), or > lmax - m
    const double* inj_y;   // [(M+1) * npair * 2] state (u_{j-2}, u_{j-1}) entering that step
    const int* segexp;     // per (m, segment s >= 1): E_s - E_{s-1}
    const int* segoff;     // [M+2] index of (m, s=0) in segexp
    const double* rst_y;   // [nrst * npair * 2] analysis restart states (ua, ub), 0 before a lane starts
    const double* tw;      // [K] complex e^{-2 pi i t / K}
    const double* rtw;     // [K+1] complex e^{+2 pi i m / (2K)}
    const int* synth_units;
    const int* analys_units;
    const unsigned* ck_mask;  // [(M+1) * nck * 2] per checkpoint: blocks starting there, blocks started
    int nblk, nck;
    int L, M, nlat, nphi, npair, K;
    long nlm;
    int n_synth_units, n_analys_units;
    int synth_lp, analys_lp, fw, pad0;
    // Longitude coefficients of one field: tile stride and size (complex).
    long f_ts, f_size;
};

struct Tiling {
    int synth_lp = 1;
    int analys_lp = 8;
    int analys_waves = 1;  // waves per analysis unit
    int fw = 1;         // fields per wave
    bool auto_fw = true;  // no tiling set: fields per wave and kernels are chosen per call
    int m_pairing = 0;  // synthesis: 1 = long and short units alternate in the launch order
    int split = 0;     // analysis: pieces of this many degrees, 0 = automatic
    int fft_rows = 0;  // latitude rows per FFT workgroup, 0 = automatic
};

// Stored-P table of a plan (Sec. 3, precomputed P_n^m; ptable.hip): P_n^m
// at the northern latitude pairs per (order, parity of n - m) in 16 x 16
// blocks of (degree row, pair), rows and pairs zero-padded to 16.  The device
// buffer holds the block offsets (boff) first, then the blocks.
struct PTable {
    int npt = 0;              // pair tiles of 16
    std::vector<long> boff;   // [(M+1) * 2] first block of (order, parity)
    long nblocks = 0;
    size_t head_bytes = 0;    // boff, padded to 256 bytes
    void* dev = nullptr;      // caller's buffer once built
    bool built = false;       // matches the plan's current lane starts
    int synth_rt = 4, synth_ct = 2;    // synthesis: pair tiles, column tiles per wave
    int analys_jt = 4, analys_ct = 2;  // analysis: block rows per parity, column tiles per wave
    // until a decomposition is set, both run one tile per wave: the waves of a
    // workgroup share the inputs through LDS, so more tiles per wave save no
    // reads and leave fewer waves (16 fields, synthesis and analysis in us, 1,
    // 2 and 4 tiles: lmax 511 71.5 and 84.6, 71.9 and 88.4, 73.2 and 90.4;
    // lmax 255 18.7 and 22.5, 21.7 and 24.8, 31.6 and 32.8)
    bool auto_tiles = true;
    int rt() const { return auto_tiles ? 1 : synth_rt; }
    int jt() const { return auto_tiles ? 1 : analys_jt; }
    // column tiles: 0 = by the number of fields (ptable.hip)
    int sct() const { return auto_tiles ? 0 : synth_ct; }
    int act() const { return auto_tiles ? 0 : analys_ct; }
};

struct Plan {
    int L = 0, M = 0, nlat = 0, nphi = 0, npair = 0, K = 0;
    long nlm = 0;
    Tiling tiling;
    int split_used = 0;
    int polar_log2 = kPolarLog2;  // lanes start where |P_n^m| first reaches 2^polar_log2
    // host tables
    std::vector<double> x, w;                 // full grid
    std::vector<double> xp, sp, wq, wfull;    // per pair
    std::vector<double> beta, gamma;          // nlm
    std::vector<double> start_y;              // (M+1) x npair: P_m^m mantissa (host emulation only)
    std::vector<int> start_k;                 // its scaled exponent
    std::vector<int> inj_j;                   // (M+1) x npair: lane start step
    bool late_starts = false;                 // some lane starts past its order's first degree
    std::vector<double> inj_y;                // (M+1) x npair x 2: state entering it
    std::vector<int> segexp, segoff;
    std::vector<double> rst_y;
    std::vector<double> tw, rtw;
    std::vector<int> synth_units, analys_units;
    std::vector<int> mf_units[kMfLists];
    std::vector<int> short_units;             // half pieces (see kShortUnits), or empty
    std::vector<int> first_pair;              // per m: first latitude pair kept by the polar cut
    double min_own_state = 0.0;               // see min_start_state
    std::vector<int> blk_first;               // (M+1) x nblk, see TB_BLK_FIRST
    std::vector<unsigned> ck_mask;            // (M+1) x nck x 2, see TB_CK_MASK
    int nblk = 0, nck = 0;
    // device image
    std::vector<unsigned char> image;  // staged device buffer contents
    std::vector<size_t> table_off;     // byte offsets of each table inside the image
    void* dev = nullptr;               // caller's device buffer after upload
    bool uploaded = false;
    PTable ptab;
    int algo = 0;  // Legendre stage: 0 on-the-fly recurrence, 1 stored P
    // Bumped by every change that moves the plan's device state or its lane
    // starts (upload, tiling, polar threshold, stored-P build or release):
    // batches that copied the plan's device descriptor or built unit tables
    // from its lane starts compare it to refuse stale copies.
    unsigned long gen = 0;
};
// Smallest nonzero |state| at the lanes' own threshold starts, or 0 if
// none: below DBL_MIN a start state at the threshold would be a denormal
// that has lost precision (the threshold is then too low for the plan).
double min_start_state(const Plan& p);
void ptable_layout(Plan& p);  // geometry of the stored-P table

// Error reporting shared by the C-ABI sources (api.cpp): sets the detail
// string of shtn_last_error_detail and returns the code.
int set_error(int code, const std::string& msg);

// A device byte range a call touches; `written` when the call writes it.
struct Range {
    const char* what;
    const void* p;
    size_t bytes;
    bool written;
};
// SHTN_OK, or SHTN_EINVAL when a written range shares a byte with any
// other range of the list (read-only ranges may overlap); the message names
// the first such pair in list order.
int check_disjoint(const std::vector<Range>& r);
// Fields of a transform: spectra (nlm complex each) or grids (nlat x nphi).
enum class Data { spec, grid };
// Appends the device memory a plan's transforms read: its uploaded image
// and, when built, its stored-P table.
void plan_ranges(const Plan& p, std::vector<Range>& r);
int hip_error(int e, const char* where);
int rows_per_block(const Plan& p, int nfields);  // FFT rows per workgroup for a call of so many fields

// Host plan construction (plan.cpp).
Plan* build_plan(int L, int M, int nlat, int nphi, std::string& err);
// Tiling of a plan that was not given one, and its degrees per analysis piece.
Tiling automatic_tiling(const Plan& p);
int automatic_split(long nlm);
int rebuild_units(Plan& p, std::string& err);     // units + restart states for the tiling
void lane_starts(Plan& p);                        // start step and state of every (order, pair) lane
// First / last start step of the lanes [i0, i1) of order m that start in
// [lo, hi); false if none does.
bool start_range(const Plan& p, int m, int i0, int i1, int lo, int hi, int& jmin, int& jmax);
void build_image(Plan& p);                        // lays out the device buffer
inline long lm_index(int L, int n, int m) { return (long)m * (2 * L + 1 - m) / 2 + n; }
// Layout of the longitude coefficients F_m(theta_i) of one field: tiles of
// kFTile consecutive latitudes, each tile order-major with the kFTile values
// of one order adjacent:
//   offset(m, i) = (i / kFTile) f_ts + m kFTile + i % kFTile,  f_ts = (mmax+1) kFTile.
// The Legendre kernels' lanes (consecutive latitudes of one order) touch
// whole 128-byte lines, and an FFT workgroup moves its rows in contiguous
// runs (half a tile per order at K = 1024).
constexpr int kFTile = 8;
constexpr int kFTileLg = 3;
struct FLayout {
    long ts, size;  // tile stride and values per field (complex)
};
#ifdef __HIPCC__
// Complex offset of F_m(theta_i) in a field's longitude coefficients.
__device__ __forceinline__ long f_index(long ts, int m, int i)
{
    return (long)(i >> kFTileLg) * ts + m * kFTile + (i & (kFTile - 1));
}
#endif
inline FLayout f_layout(int M, int nlat)
{
    const long ts = (long)(M + 1) * kFTile;
    return {ts, ts * ((nlat + kFTile - 1) / kFTile)};
}
// XCDs of the chip: workgroup b of a launch runs on XCD b % kXcds.
constexpr int kXcds = 8;
// Unit list of a synthesis launch from one queue per XCD: each sorted longest
// first (or, with `alternate`, long and short in turn), padded with units
// without work to the length of the longest, entry k of XCD x at k kXcds + x.
void pack_synth_queues(std::vector<SynthUnit> (&q)[kXcds], int alternate, std::vector<int>& units);
size_t align256(size_t v);

// Workspace bytes of a plan call with nfields fields: F, nfields x f_layout().size
// complex (and the room for nfields spectra that the size has always had: it
// decides which calls shtn_synth_noalloc takes).
size_t work_bytes(const Plan& p, int nfields);

// Fields per wave of the analysis kernel for a (pairs per lane, waves) class:
// the largest count <= fw among the built kernels (two fields with lp <= 4
// and waves <= 2, else one).  Four-field analysis passes were slower than
// two-field ones in every class that can hold them.
inline int analys_fw(int fw, int lp, int waves)
{
    return fw >= 2 && lp <= 4 && waves <= 2 ? 2 : 1;
}

// Cost of a synthesis step of n fields, fw per wave, in FP64 instructions per
// latitude pair: 2 for the recurrence and 2 per field (a last, partial group
// runs all fw).
inline long synth_step_cost(int n, int fw) { return (long)((n + fw - 1) / fw) * (2 + 2 * fw); }
constexpr int kMaxFw = 4;
// Fields per synthesis wave for nfields fields of nunits units each: the
// cheapest step among the built kernels that still leaves three waves for each
// of the 1024 SIMDs (lmax 255, 16 fields: two per wave 18.8 us, four 19.6, one
// 21.1; lmax 511, 16 fields: 64.2, 55.6 and 84.6).
inline int synth_fw(int nfields, int nunits, int lp)
{
    int best = 1;
    for (int fw = 2; fw <= kMaxFw && fw * lp <= 8; fw *= 2)
        if (synth_step_cost(nfields, fw) <= synth_step_cost(nfields, best) &&
            (long)nunits * ((nfields + fw - 1) / fw) >= 3072)
            best = fw;
    return best;
}

// Kernel launchers (legendre.hip, fft.hip).  Return a hipError_t as int.
struct LegLaunch {
    const DevPlan* plans;  // device array of plans
    const int* units;      // device unit array
    int nunits;
    int grid_y;            // field groups of the call, 1 for batches
    const long* q_off;     // per-field offset (doubles) of the spectrum, or null (f * 2 nlm)
    const long* f_off;     // per-field offset (doubles) of F, or null (f * 2 (M+1) nlat)
    const double* in;
    double* out;
    int nfields;
    int adjoint;           // 0 forward transform, 1 adjoint variant
    int lp, fw;            // template selection
    int waves = 1;         // analysis: waves per unit (latitude pairs 64 lp waves)
    double* top = nullptr; // vector transforms: the terms with x P_L (see vector.hip), else null
    int rotate = 0;        // synthesis: a unit's field groups go to the XCDs in turn (see synth_unit)
};
// Stored-P kernels (ptable.hip).
struct PtabArgs {
    const DevPlan* plan;
    const long* boff;    // device copy of PTable::boff
    const double* tab;   // the blocks
    const double* in;    // synthesis: spectra (nfields x nlm complex); analysis: F
    double* out;         // synthesis: F; analysis: spectra
    int nfields;
    int adjoint;
    int npt;
    const long* q_off = nullptr;  // per-field spectrum offset (doubles), or null (f * 2 nlm)
    const long* f_off = nullptr;  // per-field F offset (doubles), or null (f * 2 f_size)
};
int launch_ptable_build(const DevPlan* plan, const long* boff, double* tab, int npt, int M, void* stream);
int launch_sp_synth(const PtabArgs& a, int M, int rt, int ct, void* stream);
int launch_sp_analys(const PtabArgs& a, int L, int M, int jt, int ct, void* stream);
// Vector transforms (vector.hip): spectral and latitude combinations around
// the scalar stages.
int launch_vec_spec_in(const DevPlan* plan, int L, int M, const double* S, const double* T, double* Q4, int nfields,
                       int nn, void* stream);
int launch_vec_spread(const DevPlan* plan, int L, int M, const double* S, const double* T, double* Q2, double* top,
                      int nfields, int nn, void* stream);
int launch_vec_gather(const DevPlan* plan, int L, int M, const double* A2, const double* top, double* S, double* T,
                      int nfields, int nn, void* stream);
int launch_vec_f_out(const DevPlan* plan, long f_size, const double* F4, double* Fv, int nfields, void* stream);
int launch_vec_f_in(const DevPlan* plan, long f_size, const double* Fv, double* F4, int nfields, void* stream);
int launch_vec_spec_out(const DevPlan* plan, int L, int M, const double* A4, double* S, double* T, int nfields,
                        int nn, void* stream);
int launch_legendre_synth(const LegLaunch& a, void* stream);
int launch_legendre_analys(const LegLaunch& a, void* stream);
// Waves of a unit (each covers 256 latitude pairs with up to four fields, 128 with eight).
inline int mf_waves(int npair, int fields)
{
    int w = 1;
    while ((fields == 8 ? 128 : 256) * w < npair) w *= 2;
    return w;
}
// Several fields of one plan with the sums on the matrix cores (analys_mf.hip).
// Fields per unit: 8, 4, or 0 where the vector kernel is the better one.  A
// unit of eight fields costs about as much as 6.1 fields in the vector kernel,
// one of four 3.45, whether or not all are there (lmax 1023: 8 fields 267 us
// against 348, 4 fields 152 against 178, 3 fields 148 against 136), and small
// calls are bound by latency (lmax 255: 8 fields 18.8 against 17.7, 16 fields
// 22.6 against 27.7; lmax 383, 8 fields 41 both).
// And a call has to fill the chip: of four fields per unit, or of one group of
// eight, 1,600 waves for its 2,048 slots (npieces: units of one field; us: lmax
// 1023 of 41 orders, 4 fields, 1,536 waves, 34.9 against 30.8; lmax 300 of 201
// orders and 1,000 latitudes, 4 fields, 1,472 waves, 45.1 against 37.9; lmax 450,
// 4 fields, 1,824 waves, 40.3 against 42.0; two groups of eight at lmax 1023 of
// 11 orders, 2,048 waves with the padding, 32.4 against 37.6).
inline int mf_fields(int npair, long nlm, long npieces, int nfields)
{
    if ((double)nlm * npair * nfields < 6e7) return 0;
    const double vec = nfields, four = (nfields + 3) / 4 * 3.45,
                 eight = npair <= 1024 ? (nfields + 7) / 8 * 6.1 : vec + four;
    if (vec <= four && vec <= eight) return 0;
    const int mf = eight <= four ? 8 : 4, groups = (nfields + mf - 1) / mf;
    return npieces * groups * mf_waves(npair, mf) < 1600 && (mf == 4 || groups == 1) ? 0 : mf;
}
// Fields per unit of a vector analysis of nfields components, which always
// runs there: one vector field takes a unit of its own two components.
inline int mf_vec_fields(int npair, int nfields)
{
    if (nfields == 2) return 2;
    const double four = (nfields + 3) / 4 * 3.45, eight = npair <= 1024 ? (nfields + 7) / 8 * 6.1 : 2 * four;
    return eight <= four ? 8 : 4;
}
int launch_legendre_analys_mf(const LegLaunch& a, int npair, int fields, void* stream);

struct FftLaunch {
    const DevPlan* plans;     // device plan array
    const int* rowblocks;     // device: per block {field, plan, row0, nrows} or null
    int nblocks;
    int grid_y;
    int K;                    // longest rows of the launch
    int points;               // most complex points in one block (rows x K <= 4096): sizes
                              // the workgroup (one thread per 4, 8 or 16 points) and its LDS
    int rows_per_block;
    const long* g_off;        // per-field grid offset (doubles) or null
    const long* f_off;        // per-field F offset (doubles) or null
    const double* in;
    double* out;
    double* grid2 = nullptr;  // not null: fields 2 f have grid f of the grid pointer, fields 2 f + 1 grid f here
    int nfields;
    double scale;             // r2c: output scale (2 pi/nphi or 1)
    int uniform_k = 0;        // 1: every row of the launch has K points
};
int launch_c2r(const FftLaunch& a, void* stream);
int fft_rows_cap(int K);     // rows of K complex points held by one FFT workgroup
int fft_rows_auto(int K, int nlat, int nfields);  // rows per workgroup unless the caller sets them
int launch_r2c(const FftLaunch& a, void* stream);
// Both stages of a synthesis or analysis in one launch, for plans so small that
// a field fits one workgroup (fft.hip); q: spectra.
bool small_fits(int M, int nlat, int K, long nlm);
bool small_pays(int L, int M, int nlat, int K, int nfields, bool synth);
int launch_small_analys(const FftLaunch& l, int M, int nlat, long nlm, double* q, int adjoint, void* stream);
int launch_small_synth(const FftLaunch& l, int M, int nlat, long nlm, const double* q, int adjoint, void* stream);

}  // namespace shtn

// Opaque handle behind shtn_plan_t.
struct shtn_plan_s {
    shtn::Plan* p;
};

namespace shtn {
// shtn_synth's checks and launches with `work` as the workspace (api.cpp).
int synth_on_work(shtn_plan_s* plan, const double* Q, double* grid, int nfields, void* work, void* stream);
}  // namespace shtn
