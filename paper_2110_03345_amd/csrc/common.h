// Internal definitions shared by the host code and the HIP kernels of the
// acoustic FWI library (not part of the public C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace stride {

constexpr int kMaxR = 5;        // stencil radius (10th order)
constexpr int kThreads = 256;   // 4 wave64 per block
constexpr int kTileX = 64;      // contiguous axis: one wave64 spans a tile row
constexpr int kSincHalfWidth = 4;   // windowed-sinc taps: 2 r nodes per axis

// Launch shapes of the step kernels.  2D: rows per thread x wave64s per block
// (the tile is 64 x rows * waves), the fastest measured on 1104^2.  3D: points
// of a row per thread x wave64s per block (64 x points * waves); kernels with
// one stencil field take four points, those with two (adjoint with the fused
// imaging, fourth-order adjoint correction, y = 2 medium) two.
constexpr int kRy2d = 4, kWaves2d = 4;
constexpr int kVx3dOne = 4, kVx3dTwo = 2, kWaves3d = 4;
// Planes of a 3D block (chunk_planes in stride_api.cpp).
constexpr int kZc3dMin = 4, kZc3dOne = 8, kZc3dTwo = 16;
// Infinity Cache of the part, in bytes.
constexpr long long kCacheBytes = 256ll << 20;
constexpr int kPitchAlign = 16;     // row pitch of the fields, in floats (64 B)

// Padded grid as laid out in the workspace.  Axis nd-1 is contiguous.
// 2D: axis 0 = rows, axis 1 = columns.  3D: axis 0 is the marching axis.
struct Dims {
    int nd;
    int n[3];          // padded extent per axis (unused axes = 1)
    int phys[3];       // physical extent
    int nb;            // sponge cells per side
    long long st[3];   // element strides; st[nd-1] = 1
    long long total;   // elements in one field (with row pitch)
};

// Laplacian weights already divided by dx_axis^2 (rounded once from FP64);
// c0 is the summed centre weight over all axes.
struct StencilCoef {
    float c0;
    float c[3][kMaxR + 1];
    float d[3][kMaxR + 1];   // centred first-derivative weights / dx_axis (medium steps)
};

// Sponge: eta = sum_axes e[a] * depth_a^2, e[a] = eta_max_a / nb^2.
struct SpongeCoef {
    float e[3];
    float half_dt;
};

// Injection entries grouped by step-kernel block (a 2D tile, or a 3D tile
// over one chunk of planes) of the launch shape that uses the table.  Block b
// holds ent[ptr[b] .. ptr[b+1]); entry e adds w * sig[id][step] at its
// block-local point `local` = (plane in chunk * TY + tile row) * 64 + tile
// column.  A block's entries are sorted by point, in (point, tap) order
// within a point; the first entry of a point holds the number of entries of
// that point in `run`, the others 0.
struct TileEntry {
    int local;
    int run;
    int id;
    float w;
};

struct InjTable {
    const int* ptr;
    const TileEntry* ent;
};

// Point sampling: v = scale * sum_t w[r*ntap+t] * field[idx[r*ntap+t]], stored to
// out[r * out_stride + step] or, with accumulate, added to it.
struct SampleSet {
    int count;
    const long long* idx;
    const float* w;
    float* out;
    int out_stride;
    int ntap;         // taps per point: 2^ndim (linear) or (2 r)^ndim (windowed sinc)
    float scale;
    int accumulate;
};

// Threads that sample one point: one for up to 8 taps, a wave64 (lanes over
// the taps, then a wave reduction) for the windowed-sinc tap sets.
__host__ __device__ inline int sample_lanes(int ntap)
{
    return ntap > 8 ? 64 : 1;
}

struct StepParams {
    const float* A;   // stencil field: u^n (forward) or w^{m+1} (adjoint)
    const float* B;   // u^{n-1} or w^{m+2}
    float* C;         // result; may alias B
    const float* K;   // dt^2 vp^2
    const float* U;   // adjoint only: second stencil field (u^m; p in the correction)
    float* G;         // adjoint only: imaging accumulator
    const float* D;   // correction only: point field u^n (forward) or w^{m+1} (adjoint)
    int step;         // time index of the injected / sampled signals
    InjTable inj;     // injection into C: sources (forward), receivers (adjoint)
    const float* inj_sig;
    int inj_stride;
    InjTable img;     // adjoint only: source term S^m of the imaging condition
    const float* img_sig;
    int img_stride;
    SampleSet smp;    // sampling of A at `step`
    // medium steps only: gamma_a = -D_a ln rho per axis, and the attenuation
    // field (kMediumY0: 2 alpha0 vp added to the damping; kMedium: beta = 2 alpha0 vp / dt)
    const float* gam[3];
    const float* att;
    float* V;         // kStepV: L u^n + S^n out; kImageV: that of u^m in
    const float* V2;  // kImageV: that of u^{m+1} (NULL: one imaging term per step)
};

// One slot's step in a batched launch.
struct SlotStep {
    StepParams p;
    SpongeCoef sp;
    int active;
};

struct LaunchShape {
    int ty;               // tile rows
    int ry, waves;        // 2D: rows per thread; wave64s per block
    int tiles_x, tiles_y, tiles_xy;
    int zc, nzc;          // 3D: planes per block and number of z chunks
    int tile_blocks;      // logical tile blocks (before XCD padding)
    int tile_blocks_pad;  // rounded up to a multiple of 8 XCDs
};

// Rows per thread and waves per block of the 2D step kernels for a direction
// (the tile is 64 x ry*waves).
void tile_shape_2d(bool adjoint, int* ry, int* waves);
// Whether a 3D step loads its point values with the non-temporal policy.
bool stream_3d(const Dims& d, bool adjoint, int mode);

// 2D sweeps that keep the state on the chip (step2d_resident.h): one block of
// kResidentThreads per tile of tx x ty points, tx a multiple of 4.
constexpr int kResidentThreads = 1024;
constexpr int kResidentItems = 2;    // quads per thread, at most
constexpr unsigned kResidentSteps = (1u << 21) - 1;   // highest step number of a sweep
constexpr int kResidentSide = 256;   // side of a tile with its ring, at most
// Shortest sweep worth a cooperative launch: it costs about 25 us more than a
// step's (48 x 56, us a gradient with sweeps / with a launch per step: nt 3 182 / 142,
// 9 205 / 197, 13 213 / 231, 17 228 / 268; 200^2: 177 / 150, 197 / 200, 209 / 234,
// 219 / 270).  At least 2 by its protocol: blocks of a sweep of one step do not wait
// for each other, and one could store its final state before a neighbour has loaded
// its frame.
constexpr int kResidentLeast = 10;
// Polls after which a block gives up waiting for its neighbours' words: a poll
// takes about 1 us, so about a minute of the block's own running.
constexpr int kResidentPatience = 1 << 26;

struct ResidentShape {
    int tx, ty;
    int tiles_x, tiles_y, tiles;
    int t;               // steps per exchange, 1 or 2
};

// The frame a block takes from its neighbours: t R rows above and below, the
// quads of t R columns left and right.  With two steps per exchange the first is
// computed on the tile and a ring of R rows and the quads of R columns as well.
__host__ __device__ inline int resident_frame_rows(int R, const ResidentShape& rs)
{
    return rs.t * R;
}
__host__ __device__ inline int resident_frame_quads(int R, const ResidentShape& rs)
{
    return (rs.t * R + 3) / 4;
}
__host__ __device__ inline int resident_ring_rows(int R, const ResidentShape& rs)
{
    return (rs.t - 1) * R;
}
__host__ __device__ inline int resident_ring_quads(int R, const ResidentShape& rs)
{
    return (rs.t - 1) * ((R + 3) / 4);
}

// Quads computed by a block: the tile's and the ring's.
__host__ __device__ inline int resident_items(int R, const ResidentShape& rs)
{
    return (rs.tx / 4 + 2 * resident_ring_quads(R, rs)) * (rs.ty + 2 * resident_ring_rows(R, rs));
}

// Quads of a tile that neighbours take.
__host__ __device__ inline int resident_outer_quads(int R, const ResidentShape& rs)
{
    const int fr = resident_frame_rows(R, rs);
    return 2 * fr * (rs.tx / 4) + (rs.ty - 2 * fr) * 2 * resident_frame_quads(R, rs);
}

// Quads of the frame.
__host__ __device__ inline int resident_frame(int R, const ResidentShape& rs)
{
    const int fb = resident_frame_quads(R, rs);
    return 2 * resident_frame_rows(R, rs) * (rs.tx / 4 + 2 * fb) + 2 * fb * rs.ty;
}

// Threads with items: enough for the items at J each and for the outer quads at
// one each, in whole waves.
__host__ __device__ inline int resident_compute_threads(int items, int outer, int J)
{
    const int n = (items + J - 1) / J > outer ? (items + J - 1) / J : outer;
    return (n + 63) / 64 * 64;
}

// Exchange words of a tile, three per quad: word k of outer quad i at k * stride
// + i, so that a wave's accesses are contiguous (the words of a quad in a row cost
// as many times the transactions); stride a whole number of 64-byte lines.
__host__ __device__ inline int resident_word_stride(int R, const ResidentShape& rs)
{
    return (resident_outer_quads(R, rs) + 7) / 8 * 8;
}

// Bytes of the exchange area (two buffers of words).
__host__ __device__ inline long long resident_word_bytes(int R, const ResidentShape& rs)
{
    return 2ll * rs.tiles * 3 * resident_word_stride(R, rs) * 8;
}

// Row length of the LDS region of a tile (the tile and its frame) and the region
// index of tile point (y, x).
__host__ __device__ inline int resident_row(int R, const ResidentShape& rs)
{
    return rs.tx + 8 * resident_frame_quads(R, rs);
}
__host__ __device__ inline int resident_index(int R, const ResidentShape& rs, int y, int x)
{
    return (y + resident_frame_rows(R, rs)) * resident_row(R, rs) +
           4 * resident_frame_quads(R, rs) + x;
}

// LDS of a block: two buffers of the region, two more for injected values, and
// k in an adjoint sweep with two quads per thread.
__host__ __device__ inline int resident_lds_bytes(int R, const ResidentShape& rs, bool injects,
                                                  bool adjoint)
{
    const int items = resident_items(R, rs);
    const bool k = adjoint && items > kResidentThreads;
    return ((injects ? 4 : 2) * resident_row(R, rs) * (rs.ty + 2 * resident_frame_rows(R, rs)) +
            (k ? 4 * items : 0)) * 4;
}

// Points sampled by tile b: ptr[b] .. ptr[b+1]; taps as region indices.
struct ResidentSamples {
    const int* ptr;
    const int* id;         // row of `out`
    const int* idx;        // [..][ntap]
    const float* w;        // [..][ntap]
    float* out;
    int out_stride;
    int ntap;
};

// A sweep of `count` steps (kStep, kStepV or the adjoint kImageV).
struct ResidentParams {
    const float* A;        // u^n and u^{n-1} at the start (NULL: both zero)
    const float* B;
    float* A2;             // the two states at the end (NULL: not kept)
    float* B2;
    const float* K;
    float* G;              // adjoint: imaging accumulator
    float* V;              // kStepV: v of step v_from (out); adjoint: v of the first step (in)
    long long vstride;     // elements from one step's V to the next step's
    int v_from;            // kStepV: first step whose v is stored
    int step;              // signal / sample index of the first step
    int dir;               // +1 forward, -1 adjoint
    int count;             // steps
    int sample_last;       // sample the final state too (at index step + dir count)
    SpongeCoef sp;
    int injects;           // the table has entries (LDS for their values)
    InjTable inj;          // entries per tile; `local` = region index
    const float* inj_sig;
    int inj_stride;
    ResidentSamples smp;   // sampling of u^n (out NULL: none)
    unsigned long long* words;   // exchange area: no word holds a step number in
    unsigned tag;                // (tag, tag + count], the numbers of this sweep (21 bits)
    unsigned* err;               // set by a block that gave up waiting
    int patience;                // polls after which a block gives up
};

// Sweeps of one launch, on rs.tiles blocks each.
constexpr int kResidentSlots = 12;   // kernel arguments hold 4 KB
struct ResidentBatch {
    int n;
    ResidentParams p[kResidentSlots];
};

// What a step launch computes.  Fourth-order time runs two launches per
// forward step and three per adjoint step (kPrep on u^m and on w^{m+1}, then
// the adjoint kCorrect).
enum StepMode {
    kStep = 0,    // C = a (2 A + k (L A + S)) - b B                 (leapfrog step)
    kPrep = 1,    // C = k (L A + St), St: source filtered in time   (p of the corrected step)
    kCorrect = 2, // C = a (2 D + A + (k/12) L A) - b B, A = p, D = u^n;
                  // adjoint: C = a (2 D + A + (k/12) L A + k R^T g) - b B with A = q,
                  // D = w^{m+1}, and G += U (D + A/12) + (k/12) D L U with U = p
    kMedium = 3,  // forward step in a heterogeneous medium (y = 2), B a stencil field too:
                  // C = a (2 A + k (L A + sum_a gam_a D_a A + S + att (L A - L B))) - b B;
                  // with V given it also stores the imaging factor of the vp gradient there
    kStepV = 4,   // forward kStep that also stores V = L A + S (full-history gradients)
    kImageV = 5,  // adjoint kStep whose imaging reads V = L u^m + S^m instead of the
                  // stencil of u^m: G += A V, and with V2 the previous step's term as
                  // well, G = fma(A, V, fma(B, V2, G)) (B = w^{m+2})
    kAdjPlain = 6,// adjoint kStep without imaging (the step before a kImageV with V2)
    kMediumY0 = 7 // kMedium with att added to the damping (y = 0): B is a point value
};

// Perfectly matched layer: the memory-variable correction of one step, for
// the points of the padded layer (the plain leapfrog without damping has
// already written u^{n+1}; see stride_grid_t.boundary).
struct PmlParams {
    const float* u;          // u^n
    float* un;               // u^{n+1}: += k (sum_a (-D_a psi_a^n - chi_a^n))
    const float* k;
    const float* psi[3];     // psi_a^n
    float* psin[3];          // psi_a^{n+1}
    float* chi[3];           // chi_a^{n-1} -> chi_a^n (in place)
    float c0[3];             // second-derivative centre weight / dx_a^2 per axis
    float zmax[3];           // zeta_max per axis (1/s)
    float dt;
};

// One adjoint step of the heterogeneous-medium gradient (the exact transpose
// of kMedium): w^m = a (2 w^{m+1} + k (L y - sum_a D_a (gam_a w^{m+1}))) - b w^{m+2},
// y = (1 + beta) w^{m+1} - beta w^{m+2} (beta = att when att_power is 2, else 0;
// with att_power 0 att joins the damping), and G += w^{m+1} H.  The receiver
// residual is added afterwards by launch_inject_table.
struct MediumAdjParams {
    const float* w1;         // w^{m+1}
    const float* w2;         // w^{m+2}
    float* w0;               // w^m
    const float* k;
    const float* gam[3];
    const float* att;        // 2 alpha0 vp (att_power 0) or beta (2); NULL: none
    int att_power;
    const float* H;          // imaging factor of step m; NULL: no imaging
    float* G;
};

// Kernel launchers (stride_kernels.hip).
// max_sample_threads: the largest count * sample_lanes(ntap) over the slots.
void launch_step_batched(const Dims& d, int R, bool adjoint, int mode, const StencilCoef& cf,
                         const LaunchShape& ls, const SlotStep* table, int nslots,
                         int max_sample_threads, hipStream_t s);
void launch_accumulate(float* dst, const float* src, long long n, hipStream_t s);
void launch_step(const Dims& d, int R, bool adjoint, const StencilCoef& cf, const SpongeCoef& sp,
                 const LaunchShape& ls, const StepParams& p, hipStream_t s);
// Launches of the mode steps: forward kPrep, kCorrect, kMedium[Y0] or kStepV; adjoint
// kCorrect or kImageV.
void launch_step_mode(const Dims& d, int R, bool adjoint, int mode, const StencilCoef& cf,
                      const SpongeCoef& sp, const LaunchShape& ls, const StepParams& p, hipStream_t s);

// One sweep kept on the chip; hipSuccess, or the launch error (nothing ran).
// No exchange word (resident_word_bytes of them) may hold a step number of the sweep,
// (tag, tag + count]: zero before the first, numbered on after that.
hipError_t launch_resident(const Dims& d, int R, int mode, const StencilCoef& cf,
                           const ResidentShape& rs, const ResidentBatch& b, hipStream_t s);
// Outputs of a solve (p NULL: none).
struct Outputs {
    float* p[3];
    long long n[3];
};
// Fills them with NaN where *err is set (a sweep whose blocks gave up waiting), and
// sets *report (pinned; NULL: none).
void launch_poison(const unsigned* err, const Outputs& out, hipStream_t s, unsigned* report = nullptr);

void launch_pml_correction(const Dims& d, int R, const StencilCoef& cf, const PmlParams& pp,
                           hipStream_t s);
void launch_medium_adjoint(const Dims& d, int R, const StencilCoef& cf, const SpongeCoef& sp,
                           const LaunchShape& ls, const MediumAdjParams& mp, hipStream_t s);
// out[p] += a(p) k(p) (sum of the signals injected at p), for every point of an
// injection table built for the launch shape ls; a(p) the damping factor of
// the sponge and (att_power 0) the attenuation field att.
void launch_inject_table(const Dims& d, const LaunchShape& ls, const InjTable& T, const float* sig,
                         int stride, int step, const float* k, const float* att, int att_power,
                         const SpongeCoef& sp, float* out, hipStream_t s);
void launch_sample(const SampleSet& smp, const float* field, int step, hipStream_t s);
void launch_fill(float* p, long long n, float v, hipStream_t s);
// In place, per [nt] row: h[j] = (h[j-1] + 10 h[j] + h[j+1]) / 12 (zero outside),
// the transpose of the fourth-order scheme's source filter.
void launch_time_filter3(float* rows, int count, int nt, hipStream_t s);
// Zero-phase FIR low-pass of [count][nt] rows (out may alias in); K taps per side.
int lowpass_taps(double dt, double f_max);
void launch_lowpass(const float* in, float* out, int count, int nt, double dt, double f_max,
                    hipStream_t s);
// vp = clamp(vp - step m g / max|m g|, vmin, vmax); work: one device word.
void launch_descent(float* vp, const float* g, const float* mask, long long n, float step,
                    float vmin, float vmax, unsigned* work, hipStream_t s);
void launch_prep_k(const Dims& d, const float* vp, double dt, float* k, hipStream_t s);
// First-derivative weights in FP64 for the medium preparation.
struct Fd1 {
    double d[kMaxR + 1];
    double inv_dx[3];
    int r;
};

// Medium fields on the padded grid: gam[a] = -D_a ln rho_pad (rho NULL: zero;
// ln rho repeats its edge value beyond the array) and att (alpha0 NULL: zero;
// att_power 0: 2 alpha0 vp, 2: 2 alpha0 vp / dt), computed in FP64, rounded once;
// lr: scratch, a double per physical point.
void launch_prep_medium(const Dims& d, const Fd1& fd, const float* vp, const float* rho,
                        const float* alpha0, int att_power, double dt, float* const gam[3],
                        float* att, double* lr, hipStream_t s);
// flags[2] = 1 if rho has a non-positive or non-finite value or alpha0 a negative
// or non-finite one; flags[3] = max over points of vp^2 (1 + 2 beta) as float bits
// (beta = 2 alpha0 vp / dt for att_power 2, else 0).
void launch_medium_check(const float* vp, const float* rho, const float* alpha0, long long n,
                         int att_power, double dt, unsigned* flags, hipStream_t s);
// Misfit partial sums: kMisfitParts doubles of scratch.
constexpr int kMisfitParts = 256;
void launch_residual_misfit(const float* traces, const float* observed, float* residual,
                            long long n, double* misfit, double* partial, hipStream_t s);
// dvp = P^T (2 G / vp_pad), with G = H / kdiv where kdiv is given (else G = H);
// tmp0 and tmp1 hold intermediates of up to one field each.
void launch_finalize_dvp(const Dims& d, const float* H, const float* kdiv, const float* vp,
                         float* dvp, float* tmp0, float* tmp1, hipStream_t s);
void launch_copy(float* dst, const float* src, long long n, hipStream_t s);
// *flag |= bit if any of the n values is NaN or infinite (flag cleared by the caller).
void launch_finite_scan(const float* p, long long n, unsigned* flag, unsigned bit, hipStream_t s);
void launch_finite_scan(const double* p, long long n, unsigned* flag, unsigned bit, hipStream_t s);
// flags[0] = bits of max(vp) (vp > 0), flags[1] = 1 if any vp <= 0 or non-finite.
void launch_vp_check(const float* vp, long long n, unsigned* flags, hipStream_t s);

}  // namespace stride
