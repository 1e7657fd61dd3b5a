// Internal declarations shared by the kernels and the host runtime of the
// gfx950 simplified-string-method library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssm_fft.hpp"

namespace ssm {

// Twiddle table: tw[e] = exp(-2 pi i e / kTwM).  A length-L root W_L^e is
// tw[e * (kTwM / L)]; every padded length 2m (m = 2^a <= 1024 or
// m = 3 2^a <= 768) and every sub-length divides kTwM = 3 * 2^11.
constexpr int kTwM = 3 << 11;
constexpr int kMaxLogM = 10;   // half padded length m <= 1024, padded P = 2m <= 2048
// The FFT kernels read their twiddles from a compact table: for every half
// length m = 2^lg (lg <= 10) and m = 3 2^lg (lg <= 8), the 2m values
// W_{2m}^e, e < 2m, contiguous, starting at tw_off(lg, f3).
__host__ __device__ constexpr int tw_off(int lg, int f3)
{
    return f3 ? (4 << kMaxLogM) - 2 + 6 * ((1 << lg) - 1) : (2 << lg) - 2;
}
constexpr int kTwCompact = tw_off(9, 1);  // entries of the compact table
constexpr int kNT = 256;       // threads per workgroup (k_conv1: Conv1Cfg::nt; k_xinv of short rows: kXinvWide)
constexpr int kConvElems = 24 * kNT;  // complex values per convolution workgroup (slice batching cap)
constexpr int kArcEPT = 8;     // flat elements per thread in the arc-length kernel
constexpr int kNTerm = 5;      // energy partial slots: E, T_J, T_d, T_ku, T_dip
constexpr int kMaxImages = 1024;  // images per problem (the ABI's limit)
// Reduction in one workgroup per problem (k_reduce1) for problems of at
// most kRed1MaxK images with at most kRed1MaxPart energy and arc partials
// per image; kRedLanes lanes sum one image's partials there.
#ifndef SSM_RED_LANES
#define SSM_RED_LANES 4
#endif
constexpr int kRed1MaxK = 64, kRed1MaxPart = 256, kRedLanes = SSM_RED_LANES;

// The convolution has a build for each compile-time y length (32..256 and 48,
// 96, 192; up to 8 layers) and one with a runtime length for every other shape.
// They are separate kernels so that each gets its own register allocation; a
// launch covers a problem with whichever serves its shape (conv_inplace and
// conv_halves: which kernel of a build).
#ifndef SSM_CONV_CT
#define SSM_CONV_CT 1
#endif
__host__ __device__ constexpr bool conv_ct_shape(int mz, int lmy, int f3y)
{
    return SSM_CONV_CT && !f3y && mz <= 8 && lmy >= 5 && lmy <= 8;
}
// y lengths 3 2^lmy with compile-time sub-line passes (48, 96, 192)
__host__ __device__ constexpr bool conv_ct3_shape(int mz, int lmy, int f3y)
{
    return SSM_CONV_CT && f3y && mz <= 8 && lmy >= 4 && lmy <= 6;
}
// build serving a problem: the y length's log2 (5..8) for the compile-time
// power-of-two builds, 16 + log2 of the power-of-two factor (20..22) for the
// compile-time 3 2^a builds, 0 for the runtime-length one
__host__ __device__ constexpr int conv_build(int mz, int lmy, int f3y)
{
    return conv_ct_shape(mz, lmy, f3y) ? lmy : conv_ct3_shape(mz, lmy, f3y) ? 16 + lmy : 0;
}

// The monolayer convolution's split of the y length m = A B, by build: a lane
// transforms A inputs at stride B (A = 12 for lengths 3 2^a) in the first
// step.  nt threads and at most g slices per workgroup: 3 B g items in the
// first step, near nt, in an LDS share that leaves three workgroups to a CU
// (256 and 384: more, of two wavefronts); twlds: the twiddle table has a copy
// in LDS (0 where that would cost a workgroup).
struct Conv1Cfg {
    int A, B, nt, g, twlds;
};
__host__ __device__ constexpr Conv1Cfg conv1_cfg(int build, int tsize)
{
    return build == 5    ? Conv1Cfg{8, 4, 256, 16, 1}
           : build == 20 ? Conv1Cfg{12, 4, 256, 10, 1}
           : build == 6  ? (tsize == 4 ? Conv1Cfg{16, 4, 256, 10, 1} : Conv1Cfg{16, 4, 128, 5, 1})
           : build == 21 ? (tsize == 4 ? Conv1Cfg{12, 8, 256, 10, 1} : Conv1Cfg{12, 8, 128, 5, 1})
           : build == 7  ? (tsize == 4 ? Conv1Cfg{16, 8, 256, 8, 1} : Conv1Cfg{16, 8, 128, 4, 0})
           : build == 22 ? (tsize == 4 ? Conv1Cfg{12, 16, 256, 5, 1} : Conv1Cfg{12, 16, 128, 2, 1})
                         : (tsize == 4 ? Conv1Cfg{16, 16, 128, 2, 1} : Conv1Cfg{16, 16, 128, 2, 0});
}
// LDS elements of one line: B rows of the 2A values of both halves, an odd
// stride apart (strided writes and contiguous reads both meet distinct banks)
__host__ __device__ constexpr int conv1_line(Conv1Cfg c) { return c.B * (2 * c.A + 1); }
__host__ __device__ constexpr size_t conv1_lds(Conv1Cfg c, int G, int tsize)
{
    return (size_t)((c.twlds ? 2 * c.A * c.B : 0) + G * 3 * conv1_line(c)) * 2 * tsize;
}
// the same split for several layers (k_convz): G slices of 3 nz lines
__host__ __device__ constexpr int convz_twlds(int build, int tsize) { return build >= 16 || (build <= 8 ? (1 << build) : 0) * tsize <= 512; }
__host__ __device__ constexpr size_t convz_lds(int build, int G, int nz, int tsize)
{
    const Conv1Cfg c = conv1_cfg(build, tsize);
    return (size_t)((convz_twlds(build, tsize) ? 2 * c.A * c.B : 0) + G * 3 * nz * conv1_line(c)) * 2 * tsize;
}

// k_convh (FP64, 4 padded layers, one half at a time, one slice to a
// workgroup): where it serves the slices that k_convz doesn't hold (4 layers of
// 192 and 256 points), and LDS for up to nz layers
__host__ __device__ constexpr bool conv_halves(int mz, int build, int tsize)
{
    return tsize == 8 && mz == 4 && build > 0;
}
__host__ __device__ constexpr int convh_line(Conv1Cfg c) { return c.B * (c.A + 1); }
__host__ __device__ constexpr size_t convh_lds(int build, int nz)
{
    const Conv1Cfg c = conv1_cfg(build, 8);
    return (size_t)(2 * c.A * c.B + 3 * nz * convh_line(c)) * 16;
}

// Whether the in-place kernels can take a problem: monolayers always (of the
// lengths with a build); several layers where one slice's lines of both halves
// fit kConvzLds, two workgroups to a CU; one to a CU would hold fewer wavefronts
// than k_conv's three (256 x 256 x 8) or, in FP64, not fit.  3 layers of 192 and 256
// points in FP64 fit and are the faster there (us a launch, k_convz, k_convh,
// k_conv: 250 x 250 x 3, 20 images 208, 273, 377; 180 x 180 x 3, 20 images 112, 147,
// 172).  5 and 6 layers of 256 points in FP32 fit and aren't: the plan decides
// (conv_apart).  (_all, _min: every layer count, the smallest one, of a padded
// count mz.)
constexpr size_t kConvzLds = 80 * 1024;
__host__ __device__ constexpr int conv_inplace(int nz, int mz, int build, int tsize)
{
    return build == 0 || mz > 8 ? 0 : mz == 1 ? 1 : convz_lds(build, 1, nz, tsize) <= kConvzLds ? 2 : 0;
}
__host__ __device__ constexpr bool conv_inplace_all(int mz, int build, int tsize) { return conv_inplace(mz, mz, build, tsize) != 0; }
__host__ __device__ constexpr bool conv_inplace_min(int mz, int build, int tsize)
{
    return conv_inplace(mz / 2 + 1, mz, build, tsize) != 0;
}

// LDS layout of the line buffers (pad_for, padx in ssm_fft.hpp).  The
// compile-time-length transforms can store lines with one pad element per
// 2^PADL (PADL = 0: dense), which spreads their strided accesses over the
// banks; the runtime-length ones use the dense layout.
#ifndef SSM_X_CT
#define SSM_X_CT 1
#endif
#ifndef SSM_X_PADL
#define SSM_X_PADL 4
#endif
#ifndef SSM_CONV_PADL
#define SSM_CONV_PADL 0
#endif
#ifndef SSM_CONV3_PADL
#define SSM_CONV3_PADL 4
#endif
// the x kernels' 3 2^a layout in FP32: one pad per 8 elements (fewer bank
// conflicts on its 8-byte elements; FP64 keeps one per 16)
#ifndef SSM_X3_PADL_F32
#define SSM_X3_PADL_F32 3
#endif
// x lengths with compile-time passes: powers of two 32..512 (lm = log2 m)
// and 3 2^lm for 48..384, in the pad-SSM_X_PADL layout (3 2^lm in FP32:
// pad-SSM_X3_PADL_F32); tsize: bytes per real value
__host__ __device__ constexpr bool x_ct_len(int lm, int f3) { return SSM_X_CT && !f3 && lm >= 5 && lm <= 9; }
__host__ __device__ constexpr bool x_ct3_len(int lm, int f3) { return SSM_X_CT && f3 && lm >= 4 && lm <= 7; }
__host__ __device__ constexpr int x_padl(int lm, int f3, int tsize)
{
    return x_ct_len(lm, f3)    ? pad_for(SSM_X_PADL, lm)
           : x_ct3_len(lm, f3) ? pad_for(tsize == 4 ? SSM_X3_PADL_F32 : SSM_X_PADL, lm)
                               : 0;
}
__host__ __device__ constexpr int conv_padl(int mz, int lmy, int f3y)
{
    return conv_ct_shape(mz, lmy, f3y)    ? pad_for(SSM_CONV_PADL, lmy)
           : conv_ct3_shape(mz, lmy, f3y) ? pad_for(SSM_CONV3_PADL, lmy)
                                          : 0;
}
// The inverse x kernel's transform in two register steps (xinv_two_step), for
// the lengths whose passes are two: m = 2^lm (32..256; FP64 32..128, whose
// 256 would spill: 256 x 256 x 8, 48 images 0.90 ms against 0.76) and 3 2^lm
// (48, 96, 192).  The first pass has radix r1 and nb values at stride nb to a lane;
// the rest of the transform gives nout outputs to each of r1 lanes.
struct Xinv2 {
    int r1, nb, nout;
};
__host__ __device__ constexpr bool xinv2_len(int lm, int f3, int tsize)
{
    return SSM_X_CT && (f3 ? lm >= 4 && lm <= 6 : lm >= 5 && lm <= (tsize == 4 ? 8 : 7));
}
__host__ __device__ constexpr Xinv2 xinv2_cfg(int lm, int f3)
{
    const int m = (f3 ? 3 : 1) << lm, r1 = lm == 5 ? 8 : 16;
    return Xinv2{r1, m / r1, m / r1};
}
// its rounds of second-step items per thread (tiles of at most 2048 elements
// and workgroups of nt threads)
__host__ __device__ constexpr int xinv2_rounds(Xinv2 c, int nt)
{
    const int per = c.nout * (nt / 256);
    return (12 + per - 1) / per;
}
// LDS elements from one row pair to the next: nb rows of 2 r1 + 1 values, made
// an odd multiple of what spreads hp row pairs (consecutive lanes) over the
// banks
__host__ __device__ constexpr int xinv2_line(Xinv2 c, int hp, int tsize)
{
    const int n = c.nb * (2 * c.r1 + 1), w = tsize == 4 ? 32 : 16, u = hp < w ? w / hp : 1;
    const int k = (n + u - 1) / u;
    return u * (k | 1);
}
// Threads of the inverse x transform's workgroups, and the lengths with such
// workgroups (Prob::xi2 = 2, in two steps), whose lattices have the fewest
// tiles: twice the wavefronts halve each lane's chain of rows where few
// workgroups share a CU.  k_xinv, us, 256 -> 512 threads: FP32 64 x 64, 20
// images 16.4 -> 13.2, 200 20.6 -> 18.8, 1000 57 -> 60; 32 x 32, 10 images
// 12.0 -> 10.8; FP64 32 x 32, 10 images 13.0 -> 11.3, 1000 30.8 -> 29.9.  Longer
// lines lose on large batches what they gain on small ones (FP32 112 x 112,
// 60 images 20.6 -> 18.9 but 240 50.8 -> 54.1; 72 x 72, 1000 107 -> 125; 256 x
// 256 x 8, 48 images 413 -> 470; FP64 64 x 64, 1000 92 -> 117), and the choice is
// the problem's alone, since the order of its energy sums follows from it.
// 1024 threads: 64 x 64, 1000 images 87.
constexpr int kXinvWide = 512;
__host__ __device__ constexpr bool xinv2_wide(int lm, int f3, int tsize)
{
    return !f3 && lm <= (tsize == 4 ? 6 : 5);
}
// row stride of the tile's real field, likewise
__host__ __device__ constexpr int xinv2_hrow(int nx, int hp)
{
    const int r = hp < 32 ? 32 / hp : 1;
    return nx + ((r - nx) & 31);
}
// 1: its twiddles have a copy in LDS (0 where that would cost a workgroup)
__host__ __device__ constexpr int xinv2_twlds(int m, int f3, int tsize) { return f3 || m * tsize <= 512; }

// elements of a buffer of n elements in the pad-padl layout
__host__ __device__ constexpr int padded_len(int n, int padl) { return padl ? n + (n >> padl) + 1 : n; }

// Kernel kinds (profiling slots; names in the runtime).
enum KernelKind {
    KK_XFWD = 0, KK_CONV, KK_XINV, KK_ARC, KK_REDUCE, KK_INTERP,
    KK_TAN1, KK_TAN2, KK_TANRED, KK_SPEC, KK_UTIL, KK_GRAPH, KK_RK, KK_COUNT_
};

// Per-problem descriptor, resident in device memory (read-only in kernels).
struct Prob {
    int nx, ny, nz, K;
    int mx, my, mz;        // half padded lengths >= nx, ny, nz: 2^a, or 3 2^a (a >= 4) along x and y
    int lmx, lmy, lmz;     // log2 of their power-of-two factor
    int f3x, f3y;          // 1: mx (my) = 3 2^lmx (3 2^lmy)
    int pz;                // padded z length: 2*mz when nz > 1, else 1
    int nhz;               // z halves of the padded z spectrum: 2 when nz > 1, else 1
    int yt;                // lattice rows per tile of the inverse-x / epilogue kernel
    int nty;               // ceil(ny / yt)
    int tiles;             // inverse-x tiles per image = nz * nty (energy partials)
    int ytf, ntyf, tilesf; // the same for the forward x kernel
    int wgf, wgi;          // forward / inverse x workgroups (K * tiles, forward times 3 with csplit; padded to 8)
    int csplit;            // 1: a forward x workgroup takes one component of its tile, else all three
    int img0;              // index of this problem's first image in batch-wide arrays
    int gconv;             // (image, kx) slices per convolution workgroup: consecutive ones (kx fastest),
                           // or images of one kx (in place)
    int conv1;             // convolution in place, both halves together: 1 by k_conv1, 2 by k_convz
    int xi2;               // inverse x transform by xinv_two_step: 1, or 2 with kXinvWide threads
    int arc_chunks;        // arc-length workgroups (flat chunks of 3N) per image
    int xcd_remap;         // convolution kernel: group same-kx slices on one XCD
    long long N;           // sites per image
    long long s_off;       // element offset of image 0 in spin / field buffers
    long long x_off;       // complex-element offset in the x-spectrum buffer X
    long long xo_off;      // offset of the convolved spectra from the same base: x_off where the
                           // convolution works in place (conv1), in X' after X otherwise
    long long nh_off;      // element offset of this shape's dipole-kernel spectrum
    long long ep_off;      // offset (doubles) of energy partials: [K][tiles][kNTerm]
    long long ap_off;      // offset (doubles) of arc partials: [K][arc_chunks*4]
    long long fp_off;      // offset (doubles) of tangent partials: [K][ichunks][2]
    long long fm_off;      // offset (doubles) of per-workgroup force maxima: [K][ichunks]
    int ichunks;           // per-site workgroups per image (interp / tangents)
    int vec4;              // FP32 images of N divisible by 4, 16-byte aligned: 4 sites per thread
    int vec2;              // FP64 images of even N, 16-byte aligned: 2 sites per thread
    int ichunks4;          // interpolation workgroups per image (ichunks / 4 with vec4, / 2 with vec2)
    int arc_g;             // images per arc-length workgroup (image groups of arc_g)
    int arc_ng;            // image groups: arc-length workgroups = arc_chunks * arc_ng
    int red1;              // 1: reduced by one workgroup (k_reduce1), else one per image (k_reduce)
    double J, d, ku, D;    // eq. (1) parameters
};

// Work maps: workgroup ranges per problem for each kernel kind.
struct WorkMap {
    int* start;      // device: [nprob + 1] prefix sums of workgroup counts
    int total;
    size_t lds;      // dynamic LDS bytes (inverse x, in-place convolution builds)
};

// ------------------------------------------------------------------------
// launchers (ssm_kernels.hip); all enqueue on `st` and return the HIP error
// ------------------------------------------------------------------------
// The FFT kernels come in kinds (x: power-of-two or 3 2^a length;
// convolution: one build per conv_build value) and each kind has a work map
// of its own, in which the problems of other kinds have no workgroups; a
// kind whose map is empty is not launched.  wm[0..1]: x length kinds
// (f3x), inverse x also wm[2] (Prob::xi2 = 2); wm[conv_slot(b)]: convolution
// build b.
// (the in-place kernels have slots of their own, kConvSlots / 2 further on)
constexpr int kConvSlots = 16;
__host__ __device__ constexpr int conv_slot(int b, int inplace)
{
    return (inplace ? kConvSlots / 2 : 0) + (b == 0 ? 0 : (b <= 8 ? b - 4 : b - 15));
}
template <typename T>
hipError_t launch_xfwd(const Prob* P, int np, const WorkMap* wm, const T* s, void* X,
                       const void* tw, const int* done, size_t lds, hipStream_t st);
// the convolved x half-spectra go to Prob::xo_off of the same buffer
template <typename T>
hipError_t launch_conv(int mz, const Prob* P, int np, const WorkMap* wm, void* X, const T* nhat, const void* tw,
                       const int* done, size_t lds, hipStream_t st);
// mode bits for the inverse/epilogue kernel: EPI_STEP writes the stepped
// string, EPI_FIELD the field h, EPI_FORCE the damping right-hand side
// (s.s) h - (s.h) s in place of h, EPI_TERMS the four term partials
enum { EPI_STEP = 1, EPI_FIELD = 2, EPI_TERMS = 4, EPI_FORCE = 8 };
template <typename T>
// fcp, fcd: coefficients of EPI_FORCE (precession, damping)
hipError_t launch_xinv(const Prob* P, int np, const WorkMap* wm, const void* Xp, const T* s,
                       T* s_star, T* h, double* epart, const void* tw, const int* done,
                       int mode, double tau, double fcp, double fcd, hipStream_t st);
template <typename T>
hipError_t launch_arc(const Prob* P, int np, const WorkMap& wm, const T* ss, double* apart,
                      const int* done, hipStream_t st);
// Step-2 options of the reduction's last workgroup (ssm_set_reparam): bit 0
// natural cubic spline, bit 1 climbing image.  E: the current energies
// (climbing image choice); per problem: kci (climbing image or -1), spl_ok
// (spline factors valid); per image: interval widths hh, Thomas factors
// (sa, den, cp); per target image: spline weights A, B and interval width H.
struct Step2 {
    int opts = 0;
    const double* E = nullptr;
    int* kci = nullptr;
    int* spl_ok = nullptr;
    double* hh = nullptr;
    double* sa = nullptr;
    double* den = nullptr;
    double* cp = nullptr;
    double* A = nullptr;
    double* B = nullptr;
    double* H = nullptr;
    // the one-pass spline step's K x K operator of every problem of at most
    // wmax images (row k of problem pi at Wm + (img0 + k) kWRow), formed by
    // the end of step 2; wmax = 0: not formed
    double* Wm = nullptr;
    int wmax = 0;
};
constexpr int kWRow = 32;  // row stride of Step2::Wm (the largest one-pass image count)
// kinds: bit 0 problems reduced per image, bit 1 problems reduced by one
// workgroup (Prob::red1)
hipError_t launch_reduce(const Prob* P, int np, int nimg, int kinds, const int* istart, const double* epart,
                         const double* apart, double* E, double* Tm, double* E_out, double* T_out,
                         double* seg, double* alpha, int* jidx, double* wgt, int* skip, int* done,
                         int* iters, int* count, int* flags, int with_arc, hipStream_t st,
                         Step2 s2 = Step2{});
// launch_reduce (with_arc, no options) and launch_interp in one, for batches of
// red1 problems only
template <typename T>
hipError_t launch_interp1(const Prob* P, int np, const WorkMap& wm, const T* ss, T* s, const int* done,
                          const double* epart, const double* apart, double* E, double* seg, double* alpha,
                          int* jidx, double* wgt, int* skip, int* iters, int* flags, hipStream_t st, Step2 s2);
template <typename T>
// kci (or NULL): per-problem climbing image, copied like the endpoints;
// skip_if (or NULL): problems whose flag is set are left to the spline
hipError_t launch_interp(const Prob* P, int np, const WorkMap& wm, const T* ss, T* s,
                         const int* jidx, const double* wgt, const int* skip, const int* done,
                         int* flags, hipStream_t st, const int* kci = nullptr,
                         const int* skip_if = nullptr);
// natural cubic spline: second derivatives M of every site and component
// (M buffer in the spin layout), then the interpolation at the targets;
// problems of at most kskip images are left to launch_interp_splw
template <typename T>
hipError_t launch_spline_m(const Prob* P, int np, const WorkMap& wm_sitep, const T* ss, T* M, Step2 s2,
                           const int* done, int kskip, hipStream_t st);
template <typename T>
hipError_t launch_interp_spline(const Prob* P, int np, const WorkMap& wm, const T* ss, const T* M, T* s,
                                const int* jidx, const double* wgt, Step2 s2, const int* done, int* flags,
                                int kskip, hipStream_t st);
// the spline step in one pass for the problems of at most kSplwMax images
// (one thread per site, wm_sitep); kmax: the largest of their image
// counts; problems with more images are left to the two kernels above, so
// each problem takes the same path whatever else is in the batch
// (lin, or NULL: the skip flags; a problem with a degenerate spline then takes
// the linear step there as well, the same bits as launch_interp's)
template <typename T>
constexpr int kSplwMax = sizeof(T) == 4 ? 32 : 16;
static_assert(kSplwMax<float> <= kWRow && kSplwMax<double> <= kWRow, "operator rows");
template <typename T>
hipError_t launch_interp_splw(const Prob* P, int np, const WorkMap& wm_sitep, int kmax, const T* ss, T* s,
                              const int* jidx, const double* wgt, Step2 s2, const int* done, int* flags,
                              const int* lin, hipStream_t st);
// climbing image: partial sums (|t~|^2, F.t~) over image kci, their
// per-problem reduction to c = F.t~ / |t~|^2, and the step
// normalise(s + tau (F - 2 c t~)) into ss
template <typename T>
hipError_t launch_ci_part(const Prob* P, int np, const WorkMap& wm, const T* s, const T* h, const double* E,
                          double* part, int* kci, const int* done, hipStream_t st);
hipError_t launch_ci_red(const Prob* P, int np, const double* part, const int* kci, double* coef,
                         const int* done, hipStream_t st);
template <typename T>
hipError_t launch_ci_step(const Prob* P, int np, const WorkMap& wm, const T* s, const T* h, T* ss,
                          const int* kci, const double* coef, double tau, const int* done, hipStream_t st);
template <typename T>
hipError_t launch_tan1(const Prob* P, int np, const WorkMap& wm, const T* s, const T* h,
                       T* tt, double* fpart, hipStream_t st);
hipError_t launch_tanred(const Prob* P, int np, const double* fpart, double* tcoef,
                         hipStream_t st);
template <typename T>
hipError_t launch_tan2(const Prob* P, int np, const WorkMap& wm, const T* s, const T* h,
                       const T* tt, T* t_out, const double* tcoef, double* fmax,
                       hipStream_t st);
hipError_t launch_fmax(const Prob* P, int np, const double* fmax, double* fnorm, int* done,
                       double tol, double* out, hipStream_t st);
template <typename T>
hipError_t launch_spectrum(const Prob& p, T* nhat, double* f1, double* f2, const double* tw64,
                           hipStream_t st);
hipError_t launch_barrier(const Prob* P, int np, const double* E, const double* Tm,
                          double* out, hipStream_t st);
hipError_t launch_iters_out(int np, const int* iters, const int* iters0, int* out,
                            hipStream_t st);
hipError_t launch_fill_int(int* p, int n, int v, hipStream_t st);
// up to kBlobBytes bytes copied to device memory by a kernel whose argument
// carries them
constexpr int kBlobBytes = 2048;
struct Blob {
    int n;
    unsigned char b[kBlobBytes];
};
hipError_t launch_put(void* dst, const Blob& b, hipStream_t st);
hipError_t launch_fill_double(double* p, int n, double v, hipStream_t st);

// Adaptive Dormand-Prince 5(4) step 1.  Per image (batch-wide index g):
// t[g] time reached in the interval, dtp[g] proposed step, dtu[g] step of
// the current attempt, capped[g] whether that attempt ends the interval,
// act[g] still integrating, acc[g] current attempt accepted, cnt[2g..]
// accepted / rejected steps; nact counts active images after control.
struct RkState {
    double* t;
    double* dtp;
    double* dtu;
    int* capped;
    int* act;
    int* acc;
    int* cnt;
    int* nact;
};
template <typename T>
struct RkSlopes {
    T* k[7];
};
hipError_t launch_rk_init(const Prob* P, int np, int nimg, const int* istart, RkState rs, double Tint,
                          const int* done, hipStream_t st);
template <typename T>
hipError_t launch_rk_stage(const Prob* P, int np, const WorkMap& wm, const T* s, RkSlopes<T> ks, int stage,
                           RkState rs, T* y, const int* done, hipStream_t st);
template <typename T>
hipError_t launch_rk_err(const Prob* P, int np, const WorkMap& wm, const T* s, const T* y, RkSlopes<T> ks,
                         RkState rs, double rtol, double atol, double* part, const int* done, hipStream_t st);
hipError_t launch_rk_ctrl(const Prob* P, int np, int nimg, const int* istart, const double* part, RkState rs,
                          double Tint, const int* done, int* flags, hipStream_t st);
template <typename T>
hipError_t launch_rk_apply(const Prob* P, int np, const WorkMap& wm, T* s, const T* y, RkSlopes<T> ks,
                           RkState rs, const int* done, hipStream_t st);
template <typename T>
hipError_t launch_rk_norm(const Prob* P, int np, const WorkMap& wm, const T* s, T* ss, const int* done,
                          int* flags, hipStream_t st);

}  // namespace ssm
