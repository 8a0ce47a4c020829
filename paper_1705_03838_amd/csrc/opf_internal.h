// Internal definitions shared by the host code and the HIP kernels of the
// pipe-flow time-step library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "../../include/opf.h"

namespace opf {

constexpr int W9 = 9;     // finite-difference stencil width (Section 2: 9 points)
constexpr int HALF = 4;   // points on each side of a centred stencil
constexpr int FACW = 14;  // doubles per LU factor row: 8 of L, 4 of U, 1/U_ii, pad
// The N rows of one factor are FMAIN-double main records (L[i+1..i+4][i],
// U[i-1..i-4][i], 1/U_ii, pad) followed by FTAIL-double tail records
// (L[i+5..i+8][i]), N FACW doubles in all.  They make the influence data and the
// Green's function; the substep solve uses the images.
constexpr int FMAIN = 10;
constexpr int FTAIL = 4;
constexpr int NHOM = 7;   // real radial lines of influence data per (m,|k|)
// Block form of the radial operators.  The rows are taken in tiles of four,
// aligned to the wall, the last eight rows as one block: a 9-point stencil
// reaches at most four rows either way, and the clamped wall stencils (rows
// N-4..N-2, columns from N-9 on) stay within the last block and the tile
// before it, so every operator is block tridiagonal.  nt = btd_nt(N) tiles
// precede the last block; zero rows pad the axis end, btd_rows(nt) rows in
// all.  With the diagonal blocks D_I of the block elimination
//   D_0 = A_00,  D_I = A_II - B_I D_{I-1}^{-1} C_{I-1}
// (B_I = A_{I,I-1}, C_I = A_{I,I+1}), A x = b is solved by
//   v_I = D_I^{-1} (b_I - B_I v_{I-1}) upwards, x_I = v_I - D_I^{-1} C_I x_{I+1} downwards.
// Only the D_I^{-1} depend on the operator (its image: nt tiles of 16
// doubles, then the 8 x 8 block as four tiles, rows by columns; tiles 2 p and
// 2 p + 1 interleaved, element [i][k] of theirs at 32 p + 2 (4 k + i) + 0, 1, so
// that a lane's elements of two tiles are one 16-byte load).  The couplings are those of
// d^2/dr^2 + (1/r) d/dr, the same for every operator of one axis parity,
// because the Helmholtz systems are solved as L - Re / (c dt) (scaled by
// -Re / c): -B_1..-B_nt (B_nt the rows of the last block's first half), the
// second half's tile, then -C_0..-C_{nt-1}.  Only stencils folded at the axis
// depend on the parity, entries with row + column <= 3; with at most seven
// rows of padding those lie in B_1, B_2, C_0 and C_1, which follow for the
// even and then for the odd parity (element [i][k] of a tile at 4 k + i).
// nt is rounded up to even so that few kernels cover 12 <= N <= 64.
__host__ __device__ constexpr int btd_nt(int N) { return ((N - 5) / 4 + 1) / 2 * 2; }
__host__ __device__ constexpr int btd_rows(int nt) { return 4 * nt + 8; }
__host__ __device__ constexpr int btd_image(int nt) { return 16 * (nt + 4); }
__host__ __device__ constexpr int btd_coupling(int nt) { return 16 * (2 * nt + 9); }
static_assert(btd_nt(12) == 2 && btd_nt(16) == 2 && btd_nt(17) == 4 && btd_nt(64) == 14, "tiles before the last block");
static_assert(btd_rows(btd_nt(64)) == 64 && btd_rows(btd_nt(12)) == 16, "padded rows");
constexpr int NMAX = 64;  // radial points handled by one solve workgroup
// First column of row n's 9-point window: centred, clamped at the wall, folded at the axis.
__host__ __device__ constexpr int stencil_column(int n, int N) {
    const int e = n - 4 < N - 9 ? n - 4 : N - 9;
    return e < 0 ? 0 : e;
}

// Complex number used by the kernels (interleaved re/im, same layout as
// complex128 / complex64 in memory).  Aligned to its full size so that one
// value is one 16-byte (FP64) or 8-byte (FP32) load or store, in HBM and LDS.
template <typename T>
struct alignas(2 * sizeof(T)) cpx {
    T x, y;
};

// Device-resident tables built at create time (all pointers into the
// caller's workspace).
struct Tables {
    const double* r;      // [N] radial nodes
    const double* rinv;   // [N] 1/r
    const double* quad;   // [N] weights of int_0^1 g(r) r dr (g even in r)
    const double* d1;     // [2][N][9] folded first-derivative weights, parity 0 even / 1 odd
    const double* d2;     // [2][N][9] folded second-derivative weights
    const int* s0;        // [N] first column of row n's 9-point window
    const double* img;    // inverse diagonal blocks: [K][MU] Helmholtz, then [K][M] pressure (btd_image doubles each)
    const double* coup;   // coupling tiles (btd_coupling doubles)
    const double* wl;     // [2][N][9] folded weights of d2/dr2 + (1/r) d/dr, parity 0 even / 1 odd; then 0, 1
    const double* hom;    // [M][K][NHOM][N] influence data (h1+, h1-, q, h2, h3, h4, P1)
    const double* ainv;   // [M][2K-1][16][2] inverse influence matrices (complex)
    const double* green;  // [N] flux Green's function: H_0 u_G = 1, u_G(1) = 0
    double qG_inv;        // 1 / int_0^1 u_G r dr
};

// Arguments of one nonlinear-term evaluation (three transform kernels).
struct NLArgs {
    int N, M, K, nk;
    const void* in[6];  // spectral u_r,u_t,u_z,w_r,w_t,w_z  [M][nk][N] (storage type)
    void* H;            // z-transformed fields [6][N][M][3K] (compute type)
    void* G;            // theta-transformed products [3][N][M][3K] (compute type)
    void* out[3];       // spectral N_r, N_t, N_z [M][nk][N] (storage type)
    const void* twz;    // e^{-2 pi i t / 3K}, t < 3K (compute type)
    const void* twt;    // e^{-2 pi i t / 3M}, t < 3M (compute type)
    double scale;       // 1 / (9 K M)
    double rot[3];      // rotation vector Omega (Cartesian, z the pipe axis) of the Coriolis force
    int rotating;       // nonzero: add -2 Omega x u to u x omega (mp = 1 unless Omega is axial)
    int tz;             // axial points per theta-stage workgroup (tile shape), see tz_ok
    int ztile;          // radial lines per z-transform workgroup (tile shape), see ztile_ok
};

// Arguments of one substep solve (one kernel).
struct SolveArgs {
    int N, M, K, nk, mp, MU;
    int gm;             // consecutive m per workgroup (tile shape), see gm_ok
    int kind;           // OPF_SOLVE_PRED / CORR / RAW
    int fixed_flux;
    double alpha, Re, c, inv_dt, aexp, force;
    double hscale;      // -Re / c: the Helmholtz systems are solved as L - Re / (c dt) (see helmholtz_scale)
    const double* u0;   // u^n (external layout, complex128); PRED / CORR
    const void* n0;     // N^n (nonlinear storage type), or R (complex128) for RAW
    const void* n1;     // N^p for CORR
    double* u_out;      // complex128 output state (nullable)
    float* u_out32;     // complex64 shadow of the output state (nullable)
    void* w_out;        // vorticity of the output (nonlinear storage type, nullable)
    double* p_out;      // pressure head [M][nk][N] complex128 (nullable)
    double* beta_out;   // flux correction beta (device scalar)
    const double* wall; // wall velocity [3][M][nk] complex (r, theta, z) at r = 1, or null (no slip)
    Tables t;
};

// Arguments of the vorticity / diagnostics kernels.
struct AuxArgs {
    int N, M, K, nk, mp;
    int mirror;         // vorticity: m = 0, k < 0 written as conjugates of k > 0
    double alpha;
    const double* u;    // complex128 external layout
    double* w;          // complex128 output (vorticity)
    double* partial;    // [M nk][4] diagnostics per mode (k_diag)
    const double* wall; // wall velocity as in SolveArgs, or null
    Tables t;
};

// Arguments of the operator-table kernels (banded LU factors, influence
// data, flux Green's function), written into the workspace tables.
struct FactorArgs {
    int N, M, K, MU, mp;
    double alpha;
    double cr;          // c / Re
    double inv_dt;      // 1 / dt
    double shift;       // Re / (c dt), consistent with SolveArgs::hscale
    const double* rinv;
    const double* wl;   // Tables::wl
    const double* quad;
    const double* d1;
    const double* d2;
    const int* s0;
    double* fac;        // [MU K + M K] factors of N FACW doubles: H_{|mu|,|k|} then L_{m,|k|}
    double* img;        // inverse diagonal blocks (Tables::img)
    int nt;             // btd_nt(N)
    double* hom;        // [M][K][NHOM][N]
    double* ainv;       // [M][2K-1][16][2]
    double* green;      // [N]
    int* flags;         // [MU K + M K] factor status, then [M (2K-1)] influence status
    int* image_flags;   // [MU K + M K] image status
    double* qg;         // int_0^1 u_G r dr (device scalar)
};
// Factor the Helmholtz operators (and, with pressure, the pressure
// operators and the unit-wall pressure P1), then the homogeneous solutions,
// inverse influence matrices and Green's function.
hipError_t launch_operator_tables(const FactorArgs& a, bool pressure, hipStream_t s);

// Kernel-only timing of one launch: when start is set, the launch goes
// through hipExtLaunchKernelGGL, which records start and stop around the
// kernel itself (no dispatch gap), for opf_profile_steps.
struct KernelTiming {
    hipEvent_t start = nullptr, stop = nullptr;
};
template <typename... Args, typename F = void (*)(Args...)>
inline void launch_timed(F kernel, const dim3& grid, const dim3& block, uint32_t lds, hipStream_t s,
                         const KernelTiming& kt, Args... args) {
    if (kt.start) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, kt.start, kt.stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
}

// Launchers (return the first HIP error).
hipError_t launch_nonlinear(const NLArgs& a, int precision, hipStream_t s);
// One of the three transform kernels: 0 z-inverse, 1 theta + product, 2 z-forward.
hipError_t launch_nonlinear_stage(const NLArgs& a, int precision, int stage, hipStream_t s,
                                  const KernelTiming& kt = KernelTiming{});
bool nonlinear_supported(int M, int K);
// Admissible transform tile shapes: tz in {2, 4, 8} axial points per theta
// workgroup, zt in {4, 8, 16} radial lines per z workgroup, each while the
// longer radix pass fits the workgroup.
bool tz_ok(int tz, int M);
bool theta_wide(int N, int M, int K, bool fp32);  // the theta stage takes 16 axial points whatever tz is
bool ztile_ok(int zt, int K);
constexpr int DEFAULT_TZ = 4, DEFAULT_ZTILE = 8;
// Radial lines per z workgroup before any tuning: 16 with FP32 transforms
// (half the bytes per line, so the same bytes per workgroup as 8 lines in
// FP64), else 8.
inline int default_ztile(int precision) { return precision == OPF_MIXED ? 16 : DEFAULT_ZTILE; }
hipError_t launch_solve(const SolveArgs& a, int precision, hipStream_t s, const KernelTiming& kt = KernelTiming{});
// Batched forms: one launch for `members` argument records in device memory
// (grid.y = member); `proto` gives the shared sizes.
hipError_t launch_nonlinear_batch(const NLArgs& proto, const NLArgs* dev_args, int members, int precision,
                                  int stage, hipStream_t s);
hipError_t launch_solve_batch(const SolveArgs& proto, const SolveArgs* dev_args, int members, int precision,
                              hipStream_t s);
int default_gm(int mp);                  // of an ensemble class
int context_gm(int mp, int M, int K);    // of a single context
bool gm_ok(int gm, int mp);
constexpr int GM_SPAN = 6;  // Helmholtz operators that the m of one solve workgroup may use, see gm_ok
hipError_t launch_vorticity(const AuxArgs& a, hipStream_t s);
hipError_t launch_diag(const AuxArgs& a, hipStream_t s);
// out[2M + 2N + 4]: see k_diag_pack
hipError_t launch_diag_pack(const AuxArgs& a, const double* cpart, int ncp, const double* beta, double* out, hipStream_t s);
// Largest |u_r| wr[n] + |u_theta| wt[n] + |u_z| wz over the physical points
// of each (n, 4-point z tile) workgroup into out[block], from the
// z-transformed fields in a.H (stage 0 of the nonlinear term).
hipError_t launch_cfl(const NLArgs& a, int precision, const double* wr, const double* wt, double wz, double* out,
                      hipStream_t s);

// Context accessors for translation units other than the host core.
hipStream_t ctx_stream(const opf_ctx* c);
const opf_params& ctx_params(const opf_ctx* c);
void ctx_set_error(opf_ctx* c, const std::string& msg);

}  // namespace opf
