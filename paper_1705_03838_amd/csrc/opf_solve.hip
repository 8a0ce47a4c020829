// Radial solves of one substep on MI355X: right-hand side, pressure-Poisson
// equation, Helmholtz equations, influence-matrix boundary correction,
// fixed flux and vorticity, for every Fourier mode.
//
// Section 2 of the paper: a pressure-Poisson formulation with an influence-
// matrix enforcement of the boundary conditions (g = 0 when satisfied);
// Section 2.2: the implicit viscous terms are banded systems solved by LU
// decomposition for each Fourier mode.  With u+- = u_r +- i u_theta the
// vector Laplacian decouples (L_{m+-1} on u+-, L_m on u_z and P), so every
// system is a real banded matrix acting on complex data.
//
// One wave handles |k| and one m, both signs of k: two modes, four real
// right-hand sides per system.  Lanes are radial nodes for the stencil work;
// the banded systems are solved in block form (btd_nt in opf_internal.h) on
// the FP64 matrix cores.  The waves of a workgroup share the coupling
// tiles and an L1 and meet at one barrier.  m = 0 solves k >= 0 only and writes the
// conjugate into -k (Hermitian symmetry of a real field); mode (0,0) has
// u_r = 0, no pressure and the fixed-flux correction.
#include "opf_internal.h"

namespace opf {

constexpr int LSTR = NMAX + 2;            // LDS line stride (complex): avoids bank aliasing

struct dcplx {
    double x, y;
};
__device__ __forceinline__ dcplx operator+(dcplx a, dcplx b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ dcplx operator-(dcplx a, dcplx b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ dcplx operator*(double s, dcplx a) { return {s * a.x, s * a.y}; }
__device__ __forceinline__ dcplx cm(dcplx a, dcplx b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ dcplx ix(dcplx a) { return {-a.y, a.x}; }  // i * a

typedef double dpair __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ dcplx load_c(const void* base, size_t idx) {
    const T* p = reinterpret_cast<const T*>(base) + 2 * idx;
    return {double(p[0]), double(p[1])};
}
// A complex value as stored (two T), read now and widened where it is used.
template <typename T>
struct vec2 {
    T x, y;
};
// The value at a wave-uniform base plus a lane's 32-bit byte offset (one address register per lane).
template <typename T>
__device__ __forceinline__ vec2<T> load_v(const void* base, unsigned bytes) {
    const T* p = reinterpret_cast<const T*>(static_cast<const char*>(base) + bytes);
    return {p[0], p[1]};
}
template <typename T>
__device__ __forceinline__ dcplx to_c(vec2<T> v) {
    return {double(v.x), double(v.y)};
}
template <typename T>
__device__ __forceinline__ void store_c(void* base, size_t idx, dcplx v) {
    T* p = reinterpret_cast<T*>(base) + 2 * idx;
    p[0] = T(v.x);
    p[1] = T(v.y);
}

// Rounds v here: the compiler may not contract the operations before with
// those after into one multiply-add.
__device__ __forceinline__ void settle(dcplx& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// Vorticity of mode (m, kappa) at one radial node, the cylindrical curl
// (the rotational form of the nonlinear term, Section 2.2):
//   w_r = (i m / r) u_z - i kappa u_theta,  w_theta = i kappa u_r - u_z',
//   w_z = u_theta' + (u_theta - i m u_r) / r,
// from the node's values and the radial derivatives duz = u_z' (parity of
// m) and dut = u_theta' (parity of m +- 1).
__device__ __forceinline__ void curl_row(dcplx duz, dcplx dut, double rinv, int m, double kap, dcplx ur, dcplx ut,
                                         dcplx uz, dcplx& wr, dcplx& wt, dcplx& wz) {
    // explicit multiply-adds: the solve's vorticity and k_vorticity's are the same to the last bit
    const double mr = double(m) * rinv, dm = double(m);
    wr = {fma(kap, ut.y, -(mr * uz.y)), fma(-kap, ut.x, mr * uz.x)};
    wt = {fma(-kap, ur.y, -duz.x), fma(kap, ur.x, -duz.y)};
    wz = {fma(rinv, fma(dm, ur.y, ut.x), dut.x), fma(rinv, fma(-dm, ur.x, ut.y), dut.y)};
}

__device__ __forceinline__ void load_pair(const double* p, double& a, double& b) {
    const dpair v = *reinterpret_cast<const dpair*>(p);
    a = v.x;
    b = v.y;
}

// v_mfma_f64_4x4x4_4b_f64: four independent 4 x 4 x 4 products.  Lane
// l = i + 4 blk + 16 k supplies A[i][k], lane l = j + 4 blk + 16 k supplies
// B[k][j], and lane l = j + 4 blk + 16 i receives C[i][j] + sum_k A[i][k] B[k][j]:
// results arrive in the layout of the B operand, so products chain without
// any exchange between lanes.
__device__ __forceinline__ double mm4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Solve four block-tridiagonal systems (one per matrix block, each with four
// real right-hand sides) in place: D is this lane's element of each inverse
// diagonal block, cp its element of the first coupling tile in LDS and ap that
// of its parity's first one (layout at btd_coupling, tiles 16 doubles apart),
// col its element of the right-hand side's first tile in LDS (tiles 8 doubles
// apart).
//
// The chain is 4 NT + 4 dependent matrix instructions at about 28 cycles
// each (60 at 64 rows: 1.7k cycles).  One lane per right-hand side walking
// the scalar LU factors took 6.4k cycles for the pressure and 7.0k for the
// Helmholtz systems even with two lanes meeting in the middle, bound by the
// latency of four LDS instructions per row.  LDS reads run AHEAD tiles ahead,
// held there by a scheduling barrier per tile (free scheduling hoists them
// all and spills).
template <int NT>
__device__ __forceinline__ void btd_solve(const double* D, const double* cp, const double* ap, double* col) {
    constexpr int AHEAD = 4;
    double r[NT + 2], cb[NT + 1], cc[NT], v[NT];
    auto fload = [&](int q) {
        if (q <= NT) {
            cb[q] = q < 2 ? ap[16 * q] : cp[16 * q];
            r[q + 1] = col[8 * (q + 1)];
        }
    };
    auto bload = [&](int q) {
        if (q >= 0) {
            cc[q] = q < 2 ? ap[16 * (2 + q)] : cp[16 * (NT + 1 + q)];
        }
    };
    double w = col[0];
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) fload(q);
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        fload(q + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        v[q] = mm4(D[q], w, 0.0);
        w = mm4(cb[q], v[q], r[q + 1]);
    }
#pragma unroll
    for (int q = NT - 1; q >= NT - AHEAD; --q) bload(q);
    const double w1 = mm4(cb[NT], v[NT - 1], r[NT + 1]);
    double x = mm4(D[NT + 1], w1, mm4(D[NT], w, 0.0));
    col[8 * (NT + 1)] = mm4(D[NT + 3], w1, mm4(D[NT + 2], w, 0.0));
    col[8 * NT] = x;
#pragma unroll
    for (int q = NT - 1; q >= 0; --q) {
        bload(q - AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        x = mm4(D[q], mm4(cc[q], x, 0.0), v[q]);
        col[8 * q] = x;
    }
}

// Sum over the 16 lanes of a DPP row, in every lane of the row.
template <int CTRL>
__device__ __forceinline__ double dpp_rotate(double v) {
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double row_sum(double v) {  // row_ror by 8, 4, 2, 1
    v += dpp_rotate<0x128>(v);
    v += dpp_rotate<0x124>(v);
    v += dpp_rotate<0x122>(v);
    return v + dpp_rotate<0x121>(v);
}
__device__ __forceinline__ double quad_sum(double v) {  // quad_perm [1,0,3,2], [2,3,0,1]
    v += dpp_rotate<0xB1>(v);
    return v + dpp_rotate<0x4E>(v);
}
// 9 weights of one parity for row n, in registers.
struct Row9 {
    double e[W9];
    __device__ __forceinline__ void load(const double* tab, int N, int par, int n) {
        // wave-uniform base, 32-bit lane offset, constant offsets: one address for all nine loads
        const double* p = tab + par * N * W9 + unsigned(n * W9);
#pragma unroll
        for (int j = 0; j < W9; ++j) e[j] = p[j];
    }
    __device__ __forceinline__ dcplx apply(const dcplx* line, int s0) const {
        dcplx acc = e[0] * line[s0];
#pragma unroll
        for (int j = 1; j < W9; ++j) acc = acc + e[j] * line[s0 + j];
        return acc;
    }
};

// LDS of one wave: the six lines (2 modes x 3 components) and the two
// pressure lines, zero rows in front of row 0.  The line stride, 4 mod 8
// complex, starts consecutive lines 16 (or 48) banks apart, so that the
// matrix layout's reads of four rows and several lines spread over the banks.
__host__ __device__ constexpr int solve_line(int nt) { return btd_rows(nt) + 4; }
// A workgroup's LDS: its waves' lines, then the coupling tiles.
constexpr size_t solve_lds(int nt, int gm) {
    return (size_t)gm * 8 * solve_line(nt) * sizeof(dcplx) + btd_coupling(nt) * sizeof(double);
}

// A workgroup of GM waves handles |k| = kabs and GM consecutive m, which share
// the coupling tiles in LDS and read neighbouring Helmholtz operators
// (wavenumbers mp m - 1 .. mp m + 1) through one L1; wave w handles m0 + w,
// modes s = 0, 1 at +k and -k.
//
// What bounds it: HBM (the spectral fields once, a third more for the tables)
// and, on small grids, the length of one wave's phases.  Predictor / corrector
// at 64 x 48 x 127 modes: 22.5 / 24.6 us in FP64 (26.0 / 28.1 with scalar
// banded factors shared through LDS and substituted by one wave of each
// workgroup), 21.2 / 22.9 in mixed precision (25.1 / 27.0); 24 x 8 x 15: 5.8 us
// (12.4); 41 x 18 x 23, mp = 3: 8.1 us (14.1); 48 x 24 x 63, mp = 2: 10.8 us
// (15.5).  Measured and dropped: every request made at the start with two waves
// per SIMD (42 us at 64 x 48 x 127), four waves per SIMD (38 us, spills), the
// coupling tiles by LDS DMA (the compiler then waits for every load in flight
// at each LDS read) and v kept in LDS instead of registers.
template <typename TNL, int NT>
__device__ __forceinline__ void k_solve_body(const SolveArgs& a) {
    constexpr int XS = solve_line(NT), IMG = btd_image(NT);
    extern __shared__ __align__(16) unsigned char solve_smem[];
    const Tables& t = a.t;
    const int N = a.N, K = a.K, nk = a.nk, mp = a.mp, GM = a.gm;
    const int nblk = (a.M + GM - 1) / GM;
    // Consecutive block indices go round-robin to the 8 XCDs; each XCD takes
    // a contiguous range of tiles instead, so the m-blocks of one |k|, which
    // share Helmholtz operators, meet in its L2.
    const int ntiles = (int)gridDim.x;
    const int tile = ntiles % 8 == 0 ? (blockIdx.x % 8) * (ntiles / 8) + blockIdx.x / 8 : (int)blockIdx.x;
    const int kabs = tile / nblk;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // a wave past the last m works on that one without writing anything, up
    // to the workgroup's one barrier
    const int mi = min((tile % nblk) * GM + wv, a.M - 1);
    const bool live = (tile % nblk) * GM + wv < a.M;
    const int lane = tid & 63, m = mp * mi, pad = btd_rows(NT) - N;
    // Row work: lanes are radial nodes.  Up to 32 rows the two modes lie side by
    // side in the wave and are done in one pass, otherwise in two.
    constexpr bool HALF = btd_rows(NT) <= 32;
    constexpr int PASSES = HALF ? 1 : 2;
    const int n = HALF ? lane & 31 : lane, half = lane >> 5;
    auto mode_of = [&](int p) { return HALF ? half : p; };
    const bool two = kabs > 0 && mi > 0;     // the -k mode is solved on its own
    const bool zero = kabs == 0 && mi == 0;  // mode (0,0)
    const size_t S = (size_t)a.M * nk * N;
    const int nr = n < N ? n : N - 1;  // lanes past the last row read a valid row
    const int s0r = t.s0[nr] + pad;
    const double rinvr = t.rinv[nr];
    const double kap0 = a.alpha * kabs;
    auto kap_of = [&](int p) { return mode_of(p) ? -kap0 : kap0; };
    dcplx* const X = reinterpret_cast<dcplx*>(solve_smem) + wv * 8 * XS;  // line 3 s + c, then 6 + s
    auto line = [&](int p, int c) { return X + (3 * mode_of(p) + c) * XS; };
    auto pline = [&](int p) { return X + (6 + mode_of(p)) * XS; };
    auto mode_row = [&](int s) {  // row 0 of mode s in one field
        return (unsigned)((mi * nk + (K - 1 + (s ? -kabs : kabs))) * N);
    };
    // matrix layout: row ti of a tile, block blk, column j = (mode, real or imaginary part)
    const int ti = lane >> 4, blk = (lane >> 2) & 3, mode = (lane >> 1) & 1, part = lane & 1;
    const int te = 4 * ti + (lane & 3);  // this lane's element of a stored tile

    // ---- requests, in the order the phases need them: the coupling tiles
    //      (shared by the workgroup, 16 bytes per thread and load), the stencil
    //      weights, then u^n and the nonlinear terms of this lane's rows
    constexpr int CN = btd_coupling(NT) / 2, CQ = (CN + 63) / 64;
    double* const coup = reinterpret_cast<double*>(solve_smem) + GM * 16 * XS;
    dpair cl[CQ];
#pragma unroll
    for (int q = 0; q < CQ; ++q) cl[q] = reinterpret_cast<const dpair*>(t.coup)[min(tid + q * 64 * GM, CN - 1)];
    Row9 Lo, Le;  // weights of d2/dr2 + (1/r) d/dr, parity of m +- 1 and of m
    Lo.load(t.wl, N, (m + 1) & 1, nr);
    Le.load(t.wl, N, m & 1, nr);
    const double* src = a.kind == OPF_SOLVE_RAW ? static_cast<const double*>(a.n0) : a.u0;
    // the terms a kind does not use (N^p for PRED, both for RAW) read one
    // fixed location instead: one cache line for the whole wave
    const bool use0 = a.kind != OPF_SOLVE_RAW, use1 = a.kind == OPF_SOLVE_CORR;
    const void* nl0 = use0 ? a.n0 : static_cast<const void*>(t.rinv);
    const void* nl1 = use1 ? a.n1 : static_cast<const void*>(t.rinv);
    const unsigned mask0 = use0 ? ~0u : 0u, mask1 = use1 ? ~0u : 0u;
    vec2<double> ul[PASSES][3];              // u^n (RAW: R)
    vec2<TNL> x0[PASSES][3], x1[PASSES][3];  // N^n and N^p as stored
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        if (p == 1) {
            // The second mode is requested once the first has arrived: the
            // launch's load burst is served roughly in the order the requests
            // reach the memory system, so every wave then has its first mode by
            // the middle of the burst and works on it while the rest arrives
            // (FP64 corrector 25.4 us against 25.6 with both at once, mixed
            // 23.6 against 24.6, at 64 x 48 x 127 modes).
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
        }
        const unsigned row = mode_row(mode_of(p)) + nr;
#pragma unroll
        for (int c = 0; c < 3; ++c) ul[p][c] = load_v<double>(src, (row + c * (unsigned)S) * 16u);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const unsigned off = (row + c * (unsigned)S) * (unsigned)(2 * sizeof(TNL));
            x0[p][c] = load_v<TNL>(nl0, off & mask0);
            x1[p][c] = load_v<TNL>(nl1, off & mask1);
        }
    }
    double Dp[NT + 4], Dh[NT + 4];  // inverse diagonal blocks: the pressure's; u+, u-, u_z in matrix blocks 0, 1, 2
    Row9 W1o, W1e;                  // first-derivative weights of this lane's row, parity of m +- 1 and of m
    double hv[NHOM];                // homogeneous solutions at this row
    const int e16 = lane & 15;
    double wwall;                   // the wall row's weights (nine lanes of 16)
    dcplx Ai;                       // element [i][j] of mode s's A^-1 in lane 32 s + 4 i + j
    auto request_pressure = [&] {
        const double* ip = t.img + ((size_t)a.MU * K + (size_t)kabs * a.M + mi) * IMG + unsigned(2 * te);
#pragma unroll
        for (int q = 0; q < NT + 4; q += 2) load_pair(ip + 16 * q, Dp[q], Dp[q + 1]);
    };
    auto request_helmholtz = [&] {
        const unsigned mu = blk == 0 ? m + 1 : (blk == 1 ? abs(m - 1) : m);
        const double* ip = t.img + (size_t)kabs * a.MU * IMG + (mu * IMG + 2 * te);
#pragma unroll
        for (int q = 0; q < NT + 4; q += 2) load_pair(ip + 16 * q, Dh[q], Dh[q + 1]);
    };
    auto request_influence = [&] {
        const double* h = t.hom + ((size_t)mi * K + kabs) * NHOM * N + unsigned(nr);
#pragma unroll
        for (int j = 0; j < NHOM; ++j) hv[j] = j < NHOM - 1 || a.p_out ? h[j * N] : 0.0;
        wwall = e16 < W9 ? t.d1[(((m + 1) & 1) * N + N - 1) * W9 + e16] : 0.0;
        Ai = load_c<double>(t.ainv, ((size_t)mi * nk + (K - 1 + (half ? -kabs : kabs))) * 16 + e16);
    };
#pragma unroll
    for (int q = 0; q < CQ; ++q)
        if (tid + q * 64 * GM < CN) reinterpret_cast<dpair*>(coup)[tid + q * 64 * GM] = cl[q];
    // the only workgroup barrier: from here on the waves share nothing.  It
    // publishes LDS only (a full barrier would wait for the loads in flight).
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (!live) return;
#pragma unroll
    for (int l = 0; l < 8; ++l)
        if (lane < pad) X[l * XS + lane] = dcplx{0.0, 0.0};

    // ---- R = [1/dt + (1-c) L / Re] u^n + N (+ forcing) in the (+,-,z) form
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        dcplx *l0 = line(p, 0), *l1 = line(p, 1), *l2 = line(p, 2), *lp = pline(p);
        dcplx na[3];  // PRED: N^n; CORR: (1-c) N^n + c N^p
        if (a.kind == OPF_SOLVE_CORR) {
            const double cc = a.c, c1 = 1.0 - a.c;
#pragma unroll
            for (int c = 0; c < 3; ++c) na[c] = c1 * to_c(x0[p][c]) + cc * to_c(x1[p][c]);
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) na[c] = to_c(x0[p][c]);
        }
        if (p == PASSES - 1) {  // requested once the other loads' registers are free
            __builtin_amdgcn_sched_barrier(0);
            request_pressure();
            __builtin_amdgcn_sched_barrier(0);
        }
        const dcplx ur = to_c(ul[p][0]), ut = to_c(ul[p][1]), uz = to_c(ul[p][2]);
        if (n < N) {
            l0[pad + n] = ur;
            l1[pad + n] = ut;
            l2[pad + n] = uz;
        }
        __builtin_amdgcn_wave_barrier();
        dcplx rr[3];
        if (a.kind == OPF_SOLVE_RAW) {
            rr[0] = ur + ix(ut);
            rr[1] = ur - ix(ut);
            rr[2] = uz;
        } else {
            const double kap2 = kap0 * kap0;
            const dcplx dr = Lo.apply(l0, s0r), dt = Lo.apply(l1, s0r), dz = Le.apply(l2, s0r);
            const dcplx up = ur + ix(ut), um = ur - ix(ut);
            const double r2 = rinvr * rinvr;
            const dcplx Lp = (dr + ix(dt)) - (double(m + 1) * double(m + 1) * r2 + kap2) * up;
            const dcplx Lm = (dr - ix(dt)) - (double(m - 1) * double(m - 1) * r2 + kap2) * um;
            const dcplx Lz = dz - (double(m) * double(m) * r2 + kap2) * uz;
            rr[0] = a.inv_dt * up + a.aexp * Lp + (na[0] + ix(na[1]));
            rr[1] = a.inv_dt * um + a.aexp * Lm + (na[0] - ix(na[1]));
            rr[2] = a.inv_dt * uz + a.aexp * Lz + na[2];
            if (zero) rr[2].x += a.force;
        }
        __builtin_amdgcn_wave_barrier();  // every lane has read the u^n lines
        if (n < N) {
            l0[pad + n] = rr[0];
            l1[pad + n] = rr[1];
            l2[pad + n] = rr[2];
            lp[pad + n] = 0.5 * (rr[0] + rr[1]);  // R_r, for the divergence
        }
        __builtin_amdgcn_wave_barrier();
    }

    // ---- pressure-Poisson right-hand side div R (P(1) = 0):
    //      div R = d/dr R_r + [(1+m) R+ + (1-m) R-] / (2r) + i kappa R_z, R_r = (R+ + R-)/2
    {
        W1o.load(t.d1, N, (m + 1) & 1, nr);
        dcplx d[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            d[p] = W1o.apply(pline(p), s0r) +
                   (0.5 * rinvr) * (double(1 + m) * line(p, 0)[pad + nr] + double(1 - m) * line(p, 1)[pad + nr]) +
                   kap_of(p) * ix(line(p, 2)[pad + nr]);
        __builtin_amdgcn_wave_barrier();  // every lane has read the R_r lines
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (n < N) pline(p)[pad + n] = n < N - 1 ? d[p] : dcplx{0.0, 0.0};
    }
    __builtin_amdgcn_wave_barrier();
    request_helmholtz();
    __builtin_amdgcn_sched_barrier(0);
    // every matrix block solves the pressure (same results, same addresses)
    btd_solve<NT>(Dp, coup + te, coup + 16 * (2 * NT + 1 + 4 * (m & 1)) + te, &(X + (6 + mode) * XS + ti)->x + part);
    __builtin_amdgcn_wave_barrier();

    // ---- R -= grad P, scaled by -Re/c; (0,0): u_r = 0, real R_theta and R_z
    W1e.load(t.d1, N, m & 1, nr);
    dcplx P[PASSES];
    {
        const double hs = a.hscale;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            dcplx r0 = line(p, 0)[pad + nr], r1 = line(p, 1)[pad + nr], r2 = line(p, 2)[pad + nr];
            P[p] = pline(p)[pad + nr];
            if (zero) {
                const dcplx d = r0 - r1;  // 2 i R_theta
                r0 = dcplx{0.5 * d.y, 0.0};
                r1 = dcplx{0.0, 0.0};
                r2 = dcplx{r2.x, 0.0};
            } else {
                const dcplx dP = W1e.apply(pline(p), s0r);
                const dcplx mP = (double(m) * rinvr) * P[p];
                r0 = r0 - (dP - mP);
                r1 = r1 - (dP + mP);
                r2 = r2 - kap_of(p) * ix(P[p]);
            }
            r0 = hs * r0;
            r1 = hs * r1;
            r2 = hs * r2;
            if (n == N - 1) {
                r0 = r1 = r2 = dcplx{0.0, 0.0};
                if (zero && a.wall) {  // (0,0): Dirichlet values u_theta(1), u_z(1)
                    const size_t w0 = (size_t)(K - 1) * 2, ws = (size_t)a.M * nk * 2;
                    r0 = dcplx{a.wall[ws + w0], 0.0};
                    r2 = dcplx{a.wall[2 * ws + w0], 0.0};
                }
            }
            // (0,0) solves u_theta with H_1 in the + line and u_z with H_0
            if (n < N) {
                line(p, 0)[pad + n] = r0;
                line(p, 1)[pad + n] = r1;
                line(p, 2)[pad + n] = r2;
            }
        }
    }
    request_influence();  // used after the solve
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_wave_barrier();
    btd_solve<NT>(Dh, coup + te, coup + 16 * (2 * NT + 1 + 4 * ((blk < 2 ? m + 1 : m) & 1)) + te,
                  &(X + (3 * mode + min(blk, 2)) * XS + ti)->x + part);
    __builtin_amdgcn_wave_barrier();

    // ---- influence matrix a = -A^{-1} g(u_b), lanes 32 s + 4 i + j for mode s;
    //      fixed flux on (0,0)
    double gamma = 0.0;
    dcplx* const AV = X + 6 * XS;  // a of mode s at 4 s (the pressure lines are free)
    if (zero) {  // flux of u_z,b over the radial quadrature
        double qs = lane < N ? t.quad[lane] * X[2 * XS + pad + lane].x : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) qs += __shfl_xor(qs, o, 64);
        gamma = a.fixed_flux ? (0.25 - qs) * t.qG_inv : 0.0;
        if (lane == 0 && a.beta_out) *a.beta_out = gamma * a.Re * 0.25;
    } else {
        const dcplx* li = X + 3 * half * XS + pad + N - 1;  // the wall row of this half's mode
        const int e = min(e16, W9 - 1) - (W9 - 1);
        const dcplx sr = li[e] + li[XS + e];                // u+ + u- at the wall's stencil
        const dcplx dw = {row_sum(wwall * sr.x), row_sum(wwall * sr.y)};
        dcplx g0 = li[0], g1 = li[XS], g2 = li[2 * XS];
        dcplx g3 = 0.5 * (dw + double(1 + m) * g0 + double(1 - m) * g1) + (half ? -kap0 : kap0) * ix(g2);  // r = 1
        if (a.wall) {  // drive g to the wall velocity (b_r +- i b_theta, b_z, 0) instead of 0
            const size_t wi = ((size_t)mi * nk + (K - 1 + (half ? -kabs : kabs))) * 2, ws = (size_t)a.M * nk * 2;
            const dcplx br = {a.wall[wi], a.wall[wi + 1]}, bt = {a.wall[ws + wi], a.wall[ws + wi + 1]};
            g0 = g0 - (br + ix(bt));
            g1 = g1 - (br - ix(bt));
            g2 = g2 - dcplx{a.wall[2 * ws + wi], a.wall[2 * ws + wi + 1]};
        }
        const int j = lane & 3;
        const dcplx pr = cm(Ai, j == 0 ? g0 : (j == 1 ? g1 : (j == 2 ? g2 : g3)));
        const dcplx ai = {-quad_sum(pr.x), -quad_sum(pr.y)};
        AV[4 * half + ((lane >> 2) & 3)] = ai;  // eight lanes hold and write the same value
    }
    __builtin_amdgcn_wave_barrier();
    // the weights again, for the vorticity (each use loads its own: held any
    // longer they cost registers, which measured 3% slower)
    W1o.load(t.d1, N, (m + 1) & 1, nr);
    W1e.load(t.d1, N, m & 1, nr);
    const bool mirror = mi == 0 && kabs > 0;  // m = 0: -k is the conjugate of +k
    const size_t offc = mode_row(1) + n;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        if (n >= N || (mode_of(p) && !two)) continue;
        const size_t off = mode_row(mode_of(p)) + n;
        dcplx up = line(p, 0)[pad + n], um = line(p, 1)[pad + n], uz = line(p, 2)[pad + n];
        dcplx a1 = {0.0, 0.0};
        if (zero) {
            const double ut = up.x;
            uz = dcplx{uz.x + gamma * t.green[n], 0.0};
            up = dcplx{0.0, ut};
            um = dcplx{0.0, -ut};
        } else {
            const double h1p = hv[0], h1m = hv[1], qv = hv[2], h2 = hv[3], h3 = hv[4], h4 = hv[5];
            const dcplx* av = AV + 4 * mode_of(p);
            a1 = av[0];
            const dcplx a2 = av[1], a3 = av[2], a4 = av[3];
            up = up + h1p * a1 + h2 * a2;
            um = um + h1m * a1 + h3 * a3;
            uz = uz - (kap_of(p) * qv) * ix(a1) + h4 * a4;  // h1: u_z = -i kappa q
        }
        if (a.p_out) {
            const dcplx pp = zero ? dcplx{0.0, 0.0} : P[p] + hv[6] * a1;
            store_c<double>(a.p_out, off, pp);
            if (mirror) store_c<double>(a.p_out, offc, dcplx{pp.x, -pp.y});
        }
        // ---- output u (r, theta, z); omega from the stored components
        const dcplx ur = 0.5 * (up + um), ut = 0.5 * dcplx{(up - um).y, -(up - um).x};
        dcplx uo[3] = {ur, ut, uz};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            settle(uo[c]);
            const dcplx uc = {uo[c].x, -uo[c].y};
            if (a.u_out) {
                store_c<double>(a.u_out, c * S + off, uo[c]);
                if (mirror) store_c<double>(a.u_out, c * S + offc, uc);
            }
            if (a.u_out32) {
                store_c<float>(a.u_out32, c * S + off, uo[c]);
                if (mirror) store_c<float>(a.u_out32, c * S + offc, uc);
            }
            // omega is computed from (u_r, u_theta, u_z) as stored, so it
            // equals what the standalone vorticity kernel gives for the same state
            line(p, c)[pad + n] = uo[c];
        }
    }
    __builtin_amdgcn_wave_barrier();
    if (a.w_out && n < N) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (mode_of(p) && !two) continue;
            const size_t off = mode_row(mode_of(p)) + n;
            dcplx wo[3];
            curl_row(W1e.apply(line(p, 2), s0r), W1o.apply(line(p, 1), s0r), rinvr, m, kap_of(p), line(p, 0)[pad + n],
                     line(p, 1)[pad + n], line(p, 2)[pad + n], wo[0], wo[1], wo[2]);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                store_c<TNL>(a.w_out, c * S + off, wo[c]);
                if (mirror) store_c<TNL>(a.w_out, c * S + offc, dcplx{wo[c].x, -wo[c].y});
            }
        }
    }
}

// Three waves per SIMD: at most 168 VGPRs.  The two largest forms do not quite
// fit: NT = 12 (49 <= N <= 56) spills 2 registers, 12 bytes of scratch a lane, and
// NT = 14 (N >= 57) 5, 24 bytes: 4.7 MB written and read again at 64 x 48 x 127
// modes.
template <typename TNL, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_solve(SolveArgs a) {
    k_solve_body<TNL, NT>(a);
}
template <typename TNL, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_solve_b(const SolveArgs* __restrict__ aa) {
    // the member's record is read in place (a private copy would live in scratch)
    k_solve_body<TNL, NT>(aa[blockIdx.y]);
}

// Standalone vorticity of an external-layout state.  With a.mirror set
// (states, which are real fields) the m = 0, k < 0 modes are written as the
// conjugates of k > 0, as the solve kernel does; otherwise every mode is
// computed on its own.
__global__ __launch_bounds__(64) void k_vorticity(AuxArgs a) {
    __shared__ dcplx sL[3][LSTR];
    const int N = a.N, K = a.K, nk = a.nk;
    const int mi = blockIdx.x / nk, kk = blockIdx.x % nk;
    if (a.mirror && mi == 0 && kk < K - 1) return;
    const int m = a.mp * mi, n = threadIdx.x;
    const size_t S = (size_t)a.M * nk * N;
    const size_t off = ((size_t)mi * nk + kk) * N + n;
    if (n < N) {
        sL[0][n] = load_c<double>(a.u, off);
        sL[1][n] = load_c<double>(a.u, S + off);
        sL[2][n] = load_c<double>(a.u, 2 * S + off);
    }
    __syncthreads();
    if (n < N) {
        const int s0 = a.t.s0[n];
        Row9 de, dod;
        de.load(a.t.d1, N, m & 1, n);
        dod.load(a.t.d1, N, (m + 1) & 1, n);
        dcplx wo[3];
        curl_row(de.apply(sL[2], s0), dod.apply(sL[1], s0), a.t.rinv[n], m, a.alpha * (kk - (K - 1)), sL[0][n],
                 sL[1][n], sL[2][n], wo[0], wo[1], wo[2]);
        const bool mirror = a.mirror && mi == 0 && kk > K - 1;
        const size_t offc = ((size_t)mi * nk + (2 * (K - 1) - kk)) * N + n;
        for (int c = 0; c < 3; ++c) {
            store_c<double>(a.w, c * S + off, wo[c]);
            if (mirror) store_c<double>(a.w, c * S + offc, dcplx{wo[c].x, -wo[c].y});
        }
    }
}

// Diagnostics of the state.  Per mode q = (m, k): partial[4q] = max |g| of
// (u+(1), u-(1), u_z(1), div u(1)), then max over the interior nodes of
// |div u|, and the quadrature sums of |u|^2 and |omega|^2 over the three
// components.  One wave per mode, lanes are radial nodes: u is read once and
// omega stays in registers.  (Vorticity, energies by one workgroup per m and
// divergence apart took 4.5 + 8.8 + 4.0 us at 48 x 32 x 63 modes and a launch
// each; this one 5.9.)
__global__ __launch_bounds__(64) void k_diag(AuxArgs a) {
    __shared__ dcplx sL[3][LSTR];
    const int N = a.N, K = a.K, nk = a.nk;
    const int q = blockIdx.x, mi = q / nk, kk = q % nk;
    const int m = a.mp * mi, n = threadIdx.x, nr = min(n, N - 1);
    const double kap = a.alpha * (kk - (K - 1)), rinv = a.t.rinv[nr];
    const size_t S = (size_t)a.M * nk * N, off = (size_t)q * N + nr;
    const dcplx ur = load_c<double>(a.u, off), ut = load_c<double>(a.u, S + off), uz = load_c<double>(a.u, 2 * S + off);
    Row9 de, dod;  // d/dr, parity of m and of m +- 1
    de.load(a.t.d1, N, m & 1, nr);
    dod.load(a.t.d1, N, (m + 1) & 1, nr);
    sL[0][n] = ur;
    sL[1][n] = ut;
    sL[2][n] = uz;
    __syncthreads();
    const int s0 = a.t.s0[nr];
    const dcplx dr = dod.apply(sL[0], s0), dt = dod.apply(sL[1], s0), dz = de.apply(sL[2], s0);
    dcplx w[3];
    curl_row(dz, dt, rinv, m, kap, ur, ut, uz, w[0], w[1], w[2]);
    double gv = 0.0, dv = 0.0, eu = 0.0, ew = 0.0;
    if (n < N) {
        const double wq = a.t.quad[n];
        eu = wq * ((ur.x * ur.x + ur.y * ur.y) + (ut.x * ut.x + ut.y * ut.y) + (uz.x * uz.x + uz.y * uz.y));
        ew = wq * ((w[0].x * w[0].x + w[0].y * w[0].y) + (w[1].x * w[1].x + w[1].y * w[1].y) +
                   (w[2].x * w[2].x + w[2].y * w[2].y));
        // div u from u+- = u_r +- i u_theta, as the influence matrix drives it
        const dcplx up = ur + ix(ut), um = ur - ix(ut);
        const dcplx ap = (dr + ix(dt)) + (double(1 + m) * rinv) * up;
        const dcplx am = (dr - ix(dt)) + (double(1 - m) * rinv) * um;
        const dcplx d = 0.5 * (ap + am) + kap * ix(uz);
        const double ad = sqrt(d.x * d.x + d.y * d.y);
        if (n == N - 1) {
            dcplx bp = {0.0, 0.0}, bm = {0.0, 0.0}, bz = {0.0, 0.0};
            if (a.wall) {  // residual against the wall velocity
                const size_t wi = (size_t)q * 2, ws = (size_t)a.M * nk * 2;
                const dcplx br = {a.wall[wi], a.wall[wi + 1]}, bt = {a.wall[ws + wi], a.wall[ws + wi + 1]};
                bp = br + ix(bt);
                bm = br - ix(bt);
                bz = dcplx{a.wall[2 * ws + wi], a.wall[2 * ws + wi + 1]};
            }
            const dcplx ep = up - bp, em = um - bm, ez = uz - bz;
            const double a1 = sqrt(ep.x * ep.x + ep.y * ep.y), a2 = sqrt(em.x * em.x + em.y * em.y);
            const double a3 = sqrt(ez.x * ez.x + ez.y * ez.y);
            gv = fmax(fmax(a1, a2), fmax(a3, ad));
        } else {
            dv = ad;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        gv = fmax(gv, __shfl_xor(gv, o, 64));
        dv = fmax(dv, __shfl_xor(dv, o, 64));
        eu += __shfl_xor(eu, o, 64);
        ew += __shfl_xor(ew, o, 64);
    }
    if (n == 0) {
        double* p = a.partial + 4 * (size_t)q;
        p[0] = gv;
        p[1] = dv;
        p[2] = eu;
        p[3] = ew;
    }
}

// What the host needs of the diagnostics, packed for one copy (five copies to
// host memory cost 25..30 us each): out[2m], out[2m + 1] = the sums of k_diag
// over k, then the (0,0) profile of u_z (2 N), the maxima of |g|, |div u| and of
// the ncp CFL parts, and beta.  One workgroup.
__global__ __launch_bounds__(1024) void k_diag_pack(AuxArgs a, const double* __restrict__ cpart, int ncp,
                                                    const double* __restrict__ beta, double* __restrict__ out) {
    __shared__ double red[16][3];
    const int M = a.M, N = a.N, nk = a.nk, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    double g = 0.0, d = 0.0, c = 0.0;
    for (int mi = wv; mi < M; mi += 16) {
        double eu = 0.0, ew = 0.0;
        for (int k = lane; k < nk; k += 64) {
            const double* p = a.partial + 4 * ((size_t)mi * nk + k);
            g = fmax(g, p[0]);
            d = fmax(d, p[1]);
            eu += p[2];
            ew += p[3];
        }
        for (int o = 32; o > 0; o >>= 1) {
            eu += __shfl_xor(eu, o, 64);
            ew += __shfl_xor(ew, o, 64);
        }
        if (lane == 0) {
            out[2 * mi] = eu;
            out[2 * mi + 1] = ew;
        }
    }
    for (int i = t; i < ncp; i += 1024) c = fmax(c, cpart[i]);
    const double* uz = a.u + 2 * (2 * (size_t)M * nk * N + (size_t)(a.K - 1) * N);
    for (int i = t; i < 2 * N; i += 1024) out[2 * M + i] = uz[i];
    for (int o = 32; o > 0; o >>= 1) {
        g = fmax(g, __shfl_xor(g, o, 64));
        d = fmax(d, __shfl_xor(d, o, 64));
        c = fmax(c, __shfl_xor(c, o, 64));
    }
    if (lane == 0) {
        red[wv][0] = g;
        red[wv][1] = d;
        red[wv][2] = c;
    }
    __syncthreads();
    if (t < 3) {
        double v = 0.0;
        for (int i = 0; i < 16; ++i) v = fmax(v, red[i][t]);
        out[2 * M + 2 * N + t] = v;
    }
    if (t == 3) out[2 * M + 2 * N + 3] = *beta;
}

// The largest gm admitted, by gm_ok.  Ensembles step within 2% with any, small
// members within 4% (us per step, gm 1 / 2 / 4; 24 members of 48 x 24 x 63 modes 709 /
// 704 / 708 at mp = 1, 715 / 704 at mp = 2, 720 / 716 at mp = 3; of 64 x 32 x 95 1851 /
// 1833 / 1839, 1819 / 1799, 1834 / 1822; 32 of 32 x 16 x 47, mixed, 249 / 257 / 260).
int default_gm(int mp) { return mp == 1 ? 4 : (mp <= 3 ? 2 : 1); }

// A grid of at most one wave per compute unit is spread over all of them (24 x
// 8 x 15 modes: 5.8 us against 6.2 with four waves to a workgroup, 41 x 18 x 23:
// 8.1 against 8.4); beyond that neighbouring m gain more from sharing an L1
// (48 x 32 x 63 modes, 1024 waves: 10.6 us against 11.5).
int context_gm(int mp, int M, int K) { return M * K <= 256 ? 1 : default_gm(mp); }

// The admitted gm are part of the interface: tile caches are checked by them.
// The kernel itself takes any up to its 256 threads; the span of wavenumbers that
// the m of a workgroup use is kept to GM_SPAN.
bool gm_ok(int gm, int mp) { return gm >= 1 && gm <= 4 && mp * (gm - 1) + 3 <= GM_SPAN; }

template <int NT>
static void launch_solve_nt(const SolveArgs& a, const SolveArgs* batch, int members, int precision, hipStream_t s,
                            const KernelTiming& kt) {
    const dim3 grid(a.K * ((a.M + a.gm - 1) / a.gm), batch ? members : 1), block(64 * a.gm);
    const uint32_t lds = (uint32_t)solve_lds(NT, a.gm);
    if (precision == OPF_MIXED) {
        if (batch) hipLaunchKernelGGL((k_solve_b<float, NT>), grid, block, lds, s, batch);
        else launch_timed((k_solve<float, NT>), grid, block, lds, s, kt, a);
    } else {
        if (batch) hipLaunchKernelGGL((k_solve_b<double, NT>), grid, block, lds, s, batch);
        else launch_timed((k_solve<double, NT>), grid, block, lds, s, kt, a);
    }
}

static hipError_t launch_solve_any(const SolveArgs& a, const SolveArgs* batch, int members, int precision,
                                   hipStream_t s, const KernelTiming& kt) {
    switch (btd_nt(a.N)) {  // the members of a batch share N
#define OPF_CASE(V) case V: launch_solve_nt<V>(a, batch, members, precision, s, kt); break;
        OPF_CASE(2) OPF_CASE(4) OPF_CASE(6) OPF_CASE(8) OPF_CASE(10) OPF_CASE(12) OPF_CASE(14)
#undef OPF_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_solve_batch(const SolveArgs& a, const SolveArgs* batch, int members, int precision,
                              hipStream_t s) {
    return launch_solve_any(a, batch, members, precision, s, KernelTiming{});
}

hipError_t launch_solve(const SolveArgs& a, int precision, hipStream_t s, const KernelTiming& kt) {
    return launch_solve_any(a, nullptr, 1, precision, s, kt);
}

hipError_t launch_vorticity(const AuxArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_vorticity, dim3(a.M * a.nk), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_diag(const AuxArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_diag, dim3(a.M * a.nk), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_diag_pack(const AuxArgs& a, const double* cpart, int ncp, const double* beta, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_diag_pack, dim3(1), dim3(1024), 0, s, a, cpart, ncp, beta, out);
    return hipGetLastError();
}

}  // namespace opf
