// Operator tables built on the device: banded LU factors of every radial
// operator (Section 2: the implicit viscous terms and the pressure-Poisson
// equation are solved by banded LU per Fourier mode), the homogeneous
// solutions and inverse influence matrices of the influence-matrix
// correction, and the flux Green's function.  They are built when a context
// is created and again whenever the step size changes (the Helmholtz
// operators H = 1/dt - (c/Re) L depend on dt).
#include <cmath>

#include "opf_internal.h"
#include "opf_pair.h"

namespace opf {
namespace {

constexpr int BW = 13;  // band entries per row: offsets -8..+4 from the diagonal

__device__ inline double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// The radial operators, by number: q < MU K is H_{mu,|k|} with mu = q / K,
// |k| = q % K; q >= MU K is the pressure operator L_{m,|k|}, m = mp (q - MU K)
// / K, with P(1) = 0.  The pressure's (0,0) record is not used.
struct System {
    bool helm;
    int mu, ka;
    size_t image;  // its place among the images: [|k|][mu] (Helmholtz), then [|k|][m] (pressure)
    __device__ System(const FactorArgs& a, int q) {
        helm = q < a.MU * a.K;
        const int i = helm ? q : q - a.MU * a.K, row = i / a.K;
        ka = i - row * a.K;
        mu = helm ? row : a.mp * row;
        image = helm ? (size_t)ka * a.MU + row : (size_t)a.MU * a.K + (size_t)ka * a.M + row;
    }
    __device__ bool unused() const { return !helm && mu == 0 && ka == 0; }
};

// LDS of the block elimination of four systems.  A wave holds 4 x 4 blocks of
// four systems, entry [r][c] of system s in lane 16 s + 4 r + c, or an 8 x 8
// block of one, entry [r][c] in lane 8 r + c; two of those at a time.
struct BlockLds {
    dd d[128], inv[64];
    union {
        double x[128];
        dd gc[64];
    };
};

template <int q>
__device__ inline double quad_broadcast(double v) {  // lane q of each four
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, 0x55 * q, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), 0x55 * q, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Step q of Gauss-Jordan elimination in place: m becomes the inverse after all.
template <int n, int q, int T>
__device__ inline void eliminate(double (&m)[T], int (&bad)[T], int base, int r, int c) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const double row = __shfl(m[t], base + n * q + c);
        double f, piv;  // column q of this row, the pivot
        if constexpr (n == 4) f = quad_broadcast<q>(m[t]), piv = quad_broadcast<q>(row);
        else f = __shfl(m[t], base + n * r + q), piv = __shfl(m[t], base + (n + 1) * q);
        if (!(fabs(piv) > 0.0) || isinf(piv)) bad[t] = 2;
        double ip = __builtin_amdgcn_rcp(piv);  // two Newton steps: to a unit in the last place
        ip = fma(fma(-piv, ip, 1.0), ip, ip);
        ip = fma(fma(-piv, ip, 1.0), ip, ip);
        const double rm = c == q ? ip : row * ip;
        m[t] = r == q ? rm : fma(-f, rm, c == q ? 0.0 : m[t]);
    }
    if constexpr (q + 1 < n) eliminate<n, q + 1, T>(m, bad, base, r, c);
}

// Inverses of n x n matrices, D[t] this lane's entries: Gauss-Jordan elimination
// in double precision (the pivots are those of the operator's LU factors, which
// are checked), then one Newton step X + X (I - D X) with the residual in
// pairs.  T matrices per lane, whose chains run side by side.  Called by all 64
// lanes of one wave; bad is set in the lanes of a matrix with a pivot that is
// zero or not finite.
template <int n, int T>
__device__ inline void small_inverse(BlockLds& w, int lane, const dd (&D)[T], dd (&out)[T], int (&bad)[T]) {
    const int l = lane & (n * n - 1), base = lane - l, r = l / n, c = l % n;
    double m[T];
#pragma unroll
    for (int t = 0; t < T; ++t) m[t] = D[t].hi;
    eliminate<n, 0, T>(m, bad, base, r, c);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        w.d[64 * t + lane] = D[t];
        w.x[64 * t + lane] = m[t];
    }
    __builtin_amdgcn_wave_barrier();
    double e[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        dd s = {r == c ? 1.0 : 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < n; ++k) s = madd(s, w.d[64 * t + base + n * r + k], -w.x[64 * t + base + n * k + c]);
        e[t] = s.hi + s.lo;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < T; ++t) w.d[64 * t + lane].hi = e[t];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < T; ++t) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) s += w.x[64 * t + base + n * r + k] * w.d[64 * t + base + n * k + c].hi;
        out[t] = two_sum(m[t], s);
    }
    __builtin_amdgcn_wave_barrier();
}

// The images of systems q0..q0+3 (those past the last one repeat it): the
// block elimination described at btd_nt, of L - shift with the couplings of
// the table wl, as the solve uses them, and the identity's wall row.  It runs
// on pairs of doubles, so that the inverse blocks are right to a unit in the
// last place (0.8e-15 of a block's largest entry with the diagonal entries' own
// rounding; 5e-15 in plain double): their errors act on every step in the same
// way.  100 diffusion steps of u_theta(0,0) at N = 64 stay within 0.8e-14 of the
// same steps in extended precision (banded LU factors: 3.5e-14).
//
// Bound by the latency of one tile after the other, so four systems share a
// wave, 16 lanes each, and their last blocks, 64 entries each, run in pairs side
// by side.  The next tile's entries are requested a tile ahead.  The factor
// kernel takes 53 us for the 3136 Helmholtz operators of 64 x 48 x 127 modes (115
// with a wave to each system, of which 4 x 4 blocks use a quarter) and 29 us for
// the 1600 of 48 x 24 x 63 (46).  Called by all 64 lanes of one wave.
__device__ void block_images(const FactorArgs& a, int q0, int nsys, BlockLds& w, int lane) {
    const int N = a.N, nt = a.nt, pad = btd_rows(nt) - N;
    // Entry of L at a padded row and column, but for the diagonal terms; padding
    // rows and the wall row are the identity's.  No select follows the loads, so
    // that they need no branch and no early wait.
    const int none = 2 * N * W9;  // 0, then 1
    auto at = [&](const System& S, int row, int col) {
        const int n = row - pad, off = col - pad - stencil_column(n, N);
        const bool in = n >= 0 && n < N - 1 && off >= 0 && off < W9;
        return a.wl[in ? ((S.mu & 1) * N + n) * W9 + off : none + (row == col && (n < 0 || n >= N - 1))];
    };
    auto rinv_at = [&](int row) { return a.rinv[min(max(row - pad, 0), N - 1)]; };
    // v = at(row, col) of a diagonal block, with - mu^2 / r^2 - |k|^2 - shift
    auto diagonal = [&](const System& S, int row, int col, double v, double ri) {
        const double on = row == col && row >= pad && row < pad + N - 1 ? 1.0 : 0.0, kap = a.alpha * S.ka;
        return two_sum(v - on * (double(S.mu) * S.mu * ri * ri + kap * kap), S.helm ? -on * a.shift : 0.0);
    };
    auto at_image = [](int tile, int i, int k) { return 32 * (tile >> 1) + 2 * (4 * k + i) + (tile & 1); };
    int bad = 0;
    {
        const int g = lane & 48, r = (lane >> 2) & 3, c = lane & 3;
        const System S(a, min(q0 + (lane >> 4), nsys - 1));
        double* G = a.img + S.image * btd_image(nt);
        double v0, ri, b[4], u[4];  // the tile's entry and 1 / r, row r of B and column c of the C before it
        auto request = [&](int I) {
            v0 = at(S, 4 * I + r, 4 * I + c);
            ri = rinv_at(4 * I + r);
            const int J = max(I, 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                b[k] = at(S, 4 * J + r, 4 * J - 4 + k);
                u[k] = at(S, 4 * J - 4 + k, 4 * J + c);
            }
        };
        request(0);
        for (int I = 0; I < nt; ++I) {
            dd d = diagonal(S, 4 * I + r, 4 * I + c, v0, ri), s = {0.0, 0.0};  // s: D_{I-1}^{-1} C_{I-1}
            if (I > 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) s = madd(s, w.inv[g + 4 * r + k], u[k]);
                w.gc[lane] = s;
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k = 0; k < 4; ++k) d = madd(d, w.gc[g + 4 * k + c], -b[k]);
                __builtin_amdgcn_wave_barrier();
            }
            request(min(I + 1, nt - 1));
            const dd D[1] = {two_sum(d.hi, d.lo)};
            dd v[1];
            int wrong[1] = {bad};
            small_inverse<4, 1>(w, lane, D, v, wrong);
            bad = wrong[0];
            w.inv[lane] = v[0];
            __builtin_amdgcn_wave_barrier();
            G[at_image(I, r, c)] = S.unused() ? 0.0 : v[0].hi;
        }
    }
    const int r = lane >> 3, c = lane & 7, r0 = 4 * nt;
#pragma unroll 1
    for (int h = 0; h < 4; h += 2) {
        dd D[2], v[2];
        int wrong[2];
        if (r < 4 && c < 4)  // C reaches the first four columns of the last block only
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const System S(a, min(q0 + h + t, nsys - 1));
                dd s = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 4; ++k) s = madd(s, w.inv[16 * (h + t) + 4 * r + k], at(S, r0 - 4 + k, r0 + c));
                w.gc[16 * t + 4 * r + c] = s;
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const System S(a, min(q0 + h + t, nsys - 1));
            dd d = diagonal(S, r0 + r, r0 + c, at(S, r0 + r, r0 + c), rinv_at(r0 + r));
            if (c < 4)
#pragma unroll
                for (int k = 0; k < 4; ++k) d = madd(d, w.gc[16 * t + 4 * k + c], -at(S, r0 + r, r0 - 4 + k));
            D[t] = two_sum(d.hi, d.lo);
            wrong[t] = __shfl(bad, 16 * (h + t));
        }
        __builtin_amdgcn_wave_barrier();
        small_inverse<8, 2>(w, lane, D, v, wrong);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = min(q0 + h + t, nsys - 1);
            const System S(a, q);
            double* G = a.img + S.image * btd_image(nt);
            G[at_image(nt + 2 * (r >> 2) + (c >> 2), r & 3, c & 3)] = S.unused() ? 0.0 : v[t].hi;
            if (lane == 0) a.image_flags[q] = S.unused() ? 0 : wrong[t];
        }
    }
}

// The first (nsys + 3) / 4 workgroups make the images, four systems each
// (image_flags[q] 2: a pivot that is zero or not finite); the others the LU factors,
// one system each, which eliminate the band (rows in LDS) without pivoting,
// one column per pass (8 rows x 4 columns of updates in parallel), and write it
// as column records: main record i holds L[i+1..i+4][i], U[i-1..i-4][i] and
// 1/U_ii, tail record i holds L[i+5..i+8][i] (the unused record gets 1/U = 1).
// flags[q]: 0 ok, 1 entry outside the band, 2 pivot below 1e-14 max|A|, 3
// element growth (|U| > 1e3 max|A| or |L| > 1e3).
__global__ __launch_bounds__(64) void k_factor(FactorArgs a, int nsys) {
    __shared__ union {
        double B[NMAX * BW];
        BlockLds blk;
    } sm;
    const int nimg = (nsys + 3) / 4;
    const int N = a.N, n = threadIdx.x;
    if ((int)blockIdx.x < nimg) {
        block_images(a, 4 * blockIdx.x, nsys, sm.blk, n);
        return;
    }
    double* const B = sm.B;
    const int q = blockIdx.x - nimg;
    const System S(a, q);
    const bool helm = S.helm;
    const int mu = S.mu, ka = S.ka;
    double* F = a.fac + (size_t)q * N * FACW;
    if (S.unused()) {
        if (n < N) {
            for (int d = 0; d < FMAIN; ++d) F[(size_t)n * FMAIN + d] = d == 8 ? 1.0 : 0.0;
            for (int d = 0; d < FTAIL; ++d) F[(size_t)N * FMAIN + (size_t)n * FTAIL + d] = 0.0;
        }
        if (n == 0) a.flags[q] = 0;
        return;
    }
    const double kap = a.alpha * ka;
    const int par = mu & 1;
    int bad = 0;
    double amax = 0.0;
    if (n < N) {
        for (int d = 0; d < BW; ++d) B[n * BW + d] = 0.0;
        if (n == N - 1) {
            B[n * BW + 8] = 1.0;  // wall row: the boundary value
            amax = 1.0;
        } else {
            const int s = a.s0[n];
            const double ri = a.rinv[n];
            for (int j = 0; j < W9; ++j) {
                const int col = s + j;
                double v = a.d2[(par * N + n) * W9 + j] + ri * a.d1[(par * N + n) * W9 + j];
                if (col == n) v -= double(mu) * mu * ri * ri + kap * kap;
                if (helm) {
                    v = -a.cr * v;
                    if (col == n) v += a.inv_dt;
                }
                const int off = col - n;
                if (off < -8 || off > 4) {
                    if (v != 0.0) bad = 1;
                } else {
                    B[n * BW + off + 8] = v;
                }
                amax = fmax(amax, fabs(v));
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    amax = wave_max(amax);
    // elimination: lane t updates row j+1+t/4, column j+1+t%4
    const int ti = 1 + (n & 31) / 4, tc = 1 + (n & 3);
    for (int j = 0; j < N; ++j) {
        const double piv = B[j * BW + 8];
        if (!(fabs(piv) > 1e-14 * amax)) bad = bad ? bad : 2;
        const int i = j + ti, col = j + tc;
        if (n < 32 && i < N) {
            const double l = B[i * BW + (j - i + 8)] / piv;
            if (col < N && col - i >= -8) B[i * BW + (col - i + 8)] -= l * B[j * BW + (col - j + 8)];
            __builtin_amdgcn_wave_barrier();  // every lane has read its multiplier's entry
            if (tc == 1) B[i * BW + (j - i + 8)] = l;
        }
        __builtin_amdgcn_wave_barrier();
    }
    double umax = 0.0, lmax = 0.0;
    if (n < N)
        for (int d = 0; d < BW; ++d) {
            const double v = fabs(B[n * BW + d]);
            if (d >= 8) umax = fmax(umax, v);
            else lmax = fmax(lmax, v);
        }
    umax = wave_max(umax);
    lmax = wave_max(lmax);
    if (n < N) {
        double* f = F + (size_t)n * FMAIN;
        double* tl = F + (size_t)N * FMAIN + (size_t)n * FTAIL;
        for (int d = 0; d < 8; ++d) {
            const double l = n + 1 + d < N ? B[(n + 1 + d) * BW + (7 - d)] : 0.0;
            if (d < 4) f[d] = l;
            else tl[d - 4] = l;
        }
        for (int d = 0; d < 4; ++d) f[4 + d] = n - 1 - d >= 0 ? B[(n - 1 - d) * BW + (9 + d)] : 0.0;
        f[8] = 1.0 / B[n * BW + 8];
        f[9] = 0.0;
    }
    // the band check is per row: any lane's flag marks the system
    for (int o = 32; o > 0; o >>= 1) bad = max(bad, __shfl_xor(bad, o));
    if (bad == 0 && (umax > 1e3 * amax || lmax > 1e3)) bad = 3;
    if (n == 0) a.flags[q] = bad;
}

// Forward and backward substitution with column records, on a vector held
// in LDS column `lane` of v[n * 64 + lane].
__device__ void rec_solve(const double* __restrict__ F, int N, double* v, int lane) {
    for (int i = 0; i < N; ++i) {
        const double* f = F + (size_t)i * FMAIN;
        const double* tl = F + (size_t)N * FMAIN + (size_t)i * FTAIL;
        const double x = v[i * 64 + lane];
        for (int d = 0; d < 8; ++d)
            if (i + 1 + d < N) v[(i + 1 + d) * 64 + lane] -= (d < 4 ? f[d] : tl[d - 4]) * x;
    }
    for (int i = N - 1; i >= 0; --i) {
        const double* f = F + (size_t)i * FMAIN;
        const double x = v[i * 64 + lane] * f[8];
        v[i * 64 + lane] = x;
        for (int d = 0; d < 4; ++d)
            if (i - 1 - d >= 0) v[(i - 1 - d) * 64 + lane] -= f[4 + d] * x;
    }
}

__device__ inline const double* hfac(const FactorArgs& a, int mu, int ka) {
    return a.fac + ((size_t)abs(mu) * a.K + ka) * a.N * FACW;
}

// P1 = L_{m,|k|}^{-1} e_{N-1} (unit wall pressure) into slot 6 of the
// influence data; the (0,0) pair gets zeros in every slot.  One thread per
// (m, |k|) pair.
__global__ __launch_bounds__(64) void k_hom_pressure(FactorArgs a) {
    __shared__ double v[NMAX * 64];
    const int lane = threadIdx.x, pr = blockIdx.x * 64 + lane;
    const int N = a.N;
    if (pr >= a.M * a.K) return;
    const int mi = pr / a.K, ka = pr % a.K;
    double* h = a.hom + (size_t)pr * NHOM * N;
    if (mi == 0 && ka == 0) {
        for (int s = 0; s < NHOM * N; ++s) h[s] = 0.0;
        return;
    }
    for (int i = 0; i < N; ++i) v[i * 64 + lane] = i == N - 1 ? 1.0 : 0.0;
    rec_solve(a.fac + ((size_t)a.MU * a.K + pr) * N * FACW, N, v, lane);
    for (int i = 0; i < N; ++i) h[6 * N + i] = v[i * 64 + lane];
}

// Flux Green's function H_{0,0} u_G = 1 inside, u_G(1) = 0, and
// qg = int_0^1 u_G r dr (lane 0).
__device__ void green(const FactorArgs& a, double* v, int lane) {
    if (lane != 0) return;
    const int N = a.N;
    for (int i = 0; i < N; ++i) v[i * 64] = i == N - 1 ? 0.0 : 1.0;
    rec_solve(hfac(a, 0, 0), N, v, 0);
    double s = 0.0;
    for (int i = 0; i < N; ++i) {
        a.green[i] = v[i * 64];
        s += a.quad[i] * v[i * 64];
    }
    *a.qg = s;
}

// The six Helmholtz solves of the homogeneous solutions of pair (m, |k|):
// slot 0 h1+ = H_{m+1}^{-1}(-(P1' - m P1/r)), slot 1 h1- = H_{m-1}^{-1}(-(P1'
// + m P1/r)), slot 2 q = H_m^{-1} P1 (wall values 0), and slots 3..5 the unit
// wall values through H_{m+1}, H_{m-1}, H_m.  One thread per (pair, slot); the
// first workgroup solves for the flux Green's function meanwhile (a launch of
// its own took 23 us at 24 rows and 47 at 64, a seventh of a rebuild).
__global__ __launch_bounds__(64) void k_hom_helmholtz(FactorArgs a) {
    __shared__ double v[NMAX * 64];
    const int lane = threadIdx.x, id = (blockIdx.x - 1) * 64 + lane;
    const int N = a.N;
    if (blockIdx.x == 0) {
        green(a, v, lane);
        return;
    }
    if (id >= a.M * a.K * 6) return;
    const int pr = id / 6, slot = id % 6;
    const int mi = pr / a.K, ka = pr % a.K;
    if (mi == 0 && ka == 0) return;
    const int m = a.mp * mi;
    double* h = a.hom + (size_t)pr * NHOM * N;
    const double* P1 = h + 6 * N;
    for (int i = 0; i < N; ++i) {
        double r = 0.0;
        if (i == N - 1) {
            r = slot >= 3 ? 1.0 : 0.0;
        } else if (slot < 2) {
            double dP = 0.0;
            for (int j = 0; j < W9; ++j) dP += a.d1[((m & 1) * N + i) * W9 + j] * P1[a.s0[i] + j];
            const double t = m * P1[i] * a.rinv[i];
            r = slot == 0 ? -(dP - t) : -(dP + t);
        } else if (slot == 2) {
            r = P1[i];
        }
        v[i * 64 + lane] = r;
    }
    const int mu = (slot == 0 || slot == 3) ? m + 1 : (slot == 1 || slot == 4) ? m - 1 : m;
    rec_solve(hfac(a, mu, ka), N, v, lane);
    for (int i = 0; i < N; ++i) h[slot * N + i] = v[i * 64 + lane];
}

struct c2 {
    double x, y;
};
__device__ inline c2 cmul(c2 p, c2 q) { return {p.x * q.x - p.y * q.y, p.x * q.y + p.y * q.x}; }
__device__ inline c2 csub(c2 p, c2 q) { return {p.x - q.x, p.y - q.y}; }
__device__ inline double cabs2(c2 p) { return sqrt(p.x * p.x + p.y * p.y); }
__device__ inline c2 cdiv(c2 p, c2 q) {
    const double d = q.x * q.x + q.y * q.y;
    return {(p.x * q.x + p.y * q.y) / d, (p.y * q.x - p.x * q.y) / d};
}

// Inverse influence matrix of mode (m, k): A_ij = g_i(h_j) with
// g(v) = (v+(1), v-(1), v_z(1), div v(1)) and h_1 = (h1+, h1-, -i kappa q),
// h_2..h_4 the unit wall solutions, inverted by Gauss-Jordan elimination
// with partial pivoting.  One thread per (m, signed k); (0,0) gets zeros,
// and a singular matrix sets flags[mode].
__global__ __launch_bounds__(64) void k_influence(FactorArgs a) {
    int* flags = a.flags + a.MU * a.K + a.M * a.K;
    const int id = blockIdx.x * 64 + threadIdx.x;
    const int N = a.N, K = a.K, nk = 2 * K - 1;
    if (id >= a.M * nk) return;
    const int mi = id / nk, k = id % nk - (K - 1), ka = abs(k);
    double* dst = a.ainv + (size_t)id * 32;
    flags[id] = 0;
    if (mi == 0 && ka == 0) {
        for (int s = 0; s < 32; ++s) dst[s] = 0.0;
        return;
    }
    const int m = a.mp * mi, e = N - 1, po = (m + 1) & 1;
    const double kap = a.alpha * k, re = a.rinv[e];
    const double* h = a.hom + ((size_t)mi * K + ka) * NHOM * N;
    auto d1row = [&](const double* v) {
        double acc = 0.0;
        for (int j = 0; j < W9; ++j) acc += a.d1[(po * N + e) * W9 + j] * v[a.s0[e] + j];
        return acc;
    };
    const double* h1p = h;
    const double* h1m = h + N;
    const double* q = h + 2 * N;
    const double* h2 = h + 3 * N;
    const double* h3 = h + 4 * N;
    const double* h4 = h + 5 * N;
    const double dp1 = 0.5 * (d1row(h1p) + (1 + m) * h1p[e] * re) + 0.5 * (d1row(h1m) + (1 - m) * h1m[e] * re);
    c2 A[4][8];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 8; ++j) A[i][j] = {j - 4 == i ? 1.0 : 0.0, 0.0};
    A[0][0] = {h1p[e], 0.0};
    A[1][0] = {h1m[e], 0.0};
    A[2][0] = {0.0, -kap * q[e]};               // -i kappa q
    A[3][0] = {dp1 + kap * kap * q[e], 0.0};    // div h1: + i kappa (-i kappa q)
    A[0][1] = {h2[e], 0.0};
    A[3][1] = {0.5 * (d1row(h2) + (1 + m) * h2[e] * re), 0.0};
    A[1][2] = {h3[e], 0.0};
    A[3][2] = {0.5 * (d1row(h3) + (1 - m) * h3[e] * re), 0.0};
    A[2][3] = {h4[e], 0.0};
    A[3][3] = {0.0, kap * h4[e]};               // i kappa h4
    for (int c = 0; c < 4; ++c) {
        int piv = c;
        for (int i = c + 1; i < 4; ++i)
            if (cabs2(A[i][c]) > cabs2(A[piv][c])) piv = i;
        if (cabs2(A[piv][c]) == 0.0) {
            flags[id] = 1;
            for (int s = 0; s < 32; ++s) dst[s] = 0.0;
            return;
        }
        for (int j = 0; j < 8; ++j) {
            const c2 t = A[c][j];
            A[c][j] = A[piv][j];
            A[piv][j] = t;
        }
        const c2 d = A[c][c];
        for (int j = 0; j < 8; ++j) A[c][j] = cdiv(A[c][j], d);
        for (int i = 0; i < 4; ++i)
            if (i != c) {
                const c2 f = A[i][c];
                for (int j = 0; j < 8; ++j) A[i][j] = csub(A[i][j], cmul(f, A[c][j]));
            }
    }
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
            dst[2 * (4 * i + j)] = A[i][4 + j].x;
            dst[2 * (4 * i + j) + 1] = A[i][4 + j].y;
        }
}

}  // namespace

hipError_t launch_operator_tables(const FactorArgs& a, bool pressure, hipStream_t s) {
    const int nh = a.MU * a.K, np = a.M * a.K, nsys = pressure ? nh + np : nh;
    hipLaunchKernelGGL(k_factor, dim3((nsys + 3) / 4 + nsys), dim3(64), 0, s, a, nsys);
    hipError_t he = hipGetLastError();
    if (he != hipSuccess) return he;
    if (pressure) {
        hipLaunchKernelGGL(k_hom_pressure, dim3((np + 63) / 64), dim3(64), 0, s, a);
        if ((he = hipGetLastError()) != hipSuccess) return he;
    }
    hipLaunchKernelGGL(k_hom_helmholtz, dim3((np * 6 + 63) / 64 + 1), dim3(64), 0, s, a);
    if ((he = hipGetLastError()) != hipSuccess) return he;
    const int modes = a.M * (2 * a.K - 1);
    hipLaunchKernelGGL(k_influence, dim3((modes + 63) / 64), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace opf
