// Learned preconditioner of the Newton-Krylov solver: a residual MLP whose
// dense layers run on the matrix cores (bfloat16 operands, FP32
// accumulation), its backward pass and Adam; the network turns the features
// of each Fourier mode into the factors of a rank-R correction of -I, which
// k_lowrank_apply applies to the mode's radial profile, and k_head is the
// loss of that map on recorded (z, J z) pairs.
//
// Network (weights [out][in] row-major, L residual layers of width H):
//   h_0 = W_in x + b_in;  h_l = h_{l-1} + relu(W_l h_{l-1} + b_l);  y = W_out h_L + b_out.
// Every GEMM here computes C[i][j] = sum_k A[i][k] B[j][k] with both operands
// stored k-contiguous, so that each lane of a wave loads 8 consecutive
// bfloat16 values of A and of B straight into the operand registers of
// v_mfma_f32_32x32x16_bf16: the forward pass takes B = W, the input gradient
// takes B = W^T (a transposed bfloat16 copy kept beside each weight), and the
// weight gradient takes A = dZ^T, B = H^T (transposed activations written by
// the chains that take a tile of rows through the residual layers).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "opf_internal.h"

using namespace opf;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // storage of one bfloat16 value

constexpr int NCOND = 32;  // conditioning features per row
constexpr int GT = 32;     // rows and columns of C per GEMM workgroup
constexpr int MAXL = 8;    // residual layers
constexpr int MAXSEG = 2 * MAXL + 4;

// float -> bfloat16, round to nearest, ties to even (finite inputs)
__host__ __device__ inline bf16_t f2bf(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// Where the GEMM epilogue puts v = acc (+ bias[col]): out[row][col].
struct Epi {
    const float* bias;  // may be null
    float* out;
    int ldo;
};

__device__ __forceinline__ void epilogue(const Epi& e, int row, int col, float s) {
    e.out[(size_t)row * e.ldo + col] = s + (e.bias ? e.bias[col] : 0.0f);
}

// C[rows][cols] = A[rows][K] B[cols][K]^T on v_mfma_f32_32x32x16_bf16.
// One workgroup per 32x32 tile of C; its four waves split the workgroup's
// K range [k_begin, k_end) (wave w takes the 16-wide slices w, w+4, ...) and
// their partial tiles are summed in LDS in a fixed order.  Lane l of a wave
// supplies row l%32 of the A slice and row l%32 of the B slice, elements
// 8*(l/32)..+7 (the operand layout of the instruction); accumulator entry i
// of lane l is C[8(i/4) + 4(l/32) + i%4][l%32].  The next slice's operands
// are loaded before the current product is issued.  Without a split
// (part == null) the tile goes through the epilogue; with a split over
// gridDim.z ranges of kc, workgroup z writes its raw partial tile to
// part[z][rows][cols] for k_gemm_reduce.
// Requires rows, cols multiples of 32, K and kc of 16, lda, ldb multiples of 8.
template <typename Store>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B, int ldb,
                                          int m0, int n0, int kb, int ke, Store store) {
    __shared__ float red[4][16][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rr = lane & 31, kq = (lane >> 5) * 8;
    f32x16 acc = {};
    const bf16_t* ap = A + (size_t)(m0 + rr) * lda + kq;
    const bf16_t* bp = B + (size_t)(n0 + rr) * ldb + kq;
    int k0 = kb + wv * 16;
    u32x4 an = {}, bn = {};
    if (k0 < ke) {
        an = *reinterpret_cast<const u32x4*>(ap + k0);
        bn = *reinterpret_cast<const u32x4*>(bp + k0);
    }
    for (; k0 < ke; k0 += 64) {
        const u32x4 ac = an, bc = bn;
        if (k0 + 64 < ke) {
            an = *reinterpret_cast<const u32x4*>(ap + k0 + 64);
            bn = *reinterpret_cast<const u32x4*>(bp + k0 + 64);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ac), __builtin_bit_cast(bf16x8, bc),
                                                      acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) red[wv][i][lane] = acc[i];
    __syncthreads();
    for (int q = threadIdx.x; q < 1024; q += 256) {
        const int i = q >> 6, l = q & 63;
        const float s = ((red[0][i][l] + red[1][i][l]) + red[2][i][l]) + red[3][i][l];
        store(m0 + 8 * (i >> 2) + 4 * (l >> 5) + (i & 3), n0 + (l & 31), s);
    }
}
__global__ __launch_bounds__(256) void k_gemm(const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ B,
                                              int ldb, int K, int kc, Epi e, float* __restrict__ part) {
    const int kb = blockIdx.z * kc, cols = gridDim.x * GT, rows = gridDim.y * GT;
    gemm_tile(A, lda, B, ldb, blockIdx.y * GT, blockIdx.x * GT, kb, min(K, kb + kc), [&](int row, int col, float s) {
        if (part)
            part[((size_t)blockIdx.z * rows + row) * cols + col] = s;
        else
            epilogue(e, row, col, s);
    });
}

// The same product for large shapes: one 128 x 128 tile of C per workgroup,
// each wave a 64 x 64 quarter (2 x 2 instruction tiles of 32 x 32, 64
// accumulators per lane).  K advances 32 at a time through double-buffered
// LDS tiles of A and B (rows padded to 40 bf16, 80 bytes, so the 16-byte
// operand reads of 16 consecutive lanes hit distinct banks); the next
// slice's global loads are issued before the current slice's products.
// Every wave takes its 64 x 64 quarter through all of K, so a C entry is the
// same K-ordered sum for every launch shape; with a split (part != null)
// workgroup z writes its raw partial tile for k_gemm_reduce.
// Requires rows, cols multiples of 128, K and kc of 32, lda, ldb of 8.
constexpr int G2 = 128, GK2 = 32, GLS2 = 40;
__global__ __launch_bounds__(256) void k_gemm128(const bf16_t* __restrict__ A, int lda,
                                                 const bf16_t* __restrict__ B, int ldb, int K, int kc, Epi e,
                                                 float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) bf16_t sa[2][G2 * GLS2];
    __shared__ __attribute__((aligned(16))) bf16_t sb[2][G2 * GLS2];
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m0 = blockIdx.y * G2, n0 = blockIdx.x * G2;
    const int kb = blockIdx.z * kc, ke = min(K, kb + kc);
    const int lr = t >> 2, lk = 8 * (t & 3);  // loader: rows lr and lr + 64, k lk..lk+7
    const bf16_t* ag = A + (size_t)(m0 + lr) * lda + lk;
    const bf16_t* bg = B + (size_t)(n0 + lr) * ldb + lk;
    const size_t a64 = (size_t)64 * lda, b64 = (size_t)64 * ldb;
    u32x4 ra0, ra1, rb0, rb1;
    ra0 = *reinterpret_cast<const u32x4*>(ag + kb);
    ra1 = *reinterpret_cast<const u32x4*>(ag + a64 + kb);
    rb0 = *reinterpret_cast<const u32x4*>(bg + kb);
    rb1 = *reinterpret_cast<const u32x4*>(bg + b64 + kb);
    *reinterpret_cast<u32x4*>(&sa[0][lr * GLS2 + lk]) = ra0;
    *reinterpret_cast<u32x4*>(&sa[0][(lr + 64) * GLS2 + lk]) = ra1;
    *reinterpret_cast<u32x4*>(&sb[0][lr * GLS2 + lk]) = rb0;
    *reinterpret_cast<u32x4*>(&sb[0][(lr + 64) * GLS2 + lk]) = rb1;
    __syncthreads();
    const int wm = (wv >> 1) * 64, wn = (wv & 1) * 64;
    const int rr = lane & 31, kq = (lane >> 5) * 8;
    f32x16 acc[2][2] = {};
    int buf = 0;
    for (int k0 = kb; k0 < ke; k0 += GK2) {
        const bool more = k0 + GK2 < ke;
        if (more) {
            ra0 = *reinterpret_cast<const u32x4*>(ag + k0 + GK2);
            ra1 = *reinterpret_cast<const u32x4*>(ag + a64 + k0 + GK2);
            rb0 = *reinterpret_cast<const u32x4*>(bg + k0 + GK2);
            rb1 = *reinterpret_cast<const u32x4*>(bg + b64 + k0 + GK2);
        }
#pragma unroll
        for (int ks = 0; ks < GK2; ks += 16) {
            bf16x8 av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                av[i] = *reinterpret_cast<const bf16x8*>(&sa[buf][(wm + 32 * i + rr) * GLS2 + ks + kq]);
                bv[i] = *reinterpret_cast<const bf16x8*>(&sb[buf][(wn + 32 * i + rr) * GLS2 + ks + kq]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        if (more) {
            *reinterpret_cast<u32x4*>(&sa[buf ^ 1][lr * GLS2 + lk]) = ra0;
            *reinterpret_cast<u32x4*>(&sa[buf ^ 1][(lr + 64) * GLS2 + lk]) = ra1;
            *reinterpret_cast<u32x4*>(&sb[buf ^ 1][lr * GLS2 + lk]) = rb0;
            *reinterpret_cast<u32x4*>(&sb[buf ^ 1][(lr + 64) * GLS2 + lk]) = rb1;
        }
        __syncthreads();
        buf ^= 1;
    }
    const int cols = gridDim.x * G2, rows = gridDim.y * G2;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                const int col = n0 + wn + 32 * j + rr;
                if (part)
                    part[((size_t)blockIdx.z * rows + row) * cols + col] = acc[i][j][v];
                else
                    epilogue(e, row, col, acc[i][j][v]);
            }
}

// Products k_gemm128 takes.
inline bool large_product(int rows, int cols, int K) {
    return rows % G2 == 0 && cols % G2 == 0 && K % GK2 == 0 && (double)rows * cols * K >= (double)(1L << 30);
}

// Sum of the split partial tiles in order, then the epilogue.
__global__ void k_gemm_reduce(const float* __restrict__ part, int rows, int cols, int nsplit, Epi e) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)rows * cols) return;
    float s = 0.0f;
    for (int z = 0; z < nsplit; ++z) s += part[(size_t)z * rows * cols + i];
    epilogue(e, (int)(i / cols), (int)(i % cols), s);
}

// FP32 rows [nrows][d] -> bfloat16 rows [rp][d] and transposed [d][ldt];
// rows nrows..rp-1 become zero.
__global__ void k_rows_bf16(const float* __restrict__ x, int nrows, int rp, int d, bf16_t* xb, bf16_t* xt,
                            int ldt) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)rp * d) return;
    const int row = (int)(i / d), col = (int)(i % d);
    const bf16_t b = f2bf(row < nrows ? x[i] : 0.0f);
    if (xb) xb[i] = b;
    if (xt) xt[(size_t)col * ldt + row] = b;
}

__device__ inline float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ inline double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// sum of om[0..n) (or n when om is null) into *out; one workgroup.
__global__ __launch_bounds__(256) void k_weight_sum(const float* __restrict__ om, int n, float* out) {
    __shared__ float part[4];
    float s = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) s += om ? om[i] : 1.0f;
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *out = ((part[0] + part[1]) + part[2]) + part[3];
}

// Weighted squared error, rows < nrows: loss_r = om_r sum_j (y - t)^2,
// dY = 2 om_r (y - t) / W with W = sum_r om_r (om null: om_r = 1).  dY
// replaces Y in place; bfloat16 copies go to dyb [rp][d] and dyt [d][ldt].
// Rows nrows..rp-1 get dY = 0.  One wave per row.
__global__ __launch_bounds__(256) void k_loss(float* __restrict__ y, const float* __restrict__ t,
                                              const float* __restrict__ om, const float* __restrict__ wsum,
                                              int nrows, int rp, int d, bf16_t* dyb, bf16_t* dyt, int ldt,
                                              float* __restrict__ lrow) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rp) return;
    const bool live = row < nrows;
    const float w = live ? (om ? om[row] : 1.0f) : 0.0f;
    const float g = 2.0f * w / *wsum;
    float acc = 0.0f;
    for (int j = lane; j < d; j += 64) {
        const size_t i = (size_t)row * d + j;
        const float r = live ? y[i] - t[i] : 0.0f;
        acc += r * r;
        const float dy = g * r;
        y[i] = dy;
        const bf16_t b = f2bf(dy);
        dyb[i] = b;
        dyt[(size_t)j * ldt + row] = b;
    }
    acc = wave_sum(acc);
    if (lane == 0) lrow[row] = w * acc;
}

constexpr int CS_CHUNKS = 64;  // largest number of row chunks of a column sum
constexpr int GSPLIT = 8;                     // largest K split of a GEMM
constexpr size_t GPART = (size_t)1 << 23;     // floats of split partial tiles (split x rows x cols)

// Parameter segments: weight matrices [rows][cols] and bias vectors.
struct Segs {
    int n;
    long off[MAXSEG + 1];
    int rows[MAXSEG], cols[MAXSEG], mat[MAXSEG];  // mat: 0 bias, 1 weights, 2 weights of a residual layer
    int blk[MAXSEG + 1];                          // first workgroup of the segment (k_adam, k_refresh)
};

// bfloat16 weights of a residual layer [n][k], k < H, as the operand requests
// of a chain read them: 32 x 16 tiles of 1 KB, entry (n, k) of a tile with
// lane n + 32 (k / 8), element k % 8, so that a wave's request of 16 bytes a
// lane is 1 KB in a row (row-major weights give 32 pieces of 32 bytes; the
// chains took 25.7 and 31.8 us then, 1536 rows x 256 x 4 layers).
__host__ __device__ inline long frag_at(int n, int k, int H) {
    return ((long)(n / 32) * (H / 16) + k / 16) * 512 + (n % 32 + 32 * (k % 16 / 8)) * 8 + k % 8;
}

// One workgroup of k_adam and k_refresh: 64 x 32 parameters of a weight
// matrix, or 2048 of a bias.  A matrix tile's bfloat16 copies wb ([rows][cols]
// at the parameter offset) and wt ([cols][rows], through LDS) are written in
// runs of 64 and 128 bytes, both in frag_at's order for a residual layer.
// step(j, i) returns the new values of parameters i..i+3 of segment j.
constexpr int PT = 64;  // rows of a tile
template <typename Step>
__device__ __forceinline__ void param_tile(const Segs& s, bf16_t* __restrict__ wb, bf16_t* __restrict__ wt, Step step) {
    __shared__ bf16_t tile[32][PT + 4];
    int j = 0;
    while (j + 1 < s.n && (int)blockIdx.x >= s.blk[j + 1]) ++j;
    const int b = blockIdx.x - s.blk[j], t = threadIdx.x;
    const long off = s.off[j];
    if (!s.mat[j]) {
        for (int i = b * 2048 + 4 * t; i < min(s.cols[j], (b + 1) * 2048); i += 1024) step(j, off + i);
        return;
    }
    const int rows = s.rows[j], cols = s.cols[j];
    const int r0 = b / (cols / 32) * PT, c0 = b % (cols / 32) * 32;
    const int c = 4 * (t & 7);
#pragma unroll
    for (int h = 0; h < PT; h += 32) {
        const int r = r0 + h + (t >> 3);
        if (r >= rows) break;  // rows is a multiple of 32
        const long i = off + (long)r * cols + c0 + c;
        const f32x4 p = step(j, i);
        bf16_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) tile[c + q][h + (t >> 3)] = v[q] = f2bf(p[q]);
        uint2 u;
        u.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
        u.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
        *reinterpret_cast<uint2*>(wb + (s.mat[j] == 2 ? off + frag_at(r, c0 + c, cols) : i)) = u;
    }
    __syncthreads();
    const int rq = 4 * (t & 15);
    if (r0 + rq >= rows) return;
#pragma unroll
    for (int q = t >> 4; q < 32; q += 16) {
        const uint2 u = *reinterpret_cast<const uint2*>(&tile[q][rq]);
        const long at = s.mat[j] == 2 ? frag_at(c0 + q, r0 + rq, rows) : (long)(c0 + q) * rows + r0 + rq;
        *reinterpret_cast<uint2*>(wt + off + at) = u;
    }
}

__global__ __launch_bounds__(256) void k_refresh(const float* __restrict__ p, Segs s, bf16_t* wb, bf16_t* wt) {
    param_tile(s, wb, wt, [&](int, long i) { return *reinterpret_cast<const f32x4*>(p + i); });
}

// The residual layers, forward and backward, run as chains: a workgroup keeps
// 32 rows and takes them through all layers, so a layer costs one barrier
// instead of a launch (1536 rows x 256 x 4 layers, the mode rows of a
// 48 x 24 x 32 grid: a launch per layer and direction took 7.2..9.5 us, the
// chains 16.4 and 24.2 us for all layers).  The FP32 residual stays in the
// registers of the lane that owns the entry, the bfloat16 operand goes
// through a double-buffered LDS tile (rows padded by 16 bytes, so that the
// 16-byte operand reads of 16 consecutive lanes hit distinct banks), and the
// weights, which do not depend on the rows, are requested one tile ahead
// straight into operand registers.  Each wave owns a 32 x 32 tile: its
// four accumulators take the 16-wide K slices s = 0..3 mod 4 and are added in
// that order, which is the sum of k_gemm's four waves.  Few rows leave most
// of the chip idle; what bounds a chain there is the latency of a layer.
// WIDE (H > 256): up to 16 waves of 128 registers, which hold one accumulator
// and 8 slices.  FULL: every slice of every chunk exists.
template <bool WIDE>
constexpr int chain_waves() { return WIDE ? 16 : 8; }  // at most: a 32 x 32 tile each

__device__ __forceinline__ void lds_barrier() {  // orders LDS only: requests and stores stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Where a lane's 16 entries of a tile lie, and the operand requests.
template <bool WIDE, bool FULL>
struct Chain {
    static constexpr int SC = WIDE ? 8 : 16, KC = 16 * SC, NC = WIDE ? 4 : 1;  // K chunks of a tile
    static constexpr int NA = WIDE ? 1 : 4;                                    // accumulators
    int lane, rr, kq, wv, H, HS;
    uint32_t off;
    u32x4 b[SC];  // one chunk of the weights, requested ahead
    __device__ __forceinline__ Chain(int H_)
        : lane(threadIdx.x & 63), rr(lane & 31), kq((lane >> 5) * 8),
          wv(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), H(H_), HS(H_ + 8), off(4 * (lane >> 5) * H_ + wv * 32 + rr) {}
    __device__ __forceinline__ int col() const { return wv * 32 + rr; }
    // entry i of the tile lies in row row0(i) + 4 (lane / 32), column col():
    // at(x, i)[off] for x the first of the workgroup's rows (one offset per
    // lane from a pointer per i that all lanes share)
    static __device__ __forceinline__ constexpr int row0(int i) { return 8 * (i >> 2) + (i & 3); }
    template <typename T> __device__ __forceinline__ T* at(T* x, int i) const { return x + (size_t)row0(i) * H; }
    __device__ __forceinline__ void fetch(const bf16_t* __restrict__ w, int c) {
        const bf16_t* p = w + ((size_t)wv * (H / 16) + c * SC) * 512 + lane * 8;
#pragma unroll
        for (int i = 0; i < SC; ++i)
            if (FULL || c * KC + 16 * i < H) b[i] = *reinterpret_cast<const u32x4*>(p + 512 * i);
    }
    __device__ __forceinline__ void multiply(const bf16_t* hs, int c, f32x16* acc) const {
        const bf16_t* p = hs + rr * HS + kq;
#pragma unroll
        for (int i = 0; i < SC; ++i)
            if (FULL || c * KC + 16 * i < H)
                acc[i % NA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    *reinterpret_cast<const bf16x8*>(p + c * KC + 16 * i), __builtin_bit_cast(bf16x8, b[i]), acc[i % NA], 0, 0, 0);
    }
    __device__ __forceinline__ float sum(const f32x16* acc, int i) const {
        if constexpr (WIDE) return acc[0][i];
        else return ((acc[0][i] + acc[1][i]) + acc[2][i]) + acc[3][i];
    }
    // the bfloat16 entries w[16] of the tile: into the LDS tile and, transposed, to dst[col][m0 + row]
    __device__ __forceinline__ void publish(const float* w, bf16_t* hs, bf16_t* dst, int R, int m0) const {
        const int hi = 4 * (lane >> 5), cc = col();
        const uint32_t to = (uint32_t)cc * R + hi;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = f2bf(w[4 * g + i]);
                if (hs) hs[(hi + row0(4 * g + i)) * HS + cc] = h[i];
            }
            if (dst) {
                uint2 u;
                u.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
                u.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
                *reinterpret_cast<uint2*>((dst + m0 + 8 * g) + to) = u;
            }
        }
    }
};

struct ChainArgs {
    const bf16_t* X;  // [rows][NCOND]
    const bf16_t* W;  // bfloat16 weights: Wb forward, Wt backward
    const float* P;   // parameters (biases)
    long woff[MAXL + 1], boff[MAXL + 1];
    int H, L, R, rows;
    float* Z;      // [L][R][H] pre-activations (forward, training only: else null; backward: read)
    bf16_t* HT;    // [L + 1][H][R] transposed activations (training only, else null)
    bf16_t* HL;    // [R][H] activations of the last layer
    const float* src;  // backward: dL/dh_L as nsplit partial products [rows][H], stride floats apart
    size_t stride;
    int nsplit;
    float* D;    // [L + 1][R][H] dL/dh_l
    bf16_t* DT;  // [L + 1][H][R] dL/dh_l where z_{l-1} > 0 (all of it for l = 0), transposed
};

// h_0 = W_in x + b_in; z_l = W_l h_l + b_l; h_{l+1} = h_l + relu(z_l).
template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * chain_waves<WIDE>()) __attribute__((amdgpu_waves_per_eu(WIDE ? 4 : 2, WIDE ? 4 : 2)))
void k_chain_fwd(ChainArgs a) {
    extern __shared__ __attribute__((aligned(16))) bf16_t hsm16[];
    Chain<WIDE, FULL> q(a.H);
    const int H = a.H, m0 = blockIdx.x * 32, buf = 32 * q.HS;
    const size_t RH = (size_t)a.R * H;
    q.fetch(a.W + a.woff[1], 0);
    float res[16];
    {
        const bf16_t* ap = a.X + (size_t)(m0 + q.rr) * NCOND + q.kq;
        const bf16_t* bp = a.W + a.woff[0] + (size_t)q.col() * NCOND + q.kq;
        f32x16 acc[2] = {};
#pragma unroll
        for (int i = 0; i < 2; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(ap + 16 * i),
                                                             *reinterpret_cast<const bf16x8*>(bp + 16 * i), acc[i], 0, 0, 0);
        const float bias = a.P[a.boff[0] + q.col()];
#pragma unroll
        for (int i = 0; i < 16; ++i) res[i] = (acc[0][i] + acc[1][i]) + bias;
        q.publish(res, hsm16, a.HT, a.R, m0);
    }
    lds_barrier();
    for (int l = 0; l < a.L; ++l) {
        const bf16_t* in = hsm16 + (l & 1) * buf;
        bf16_t* out = hsm16 + ((l + 1) & 1) * buf;
        const float bias = a.P[a.boff[l + 1] + q.col()];
        f32x16 acc[q.NA] = {};
#pragma unroll
        for (int c = 0; c < q.NC; ++c) {
            q.multiply(in, c, acc);
            if (c + 1 < q.NC) q.fetch(a.W + a.woff[l + 1], c + 1);
            else if (l + 1 < a.L) q.fetch(a.W + a.woff[l + 2], 0);
        }
        float z[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            z[i] = q.sum(acc, i) + bias;
            res[i] += fmaxf(z[i], 0.0f);
        }
        if (a.HT) {
            float* zp = a.Z + (size_t)l * RH + (size_t)m0 * H;
#pragma unroll
            for (int i = 0; i < 16; ++i) q.at(zp, i)[q.off] = z[i];
        }
        q.publish(res, out, a.HT ? a.HT + (size_t)(l + 1) * RH : nullptr, a.R, m0);
        lds_barrier();
    }
    const bf16_t* h = hsm16 + (a.L & 1) * buf;
    for (int i = threadIdx.x; i < 4 * H; i += blockDim.x) {  // 16 bytes each
        const int r = i / (H / 8), c = (i - r * (H / 8)) * 8;
        *reinterpret_cast<u32x4*>(a.HL + (size_t)(m0 + r) * H + c) = *reinterpret_cast<const u32x4*>(h + r * q.HS + c);
    }
}

// D_L = the sum of src's partial products; dz_l = D_{l+1} where z_l > 0;
// D_l = D_{l+1} + W_l^T dz_l.
template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * chain_waves<WIDE>()) __attribute__((amdgpu_waves_per_eu(WIDE ? 4 : 2, WIDE ? 4 : 2)))
void k_chain_bwd(ChainArgs a) {
    extern __shared__ __attribute__((aligned(16))) bf16_t hsm16[];
    Chain<WIDE, FULL> q(a.H);
    const int H = a.H, L = a.L, m0 = blockIdx.x * 32, buf = 32 * q.HS;
    const size_t RH = (size_t)a.R * H, at = (size_t)m0 * H;
    q.fetch(a.W + a.woff[L], 0);
    float res[16], zm[16], w[16];
    auto mask = [&](int l) {  // request z_l
        const float* zp = a.Z + (size_t)l * RH + at;
#pragma unroll
        for (int i = 0; i < 16; ++i) zm[i] = q.at(zp, i)[q.off];
    };
    mask(L - 1);
#pragma unroll
    for (int i = 0; i < 16; ++i) res[i] = 0.0f;
#pragma unroll 2
    for (int p = 0; p < a.nsplit; ++p)
#pragma unroll
        for (int i = 0; i < 16; ++i) res[i] += q.at(a.src + (size_t)p * a.stride + at, i)[q.off];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        q.at(a.D + (size_t)L * RH + at, i)[q.off] = res[i];
        w[i] = zm[i] > 0.0f ? res[i] : 0.0f;
    }
    q.publish(w, hsm16, a.DT + (size_t)L * RH, a.R, m0);
    lds_barrier();
    for (int l = L - 1; l >= 0; --l) {
        const bf16_t* in = hsm16 + ((L - 1 - l) & 1) * buf;
        bf16_t* out = hsm16 + ((L - l) & 1) * buf;
        mask(l > 0 ? l - 1 : 0);
        f32x16 acc[q.NA] = {};
#pragma unroll
        for (int c = 0; c < q.NC; ++c) {
            q.multiply(in, c, acc);
            if (c + 1 < q.NC) q.fetch(a.W + a.woff[l + 1], c + 1);
            else if (l > 0) q.fetch(a.W + a.woff[l], 0);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            res[i] += q.sum(acc, i);
            q.at(a.D + (size_t)l * RH + at, i)[q.off] = res[i];
            w[i] = l == 0 || zm[i] > 0.0f ? res[i] : 0.0f;
        }
        q.publish(w, l > 0 ? out : nullptr, a.DT + (size_t)l * RH, a.R, m0);
        lds_barrier();
    }
}

// What is left of the gradients once the chain has run, in one launch of
// independent workgroups whose partial sums the reader adds (a launch each
// cost 4.5 us or more at 1536 rows, whatever it did; 31 in all):
//  - the first ngemm workgroups: 32 x 32 tiles of the weight gradients of the
//    input layer and of nhid residual layers, dW = DT HT^T with K = rows split
//    over nsplit ranges of kc, raw partial tiles to gpart[split][parameter];
//  - then the column sums over row chunks of ch (32 columns x 8 row groups
//    per workgroup, part[chunk][column]): columns of dL/dY, then of D_l where
//    z_{l-1} > 0 (D_0: all), l = 0..L;
//  - the last workgroup: the loss, *loss = sum_r lrow[r] / (*wsum or count).
struct GradArgs {
    const bf16_t *DT, *HT, *XT;
    const float *D, *Z, *Y;
    long woff[MAXL + 1];
    int H, L, R, dout, rows;
    int nhid, nsplit, kc, ngemm;
    int ch, nch, col0;  // columns before col0 are in part already
    float* gpart;
    long nph;  // parameters before the output layer's
    float* part;
    const float *lrow, *wsum;
    float count;
    int nlive;
    float* loss;
    // for grad_of
    float* G;
    long wout, bout;
    int osplit;          // partial products of the output layer's weight gradient in opart (0: already in G)
    const float* opart;  // [osplit][dout][H]
};

__global__ __launch_bounds__(256) void k_grad_parts(GradArgs a) {
    const int H = a.H, R = a.R, th = H / GT;
    int b = blockIdx.x;
    if (b < a.ngemm) {
        const int z = b % a.nsplit, kb = z * a.kc, ke = min(a.rows, kb + a.kc);
        b /= a.nsplit;
        const bf16_t *A = a.DT, *B = a.XT;
        long off = a.woff[0];
        int m0 = b * GT, n0 = 0, ldc = NCOND;
        if (b >= th) {  // (the input layer's th tiles come first)
            b -= th;
            const int l = b / (th * th);
            b -= l * th * th;
            m0 = b / th * GT, n0 = b % th * GT, ldc = H;
            A = a.DT + (size_t)(l + 1) * H * R;
            B = a.HT + (size_t)l * H * R;
            off = a.woff[l + 1];
        }
        float* out = a.gpart + (size_t)z * a.nph + off;
        gemm_tile(A, R, B, R, m0, n0, kb, ke, [&](int row, int col, float s) { out[(size_t)row * ldc + col] = s; });
        return;
    }
    b -= a.ngemm;
    const int ncol = a.dout + (a.L + 1) * H;
    __shared__ float red[8][32];
    const int c1 = (ncol - a.col0) / 32;
    if (b < a.nch * c1) {
        const int cb = a.col0 / 32 + b % c1, k = b / c1;
        const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
        const float *src = a.Y, *mask = nullptr;
        int col = cb * 32, ld = a.dout;
        if (col >= a.dout) {
            const int l = (col - a.dout) / H;
            col -= a.dout + l * H;
            ld = H;
            src = a.D + (size_t)l * R * H;
            if (l > 0) mask = a.Z + (size_t)(l - 1) * R * H;
        }
        const int r1 = min(a.rows, (k + 1) * a.ch);
        float s = 0.0f;
#pragma unroll 4
        for (int r = k * a.ch + g; r < r1; r += 8) {
            const size_t i = (size_t)r * ld + col + c;
            const float v = src[i];
            s += (!mask || mask[i] > 0.0f) ? v : 0.0f;
        }
        red[g][c] = s;
        __syncthreads();
        if (g == 0) {
            float t = 0.0f;
            for (int r = 0; r < 8; ++r) t += red[r][c];
            a.part[(size_t)k * ncol + cb * 32 + c] = t;
        }
        return;
    }
    float s = 0.0f;
    for (int i = threadIdx.x; i < a.nlive; i += 256) s += a.lrow[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *a.loss = (((red[0][0] + red[0][1]) + red[0][2]) + red[0][3]) / (a.wsum ? *a.wsum : a.count);
}

// Gradients of parameters i..i+3, segment j: their partial sums added in order.
__device__ __forceinline__ f32x4 grad_of(const GradArgs& a, int j, long i) {
    const int l = j >> 1, ncol = a.dout + (a.L + 1) * a.H;
    const float* p = a.G + i;  // (a product that was not split, or was added up by k_gemm_reduce)
    size_t stride = 0;
    int n = 1;
    if (j & 1) {
        p = a.part + (l > a.L ? i - a.bout : a.dout + l * a.H + (i - a.woff[l] - (long)a.H * (l ? a.H : NCOND)));
        stride = ncol;
        n = a.nch;
    } else if (l > a.L ? a.osplit > 0 : l <= a.nhid) {
        p = l > a.L ? a.opart + (i - a.wout) : a.gpart + i;
        stride = l > a.L ? (size_t)a.dout * a.H : a.nph;
        n = l > a.L ? a.osplit : a.nsplit;
    }
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
    for (int z = 0; z < n; ++z) s += *reinterpret_cast<const f32x4*>(p + z * stride);
    return s;
}

// G = the gradients, for a caller that wants them: four parameters per thread.
__global__ __launch_bounds__(256) void k_grad_sum(GradArgs a, Segs s) {
    const long i = 4 * ((long)blockIdx.x * 256 + threadIdx.x);
    if (i >= s.off[s.n]) return;
    int j = 0;
    while (j + 1 < s.n && i >= s.off[j + 1]) ++j;
    *reinterpret_cast<f32x4*>(a.G + i) = grad_of(a, j, i);
}

// Adam (Kingma & Ba 2015): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// p -= lr (m c1) / (sqrt(v c2) + eps), c1 = 1/(1-b1^t), c2 = 1/(1-b2^t).
// It adds up the gradient's partial sums itself, so G is neither written nor
// read.  Bound by the 28 bytes a parameter that it moves besides: 2.64 M
// parameters take 23 us (20 after a k_grad_sum of 11 us; 33 with one thread
// per parameter, whose 2-byte stores of wt were a row apart).
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, GradArgs g, float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                              float b2, float c1, float c2, float eps, Segs s, bf16_t* wb, bf16_t* wt) {
    param_tile(s, wb, wt, [&](int j, long i) {
        const f32x4 gi = grad_of(g, j, i);
        f32x4 mi = *reinterpret_cast<const f32x4*>(m + i), vi = *reinterpret_cast<const f32x4*>(v + i);
        f32x4 pi = *reinterpret_cast<const f32x4*>(p + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            mi[q] = b1 * mi[q] + (1.0f - b1) * gi[q];
            vi[q] = b2 * vi[q] + (1.0f - b2) * gi[q] * gi[q];
            pi[q] = pi[q] - lr * (mi[q] * c1) / (sqrtf(vi[q] * c2) + eps);
        }
        *reinterpret_cast<f32x4*>(m + i) = mi;
        *reinterpret_cast<f32x4*>(v + i) = vi;
        *reinterpret_cast<f32x4*>(p + i) = pi;
        return pi;
    });
}

}  // namespace

// ---------------------------------------------------------------------------
// The preconditioner: per-mode low-rank corrections generated by the network.
namespace {

constexpr int RMAX = 32;  // largest rank

// Conditioning features of mode (m, k): mu = mp m (azimuthal wavenumber),
// kappa = alpha k (axial wavenumber).
__device__ inline float cond_feature(int j, int mi, int k, int mp, double alpha) {
    const double mu = (double)mp * mi, ka = alpha * k;
    switch (j) {
        case 0: return 1.0f;
        case 1: return (float)(mu / 48.0);
        case 2: return (float)(ka / 40.0);
        case 3: return (float)(fabs(ka) / 40.0);
        case 4: return (float)((ka > 0) - (ka < 0));
        case 5: return (float)((mu / 48.0) * (mu / 48.0));
        case 6: return (float)((ka / 40.0) * (ka / 40.0));
        case 7: return (float)(mu * fabs(ka) / 1920.0);
        default: break;
    }
    if (j < 16) return mi == j - 8 ? 1.0f : 0.0f;
    if (j < 31) return k == j - 23 ? 1.0f : 0.0f;
    return (k > 7 || k < -7) ? 1.0f : 0.0f;
}

// One row of NCOND features per mode q = m (2K-1) + k + K-1; rows past M(2K-1)
// are zero.
__global__ void k_features(float* __restrict__ fx, int rows, int rp, int nk, int K, int mp, double alpha) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= rp * NCOND) return;
    const int q = i / NCOND, j = i % NCOND;
    fx[i] = q < rows ? cond_feature(j, q / nk, q % nk - (K - 1), mp, alpha) : 0.0f;
}

// Output row of mode q: A[e][j] at 2(e R + j) (+1 imaginary), e < 3N, j < R;
// B at the same places from offset 6 N R on.

// z_q = -v_q + A_q (B_q^H v_q) with v_q the profile of mode q (e = c N + n);
// (m = 0, k < 0) is the conjugate of (0, -k), (0, 0) keeps its real part.
// One wave per output mode; the waves of a workgroup share nothing.
__global__ __launch_bounds__(256) void k_lowrank_apply(const float* __restrict__ fac, int dout, int rank,
                                                       const double* __restrict__ v, double* __restrict__ z, int N,
                                                       int M, int nk, int K) {
    __shared__ double cs[4][2 * RMAX];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q0 = blockIdx.x * 4 + w;
    if (q0 >= M * nk) return;
    const int mi = q0 / nk, kk = q0 % nk;
    const bool mir = mi == 0 && kk < K - 1;
    const int q = mir ? 2 * (K - 1) - kk : q0;
    const long S = (long)M * nk * N;
    const int n3 = 3 * N;
    const float* A = fac + (long)q * dout;
    const float* B = A + 6 * N * rank;
    double yr[3], yi[3];
    for (int t = 0; t < 3; ++t) {
        const int e = lane + 64 * t;
        yr[t] = yi[t] = 0.0;
        if (e < n3) {
            const long idx = (e / N) * S + (long)q * N + e % N;
            yr[t] = v[2 * idx];
            yi[t] = v[2 * idx + 1];
        }
    }
    for (int j = 0; j < rank; ++j) {  // c_j = sum_e conj(B_ej) y_e
        double cr = 0.0, ci = 0.0;
        for (int t = 0; t < 3; ++t) {
            const int e = lane + 64 * t;
            if (e < n3) {
                const double br = B[2 * (e * rank + j)], bi = B[2 * (e * rank + j) + 1];
                cr += br * yr[t] + bi * yi[t];
                ci += br * yi[t] - bi * yr[t];
            }
        }
        // every lane holds the same sum and stores it: each lane reads back its own store
        cs[w][2 * j] = wave_sum(cr);
        cs[w][2 * j + 1] = wave_sum(ci);
    }
    for (int t = 0; t < 3; ++t) {
        const int e = lane + 64 * t;
        if (e >= n3) continue;
        double zr = -yr[t], zi = -yi[t];
        for (int j = 0; j < rank; ++j) {
            const double ar = A[2 * (e * rank + j)], ai = A[2 * (e * rank + j) + 1];
            const double cr = cs[w][2 * j], ci = cs[w][2 * j + 1];
            zr += ar * cr - ai * ci;
            zi += ar * ci + ai * cr;
        }
        if (mir) zi = -zi;
        if (mi == 0 && kk == K - 1) zi = 0.0;
        const long out = (e / N) * S + (long)q0 * N + e % N;
        z[2 * out] = zr;
        z[2 * out + 1] = zi;
    }
}

struct HeadArgs {
    const double* pairs;  // [npairs][2][3][M][2K-1][N] complex: (z, J z)
    long vec;             // doubles per vector
    const int* idx;       // pair indices of the batch
    int batch;
    int N, M, nk, rank, dout;
    int rows, rp;  // M(2K-1) live rows, rows padded to 32
    float* Y;      // in: network output rows; out: dLoss/dY
    bf16_t* dyb;   // [rp][dout]
    float* lrow;   // per-row loss
    float scale;   // 1 / (batch rows)
    int hb;        // pairs per pass (head_pairs)
};

constexpr int HB = 8;             // most pairs staged per pass of the loss head
constexpr int HOUT = 12;          // gradient outputs per thread and factor: 3N R <= 256 HOUT
constexpr int HEAD_LDS = 53248;   // LDS bytes of one loss-head workgroup at most (three per compute unit)

// float2 slots of the loss head's LDS for nb pairs per pass: U and V rows
// padded to R + 1 entries, the nb staged profiles xhat and that (then r),
// C and G, and 256 partial sums.
__host__ __device__ inline int head_slots(int n3, int R, int nb) {
    return 2 * n3 * (R + 1) + nb * (2 * n3 + 2 * R) + 256;
}
// Pairs per pass that fit HEAD_LDS, at least 1.  Every admissible grid
// (3N R <= 3072, 3N <= 192) needs at most 7200 slots (57.6 KB) for one pair,
// within the 64 KB a workgroup may take.
inline int head_pairs(int n3, int R) {
    int nb = HB;
    while (nb > 1 && head_slots(n3, R, nb) * 8 > HEAD_LDS) --nb;
    return nb;
}

// Loss head of the training pairs: the network's factors U = A, V = B model
// the Jacobian on each mode, J_q ~ -I + U V^H.  For mode q and pair p:
// s = RMS of the z_q profile (pairs with s = 0 skip), xhat = z_q / s,
// that = (J z)_q / s, c = V^H xhat, r = -xhat + U c - that;
// loss = scale sum |r|^2, dU = 2 scale sum r c^H, dV = 2 scale sum xhat (U^H r)^H.
// One workgroup of 256 threads per row.  The row's U and V are staged in LDS
// once (rows padded to R + 1 entries, so threads over consecutive e spread
// over the banks); pairs pass through LDS hb at a time (FP32).  Per pass:
// C = V^H X and G = U^H R with the sum over e split into np ranges whose
// partial sums are added in a fixed order, R = -X + U C - T by threads over
// (pair, e), and dU += R C^H, dV += X G^H in registers (each thread owns
// fixed gradient entries) until the row is written once: dY in FP32 and its
// row-major bfloat16 copy (k_head_out makes the transposed one).
// Bound by its vector instructions: 1512 rows of 3 N = 144, R = 16, 16 pairs
// take 97 us (its bytes 40 us), 127 with U, V, xhat and r addressed entry by
// entry and a branch per gradient entry (8100 instructions per wave, 4600 of
// them the sums' own).  xhat and r lie side by side, one 16-byte read for
// both updates; addresses advance by the row; entries past the last one
// repeat it instead of branching; the next pass's profiles are requested a
// pass ahead, and barriers order LDS only.  Three workgroups per compute unit
// (HEAD_LDS, 168 VGPRs): with 177 VGPRs and two it took 153 us.
// HO: gradient entries per thread and factor (3N R <= 256 HO); JFIX: R
// divides 256, so every entry of a thread has the same j and the thread
// keeps C and G of its column in registers through the dU, dV update.
template <int HO, bool JFIX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HO <= 9 ? 3 : 2, HO <= 9 ? 3 : 2)))
void k_head(HeadArgs a) {
    extern __shared__ float2 hsm[];
    __shared__ float lpart[4];
    const int q = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
    float* yrow = a.Y + (long)q * a.dout;
    const int n3 = 3 * a.N, R = a.rank, RP = R + 1, nf = n3 * R;  // complex entries of U (and of V)
    if (q >= a.rows) {  // padding rows: zero gradient
        for (int j = t; j < a.dout; j += 256) {
            yrow[j] = 0.0f;
            a.dyb[(long)q * a.dout + j] = 0;
        }
        if (t == 0) a.lrow[q] = 0.0f;
        return;
    }
    const int hb = a.hb;
    float2* sU = hsm;               // [n3][RP]
    float2* sV = sU + n3 * RP;      // [n3][RP]
    float4* xr = reinterpret_cast<float4*>(sV + n3 * RP);  // [hb][n3 + 1]: (xhat; that, then r)
    const int XP = n3 + 1;
    float2* cs = reinterpret_cast<float2*>(xr + hb * XP);  // [hb][R]
    float2* gs = cs + hb * R;       // [hb][R]
    float2* red = gs + hb * R;      // [256] partial sums
    {
        const float2* U2 = reinterpret_cast<const float2*>(yrow);
        const int ej = t / R, jj = t - ej * R;
#pragma unroll
        for (int o = 0; o < HO; ++o) {
            const int i = t + 256 * o;
            if (i >= nf) break;
            const int e = JFIX ? ej + 256 / R * o : i / R, j = JFIX ? jj : i - e * R;
            sU[e * RP + j] = U2[i];
            sV[e * RP + j] = U2[nf + i];
        }
    }
    const long S = (long)a.M * a.nk * a.N;
    float2 du[HO], dv[HO];
#pragma unroll
    for (int o = 0; o < HO; ++o) du[o] = dv[o] = make_float2(0.0f, 0.0f);
    float lsum = 0.0f;
    // z and J z of mode q of batch entry b at e = lane + 64 i < 3 N <= 192: the
    // first pair of each wave is requested a pass ahead
    double2 zz[3], jz[3];
    auto request = [&](int b) {
        const double* zv = a.pairs + (long)a.idx[min(b, a.batch - 1)] * 2 * a.vec + 2 * (long)q * a.N;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int e = min(lane + 64 * i, n3 - 1), c = e >= 2 * a.N ? 2 : e >= a.N ? 1 : 0;
            const double* ze = zv + 2 * (c * S + e - c * a.N);
            zz[i] = *reinterpret_cast<const double2*>(ze);
            jz[i] = *reinterpret_cast<const double2*>(ze + a.vec);
        }
    };
    request(w);
    for (int b0 = 0; b0 < a.batch; b0 += hb) {
        const int nb = min(hb, a.batch - b0);
        const int items = nb * R;
        const int np = items >= 256 ? 1 : 256 / items;  // e ranges of the V^H X and U^H R sums
        const int elen = (n3 + np - 1) / np;
        for (int b = w; b < nb; b += 4) {  // one wave per pair: its z and J z profiles of mode q, over s
            if (b > w) request(b0 + b);
            float2 x[3], th[3];
            float s2 = 0.0f;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                x[i] = make_float2((float)zz[i].x, (float)zz[i].y);
                th[i] = make_float2((float)jz[i].x, (float)jz[i].y);
                if (lane + 64 * i < n3) s2 += x[i].x * x[i].x + x[i].y * x[i].y;
            }
            s2 = wave_sum(s2);
            const float f = s2 > 0.0f ? 1.0f / sqrtf(s2 / n3) : 0.0f;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int e = lane + 64 * i;
                if (e >= n3) continue;
                xr[b * XP + e] = make_float4(x[i].x * f, x[i].y * f, th[i].x * f, th[i].y * f);
            }
        }
        request(b0 + hb + w);
        lds_barrier();
        for (int i = t; i < items * np; i += 256) {  // partial C = V^H X over e range p
            const int p = i / items, bj = i - p * items, b = bj / R, j = bj - b * R;
            const int e0 = p * elen, e1 = min(n3, e0 + elen);
            float cr = 0.0f, ci = 0.0f;
            const float2 *vp = sV + e0 * RP + j, *xp = reinterpret_cast<const float2*>(xr + b * XP + e0);
#pragma unroll 4
            for (int e = e0; e < e1; ++e, vp += RP, xp += 2) {
                const float2 v = *vp, x = *xp;
                cr += v.x * x.x + v.y * x.y;
                ci += v.x * x.y - v.y * x.x;
            }
            if (np == 1) cs[bj] = make_float2(cr, ci);
            else red[i] = make_float2(cr, ci);
        }
        lds_barrier();
        if (np > 1) {
            for (int bj = t; bj < items; bj += 256) {
                float2 c = red[bj];
                for (int p = 1; p < np; ++p) c.x += red[p * items + bj].x, c.y += red[p * items + bj].y;
                cs[bj] = c;
            }
            lds_barrier();
        }
        for (int i = t, b = 0, e = t; i < nb * n3; i += 256, e += 256) {  // r = -x + U c - that
            while (e >= n3) e -= n3, ++b;  // i = b n3 + e
            const float4 xt = xr[b * XP + e];
            float pr = -xt.x - xt.z, pi = -xt.y - xt.w;
#pragma unroll 4
            for (int j = 0; j < R; ++j) {
                const float2 u = sU[e * RP + j], c = cs[b * R + j];
                pr += u.x * c.x - u.y * c.y;
                pi += u.x * c.y + u.y * c.x;
            }
            reinterpret_cast<float2*>(xr + b * XP + e)[1] = make_float2(pr, pi);
            lsum += pr * pr + pi * pi;
        }
        lds_barrier();
        for (int i = t; i < items * np; i += 256) {  // partial G = U^H R over e range p
            const int p = i / items, bj = i - p * items, b = bj / R, j = bj - b * R;
            const int e0 = p * elen, e1 = min(n3, e0 + elen);
            float gr = 0.0f, gi = 0.0f;
            const float2 *up = sU + e0 * RP + j, *rp = reinterpret_cast<const float2*>(xr + b * XP + e0) + 1;
#pragma unroll 4
            for (int e = e0; e < e1; ++e, up += RP, rp += 2) {
                const float2 u = *up, r = *rp;
                gr += u.x * r.x + u.y * r.y;
                gi += u.x * r.y - u.y * r.x;
            }
            if (np == 1) gs[bj] = make_float2(gr, gi);
            else red[i] = make_float2(gr, gi);
        }
        lds_barrier();
        if (np > 1) {
            for (int bj = t; bj < items; bj += 256) {
                float2 g = red[bj];
                for (int p = 1; p < np; ++p) g.x += red[p * items + bj].x, g.y += red[p * items + bj].y;
                gs[bj] = g;
            }
            lds_barrier();
        }
        if constexpr (JFIX) {  // dU += r c^H, dV += x g^H on this thread's entries (column j0)
            const int j0 = t % R, e0 = t / R, es = 256 / R;
            const float4* at[HO];  // entries past the last one repeat it and are not stored
#pragma unroll
            for (int o = 0; o < HO; ++o) at[o] = xr + min(e0 + es * o, n3 - 1);
            for (int b = 0; b < nb; ++b) {
                const float2 c = cs[b * R + j0], g = gs[b * R + j0];
#pragma unroll
                for (int o = 0; o < HO; ++o) {
                    const float4 x = *at[o];
                    at[o] += XP;
                    du[o].x += x.z * c.x + x.w * c.y;
                    du[o].y += x.w * c.x - x.z * c.y;
                    dv[o].x += x.x * g.x + x.y * g.y;
                    dv[o].y += x.y * g.x - x.x * g.y;
                }
            }
        } else {
#pragma unroll
            for (int o = 0; o < HO; ++o) {
                const int i = t + 256 * o;
                if (i < nf) {
                    const int e = i / R, j = i - e * R;
                    for (int b = 0; b < nb; ++b) {
                        const float4 x = xr[b * XP + e];
                        const float2 c = cs[b * R + j], g = gs[b * R + j];
                        du[o].x += x.z * c.x + x.w * c.y;
                        du[o].y += x.w * c.x - x.z * c.y;
                        dv[o].x += x.x * g.x + x.y * g.y;
                        dv[o].y += x.y * g.x - x.x * g.y;
                    }
                }
            }
        }
        lds_barrier();
    }
    lsum = wave_sum(lsum);
    if (lane == 0) lpart[w] = lsum;
    __syncthreads();
    if (t == 0) a.lrow[q] = ((lpart[0] + lpart[1]) + lpart[2]) + lpart[3];
    const float g2 = 2.0f * a.scale;
    float2* y2 = reinterpret_cast<float2*>(yrow);
    uint32_t* yb = reinterpret_cast<uint32_t*>(a.dyb + (long)q * a.dout);  // bf16 pairs
#pragma unroll
    for (int o = 0; o < HO; ++o) {
        const int i = t + 256 * o;  // with JFIX: e = e0 + es o, j = j0, i.e. the same i
        if (i < nf) {
            const float2 gu = make_float2(g2 * du[o].x, g2 * du[o].y), gv = make_float2(g2 * dv[o].x, g2 * dv[o].y);
            y2[i] = gu;
            y2[nf + i] = gv;
            yb[i] = (uint32_t)f2bf(gu.x) | ((uint32_t)f2bf(gu.y) << 16);
            yb[nf + i] = (uint32_t)f2bf(gv.x) | ((uint32_t)f2bf(gv.y) << 16);
        }
    }
    for (int j = 4 * nf + t; j < a.dout; j += 256) {
        yrow[j] = 0.0f;
        a.dyb[(long)q * a.dout + j] = 0;
    }
}

// dL/dY [rows][cols] of the loss head: the transposed bfloat16 copy dst[col][row]
// and the column sums of each 128-row chunk, part[chunk][col] (the sums of
// k_grad_parts, in its order), from one reading.  64 columns x 128 rows per
// workgroup: 32 rows a thread in flight, runs of 256 bytes read and written,
// the transposition through LDS (rows of 65 words, so that neither side
// conflicts).  Bound by its bytes: 1536 x 9216 (85 MB) take 13.7 us; a
// transposition of the bfloat16 rows and column sums apart took 17 + 13 us.
constexpr int HC = 128;  // rows of a chunk
__global__ __launch_bounds__(256) void k_head_out(const float* __restrict__ Y, int rows, int cols,
                                                  bf16_t* __restrict__ dst, int ldd, float* __restrict__ part, int ncol) {
    __shared__ bf16_t tile[64][HC + 2];
    __shared__ float red[8][64];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * HC;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    float v[HC / 4], s[2] = {0.0f, 0.0f};  // this thread's rows ty + 4 i; their sums by row % 8
#pragma unroll
    for (int i = 0; i < HC / 4; ++i) {
        const int r = r0 + ty + 4 * i;
        v[i] = r < rows && c0 + tx < cols ? Y[(size_t)r * cols + c0 + tx] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < HC / 4; ++i) {
        s[i & 1] += v[i];
        tile[tx][ty + 4 * i] = f2bf(v[i]);
    }
    red[ty][tx] = s[0];
    red[ty + 4][tx] = s[1];
    __syncthreads();
    if (ty == 0 && c0 + tx < cols) {
        float t = 0.0f;
        for (int g = 0; g < 8; ++g) t += red[g][tx];
        part[(size_t)blockIdx.y * ncol + c0 + tx] = t;
    }
    for (int c = ty; c < 64; c += 4)
        if (c0 + c < cols && r0 + 2 * tx < rows)
            *reinterpret_cast<uint32_t*>(dst + (size_t)(c0 + c) * ldd + r0 + 2 * tx) =
                *reinterpret_cast<const uint32_t*>(&tile[c][2 * tx]);
}

// Preconditioner factors from the Jacobian model of each mode: with
// J_q ~ -I + U V^H, J_q^{-1} = -(I + U G^{-1} V^H), G = I_R - V^H U
// (Sherman-Morrison-Woodbury), so P(v) = -v + A (B^H v) with A = -U G^{-1},
// B = V.  G is inverted by Gauss-Jordan elimination with partial pivoting in
// FP64; a mode whose G has a zero pivot gets A = 0 (P = -I there) and
// singular[q] = 1.  One workgroup of one wave per mode.
__global__ __launch_bounds__(64) void k_woodbury(const float* __restrict__ uv, float* __restrict__ fac, int dout,
                                                 int N, int rank, int rows, int* __restrict__ singular) {
    __shared__ double g[RMAX][2 * RMAX];   // G, then its inverse (complex, row-major)
    __shared__ double gi[RMAX][2 * RMAX];
    const int q = blockIdx.x, lane = threadIdx.x;
    if (q >= rows) return;
    const int R = rank, n3 = 3 * N, nf = 6 * N * R;
    const float* U = uv + (long)q * dout;
    const float* V = U + nf;
    float* A = fac + (long)q * dout;
    float* B = A + nf;
    for (int i = 0; i < R; ++i)
        for (int j = 0; j < R; ++j) {  // (V^H U)_ij = sum_e conj(V_ei) U_ej
            double sr = 0.0, si = 0.0;
            for (int e = lane; e < n3; e += 64) {
                const double vr = V[2 * (e * R + i)], vi = V[2 * (e * R + i) + 1];
                const double ur = U[2 * (e * R + j)], ui = U[2 * (e * R + j) + 1];
                sr += vr * ur + vi * ui;
                si += vr * ui - vi * ur;
            }
            sr = wave_sum(sr);
            si = wave_sum(si);
            if (lane == 0) {
                g[i][2 * j] = (i == j ? 1.0 : 0.0) - sr;
                g[i][2 * j + 1] = -si;
            }
        }
    __shared__ int bad;
    if (lane == 0) {  // Gauss-Jordan on [G | I]
        bad = 0;
        for (int i = 0; i < R; ++i)
            for (int j = 0; j < R; ++j) {
                gi[i][2 * j] = i == j ? 1.0 : 0.0;
                gi[i][2 * j + 1] = 0.0;
            }
        for (int c = 0; c < R && !bad; ++c) {
            int piv = c;
            double best = -1.0;
            for (int i = c; i < R; ++i) {
                const double m = g[i][2 * c] * g[i][2 * c] + g[i][2 * c + 1] * g[i][2 * c + 1];
                if (m > best) {
                    best = m;
                    piv = i;
                }
            }
            if (!(best > 0.0)) {
                bad = 1;
                break;
            }
            for (int j = 0; j < 2 * R; ++j) {
                const double t = g[c][j];
                g[c][j] = g[piv][j];
                g[piv][j] = t;
                const double u = gi[c][j];
                gi[c][j] = gi[piv][j];
                gi[piv][j] = u;
            }
            const double pr = g[c][2 * c], pi = g[c][2 * c + 1];
            const double den = pr * pr + pi * pi;
            const double ir = pr / den, ii = -pi / den;  // 1 / pivot
            for (int j = 0; j < R; ++j) {
                double a = g[c][2 * j], b = g[c][2 * j + 1];
                g[c][2 * j] = a * ir - b * ii;
                g[c][2 * j + 1] = a * ii + b * ir;
                a = gi[c][2 * j];
                b = gi[c][2 * j + 1];
                gi[c][2 * j] = a * ir - b * ii;
                gi[c][2 * j + 1] = a * ii + b * ir;
            }
            for (int i = 0; i < R; ++i) {
                if (i == c) continue;
                const double fr = g[i][2 * c], fi = g[i][2 * c + 1];
                for (int j = 0; j < R; ++j) {
                    g[i][2 * j] -= fr * g[c][2 * j] - fi * g[c][2 * j + 1];
                    g[i][2 * j + 1] -= fr * g[c][2 * j + 1] + fi * g[c][2 * j];
                    gi[i][2 * j] -= fr * gi[c][2 * j] - fi * gi[c][2 * j + 1];
                    gi[i][2 * j + 1] -= fr * gi[c][2 * j + 1] + fi * gi[c][2 * j];
                }
            }
        }
        singular[q] = bad;
    }
    __syncthreads();
    for (int e = lane; e < n3; e += 64)
        for (int j = 0; j < R; ++j) {  // A = -U G^{-1}, B = V
            double ar = 0.0, ai = 0.0;
            if (!bad)
                for (int i = 0; i < R; ++i) {
                    const double ur = U[2 * (e * R + i)], ui = U[2 * (e * R + i) + 1];
                    ar -= ur * gi[i][2 * j] - ui * gi[i][2 * j + 1];
                    ai -= ur * gi[i][2 * j + 1] + ui * gi[i][2 * j];
                }
            A[2 * (e * R + j)] = (float)ar;
            A[2 * (e * R + j) + 1] = (float)ai;
            B[2 * (e * R + j)] = V[2 * (e * R + j)];
            B[2 * (e * R + j) + 1] = V[2 * (e * R + j) + 1];
        }
    for (int j = 2 * nf + lane; j < dout; j += 64) A[j] = 0.0f;
}

uint64_t splitmix64(uint64_t& state) {
    uint64_t z = (state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

double uniform01(uint64_t& state) { return (double)(splitmix64(state) >> 11) * (1.0 / 9007199254740992.0); }

int round32(int x) { return (x + 31) / 32 * 32; }

}  // namespace

struct opf_mlp {
    opf_ctx* ctx = nullptr;
    hipStream_t s = nullptr;
    int N = 0, M = 0, K = 0, nk = 0, mp = 1;
    double alpha = 1.0;
    int H = 0, L = 0, rank = 0, din = 0, dout = 0, R = 0, mode_rows = 0;
    long np = 0;
    Segs segs{};
    long woff[MAXL + 2] = {}, boff[MAXL + 2] = {};
    float lr = 1e-3f, lr_final = 1e-3f, b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    long t = 0;
    bool fac_ok = false;
    float *P = nullptr, *G = nullptr, *Am = nullptr, *Av = nullptr;
    bf16_t *Wb = nullptr, *Wt = nullptr;
    bf16_t *Xb = nullptr, *XT = nullptr;
    bf16_t *HL = nullptr, *HT = nullptr;       // h_L [R][H]; h_l transposed, l = 0..L
    float *Z = nullptr, *Y = nullptr, *D = nullptr;  // D: dL/dh_l [R][H], l = 0..L
    bf16_t *dYb = nullptr, *dYT = nullptr, *DT = nullptr;  // DT: D_l where z_{l-1} > 0, transposed
    float *fx = nullptr, *fac = nullptr;
    int* idx = nullptr;
    int* singular = nullptr;  // [rows] modes whose Woodbury matrix is singular
    float* part = nullptr;    // [CS_CHUNKS][dout + (L + 1) H] column-sum partials
    float* gpart = nullptr;   // [GPART] split-K partial tiles
    int n_singular = 0;
    float *lrow = nullptr, *wsum = nullptr, *losses = nullptr;
    int loss_cap = 0;
    std::string err;

    bf16_t* ht(int l) const { return HT + (size_t)l * H * R; }
    bf16_t* dt(int l) const { return DT + (size_t)l * H * R; }
    float* d(int l) const { return D + (size_t)l * R * H; }
};

namespace {

constexpr int LOSS_CAP = 1 << 16;  // training steps per call
constexpr int IDX_CAP = 1 << 20;   // pair indices per call (steps x batch)

#define MCHK(net, call)                                                             \
    do {                                                                            \
        hipError_t e_ = (call);                                                     \
        if (e_ != hipSuccess) {                                                     \
            (net)->err = std::string(#call) + ": " + hipGetErrorString(e_);         \
            return OPF_E_HIP;                                                       \
        }                                                                           \
    } while (0)

struct Layout {
    size_t off[32] = {};
    size_t total = 0;
    int n = 0;
    size_t take(size_t bytes) {
        const size_t o = total;
        off[n++] = o;
        total += (bytes + 255) / 256 * 256;
        return o;
    }
};

// dims, parameter segments and buffer layout of a network
Layout plan(opf_mlp* m) {
    m->din = NCOND;
    m->dout = round32(12 * m->N * m->rank);
    long o = 0;
    int j = 0, blk = 0;
    auto seg = [&](int rows, int cols, int mat) {
        m->segs.off[j] = o;
        m->segs.rows[j] = rows;
        m->segs.cols[j] = cols;
        m->segs.mat[j] = mat;
        m->segs.blk[j] = blk;
        blk += mat ? (rows + PT - 1) / PT * (cols / 32) : (cols + 2047) / 2048;
        ++j;
        const long at = o;
        o += (long)rows * cols;
        return at;
    };
    m->woff[0] = seg(m->H, m->din, 1);
    m->boff[0] = seg(1, m->H, 0);
    for (int l = 0; l < m->L; ++l) {
        m->woff[l + 1] = seg(m->H, m->H, 2);
        m->boff[l + 1] = seg(1, m->H, 0);
    }
    m->woff[m->L + 1] = seg(m->dout, m->H, 1);
    m->boff[m->L + 1] = seg(1, m->dout, 0);
    m->segs.n = j;
    m->segs.off[j] = o;
    m->segs.blk[j] = blk;
    m->np = o;
    const size_t R = m->R, H = m->H, L = m->L, np = o;
    Layout lay;
    for (int q = 0; q < 4; ++q) lay.take(np * 4);  // P, G, Am, Av
    lay.take(np * 2);                              // Wb
    lay.take(np * 2);                              // Wt
    lay.take(R * m->din * 2);                      // Xb
    lay.take(R * m->din * 2);                      // XT
    lay.take(R * H * 2);                           // HL
    lay.take((L + 1) * R * H * 2);                 // HT
    lay.take(L * R * H * 4);                       // Z
    lay.take(R * m->dout * 4);                     // Y
    lay.take((L + 1) * R * H * 4);                 // D
    lay.take(R * m->dout * 2);                     // dYb
    lay.take(R * m->dout * 2);                     // dYT
    lay.take((L + 1) * R * H * 2);                 // DT
    lay.take(R * m->din * 4);                      // fx: mode feature rows
    lay.take(R * m->dout * 4);                     // fac: factor rows in use
    lay.take((size_t)IDX_CAP * 4);                 // idx: pair indices
    lay.take(R * 4);                               // singular: per-mode flag of a singular G
    lay.take((size_t)CS_CHUNKS * (m->dout + (L + 1) * H) * 4);  // part
    lay.take(GPART * 4);                                         // gpart
    lay.take(R * 4);                               // lrow
    lay.take(256);                                 // wsum
    lay.take((size_t)LOSS_CAP * 4);                // losses
    return lay;
}

opf_status check_cfg(const opf_ctx* c, const opf_mlp_config* cfg, std::string* why) {
    if (!c || !cfg) return OPF_E_INVALID;
    const opf_params& p = ctx_params(c);
    auto bad = [&](const char* s) {
        if (why) *why = s;
        return OPF_E_INVALID;
    };
    if (cfg->width < 32 || cfg->width > 512 || cfg->width % 32) return bad("width must be a multiple of 32 in [32, 512]");
    if (cfg->layers < 1 || cfg->layers > MAXL) return bad("layers must be in [1, 8]");
    if (cfg->rank < 1 || cfg->rank > RMAX) return bad("rank must be in [1, 32]");
    if (3L * p.N * cfg->rank > 256L * HOUT) return bad("3 N rank must not exceed 3072");
    if (cfg->max_rows < 0 || cfg->max_rows > (1 << 20)) return bad("max_rows must be in [0, 2^20]");
    if (!(cfg->lr >= 0.0f) || !(cfg->lr_final >= 0.0f) || !(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f) ||
        !(cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f) || !(cfg->adam_eps > 0.0f))
        return bad("bad Adam parameters");
    return OPF_OK;
}

// A product left as nsplit partial products [rows][cols] for its reader to add
// in order (one: the product itself, at Epi::out's place).
struct Parts {
    const float* at = nullptr;
    int nsplit = 0;
};

struct Split {
    int n, kc;  // K ranges and their length
};

// K split of a GEMM whose tile count cannot fill the chip but whose K is long.
Split split_of(int rows, int cols, int K) {
    Split p{1, K};
    const size_t rc = (size_t)rows * cols;
    if (large_product(rows, cols, K)) {  // 128 x 128 tiles, until about 256 workgroups
        const long tiles = (long)(rows / G2) * (cols / G2);
        if (tiles < 256) {
            p.n = (int)std::min<long>((256 + tiles - 1) / tiles, std::min(K / 256, 2 * GSPLIT));
            if (p.n * rc > GPART) p.n = (int)(GPART / rc);
            p.n = std::max(p.n, 1);
            p.kc = ((K + p.n - 1) / p.n + GK2 - 1) / GK2 * GK2;
            p.n = (K + p.kc - 1) / p.kc;
        }
        return p;
    }
    const long tiles = (long)(rows / GT) * (cols / GT);
    if (tiles < 1024 && K >= 512) {
        p.n = (int)std::min<long>((2048 + tiles - 1) / tiles, std::min(K / 256, GSPLIT));
        p.kc = ((K + p.n - 1) / p.n + 63) / 64 * 64;
        p.n = (K + p.kc - 1) / p.kc;
        if (p.n * rc > GPART) p = {1, K};
    }
    return p;
}

// Launch a GEMM.  The partial tiles of a split go to the scratch and through
// k_gemm_reduce, or stay in the scratch when the caller takes `parts`.
hipError_t gemm(opf_mlp* m, const bf16_t* A, int lda, const bf16_t* B, int ldb, int rows, int cols, int K,
                const Epi& e, Parts* parts = nullptr) {
    if (rows % GT || cols % GT || K % 16 || lda % 8 || ldb % 8 || rows <= 0 || cols <= 0 || K <= 0)
        return hipErrorInvalidValue;
    const Split p = split_of(rows, cols, K);
    float* part = p.n > 1 ? m->gpart : nullptr;
    if (large_product(rows, cols, K))
        hipLaunchKernelGGL(k_gemm128, dim3(cols / G2, rows / G2, p.n), dim3(256), 0, m->s, A, lda, B, ldb, K, p.kc, e, part);
    else
        hipLaunchKernelGGL(k_gemm, dim3(cols / GT, rows / GT, p.n), dim3(256), 0, m->s, A, lda, B, ldb, K, p.kc, e, part);
    if (parts) {
        parts->at = part ? part : e.out;
        parts->nsplit = p.n;
    } else if (part) {
        const size_t n = (size_t)rows * cols;
        hipLaunchKernelGGL(k_gemm_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, m->s, part, rows, cols, p.n, e);
    }
    return hipGetLastError();
}

ChainArgs chain_args(const opf_mlp* m, int rp, const bf16_t* W) {
    ChainArgs a{};
    a.X = m->Xb;
    a.W = W;
    a.P = m->P;
    for (int l = 0; l <= m->L; ++l) a.woff[l] = m->woff[l], a.boff[l] = m->boff[l];
    a.H = m->H;
    a.L = m->L;
    a.R = m->R;
    a.rows = rp;
    a.Z = m->Z;
    a.HL = m->HL;
    return a;
}

// One workgroup per 32 rows, one wave per 32 columns.
hipError_t launch_chain(const ChainArgs& a, bool fwd, hipStream_t s) {
    const int H = a.H;
    auto k = H < 256    ? (fwd ? k_chain_fwd<false, false> : k_chain_bwd<false, false>)
             : H == 256 ? (fwd ? k_chain_fwd<false, true> : k_chain_bwd<false, true>)
             : H < 512  ? (fwd ? k_chain_fwd<true, false> : k_chain_bwd<true, false>)
                        : (fwd ? k_chain_fwd<true, true> : k_chain_bwd<true, true>);
    const size_t lds = (size_t)2 * 32 * (H + 8) * sizeof(bf16_t);  // 66.6 KB at H = 512
    if (lds > 65536) {
        const hipError_t st = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (st != hipSuccess) return st;
    }
    hipLaunchKernelGGL(k, dim3(a.rows / 32), dim3(2 * H), lds, s, a);
    return hipGetLastError();
}

// Forward pass over rp rows (multiple of 32) of bfloat16 rows Xb.
// train: also keep pre-activations and transposed activations.
hipError_t forward(opf_mlp* m, int rp, bool train) {
    const int H = m->H, L = m->L;
    ChainArgs a = chain_args(m, rp, m->Wb);
    a.HT = train ? m->HT : nullptr;
    const hipError_t st = launch_chain(a, true, m->s);
    if (st != hipSuccess) return st;
    Epi g{};
    g.bias = m->P + m->boff[L + 1];
    g.out = m->Y;
    g.ldo = m->dout;
    return gemm(m, m->HL, H, m->Wb + m->woff[L + 1], H, rp, m->dout, H, g);
}

// Loss (of per-row losses lrow[0..nlive) over *wsum or count) and parameter
// gradients, as the partial sums that `g` describes, from dL/dY (FP32 in Y,
// bfloat16 in dYb / dYT; ysums: its column sums already in part) after
// forward(train = true) over rp rows.  k_grad_sum or k_adam adds them up.
hipError_t backprop(opf_mlp* m, int rp, bool ysums, int nlive, const float* wsum, float count, float* loss_slot, GradArgs& g) {
    const int H = m->H, L = m->L, R = m->R, dout = m->dout;
    hipError_t st;
    Epi e{};
    Parts p;
    e.out = m->d(L);  // dL/dh_L = dY W_out, added up by the chain
    e.ldo = H;
    if ((st = gemm(m, m->dYb, dout, m->Wt + m->woff[L + 1], dout, rp, H, dout, e, &p)) != hipSuccess) return st;
    ChainArgs a = chain_args(m, rp, m->Wt);
    a.HT = m->HT;
    a.src = p.at;
    a.nsplit = p.nsplit;
    a.stride = (size_t)rp * H;
    a.D = m->D;
    a.DT = m->DT;
    if ((st = launch_chain(a, false, m->s)) != hipSuccess) return st;

    g = GradArgs{};
    g.DT = m->DT;
    g.HT = m->HT;
    g.XT = m->XT;
    g.D = m->D;
    g.Z = m->Z;
    g.Y = m->Y;
    for (int l = 0; l <= L; ++l) g.woff[l] = m->woff[l];
    g.H = H;
    g.L = L;
    g.R = R;
    g.dout = dout;
    g.rows = rp;
    g.nph = m->woff[L + 1];
    g.G = m->G;
    g.wout = m->woff[L + 1];
    g.bout = m->boff[L + 1];
    // weight gradients of the residual layers: 128 x 128 tiles where a product
    // is large (each row of the operands is then read four times less often)
    g.nhid = large_product(H, H, rp) ? 0 : L;
    for (int l = g.nhid; l < L; ++l) {
        Epi w{};
        w.out = m->G + m->woff[l + 1];
        w.ldo = H;
        if ((st = gemm(m, m->dt(l + 1), R, m->ht(l), R, H, H, rp, w)) != hipSuccess) return st;
    }
    g.nsplit = std::max(1, std::min({rp / 256, GSPLIT, (int)(GPART / g.nph)}));
    g.kc = ((rp + g.nsplit - 1) / g.nsplit + 63) / 64 * 64;
    g.nsplit = (rp + g.kc - 1) / g.kc;
    // output layer: dW = dY^T H_L; its partial products stay in the scratch
    // until k_grad_sum when the other layers' fit behind them
    e.out = m->G + g.wout;
    e.ldo = H;
    const size_t nw = (size_t)dout * H;
    const int osplit = split_of(dout, H, rp).n;
    const bool keep = osplit > 1 && osplit * nw + (size_t)g.nsplit * g.nph <= GPART;
    if ((st = gemm(m, m->dYT, R, m->ht(L), R, dout, H, rp, e, keep ? &p : nullptr)) != hipSuccess) return st;
    g.osplit = keep ? osplit : 0;
    g.opart = m->gpart;
    g.gpart = m->gpart + g.osplit * nw;

    g.ngemm = (H / GT + g.nhid * (H / GT) * (H / GT)) * g.nsplit;
    g.ch = std::max(HC, (rp + CS_CHUNKS - 1) / CS_CHUNKS);
    g.nch = (rp + g.ch - 1) / g.ch;
    g.part = m->part;
    g.lrow = m->lrow;
    g.wsum = wsum;
    g.count = count;
    g.nlive = nlive;
    g.loss = loss_slot;
    g.col0 = ysums ? dout : 0;
    hipLaunchKernelGGL(k_grad_parts, dim3(g.ngemm + g.nch * ((dout + (L + 1) * H - g.col0) / 32) + 1), dim3(256), 0, m->s, g);
    return hipGetLastError();
}

// Squared-error loss of rows (targets t, weights om) into *loss_slot and
// dL/dY, then the parameter gradients.
hipError_t backward_rows(opf_mlp* m, const float* t, const float* om, int nrows, int rp, float* loss_slot, GradArgs& g) {
    hipStream_t s = m->s;
    hipLaunchKernelGGL(k_weight_sum, dim3(1), dim3(256), 0, s, om, nrows, m->wsum);
    hipLaunchKernelGGL(k_loss, dim3(rp / 4), dim3(256), 0, s, m->Y, t, om, m->wsum, nrows, rp, m->dout, m->dYb,
                       m->dYT, m->R, m->lrow);
    const hipError_t st = hipGetLastError();
    return st != hipSuccess ? st : backprop(m, rp, false, nrows, m->wsum, 0.0f, loss_slot, g);
}

// Loss head over pairs idx[0..batch) into *loss_slot and dL/dY, then the
// parameter gradients (forward over the mode feature rows first).
hipError_t backward_pairs(opf_mlp* m, const double* pairs, const int* idx, int batch, float* loss_slot, GradArgs& g) {
    hipStream_t s = m->s;
    const int rp = round32(m->mode_rows);
    HeadArgs a{};
    a.pairs = pairs;
    a.vec = 2L * 3 * m->M * m->nk * m->N;
    a.idx = idx;
    a.batch = batch;
    a.N = m->N;
    a.M = m->M;
    a.nk = m->nk;
    a.rank = m->rank;
    a.dout = m->dout;
    a.rows = m->mode_rows;
    a.rp = rp;
    a.Y = m->Y;
    a.dyb = m->dYb;
    a.lrow = m->lrow;
    a.scale = (float)(1.0 / ((double)batch * m->mode_rows));
    a.hb = head_pairs(3 * m->N, m->rank);
    const size_t hl = (size_t)(head_slots(3 * m->N, m->rank, a.hb) + 2 * a.hb) * sizeof(float2);  // (one entry of padding per pair)
    const int nf = 3 * m->N * m->rank, ho = nf <= 768 ? 3 : nf <= 1536 ? 6 : nf <= 2304 ? 9 : 12;
    const bool jfix = 256 % m->rank == 0;
    auto kh = jfix ? (ho == 3 ? k_head<3, true> : ho == 6 ? k_head<6, true> : ho == 9 ? k_head<9, true> : k_head<12, true>)
                   : (ho == 3 ? k_head<3, false> : ho == 6 ? k_head<6, false> : ho == 9 ? k_head<9, false> : k_head<12, false>);
    hipLaunchKernelGGL(kh, dim3(rp), dim3(256), hl, s, a);
    // (a chunk of the column sums is HC rows up to CS_CHUNKS HC = 8192 rows; the
    // longest transform lines allow 64 x 127 modes)
    if (rp > CS_CHUNKS * HC) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_head_out, dim3((m->dout + 63) / 64, (rp + HC - 1) / HC), dim3(256), 0, s, m->Y, rp, m->dout,
                       m->dYT, m->R, m->part, m->dout + (m->L + 1) * m->H);
    const hipError_t st = hipGetLastError();
    return st != hipSuccess ? st : backprop(m, rp, true, m->mode_rows, nullptr, (float)((long)batch * m->mode_rows), loss_slot, g);
}

hipError_t adam(opf_mlp* m, const GradArgs& g, float lr) {
    m->t += 1;
    m->fac_ok = false;
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)m->b1, (double)m->t)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)m->b2, (double)m->t)));
    hipLaunchKernelGGL(k_adam, dim3(m->segs.blk[m->segs.n]), dim3(256), 0, m->s, m->P, g, m->Am, m->Av, lr, m->b1, m->b2, c1, c2, m->eps, m->segs, m->Wb, m->Wt);
    return hipGetLastError();
}

hipError_t grad_sum(opf_mlp* m, const GradArgs& g) {
    hipLaunchKernelGGL(k_grad_sum, dim3((unsigned)((m->np / 4 + 255) / 256)), dim3(256), 0, m->s, g, m->segs);
    return hipGetLastError();
}

hipError_t rows_bf16(opf_mlp* m, const float* x, int nrows, int rp, bool transposed) {
    const size_t n = (size_t)rp * m->din;
    hipLaunchKernelGGL(k_rows_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, m->s, x, nrows, rp, m->din,
                       m->Xb, transposed ? m->XT : nullptr, m->R);
    return hipGetLastError();
}

// The mode feature rows as GEMM input (and transposed, for training).
hipError_t feature_input(opf_mlp* m) { return rows_bf16(m, m->fx, m->mode_rows, round32(m->mode_rows), true); }

// Preconditioner factors (A, B) of the current parameters into fac: the
// network's Jacobian model (U, V) per mode, inverted by Woodbury.
hipError_t refresh_factors(opf_mlp* m) {
    if (m->fac_ok) return hipSuccess;
    const int rp = round32(m->mode_rows);
    hipError_t st = feature_input(m);
    if (st == hipSuccess) st = forward(m, rp, false);
    if (st != hipSuccess) return st;
    hipLaunchKernelGGL(k_woodbury, dim3(m->mode_rows), dim3(64), 0, m->s, m->Y, m->fac, m->dout, m->N, m->rank,
                       m->mode_rows, m->singular);
    if ((st = hipGetLastError()) != hipSuccess) return st;
    std::vector<int> flags(m->mode_rows);
    if ((st = hipMemcpyAsync(flags.data(), m->singular, flags.size() * sizeof(int), hipMemcpyDeviceToHost, m->s)) !=
            hipSuccess ||
        (st = hipStreamSynchronize(m->s)) != hipSuccess)
        return st;
    m->n_singular = 0;
    for (int f : flags) m->n_singular += f;
    m->fac_ok = true;
    return hipSuccess;
}

bool same_grid(const opf_mlp* m, const opf_ctx* c) {
    const opf_params& p = ctx_params(c);
    return p.N == m->N && p.M == m->M && p.K == m->K && p.mp == m->mp && p.alpha == m->alpha;
}

}  // namespace

extern "C" {

opf_status opf_mlp_default_config(opf_mlp_config* cfg) {
    if (!cfg) return OPF_E_INVALID;
    *cfg = opf_mlp_config{};
    cfg->width = 256;
    cfg->layers = 4;
    cfg->rank = 8;
    cfg->max_rows = 0;
    cfg->seed = 1;
    cfg->lr = 1e-3f;
    cfg->beta1 = 0.9f;
    cfg->beta2 = 0.999f;
    cfg->adam_eps = 1e-8f;
    cfg->lr_final = 1e-3f;
    return OPF_OK;
}

static void dims_for(opf_mlp* m, const opf_ctx* ctx, const opf_mlp_config* cfg) {
    const opf_params& p = ctx_params(ctx);
    m->N = p.N;
    m->M = p.M;
    m->K = p.K;
    m->nk = 2 * p.K - 1;
    m->mp = p.mp;
    m->alpha = p.alpha;
    m->H = cfg->width;
    m->L = cfg->layers;
    m->rank = cfg->rank;
    m->mode_rows = p.M * m->nk;
    m->R = round32(std::max(cfg->max_rows, m->mode_rows));
}

opf_status opf_mlp_workspace_size(const opf_ctx* ctx, const opf_mlp_config* cfg, size_t* bytes) {
    if (!bytes) return OPF_E_INVALID;
    const opf_status st = check_cfg(ctx, cfg, nullptr);
    if (st != OPF_OK) return st;
    opf_mlp m;
    dims_for(&m, ctx, cfg);
    *bytes = plan(&m).total;
    return OPF_OK;
}

opf_status opf_mlp_create(opf_ctx* ctx, const opf_mlp_config* cfg, void* dev_workspace, size_t bytes,
                          opf_mlp** out) {
    if (!out || !dev_workspace) return OPF_E_INVALID;
    *out = nullptr;
    std::string why;
    opf_status st = check_cfg(ctx, cfg, &why);
    if (st != OPF_OK) {
        if (ctx) ctx_set_error(ctx, why);
        return st;
    }
    if (reinterpret_cast<uintptr_t>(dev_workspace) % 256) return OPF_E_INVALID;
    opf_mlp* m = new (std::nothrow) opf_mlp;
    if (!m) return OPF_E_NOMEM;
    m->ctx = ctx;
    m->s = ctx_stream(ctx);
    dims_for(m, ctx, cfg);
    m->lr = cfg->lr;
    m->lr_final = cfg->lr_final;
    m->b1 = cfg->beta1;
    m->b2 = cfg->beta2;
    m->eps = cfg->adam_eps;
    const Layout lay = plan(m);
    if (bytes < lay.total) {
        delete m;
        return OPF_E_NOMEM;
    }
    unsigned char* b = static_cast<unsigned char*>(dev_workspace);
    int q = 0;
    auto at = [&](auto*& ptr) { ptr = reinterpret_cast<std::remove_reference_t<decltype(ptr)>>(b + lay.off[q++]); };
    at(m->P);
    at(m->G);
    at(m->Am);
    at(m->Av);
    at(m->Wb);
    at(m->Wt);
    at(m->Xb);
    at(m->XT);
    at(m->HL);
    at(m->HT);
    at(m->Z);
    at(m->Y);
    at(m->D);
    at(m->dYb);
    at(m->dYT);
    at(m->DT);
    at(m->fx);
    at(m->fac);
    at(m->idx);
    at(m->singular);
    at(m->part);
    at(m->gpart);
    at(m->lrow);
    at(m->wsum);
    at(m->losses);
    m->loss_cap = LOSS_CAP;
    const int rp = round32(m->mode_rows);
    hipLaunchKernelGGL(k_features, dim3((rp * NCOND + 255) / 256), dim3(256), 0, m->s, m->fx, m->mode_rows, rp, m->nk,
                       m->K, m->mp, m->alpha);
    if (hipGetLastError() != hipSuccess) {
        delete m;
        return OPF_E_HIP;
    }
    // initial weights: W ~ U(-a, a), a = 1/sqrt(fan_in) (output layer 0.01 a),
    // biases 0, from SplitMix64 (Steele, Lea & Flood 2014)
    std::vector<float> host(m->np, 0.0f);
    uint64_t state = cfg->seed;
    for (int j = 0; j < m->segs.n; ++j) {
        if (!m->segs.mat[j]) continue;
        const double a = (j == m->segs.n - 2 ? 0.01 : 1.0) / std::sqrt((double)m->segs.cols[j]);
        for (long i = m->segs.off[j]; i < m->segs.off[j + 1]; ++i) host[i] = (float)(a * (2.0 * uniform01(state) - 1.0));
    }
    st = opf_mlp_set_params(m, host.data(), m->np);
    if (st != OPF_OK) {
        ctx_set_error(ctx, m->err);
        delete m;
        return st;
    }
    *out = m;
    return OPF_OK;
}

opf_status opf_mlp_destroy(opf_mlp* net) {
    delete net;
    return OPF_OK;
}

opf_status opf_mlp_dims(const opf_mlp* net, int32_t* din, int32_t* dout, int64_t* n_params) {
    if (!net) return OPF_E_INVALID;
    if (din) *din = net->din;
    if (dout) *dout = net->dout;
    if (n_params) *n_params = net->np;
    return OPF_OK;
}

opf_status opf_mlp_set_params(opf_mlp* net, const float* host, int64_t n) {
    if (!net || !host || n != net->np) return OPF_E_INVALID;
    for (int64_t i = 0; i < n;) {
        // no exit per value, so that the test vectorises: the call takes
        // 0.48 ms for 2.64 M values, 0.88 with one
        const int64_t e = std::min<int64_t>(n, i + 4096);
        uint32_t bad = 0;
        for (; i < e; ++i) bad |= (__builtin_bit_cast(uint32_t, host[i]) & 0x7F800000u) == 0x7F800000u;
        if (bad) return OPF_E_INVALID;
    }
    MCHK(net, hipMemcpyAsync(net->P, host, (size_t)n * 4, hipMemcpyHostToDevice, net->s));
    MCHK(net, hipMemsetAsync(net->Am, 0, (size_t)n * 4, net->s));
    MCHK(net, hipMemsetAsync(net->Av, 0, (size_t)n * 4, net->s));
    hipLaunchKernelGGL(k_refresh, dim3(net->segs.blk[net->segs.n]), dim3(256), 0, net->s, net->P, net->segs,
                       net->Wb, net->Wt);
    MCHK(net, hipGetLastError());
    MCHK(net, hipStreamSynchronize(net->s));
    net->t = 0;
    net->fac_ok = false;
    return OPF_OK;
}

opf_status opf_mlp_get_params(opf_mlp* net, float* host, int64_t n) {
    if (!net || !host || n != net->np) return OPF_E_INVALID;
    MCHK(net, hipMemcpyAsync(host, net->P, (size_t)n * 4, hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));
    return OPF_OK;
}

opf_status opf_mlp_forward(opf_mlp* net, const float* x_dev, int32_t rows, float* y_dev) {
    if (!net || !x_dev || !y_dev || rows < 1 || rows > net->R) return OPF_E_INVALID;
    const int rp = round32(rows);
    MCHK(net, rows_bf16(net, x_dev, rows, rp, false));
    MCHK(net, forward(net, rp, false));
    MCHK(net, hipMemcpyAsync(y_dev, net->Y, (size_t)rows * net->dout * 4, hipMemcpyDeviceToDevice, net->s));
    return OPF_OK;
}

opf_status opf_mlp_gradient(opf_mlp* net, const float* x_dev, const float* t_dev, const float* w_dev, int32_t rows,
                            double* loss_host, float* grad_host) {
    if (!net || !x_dev || !t_dev || rows < 1 || rows > net->R) return OPF_E_INVALID;
    const int rp = round32(rows);
    MCHK(net, rows_bf16(net, x_dev, rows, rp, true));
    MCHK(net, forward(net, rp, true));
    GradArgs g;
    MCHK(net, backward_rows(net, t_dev, w_dev, rows, rp, net->losses, g));
    if (grad_host) MCHK(net, grad_sum(net, g));
    float l = 0.0f;
    MCHK(net, hipMemcpyAsync(&l, net->losses, 4, hipMemcpyDeviceToHost, net->s));
    if (grad_host) MCHK(net, hipMemcpyAsync(grad_host, net->G, (size_t)net->np * 4, hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));
    if (loss_host) *loss_host = l;
    return std::isfinite(l) ? OPF_OK : OPF_E_NUMERIC;
}

opf_status opf_mlp_train(opf_mlp* net, const float* x_dev, const float* t_dev, const float* w_dev, int32_t rows,
                         int32_t batch, int32_t epochs, uint64_t shuffle_seed, float* loss_host) {
    if (!net || !x_dev || !t_dev || rows < 1 || batch < 1 || batch > net->R || epochs < 0) return OPF_E_INVALID;
    const int nb = (rows + batch - 1) / batch;
    if ((long)nb * epochs > net->loss_cap) return OPF_E_INVALID;
    std::vector<int> order(nb);
    uint64_t state = shuffle_seed;
    int step = 0;
    for (int ep = 0; ep < epochs; ++ep) {
        for (int i = 0; i < nb; ++i) order[i] = i;
        for (int i = nb - 1; i > 0; --i) std::swap(order[i], order[(int)(uniform01(state) * (i + 1))]);
        for (int i = 0; i < nb; ++i) {
            const int r0 = order[i] * batch;
            const int n = std::min(batch, rows - r0);
            const int rp = round32(n);
            MCHK(net, rows_bf16(net, x_dev + (size_t)r0 * net->din, n, rp, true));
            MCHK(net, forward(net, rp, true));
            GradArgs g;
            MCHK(net, backward_rows(net, t_dev + (size_t)r0 * net->dout, w_dev ? w_dev + r0 : nullptr, n, rp,
                                    net->losses + step, g));
            MCHK(net, adam(net, g, net->lr));
            ++step;
        }
    }
    std::vector<float> l(step);
    if (step) MCHK(net, hipMemcpyAsync(l.data(), net->losses, (size_t)step * 4, hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));
    if (loss_host)
        for (int ep = 0; ep < epochs; ++ep) {
            double a = 0.0;
            for (int i = 0; i < nb; ++i) a += l[(size_t)ep * nb + i];
            loss_host[ep] = (float)(a / nb);
        }
    return OPF_OK;
}

opf_status opf_mlp_pair_gradient(opf_ctx* ctx, opf_mlp* net, const void* pairs_dev, int32_t npairs,
                                 const int32_t* idx_host, int32_t batch, double* loss_host, float* grad_host) {
    if (!ctx || !net || !pairs_dev || !idx_host || npairs < 1 || batch < 1 || batch > IDX_CAP) return OPF_E_INVALID;
    if (!same_grid(net, ctx)) return OPF_E_INVALID;
    for (int b = 0; b < batch; ++b)
        if (idx_host[b] < 0 || idx_host[b] >= npairs) return OPF_E_INVALID;
    MCHK(net, hipMemcpyAsync(net->idx, idx_host, (size_t)batch * 4, hipMemcpyHostToDevice, net->s));
    MCHK(net, feature_input(net));
    MCHK(net, forward(net, round32(net->mode_rows), true));
    GradArgs g;
    MCHK(net, backward_pairs(net, static_cast<const double*>(pairs_dev), net->idx, batch, net->losses, g));
    if (grad_host) MCHK(net, grad_sum(net, g));
    float l = 0.0f;
    MCHK(net, hipMemcpyAsync(&l, net->losses, 4, hipMemcpyDeviceToHost, net->s));
    if (grad_host) MCHK(net, hipMemcpyAsync(grad_host, net->G, (size_t)net->np * 4, hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));
    if (loss_host) *loss_host = l;
    return std::isfinite(l) ? OPF_OK : OPF_E_NUMERIC;
}

opf_status opf_mlp_train_pairs(opf_ctx* ctx, opf_mlp* net, const void* pairs_dev, int32_t npairs, int32_t batch,
                               int32_t steps, uint64_t seed, float* loss_host) {
    if (!ctx || !net || !pairs_dev || npairs < 1 || batch < 1 || steps < 0) return OPF_E_INVALID;
    if ((long)batch * steps > IDX_CAP || steps > net->loss_cap) return OPF_E_INVALID;
    if (!same_grid(net, ctx)) return OPF_E_INVALID;
    // pair indices of every step: consecutive batches of per-epoch shuffles
    std::vector<int> idx((size_t)batch * steps);
    std::vector<int> perm(npairs);
    uint64_t state = seed;
    size_t filled = 0;
    while (filled < idx.size()) {
        for (int i = 0; i < npairs; ++i) perm[i] = i;
        for (int i = npairs - 1; i > 0; --i) std::swap(perm[i], perm[(int)(uniform01(state) * (i + 1))]);
        for (int i = 0; i < npairs && filled < idx.size(); ++i) idx[filled++] = perm[i];
    }
    if (!idx.empty()) MCHK(net, hipMemcpyAsync(net->idx, idx.data(), idx.size() * 4, hipMemcpyHostToDevice, net->s));
    MCHK(net, feature_input(net));
    const int rp = round32(net->mode_rows);
    for (int st = 0; st < steps; ++st) {
        // cosine schedule from lr to lr_final over the call's steps
        const double c = 0.5 * (1.0 + std::cos(M_PI * st / std::max(steps, 1)));
        const float lr = (float)(net->lr_final + (net->lr - net->lr_final) * c);
        MCHK(net, forward(net, rp, true));
        GradArgs g;
        MCHK(net, backward_pairs(net, static_cast<const double*>(pairs_dev), net->idx + (size_t)st * batch, batch,
                                 net->losses + st, g));
        MCHK(net, adam(net, g, lr));
    }
    if (loss_host && steps > 0) MCHK(net, hipMemcpyAsync(loss_host, net->losses, (size_t)steps * 4,
                                                         hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));  // the host index array lives until here
    return OPF_OK;
}

opf_status opf_precondition(opf_ctx* ctx, opf_mlp* net, const void* v_dev, void* z_dev) {
    if (!ctx || !net || !v_dev || !z_dev) return OPF_E_INVALID;
    if (!same_grid(net, ctx)) return OPF_E_INVALID;
    MCHK(net, refresh_factors(net));
    hipLaunchKernelGGL(k_lowrank_apply, dim3((net->mode_rows + 3) / 4), dim3(256), 0, net->s, net->fac, net->dout,
                       net->rank, static_cast<const double*>(v_dev), static_cast<double*>(z_dev), net->N, net->M,
                       net->nk, net->K);
    MCHK(net, hipGetLastError());
    return OPF_OK;
}

opf_status opf_mlp_factors(opf_mlp* net, float* host, int64_t n, int32_t* singular_modes) {
    if (!net || (host && n != (int64_t)net->mode_rows * net->dout)) return OPF_E_INVALID;
    MCHK(net, refresh_factors(net));
    if (host) MCHK(net, hipMemcpyAsync(host, net->fac, (size_t)n * 4, hipMemcpyDeviceToHost, net->s));
    MCHK(net, hipStreamSynchronize(net->s));
    if (singular_modes) *singular_modes = net->n_singular;
    return OPF_OK;
}

const char* opf_mlp_last_error(const opf_mlp* net) { return net ? net->err.c_str() : "null network"; }

}  // extern "C"
