// k_sketch.hip -- the data-driven sketch basis V_r of the index (Sec. 4.2,
// the index entry: the rank-r sketch of the content uses V_r drawn from the
// context's own prefix queries).
//
// V_r spans the dominant r-dimensional eigenspace of the prefix content
// queries' second moment C = sum_i q_i q_i^T (512 x 512).  The index score
// (V_r^T q).(V_r^T c) = q^T V_r V_r^T c and the residual norm
// ||(I - V_r V_r^T) c|| depend on the subspace only, so any orthonormal basis
// of it serves; the basis is found by subspace (orthogonal) iteration:
//   V_0 = orth(C R) with R a fixed +-1 pattern, V_{t+1} = orth(C V_t),
// orth = Cholesky QR (W = V L^T with L L^T = W^T W), all fp64.  The rounds
// before the last need a well-conditioned basis of the same nested spans, which
// one Cholesky QR gives (its loss of orthogonality, cond^2 2^-53, only enters
// the condition number of the next round's columns); the last round applies it
// twice, so the result is orthonormal to rounding.  Measured against an
// extended-precision iteration, one pass per round and two differ from it by
// the same 1e-13 (4096 queries near 48 dimensions, r = 64).
// The error shrinks as (lambda_{r+1} / lambda_r)^t.  The basis is handed to
// vkv_digest_build as P = RNE_bf16(s V_r^T), s = 1 - 2^-6, which keeps the
// rounded basis contractive (checked there).  Not on the per-step path: it is
// part of the compression event.
//
// What bounds it: a chain of small dependent launches (20 products and 10
// factorisations at r = 64 and 8 iterations), each of a few microseconds of
// latency; the arithmetic (1.5 GFLOP fp64 at 4096 queries, r = 64) is 22 us of
// the fp64 matrix cores.  Every product runs on v_mfma_f64_16x16x4f64.  Measured
// there: 8.41 -> 0.54 ms a call (second moment 728 -> 59 us, a product 44 -> 6,
// a factorisation with its inversion or elimination 310 -> 32, and 10 instead
// of 18 of them).
#include "vkv_internal.h"

namespace vkv {

constexpr double SK_SCALE = 1.0 - 0x1p-6;
constexpr int SK_PANEL = 64;    // columns factored at a time

// C = sum_i q_i q_i^T over the m queries (bf16 products exact in fp64).  Block
// (ta <= tb) owns the 32 x 32 tile of C and its mirror image as 16 x 16 pieces,
// two waves to a piece (the halves of each chunk's queries, added at the end):
// 136 blocks x 4 SIMDs run m / 4 matrix steps each, 27 us at m = 4096, the
// floor of this form.  Chunks of 64 queries are widened to fp64 once into a
// two-stage LDS buffer while the other stage is multiplied (the chunk after it
// already loading); rows of 80 doubles give the operand reads' four k-slots
// distinct banks.
constexpr int CV_T = 32, CV_K = 64, CV_LD = 80;

__global__ __launch_bounds__(512) void cov_kernel(const uint16_t* q, int64_t m, double* C) {
    __shared__ __align__(16) double s_q[2][CV_K * CV_LD];   // [i][a columns 0..31, b columns 32..63]
    int tb = 0, ta = blockIdx.x;
    while (ta > tb) ta -= ++tb;   // block id -> (ta <= tb)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wa = (wave >> 1) & 1, wb = wave & 1, half = wave >> 2;
    // loader: two columns of rows tid / 32 + 16 e
    const int lc = 2 * (tid & 31), li = tid >> 5;
    const uint16_t* src = q + (lc < CV_T ? ta * CV_T + lc : tb * CV_T + lc - CV_T);
    uint32_t v[4];
    auto load = [&](int64_t i0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t i = i0 + li + 16 * e;
            v[e] = (i < m) ? *reinterpret_cast<const uint32_t*>(src + i * D_LAT) : 0u;
        }
    };
    auto store = [&](int st) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            *reinterpret_cast<double2*>(&s_q[st][(li + 16 * e) * CV_LD + lc]) =
                make_double2(bf16_bits_f64((uint16_t)v[e]), bf16_bits_f64((uint16_t)(v[e] >> 16)));
    };
    const int oa = (32 * half + (lane >> 4)) * CV_LD + 16 * wa + (lane & 15);
    const int ob = (32 * half + (lane >> 4)) * CV_LD + CV_T + 16 * wb + (lane & 15);
    f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
    load(0);
    store(0);
    load(CV_K);
    __syncthreads();
    int st = 0;
    for (int64_t i0 = 0; i0 < m; i0 += CV_K, st ^= 1) {
        store(st ^ 1);          // the next chunk (zeros past the last)
        load(i0 + 2 * CV_K);
        const double* pa = s_q[st] + oa;
        const double* pb = s_q[st] + ob;
#pragma unroll
        for (int s = 0; s < CV_K / 8; ++s)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[4 * s * CV_LD], pb[4 * s * CV_LD], acc, 0, 0, 0);
        __syncthreads();
    }
    f64x4_t* s_red = reinterpret_cast<f64x4_t*>(s_q);   // the first halves' pieces, [piece][lane]
    if (half) s_red[(wave & 3) * 64 + lane] = acc;
    __syncthreads();
    if (half) return;
    acc += s_red[wave * 64 + lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int a = ta * CV_T + 16 * wa + 4 * e + (lane >> 4), b = tb * CV_T + 16 * wb + (lane & 15);
        C[(int64_t)a * D_LAT + b] = acc[e];
        C[(int64_t)b * D_LAT + a] = acc[e];   // (the diagonal tiles write each entry twice, the same sum)
    }
}

__global__ __launch_bounds__(64) void sk_zero_kernel(int* p) {
    if (threadIdx.x == 0) p[0] = 0;
}

// The fixed +-1 start pattern R[i][j]: the top bit of MurmurHash3's 32-bit
// finaliser (fmix32) of i * 512 + j plus a constant.  (A hash whose low bits
// are weakly mixed gives a pattern of low rank; this one is well conditioned.)
__device__ __forceinline__ double start_pattern(int i, int j) {
    uint32_t h = (uint32_t)(i * D_LAT + j) + 0x5BD1E995u;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return (h >> 31) ? 1.0 : -1.0;
}

// Out[a][c] (-)= sum_k A(a, k) B(k, c), A(a, k) = A[a*s0 + k*s1], B(k, c) =
// B[k*s0 + c*s1] (nullptr: the start pattern); fp64, row-major Out of ldo
// columns, K = 16 NST.  Block (ta, tc) owns a 16 x 16 tile; its four waves take
// a quarter of K each with all their loads in flight together, so a 512-deep
// product is one memory round trip and a chain of 32 matrix steps (1 us); the
// quarters are added in a fixed order.
struct Mat {
    const double* p;
    int64_t s0, s1;
};

template <int NST, bool SUB>
__global__ __launch_bounds__(256) void sk_gemm_kernel(Mat A, Mat B, double* Out, int64_t ldo) {
    __shared__ f64x4_t s_red[3][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = 16 * blockIdx.x + (lane & 15), col = 16 * blockIdx.y + (lane & 15);
    const int k0 = 4 * NST * wave + (lane >> 4);
    double va[NST], vb[NST];
#pragma unroll
    for (int s = 0; s < NST; ++s) {
        const int k = k0 + 4 * s;
        va[s] = A.p[row * A.s0 + k * A.s1];
        vb[s] = B.p ? B.p[k * B.s0 + col * B.s1] : start_pattern(k, col);
    }
    f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < NST; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[s], vb[s], acc, 0, 0, 0);
    if (wave > 0) s_red[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w) acc += s_red[w][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double* o = Out + (int64_t)(16 * blockIdx.x + 4 * e + (lane >> 4)) * ldo + col;
        *o = SUB ? *o - acc[e] : acc[e];
    }
}

// ||column||^2 of Y [512 x r]: the original diagonal the pivots are held against
__global__ __launch_bounds__(64) void sk_colnorm_kernel(const double* Y, int r, double* d0) {
    double s = 0.0;
    for (int i = threadIdx.x; i < D_LAT; i += 64) {
        const double y = Y[(int64_t)i * r + blockIdx.x];
        s = fma(y, y, s);
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x == 0) d0[blockIdx.x] = s;
}

// One panel of W columns: X = Y L^{-T} with L L^T = G = Y^T Y, without forming
// L or its inverse: the elimination that turns G's columns into L^T's turns
// the rows of Y, taken as further columns, into those of X.  Wave 0's lane c
// holds column c of G, wave 1's lane l holds row 64 blk + l of Y.  A step takes
// two rows j, j + 1 of G, broadcast through LDS (double-buffered, one barrier a
// step): with d0, d1 their pivots, f0 = a0 / d0 and f1 = (a1 - u0[1] f0) / d1 a
// column loses u0 (f0 - (u0[1] / d0) f1) + u1 f1.  The arrays shift by two, so
// the pivot rows are always entries 0 and 1 and no register is indexed
// dynamically (entries past the last row hold leftovers that no valid row ever
// reads).  The 8 blocks repeat G's elimination rather than exchange it.  A pivot
// that is not finite or not above SK_PIV_REL times its column's original squared
// norm sets *bad: the columns are numerically dependent (Cholesky QR needs the
// condition number of the columns below about 1e7).  Bound by the latency of
// W / 2 dependent steps (LDS round trip, two reciprocals, barrier); the entries
// shrink in four phases of W / 8 steps, which also keeps the code small.
constexpr double SK_PIV_REL = 1e-15;

__device__ __forceinline__ void sk_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// 1 / d by two Newton steps on the hardware's estimate (d normal, as the pivots are)
__device__ __forceinline__ double recip(double d) {
    double x = __builtin_amdgcn_rcp(d);
    x = fma(fma(-d, x, 1.0), x, x);
    return fma(fma(-d, x, 1.0), x, x);
}

template <int N, int STEPS, int W>
__device__ __forceinline__ void orth_phase(double (&a)[W], double (*s_row)[2][SK_PANEL], const double* s_d0, int& j,
                                           int wave, int lane, double* s_x, double* s_piv, int* s_bad) {
#pragma unroll 1
    for (int e = 0; e < STEPS; ++e, j += 2) {
        const double* u0 = s_row[(j >> 1) & 1][0];   // rows j and j + 1 from column j on
        const double* u1 = s_row[(j >> 1) & 1][1];
        double d0 = u0[0];
        const double u01 = u0[1];
        bool bad = !(d0 > SK_PIV_REL * s_d0[j]) || !(d0 < INFINITY);
        d0 = bad ? 1.0 : d0;
        const double r0 = recip(d0), g = u01 * r0;
        double d1 = fma(-g, u01, u1[1]);
        const bool bad1 = !(d1 > SK_PIV_REL * s_d0[j + 1]) || !(d1 < INFINITY);
        d1 = bad1 ? 1.0 : d1;
        const double x0 = a[0], f0 = x0 * r0;
        const double x1 = fma(-u01, f0, a[1]), f1 = x1 * recip(d1);
        const double h0 = fma(-g, f1, f0);
        a[0] = fma(-u1[2], f1, fma(-u0[2], h0, a[2]));
        a[1] = fma(-u1[3], f1, fma(-u0[3], h0, a[3]));
        if (wave == 0 && lane > j + 1) {   // rows j + 2 and j + 3 for the next step
            s_row[((j >> 1) + 1) & 1][0][lane - j - 2] = a[0];
            s_row[((j >> 1) + 1) & 1][1][lane - j - 2] = a[1];
        }
#pragma unroll
        for (int i = 2; i < N - 2; ++i) a[i] = fma(-u1[i + 2], f1, fma(-u0[i + 2], h0, a[i + 2]));
        if (wave == 1) {
            s_x[j] = x0;
            s_x[j + 1] = x1;
        }
        if (lane == 0) {
            s_piv[j] = d0;
            s_piv[j + 1] = d1;
            if (bad || bad1) *s_bad = 1;
        }
        sk_lds_barrier();
    }
}

template <int W>
__global__ __launch_bounds__(128) void sk_orth_kernel(const double* G, const double* Y, const double* d0, double* X,
                                                      int64_t ld, int* bad) {
    constexpr int XLD = W + 1;
    __shared__ double s_row[2][2][SK_PANEL];
    __shared__ double s_d0[W], s_piv[2][W];
    __shared__ double s_x[64 * XLD];   // the block's rows of Y, then of X before their scaling
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * 64;
    if (tid == 0) s_bad = 0;
    double a[W];
    const int c = min(lane, W - 1);
    if (wave == 0) {
#pragma unroll
        for (int i = 0; i < W; ++i) a[i] = G[i * W + c];
        s_row[0][0][lane] = a[0];
        s_row[0][1][lane] = a[1];
        s_row[1][0][lane] = s_row[1][1][lane] = 0.0;
        if (lane < W) s_d0[lane] = d0 ? d0[lane] : G[lane * W + lane];
    }
    for (int p = tid; p < 64 * W; p += 128) s_x[(p / W) * XLD + p % W] = Y[(row0 + p / W) * ld + p % W];
    __syncthreads();
    if (wave == 1) {
#pragma unroll
        for (int i = 0; i < W; ++i) a[i] = s_x[lane * XLD + i];
    }
    sk_lds_barrier();
    double* xr = s_x + lane * XLD;
    double* pv = s_piv[wave];   // (both waves compute the pivots; each keeps its own copy)
    int j = 0;
    orth_phase<W, W / 8, W>(a, s_row, s_d0, j, wave, lane, xr, pv, &s_bad);
    orth_phase<3 * W / 4, W / 8, W>(a, s_row, s_d0, j, wave, lane, xr, pv, &s_bad);
    orth_phase<W / 2, W / 8, W>(a, s_row, s_d0, j, wave, lane, xr, pv, &s_bad);
    orth_phase<W / 4, W / 8, W>(a, s_row, s_d0, j, wave, lane, xr, pv, &s_bad);
    if (wave == 0 && lane < W) s_d0[lane] = 1.0 / sqrt(s_piv[0][lane]);
    __syncthreads();
    for (int p = tid; p < 64 * W; p += 128) X[(row0 + p / W) * ld + p % W] = s_x[(p / W) * XLD + p % W] * s_d0[p % W];
    if (tid == 0 && s_bad && blockIdx.x == 0) *bad = 1;
}

// P[j][i] = RNE_bf16(s V[i][j]); quot[j] = v_j^T (C v_j) (the Rayleigh quotient
// of column j) with CV = C V, unless CV is null.  Block j.
__global__ __launch_bounds__(256) void basis_out_kernel(const double* V, const double* CV, int r, uint16_t* P,
                                                        double* quot) {
    __shared__ double s_red[4];
    const int j = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    for (int i = tid; i < D_LAT; i += 256) {
        const double v = V[(int64_t)i * r + j];
        P[(int64_t)j * D_LAT + i] = f64_to_bf16_rne(SK_SCALE * v);
        if (CV) s = fma(v, CV[(int64_t)i * r + j], s);
    }
    if (!CV) return;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((tid & 63) == 0) s_red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) quot[j] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

// energy[0] = sum_j quot[j] = trace(V^T C V), energy[1] = trace(C)
__global__ __launch_bounds__(64) void energy_kernel(const double* quot, const double* C, int r, double* energy) {
    double e0 = 0.0, e1 = 0.0;
    for (int j = threadIdx.x; j < r; j += 64) e0 += quot[j];
    for (int a = threadIdx.x; a < D_LAT; a += 64) e1 += C[(int64_t)a * D_LAT + a];
    for (int o = 32; o > 0; o >>= 1) {
        e0 += __shfl_xor(e0, o);
        e1 += __shfl_xor(e1, o);
    }
    if (threadIdx.x == 0) {
        energy[0] = e0;
        energy[1] = e1;
    }
}

size_t sketch_workspace_bytes(int r) {
    return (size_t)D_LAT * D_LAT * 8 + 2 * (size_t)D_LAT * r * 8 + 2 * (size_t)r * r * 8 + 256;
}

// M x N tiles of 16 x 16; K is 512, or a whole panel's columns where the product is subtracted
template <bool SUB>
static hipError_t gemm(Mat A, Mat B, int M, int N, double* Out, int64_t ldo, hipStream_t s) {
    constexpr int NST = (SUB ? SK_PANEL : D_LAT) / 16;
    hipLaunchKernelGGL((sk_gemm_kernel<NST, SUB>), dim3((unsigned)(M / 16), (unsigned)(N / 16)), dim3(256), 0, s, A, B, Out,
                       ldo);
    return hipGetLastError();
}

hipError_t launch_sketch(const uint16_t* q, int64_t m, int r, int iters, void* ws, uint16_t* P, double* energy,
                         hipStream_t s) {
    double* C = reinterpret_cast<double*>(ws);
    double* X = C + (size_t)D_LAT * D_LAT;     // the basis (512 x r)
    double* Y = X + (size_t)D_LAT * r;         // its image / the second orthonormalisation
    double* G = Y + (size_t)D_LAT * r;         // a panel's Gram matrix, then its products with the later columns
    double* D0 = G + (size_t)r * r;            // the columns' original squared norms; the quotients at the end
    int* bad = reinterpret_cast<int*>(D0 + (size_t)r * r);
    hipLaunchKernelGGL(sk_zero_kernel, dim3(1), dim3(64), 0, s, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr unsigned NT = D_LAT / CV_T;
    hipLaunchKernelGGL(cov_kernel, dim3(NT * (NT + 1) / 2), dim3(512), 0, s, q, m, C);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // orth(src -> dst), src overwritten: panels of 64 columns (the last one of
    // 32 where r is an odd multiple of 32), each by Cholesky QR and then
    // projected out of the columns after it (with one panel: Cholesky QR)
    auto orth = [&](double* src, double* dst) -> hipError_t {
        const double* d0 = nullptr;
        hipError_t e2;
        if (r > SK_PANEL) {
            d0 = D0;
            hipLaunchKernelGGL(sk_colnorm_kernel, dim3((unsigned)r), dim3(64), 0, s, src, r, D0);
            if ((e2 = hipGetLastError()) != hipSuccess) return e2;
        }
        for (int p = 0; p < r; p += SK_PANEL) {
            const int w = r - p < SK_PANEL ? r - p : SK_PANEL, rest = r - p - w;
            double* Yp = src + p;
            if ((e2 = gemm<false>(Mat{Yp, 1, r}, Mat{Yp, r, 1}, w, w, G, w, s)) != hipSuccess) return e2;
            const double* dp = d0 ? d0 + p : nullptr;
            if (w == SK_PANEL)
                hipLaunchKernelGGL(sk_orth_kernel<SK_PANEL>, dim3(D_LAT / 64), dim3(128), 0, s, G, Yp, dp, dst + p,
                                   (int64_t)r, bad);
            else
                hipLaunchKernelGGL(sk_orth_kernel<SK_PANEL / 2>, dim3(D_LAT / 64), dim3(128), 0, s, G, Yp, dp, dst + p,
                                   (int64_t)r, bad);
            if ((e2 = hipGetLastError()) != hipSuccess) return e2;
            if (rest == 0) break;
            // T = X_p^T Y_rest, Y_rest -= X_p T
            const double* Xp = dst + p;
            if ((e2 = gemm<false>(Mat{Xp, 1, r}, Mat{Yp + w, r, 1}, w, rest, G, rest, s)) != hipSuccess) return e2;
            if ((e2 = gemm<true>(Mat{Xp, r, 1}, Mat{G, rest, 1}, D_LAT, rest, Yp + w, r, s)) != hipSuccess) return e2;
        }
        return hipSuccess;
    };
    for (int t = 0; t <= iters; ++t) {
        // Y = C X (the start pattern on the first round), then X = orth(Y)
        if ((e = gemm<false>(Mat{C, D_LAT, 1}, Mat{t == 0 ? nullptr : X, r, 1}, D_LAT, r, Y, r, s)) != hipSuccess)
            return e;
        if ((e = orth(Y, X)) != hipSuccess) return e;
    }
    if ((e = orth(X, Y)) != hipSuccess) return e;   // the second pass: the basis is in Y
    if (energy && (e = gemm<false>(Mat{C, D_LAT, 1}, Mat{Y, r, 1}, D_LAT, r, X, r, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(basis_out_kernel, dim3((unsigned)r), dim3(256), 0, s, Y, energy ? X : nullptr, r, P, D0);
    if ((e = hipGetLastError()) != hipSuccess || !energy) return e;
    hipLaunchKernelGGL(energy_kernel, dim3(1), dim3(64), 0, s, D0, C, r, energy);
    return hipGetLastError();
}

}  // namespace vkv
