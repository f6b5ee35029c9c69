// k_sigma.hip -- the query-independent tier-1 selector sigma_u (Sec. 4.1, the
// sigma equation; App. H, block close) and the tier it keeps.
//
// Per closed block of 4096 rows and per channel of the 64-dim branch r_u as
// the cache row stores it (its last 64 elements), sigma keeps the
// frequency bins [0, kappa) of the sequence-axis DFT (and their mirrors),
// inverts, and takes the norm over the channels of what that low-pass
// reconstruction misses at each row.
//
// sigma_fft_kernel: one workgroup per (8-channel group, block, sequence).  Two
// real channels travel as one complex sequence z = x + i y (the mask keeps
// f and N - f together, so masking z masks x and y alike).  The 4096-point
// transform runs in LDS in place as six radix-4 decimation-in-frequency
// stages (natural order in, base-4 digit-reversed order out); the mask is
// applied in that order; the inverse is the adjoint of the same stages taken
// in reverse (digit-reversed in, natural out), which gives N times the
// inverse transform with no permutation pass.  fp64 throughout; twiddles
// come from a quarter-wave cosine table.  The squared residuals of the
// group's 8 channels are summed per row and stored; sigma_reduce_kernel adds
// the 8 groups in order and takes the square root.
//
// sigma_lowpass_kernel: the same for the small kappa that the tier uses, the
// transform in registers and only its kept bins formed.
//
// sigma_select_kernel: one workgroup per sequence.  The tier is the first
// nsink rows plus the top-m of the other closed rows by (sigma desc, row asc):
// the m-th key over the fp64 bit patterns (sigma >= 0, so the bits order like
// the values), then one ordered pass writes the rows above it and the first
// rows equal to it, ascending.
//
// Also here: the flags of a caller's tier (for the step on a given kept set)
// and the all-layer CSR pack of row lists (offsets by one block's prefix sum,
// then one copy per list).
#include <type_traits>

#include "vkv_internal.h"

namespace vkv {

constexpr int SG_N = 4096;                 // rows per closed block
constexpr int SG_Q4 = SG_N / 4;            // quarter wave
constexpr int SG_THREADS = 256;
constexpr int SG_ROWS = SG_N / SG_THREADS; // rows per thread in the residual pass
constexpr int SG_GROUPS = 8;               // 8-channel groups of the 64-dim branch
constexpr size_t SG_LDS = (size_t)SG_N * sizeof(double2) + (size_t)(SG_Q4 + 1) * sizeof(double);

// exp(-2 pi i k / N) for k in [0, N), from ct[j] = cos(2 pi j / N), j in [0, N/4]
__device__ __forceinline__ double2 sg_twiddle(const double* ct, int k) {
    const int q = k >> 10, r = k & (SG_Q4 - 1);
    double c, s;
    if (q == 0) {
        c = ct[r];
        s = ct[SG_Q4 - r];
    } else if (q == 1) {
        c = -ct[SG_Q4 - r];
        s = ct[r];
    } else if (q == 2) {
        c = -ct[r];
        s = -ct[SG_Q4 - r];
    } else {
        c = ct[SG_Q4 - r];
        s = -ct[r];
    }
    return make_double2(c, -s);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {   // a * conj(b)
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// base-4 digit reversal of a 12-bit index (six digits)
__device__ __forceinline__ int rev4(int p) {
    int f = 0;
#pragma unroll
    for (int d = 0; d < 6; ++d) f = (f << 2) | ((p >> (2 * d)) & 3);
    return f;
}

// Stage st of the forward transform (in place): groups of 4Q = N / 4^st, the
// butterfly (a, b, c, d) at quarter offsets, twiddles w^i, w^2i, w^3i with
// w = exp(-2 pi i / 4Q).
__device__ __forceinline__ void dif_stage(double2* X, const double* ct, int st, int tid) {
    const int lq = 10 - 2 * st;            // log2 Q
    const int Q = 1 << lq;
#pragma unroll
    for (int m = 0; m < SG_N / 4 / SG_THREADS; ++m) {
        const int j = tid + SG_THREADS * m;
        const int i = j & (Q - 1);
        const int i0 = ((j >> lq) << (lq + 2)) + i;
        const double2 a = X[i0], b = X[i0 + Q], c = X[i0 + 2 * Q], d = X[i0 + 3 * Q];
        const double2 apc = cadd(a, c), amc = csub(a, c), bpd = cadd(b, d), bmd = csub(b, d);
        const int k = i << (2 * st);
        X[i0] = cadd(apc, bpd);
        X[i0 + Q] = cmul(make_double2(amc.x + bmd.y, amc.y - bmd.x), sg_twiddle(ct, k));
        X[i0 + 2 * Q] = cmul(csub(apc, bpd), sg_twiddle(ct, 2 * k));
        X[i0 + 3 * Q] = cmul(make_double2(amc.x - bmd.y, amc.y + bmd.x), sg_twiddle(ct, 3 * k));
    }
}

// The adjoint of dif_stage: conjugate twiddles first, then the conjugate butterfly.
__device__ __forceinline__ void dit_adjoint_stage(double2* X, const double* ct, int st, int tid) {
    const int lq = 10 - 2 * st;
    const int Q = 1 << lq;
#pragma unroll
    for (int m = 0; m < SG_N / 4 / SG_THREADS; ++m) {
        const int j = tid + SG_THREADS * m;
        const int i = j & (Q - 1);
        const int i0 = ((j >> lq) << (lq + 2)) + i;
        const int k = i << (2 * st);
        const double2 A = X[i0];
        const double2 B = cmulc(X[i0 + Q], sg_twiddle(ct, k));
        const double2 C = cmulc(X[i0 + 2 * Q], sg_twiddle(ct, 2 * k));
        const double2 D = cmulc(X[i0 + 3 * Q], sg_twiddle(ct, 3 * k));
        const double2 apc = cadd(A, C), amc = csub(A, C), bpd = cadd(B, D), bmd = csub(B, D);
        X[i0] = cadd(apc, bpd);
        X[i0 + Q] = make_double2(amc.x - bmd.y, amc.y + bmd.x);
        X[i0 + 2 * Q] = csub(apc, bpd);
        X[i0 + 3 * Q] = make_double2(amc.x + bmd.y, amc.y - bmd.x);
    }
}

__global__ __launch_bounds__(SG_THREADS) void sigma_fft_kernel(SigmaArgs a) {
    extern __shared__ __align__(16) uint8_t sg_lds[];
    double2* X = reinterpret_cast<double2*>(sg_lds);
    double* ct = reinterpret_cast<double*>(sg_lds + (size_t)SG_N * sizeof(double2));
    const int grp = blockIdx.x, blk = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    for (int j = tid; j <= SG_Q4; j += SG_THREADS)
        ct[j] = (j == 0) ? 1.0 : (j == SG_Q4 ? 0.0 : cospi((double)j / (double)(SG_N / 2)));
    const uint16_t* base = a.cache + (int64_t)b * a.cbs + (a.t0 + (int64_t)blk * SG_N) * a.crs + D_LAT + 8 * grp;
    double acc[SG_ROWS];
#pragma unroll
    for (int m = 0; m < SG_ROWS; ++m) acc[m] = 0.0;
    for (int pair = 0; pair < 4; ++pair) {
        float xv[SG_ROWS], yv[SG_ROWS];
#pragma unroll
        for (int m = 0; m < SG_ROWS; ++m) {
            const int t = tid + SG_THREADS * m;
            const uint32_t w = *reinterpret_cast<const uint32_t*>(base + (int64_t)t * a.crs + 2 * pair);
            xv[m] = __uint_as_float(w << 16);
            yv[m] = __uint_as_float(w & 0xFFFF0000u);
            X[t] = make_double2((double)xv[m], (double)yv[m]);
        }
        __syncthreads();
        for (int st = 0; st < 6; ++st) {
            dif_stage(X, ct, st, tid);
            __syncthreads();
        }
        // keep bins f < kappa and f > N - kappa (position p holds bin rev4(p))
        for (int p = tid; p < SG_N; p += SG_THREADS) {
            const int f = rev4(p);
            if (f >= a.kappa && f <= SG_N - a.kappa) X[p] = make_double2(0.0, 0.0);
        }
        __syncthreads();
        for (int st = 5; st >= 0; --st) {
            dit_adjoint_stage(X, ct, st, tid);
            __syncthreads();
        }
        constexpr double inv_n = 1.0 / SG_N;
#pragma unroll
        for (int m = 0; m < SG_ROWS; ++m) {
            const int t = tid + SG_THREADS * m;
            const double2 l = X[t];
            const double dx = (double)xv[m] - l.x * inv_n, dy = (double)yv[m] - l.y * inv_n;
            acc[m] += dx * dx + dy * dy;
        }
        __syncthreads();
    }
    double* out = a.part + (((int64_t)b * a.nblk + blk) * SG_GROUPS + grp) * SG_N;
#pragma unroll
    for (int m = 0; m < SG_ROWS; ++m) out[tid + SG_THREADS * m] = acc[m];
}

// The same for kappa <= SG_KLOW, the kept bins of the tier's own settings (16
// and 64): the transform in three radix-16 passes held in registers, of which
// only the kept bins' part is formed.  With t = 256 t2 + 16 t1 + t0 and
// f = f0 + 16 f1 + 256 f2, w = exp(-2 pi i / 4096):
//   A[f0; t1 t0] = w^((16 t1 + t0) f0) sum_t2 x[t] w16^(t2 f0)   thread (t1, t0)
//   B[f0 f1; t0] = sum_t1 A[f0; t1 t0] w16^(t1 f1)               thread (f0, t0)
//   X[f]         = sum_t0 B[f0 f1; t0] w256^(t0 (f1 + 16 f2))    over 16 lanes
// The bins f < 64 have f2 = 0, f1 < 4, the bins f > N - 64 have f2 = 15,
// f1 >= 12: eight values of f1, each with one f2, so a thread forms 8 of its 16
// B's, the last pass is a 16-lane sum per B, and the inverse runs back the same
// way from the same registers.  A and its inverse are the only exchanges
// through LDS, each written to and read from the thread's own places on one
// side, so two barriers serve a pair of channels (24 LDS passes and barriers in
// the stage-by-stage form above).  The rows' 8 bytes of two pairs are read at
// once.  The 8 channel groups of a block share its cache lines, so they go to
// one XCD (consecutive workgroup ids go round the 8 XCDs).
// Bound by fp64 issue (about 1400 vector instructions per thread and pair) and
// the strided 8-byte row reads.  Measured at 8 x 32 blocks of rows: 836 -> 165 us.
constexpr int SG_KLOW = 64;
constexpr int64_t SG_KLOW_STRIDE = 1 << 22;   // row stride (elements) whose lane offsets fit 32 bits
constexpr size_t SG_KLOW_LDS = SG_LDS + 128 * sizeof(double2);

template <bool INV>
__device__ __forceinline__ double2 mul_i(double2 a) {   // a * -i (forward w4) or a * i
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// four-point transform in place: (a, b, c, d) -> outputs 0..3
template <bool INV>
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
    const double2 apc = cadd(a, c), amc = csub(a, c), bpd = cadd(b, d), bmd = mul_i<INV>(csub(b, d));
    a = cadd(apc, bpd);
    b = cadd(amc, bmd);
    c = csub(apc, bpd);
    d = csub(amc, bmd);
}

// a * w16^k (forward) or a * w16^-k, k = 0..9 with k = b c, b, c < 4
template <bool INV, int K>
__device__ __forceinline__ double2 mul_w16(double2 a) {
    constexpr double C1 = 0.92387953251128675613, S1 = 0.38268343236508977173, R = 0.70710678118654752440;
    if constexpr (K == 0) return a;
    if constexpr (K == 4) return mul_i<INV>(a);
    if constexpr (K == 2) return INV ? make_double2(R * (a.x - a.y), R * (a.x + a.y)) : make_double2(R * (a.x + a.y), R * (a.y - a.x));
    if constexpr (K == 6) return mul_i<INV>(mul_w16<INV, 2>(a));
    if constexpr (K == 1 || K == 3 || K == 9) {
        constexpr double c = K == 1 ? C1 : (K == 3 ? S1 : -C1), s = K == 1 ? S1 : (K == 3 ? C1 : -S1);
        return INV ? cmulc(a, make_double2(c, -s)) : cmul(a, make_double2(c, -s));
    }
    return a;
}

// x[4 a + b] -> first layer over a, the twiddles w16^(b c): x[4 c + b]
template <bool INV>
__device__ __forceinline__ void dft16_columns(double2 (&x)[16]) {
#pragma unroll
    for (int b = 0; b < 4; ++b) dft4<INV>(x[b], x[4 + b], x[8 + b], x[12 + b]);
}
template <bool INV>
__device__ __forceinline__ void dft16_twiddles(double2 (&x)[16]) {
    x[5] = mul_w16<INV, 1>(x[5]);
    x[6] = mul_w16<INV, 2>(x[6]);
    x[7] = mul_w16<INV, 3>(x[7]);
    x[9] = mul_w16<INV, 2>(x[9]);
    x[10] = mul_w16<INV, 4>(x[10]);
    x[11] = mul_w16<INV, 6>(x[11]);
    x[13] = mul_w16<INV, 3>(x[13]);
    x[14] = mul_w16<INV, 6>(x[14]);
    x[15] = mul_w16<INV, 9>(x[15]);
}

// sum over the 16 lanes of each row of the wave, in all of them
__device__ __forceinline__ double rowsum16_f64(double v) {
    auto perm = [](double x, auto ctrl) __attribute__((always_inline)) {
        const uint64_t u = d2u(x);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, decltype(ctrl)::value, 0xF, 0xF, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), decltype(ctrl)::value, 0xF, 0xF, true);
        return u2d(((uint64_t)hi << 32) | lo);
    };
    v += perm(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
    v += perm(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
    v += perm(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
    v += perm(v, std::integral_constant<int, 0x140>{});   // row_mirror
    return v;
}

__global__ __launch_bounds__(SG_THREADS, 2) void sigma_lowpass_kernel(SigmaArgs a) {
    extern __shared__ __align__(16) uint8_t sg_lds[];
    double2* X = reinterpret_cast<double2*>(sg_lds);                             // [f0][16 t1 + t0]
    double2* ph = X + SG_N;   // [8][16] phases of the last pass: w256^(t0 (f1 + 16 f2)), f1 + 16 f2 = c, 252 + c
    double* ct = reinterpret_cast<double*>(ph + 128);
    // workgroup id -> (block of rows, channel group): 8 consecutive ids on one
    // XCD (ids 8 apart) are the 8 groups of one block
    const int64_t id = blockIdx.x, idx = id >> 3, job = (idx >> 3) * 8 + (id & 7);
    const int grp = (int)(idx & 7);
    if (job >= (int64_t)a.nblk * a.B) return;
    const int blk = (int)(job % a.nblk), b = (int)(job / a.nblk), tid = threadIdx.x;
    for (int j = tid; j <= SG_Q4; j += SG_THREADS)
        ct[j] = (j == 0) ? 1.0 : (j == SG_Q4 ? 0.0 : cospi((double)j / (double)(SG_N / 2)));
    // uniform base, one 32-bit lane offset: the 16 row addresses cost no registers
    const uint8_t* base = reinterpret_cast<const uint8_t*>(a.cache + (int64_t)b * a.cbs +
                                                           (a.t0 + (int64_t)blk * SG_N) * a.crs + D_LAT + 8 * grp);
    const uint32_t rowb = (uint32_t)(2 * a.crs), lane_off = (uint32_t)tid * rowb;
    const int f0 = tid >> 4, t0 = tid & 15;
    double acc[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) acc[m] = 0.0;
    __syncthreads();
    if (tid < 128) {
        const int c = tid >> 4;
        ph[tid] = sg_twiddle(ct, (16 * (tid & 15) * (c < 4 ? c : 248 + c)) & (SG_N - 1));
    }
    // w^(tid f), f = c + 4 d, as a product of two (all 15 do not fit the registers)
    double2 w1[4], w4[4];
#pragma unroll
    for (int f = 1; f < 4; ++f) {
        w1[f] = sg_twiddle(ct, tid * f);
        w4[f] = sg_twiddle(ct, tid * 4 * f);
    }
    auto tw = [&](int c, int d) __attribute__((always_inline)) {
        return c == 0 ? w4[d] : (d == 0 ? w1[c] : cmul(w1[c], w4[d]));
    };
    // (an opaque copy per use: the compiler would otherwise keep the 9 products,
    // and below the 16 row addresses, across the loop in scratch memory)
    auto hide = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int f = 1; f < 4; ++f) asm volatile("" : "+v"(w1[f].x), "+v"(w1[f].y), "+v"(w4[f].x), "+v"(w4[f].y));
    };
    // one pair of channels, the rows' values in w (bf16 bits, two a word)
    auto one_pair = [&](const uint32_t (&w)[16]) __attribute__((always_inline)) {
        double2 x[16];
        auto input = [&](int m) __attribute__((always_inline)) {
            return make_double2((double)__uint_as_float(w[m] << 16), (double)__uint_as_float(w[m] & 0xFFFF0000u));
        };
#pragma unroll
        for (int m = 0; m < 16; ++m) x[m] = input(m);
        dft16_columns<false>(x);
        dft16_twiddles<false>(x);
        hide();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            dft4<false>(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
#pragma unroll
            for (int d = 0; d < 4; ++d) {   // output f = c + 4 d
                const int f = c + 4 * d;
                X[SG_THREADS * f + tid] = f ? cmul(x[4 * c + d], tw(c, d)) : x[4 * c + d];
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 16; ++m) x[m] = X[SG_THREADS * f0 + 16 * m + t0];
        dft16_columns<false>(x);
        dft16_twiddles<false>(x);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // outputs f1 = c (d = 0) and f1 = 12 + c (d = 3: w4^(3b) = i^b)
            const double2 u = cadd(x[4 * c], x[4 * c + 2]), v = cadd(x[4 * c + 1], x[4 * c + 3]);
            const double2 p = csub(x[4 * c], x[4 * c + 2]), q = csub(x[4 * c + 1], x[4 * c + 3]);
            double2 lo = cadd(u, v), hi = make_double2(p.x - q.y, p.y + q.x);
            // X[f] for f = f0 + 16 c and f = 4096 - 64 + 16 c + f0
            const double2 wl = ph[16 * c + t0], wh = ph[16 * (4 + c) + t0];
            lo = cmul(lo, wl);
            hi = cmul(hi, wh);
            lo = make_double2(rowsum16_f64(lo.x), rowsum16_f64(lo.y));
            hi = make_double2(rowsum16_f64(hi.x), rowsum16_f64(hi.y));
            const double kl = (f0 + 16 * c < a.kappa) ? 1.0 : 0.0;
            const double kh = (SG_N - 64 + 16 * c + f0 > SG_N - a.kappa) ? 1.0 : 0.0;
            lo = cmulc(kl != 0.0 ? lo : make_double2(0.0, 0.0), wl);
            hi = cmulc(kh != 0.0 ? hi : make_double2(0.0, 0.0), wh);
            // the inverse's layer over d: w4^(-3 b) = (-i)^b
            x[4 * c] = cadd(lo, hi);
            x[4 * c + 1] = make_double2(lo.x + hi.y, lo.y - hi.x);
            x[4 * c + 2] = csub(lo, hi);
            x[4 * c + 3] = make_double2(lo.x - hi.y, lo.y + hi.x);
        }
        dft16_twiddles<true>(x);
        dft16_columns<true>(x);   // over c: x[4 a + b]
#pragma unroll
        for (int m = 0; m < 16; ++m) X[SG_THREADS * f0 + 16 * m + t0] = x[m];
        __syncthreads();
        hide();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int f = c + 4 * d;
                const double2 v = X[SG_THREADS * f + tid];
                x[4 * c + d] = f ? cmulc(v, tw(c, d)) : v;
            }
            dft4<true>(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
        }
        dft16_twiddles<true>(x);
        dft16_columns<true>(x);
        constexpr double inv_n = 1.0 / SG_N;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const double2 v = input(m);
            const double dx = fma(-inv_n, x[m].x, v.x), dy = fma(-inv_n, x[m].y, v.y);
            acc[m] = fma(dx, dx, fma(dy, dy, acc[m]));
        }
    };
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        uint32_t lo[16], hi[16], off = lane_off;
        const uint8_t* rows = base + 8 * half;
#pragma unroll
        for (int m = 0; m < 16; ++m, rows += (uint64_t)SG_THREADS * rowb) {
            asm volatile("" : "+s"(rows), "+v"(off));
            const uint2 v = *reinterpret_cast<const uint2*>(rows + off);
            lo[m] = v.x;
            hi[m] = v.y;
        }
        one_pair(lo);
        one_pair(hi);
    }
    double* out = a.part + (((int64_t)b * a.nblk + blk) * SG_GROUPS + grp) * SG_N;
#pragma unroll
    for (int m = 0; m < 16; ++m) out[tid + SG_THREADS * m] = acc[m];
}

__global__ __launch_bounds__(256) void sigma_reduce_kernel(SigmaArgs a) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;   // row within the closed range
    const int b = blockIdx.y;
    if (e >= (int64_t)a.nblk * SG_N) return;
    const int64_t blk = e / SG_N, t = e % SG_N;
    const double* p = a.part + ((int64_t)b * a.nblk + blk) * SG_GROUPS * SG_N + t;
    double s = 0.0;
#pragma unroll
    for (int g = 0; g < SG_GROUPS; ++g) s += p[(int64_t)g * SG_N];
    a.sigma[(int64_t)b * a.sstride + a.t0 + e] = sqrt(s);
}

size_t sigma_workspace_bytes(int64_t B, int64_t nblk) { return (size_t)(B * nblk) * SG_GROUPS * SG_N * sizeof(double); }

hipError_t launch_sigma(const SigmaArgs& a, hipStream_t s) {
    if (a.nblk == 0 || a.B == 0) return hipSuccess;
    const int64_t jobs = (a.nblk * a.B + 7) / 8 * 8 * SG_GROUPS;
    if (a.kappa <= SG_KLOW && a.crs <= SG_KLOW_STRIDE && jobs <= INT32_MAX) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&sigma_lowpass_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)SG_KLOW_LDS);
        hipLaunchKernelGGL(sigma_lowpass_kernel, dim3((unsigned)jobs), dim3(SG_THREADS), SG_KLOW_LDS, s, a);
    } else {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&sigma_fft_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)SG_LDS);
        hipLaunchKernelGGL(sigma_fft_kernel, dim3(SG_GROUPS, (unsigned)a.nblk, (unsigned)a.B), dim3(SG_THREADS),
                           SG_LDS, s, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t rows = (int64_t)a.nblk * SG_N;
    hipLaunchKernelGGL(sigma_reduce_kernel, dim3((unsigned)((rows + 255) / 256), (unsigned)a.B), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------ the sigma tier

constexpr int SS_THREADS = 1024;
constexpr int SS_WAVES = SS_THREADS / 64;
constexpr int SS_PER = 8;              // keys per thread and round, all loads in flight
constexpr int SS_LIST = 12288;         // keys near the threshold held in LDS
constexpr int SS_SAMPLE = 2048;        // keys sampled to place the bracket around it
constexpr int SS_BINS = 2048;          // bins of the sample's histogram
constexpr int SS_WORDS = 2048;         // 64-row mask words of an output segment (131072 rows)

// What bounds it: one workgroup reads its sequence's keys twice, so the time is
// that of 2 x 8 n bytes through one CU plus a few barriers (there is no scratch
// buffer through which workgroups could share a sequence).  A sample brackets
// the take-th key; the first pass counts the keys above the bracket and lists
// those inside it in LDS, where a radix select finds the threshold; the second
// writes the rows above it, and the first rows equal to it, in order: 64-row
// masks of a segment go to LDS, one scan over their counts places every word.
// A bracket that misses or a list that overflows (ties, adversarial orders)
// falls back to radix passes over all keys.  Measured at 8 x 131072 keys,
// m = 4092: 473 -> 78 us (nine passes of one load per thread and round before);
// the first pass, through a cold cache, takes about half of it.

// exclusive prefix over the threads of (lo, hi) halves of a 64-bit pair, and the totals
__device__ __forceinline__ uint64_t ss_scan(uint64_t v, uint64_t* s_w, uint64_t& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t t = __shfl_up((unsigned long long)incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    uint64_t before = 0, tot = 0;
    for (int i = 0; i < SS_WAVES; ++i) {
        const uint64_t c = s_w[i];
        before += i < w ? c : 0;
        tot += c;
    }
    __syncthreads();
    total = tot;
    return before + incl - v;
}

// in wave 0: the digit d of a 256-bin histogram where the count of entries in
// digits >= d first reaches `need`, and the count above it
__device__ __forceinline__ void ss_pick(const uint32_t* hist, int64_t need, int* s_d, int64_t* s_above) {
    const int lane = threadIdx.x & 63;
    uint32_t h[4], loc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) loc += h[j] = hist[4 * lane + j];
    uint32_t suf = loc;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_down(suf, o);
        if (lane + o < 64) suf += t;
    }
    int64_t run = suf - loc;
    if (run < need && need <= (int64_t)suf) {
#pragma unroll
        for (int j = 3; j >= 0; --j) {
            if (run < need && need <= run + (int64_t)h[j]) {
                *s_d = 4 * lane + j;
                *s_above = run;
            }
            run += h[j];
        }
    }
}

// the need-th largest of the `cnt` keys of key[0 .. cnt) that agree with
// `prefix` on the bits of `mask`, digit by digit from `shift` down; need becomes
// the rank among the keys equal to the result
template <typename Get>
__device__ __forceinline__ uint64_t ss_radix(Get key, int64_t cnt, uint64_t prefix, uint64_t mask, int shift,
                                             int64_t& need, uint32_t* hist, int* s_d, int64_t* s_above, uint64_t* s_key) {
    const int tid = threadIdx.x;
    for (;; shift -= 8) {
        const int sh = shift < 0 ? 0 : shift;   // the last digit may overlap bits already fixed
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int64_t i = tid; i < cnt; i += SS_THREADS) {
            const uint64_t k = key(i);
            if ((k & mask) == prefix) atomicAdd(&hist[(k >> sh) & 255u], 1u);
        }
        __syncthreads();
        if (tid < 64) ss_pick(hist, need, s_d, s_above);
        __syncthreads();
        prefix |= (uint64_t)*s_d << sh;
        mask |= 255ull << sh;
        need -= *s_above;
        const bool single = hist[*s_d] == 1;
        if (sh == 0) return prefix;
        if (single) {   // one key left: its other digits are read off
            for (int64_t i = tid; i < cnt; i += SS_THREADS) {
                const uint64_t k = key(i);
                if ((k & mask) == prefix) *s_key = k;
            }
            __syncthreads();
            return *s_key;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(SS_THREADS) void sigma_select_kernel(SigmaSelArgs a) {
    __shared__ __align__(16) uint64_t s_list[SS_LIST];   // then the segment's masks
    __shared__ uint32_t s_h[SS_BINS];
    __shared__ uint64_t s_w[SS_WAVES];
    __shared__ uint64_t s_br[2];
    __shared__ double s_mm[2][SS_WAVES];
    __shared__ uint32_t s_cnt[2];                        // keys above the bracket, keys inside it
    __shared__ int s_d;
    __shared__ int64_t s_above;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t* key = reinterpret_cast<const uint64_t*>(a.sigma + (int64_t)b * a.sstride);
    int32_t* out = a.kept + (int64_t)b * a.kstride;
    const int64_t lo = a.n < a.nsink ? a.n : a.nsink;
    const int64_t navail = a.n - lo;
    const int64_t take = a.m < navail ? a.m : navail;
    const bool all = take == navail;
    // the take-th largest key among rows [lo, n) and the rank `need` among its equals
    uint64_t thr = 0;
    int64_t need = take;
    if (take > 0 && !all) {
        const uint64_t* ka = key + lo;
        uint64_t blo = 0, bhi = ~0ull;   // the bracket (inclusive bits)
        if (tid < 2) s_cnt[tid] = 0;
        if (navail > SS_LIST) {
            // SS_SAMPLE keys at even spacing, in a linear histogram of their range
            uint64_t sk[2];
            double mn = INFINITY, mx = -INFINITY;
            const int64_t stride = navail / SS_SAMPLE;
#pragma unroll
            for (int j = 0; j < 2; ++j) sk[j] = ka[(int64_t)(tid + SS_THREADS * j) * stride];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                mn = fmin(mn, u2d(sk[j]));
                mx = fmax(mx, u2d(sk[j]));
            }
            for (int o = 32; o > 0; o >>= 1) {
                mn = fmin(mn, __shfl_xor(mn, o));
                mx = fmax(mx, __shfl_xor(mx, o));
            }
            if (lane == 0) {
                s_mm[0][wave] = mn;
                s_mm[1][wave] = mx;
            }
            for (int i = tid; i < SS_BINS; i += SS_THREADS) s_h[i] = 0;
            __syncthreads();
            for (int w = 0; w < SS_WAVES; ++w) {
                mn = fmin(mn, s_mm[0][w]);
                mx = fmax(mx, s_mm[1][w]);
            }
            const double range = mx - mn;
            const double sc = (range > 0.0 && range < INFINITY) ? (double)SS_BINS / range : 0.0;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const double t = (u2d(sk[j]) - mn) * sc;
                const int bin = t > 0.0 ? (t < (double)SS_BINS ? (int)t : SS_BINS - 1) : 0;
                atomicAdd(&s_h[bin], 1u);
            }
            if (tid == 0) {
                s_br[0] = 0;
                s_br[1] = ~0ull;
            }
            __syncthreads();
            // sample ranks k_s -+ (4 sqrt(k_s) + 16) around the threshold's
            const double ks = (double)take * SS_SAMPLE / (double)navail, dl = 4.0 * sqrt(ks) + 16.0;
            const int64_t c_hi = (int64_t)floor(ks - dl), c_lo = (int64_t)ceil(ks + dl);
            const uint32_t h0 = s_h[2 * tid], h1 = s_h[2 * tid + 1];
            uint64_t tot;
            const int64_t below = (int64_t)ss_scan(h0 + h1, s_w, tot);
            const int64_t suf1 = (int64_t)tot - below - h0, suf0 = (int64_t)tot - below;   // in bins >= 2 tid + 1, >= 2 tid
            auto edge = [&](int bin) { return mn + (double)bin / sc; };
            if (sc > 0.0 && mn >= 0.0) {
                // upper end: the bin where the count from the top reaches c_hi; lower end likewise c_lo
                const int64_t suf2 = suf1 - h1;
                if (c_hi >= 1) {
                    if (suf2 < c_hi && c_hi <= suf1) s_br[1] = d2u(edge(2 * tid + 2));
                    if (suf1 < c_hi && c_hi <= suf0) s_br[1] = d2u(edge(2 * tid + 1));
                }
                if (c_lo <= SS_SAMPLE) {
                    if (suf2 < c_lo && c_lo <= suf1) s_br[0] = d2u(edge(2 * tid + 1));
                    if (suf1 < c_lo && c_lo <= suf0) s_br[0] = d2u(edge(2 * tid));
                }
            }
            __syncthreads();
            blo = s_br[0];
            bhi = s_br[1];
        } else {
            __syncthreads();
        }
        // count the keys above the bracket, list those inside it
        uint32_t nab = 0;
        // (the next round's keys load while this one's are sorted out; one
        // list append per wave and round)
        constexpr int64_t ROUND = (int64_t)SS_THREADS * SS_PER;
        uint64_t k[SS_PER];
        auto load = [&](int64_t u0) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) k[j] = ka[min(u0 + tid + (int64_t)SS_THREADS * j, navail - 1)];
        };
        load(0);
        for (int64_t u0 = 0; u0 < navail; u0 += ROUND) {
            uint64_t c[SS_PER];
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) c[j] = k[j];
            if (u0 + ROUND < navail) load(u0 + ROUND);
            uint64_t bal[SS_PER];
            uint32_t found = 0;
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) {
                const bool live = u0 + tid + (int64_t)SS_THREADS * j < navail;
                nab += live && c[j] > bhi;
                bal[j] = __ballot(live && c[j] >= blo && c[j] <= bhi);
                found += __popcll(bal[j]);
            }
            if (found == 0) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&s_cnt[1], found);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) {
                const uint32_t p = at + __popcll(bal[j] & ((1ull << lane) - 1ull));
                if (((bal[j] >> lane) & 1) && p < SS_LIST) s_list[p] = c[j];
                at += __popcll(bal[j]);
            }
        }
        for (int o = 32; o > 0; o >>= 1) nab += __shfl_xor(nab, o);
        if (lane == 0 && nab) atomicAdd(&s_cnt[0], nab);
        __syncthreads();
        const int64_t above = s_cnt[0], inside = s_cnt[1];
        if (inside <= SS_LIST && above < take && take <= above + inside) {
            need = take - above;
            // the digits start at the first bit in which the bracket's ends differ
            const uint64_t diff = blo ^ bhi;
            const int top = diff ? 63 - __clzll((long long)diff) : 0;
            const int shift = top < 7 ? 0 : top - 7;
            const uint64_t mask = shift + 8 >= 64 ? 0ull : ~0ull << (shift + 8);
            thr = ss_radix([&](int64_t i) { return s_list[i]; }, inside, blo & mask, mask, shift, need, s_h, &s_d,
                           &s_above, &s_br[0]);
        } else {
            thr = ss_radix([&](int64_t i) { return ka[i]; }, navail, 0ull, 0ull, 56, need, s_h, &s_d, &s_above,
                           &s_br[0]);
        }
    }
    // ordered output: sinks, keys above the threshold, and the first `need` rows equal to it
    uint64_t* s_gt = s_list;               // per 64 rows: rows certainly in
    uint64_t* s_eq = s_list + SS_WORDS;    // rows equal to the threshold
    int64_t base = 0, eq_seen = 0;
    constexpr int64_t SEG = 64ll * SS_WORDS;
    __syncthreads();
    for (int64_t g0 = 0; g0 < a.n; g0 += SEG) {
        const int nw = (int)((min(a.n - g0, SEG) + 63) / 64);
        uint64_t k[SS_PER];
        auto load = [&](int w0) __attribute__((always_inline)) {
            if (take == 0 || all) return;   // no key decides
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) k[j] = key[min(g0 + (int64_t)64 * (w0 + SS_WAVES * j) + lane, a.n - 1)];
        };
        load(wave);
        for (int w0 = wave; w0 < nw; w0 += SS_WAVES * SS_PER) {
            uint64_t c[SS_PER];
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) c[j] = k[j];
            if (w0 + SS_WAVES * SS_PER < nw) load(w0 + SS_WAVES * SS_PER);
#pragma unroll
            for (int j = 0; j < SS_PER; ++j) {
                const int w = w0 + SS_WAVES * j;
                const int64_t u = g0 + 64ll * w + lane;
                const bool cand = u >= lo && u < a.n && take > 0;
                const bool in = u < a.n && (u < lo || (cand && (all || c[j] > thr)));
                const uint64_t gt = __ballot(in), eq = __ballot(cand && !all && c[j] == thr);
                if (w < nw && lane == 0) {
                    s_gt[w] = gt;
                    s_eq[w] = eq;
                }
            }
        }
        __syncthreads();
        // words 2 tid and 2 tid + 1: rows in, and equal rows, before them
        uint64_t cnt = 0;
        uint64_t gt[2], eq[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int w = 2 * tid + j;
            gt[j] = w < nw ? s_gt[w] : 0;
            eq[j] = w < nw ? s_eq[w] : 0;
            cnt += (uint64_t)__popcll(gt[j]) | ((uint64_t)__popcll(eq[j]) << 32);
        }
        uint64_t tot;
        const uint64_t before = ss_scan(cnt, s_w, tot);
        int64_t ng = (int64_t)(before & 0xFFFFFFFFull), ne = eq_seen + (int64_t)(before >> 32);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint64_t bits = gt[j] | eq[j];
            int64_t pos = base + ng + min(ne, need) - min(eq_seen, need);
            const int64_t u0 = g0 + 64ll * (2 * tid + j);
            while (bits) {
                const int e = __ffsll((unsigned long long)bits) - 1;
                bits &= bits - 1;
                if ((gt[j] >> e) & 1) {
                    out[pos++] = (int32_t)(u0 + e);
                } else if (ne++ < need) {
                    out[pos++] = (int32_t)(u0 + e);
                }
            }
            ng += __popcll(gt[j]);
            ne = eq_seen + (int64_t)(before >> 32) + __popcll(eq[0]);   // before word 2 tid + 1
        }
        const int64_t eq_after = eq_seen + (int64_t)(tot >> 32);
        base += (int64_t)(tot & 0xFFFFFFFFull) + min(eq_after, need) - min(eq_seen, need);
        eq_seen = eq_after;
        __syncthreads();
    }
}

hipError_t launch_sigma_select(const SigmaSelArgs& a, hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    hipLaunchKernelGGL(sigma_select_kernel, dim3((unsigned)a.B), dim3(SS_THREADS), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------ a caller's tier into the flags

// flags[b][u] = 1 for the k rows of sel[b] inside [0, A), 0 for the other rows
// The per-row tier flags of a kept table (ascending rows in [0, A)), in one
// pass: block (c, b) owns rows [4096 c, 4096 (c + 1)) of sequence b, clears
// their flags, finds the table's entries inside its range by two searches of
// the ascending list, and marks them.  No block depends on another's writes.
constexpr int TF_ROWS = 4096;

// first position i of the ascending list ks[0, k) with ks[i] >= v (k if none),
// by one wave: each round probes 64 evenly spaced positions and keeps the
// interval between the last probe below v and the first one at or above it
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t* ks, int64_t k, int64_t v, int lane) {
    int64_t lo = 0, hi = k;   // the answer lies in [lo, hi]
    while (hi - lo > 64) {
        const int64_t step = (hi - lo + 63) / 64;
        const int64_t p = lo + (int64_t)lane * step;
        const bool below = p < hi && (int64_t)ks[p] < v;
        const int cnt = __popcll(__ballot(below));   // the probes below v are a prefix of the lanes
        const int64_t nlo = cnt == 0 ? lo : lo + (int64_t)(cnt - 1) * step + 1;
        hi = min(hi, lo + (int64_t)cnt * step);
        lo = nlo;
    }
    const int64_t p = lo + lane;
    const bool below = p < hi && (int64_t)ks[p] < v;
    return lo + __popcll(__ballot(below));
}

__global__ __launch_bounds__(256) void tier_flags_kernel(uint8_t* flags, int64_t fstride, int64_t A, const int32_t* sel,
                                                         int64_t k) {
    __shared__ int64_t s_range[2];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t u0 = (int64_t)blockIdx.x * TF_ROWS, u1 = min(A, u0 + TF_ROWS);
    uint8_t* fb = flags + (int64_t)b * fstride;
    const int32_t* ks = sel + (int64_t)b * k;
    for (int64_t u = u0 + tid; u < u1; u += 256) fb[u] = 0;
    if (wave < 2) {   // wave 0: the first entry >= u0, wave 1: the first entry >= u1
        const int64_t pos = wave_lower_bound(ks, k, wave == 0 ? u0 : u1, lane);
        if (lane == 0) s_range[wave] = pos;
    }
    __syncthreads();   // the clears are done before any mark, and the range is known
    for (int64_t i = s_range[0] + tid; i < s_range[1]; i += 256) {
        const int32_t u = ks[i];
        if (u >= u0 && u < u1) fb[u] = 1;
    }
}

hipError_t launch_mark_tier(uint8_t* flags, int64_t fstride, int64_t A, int B, const int32_t* sel, int64_t k,
                            hipStream_t s) {
    if (B == 0 || A == 0) return hipSuccess;
    const unsigned g = (unsigned)((A + TF_ROWS - 1) / TF_ROWS);
    hipLaunchKernelGGL(tier_flags_kernel, dim3(g, (unsigned)B), dim3(256), 0, s, flags, fstride, A, sel, k);
    return hipGetLastError();
}

}  // namespace vkv

namespace vkv {

// ------------------------------------------------ all-layer CSR pack of row lists

// offsets[i] = sum_{j < i} min(max(counts[j], 0), cap), i in [0, n]; one block, 1024 threads
__global__ __launch_bounds__(1024) void pack_offsets_kernel(const int32_t* counts, int64_t n, int64_t cap,
                                                            int32_t* offsets) {
    __shared__ int64_t s_part[1024];
    const int tid = threadIdx.x;
    const int64_t per = (n + 1023) / 1024;
    const int64_t i0 = tid * per, i1 = min(n, i0 + per);
    int64_t s = 0;
    for (int64_t i = i0; i < i1; ++i) {
        const int64_t c = counts[i];
        s += c < 0 ? 0 : (c < cap ? c : cap);
    }
    s_part[tid] = s;
    __syncthreads();
    int64_t base = 0;
    for (int j = 0; j < tid; ++j) base += s_part[j];
    for (int64_t i = i0; i < i1; ++i) {
        offsets[i] = (int32_t)base;
        const int64_t c = counts[i];
        base += c < 0 ? 0 : (c < cap ? c : cap);
    }
    if (tid == 1023) offsets[n] = (int32_t)base;
}

__global__ __launch_bounds__(256) void pack_copy_kernel(const int32_t* lists, const int32_t* offsets, int64_t cap,
                                                        int32_t* packed) {
    const int64_t i = blockIdx.y;
    const int64_t len = offsets[i + 1] - offsets[i];
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < len; t += (int64_t)gridDim.x * 256)
        packed[offsets[i] + t] = lists[i * cap + t];
}

hipError_t launch_pack_rows(const int32_t* lists, const int32_t* counts, int64_t n, int64_t cap, int32_t* offsets,
                            int32_t* packed, hipStream_t s) {
    hipLaunchKernelGGL(pack_offsets_kernel, dim3(1), dim3(1024), 0, s, counts, n, cap, offsets);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n == 0 || cap == 0) return e;
    const unsigned gx = (unsigned)((cap + 255) / 256 < 64 ? (cap + 255) / 256 : 64);
    hipLaunchKernelGGL(pack_copy_kernel, dim3(gx, (unsigned)n), dim3(256), 0, s, lists, offsets, cap, packed);
    return hipGetLastError();
}

}  // namespace vkv
