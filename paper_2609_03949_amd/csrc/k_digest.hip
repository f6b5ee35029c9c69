// k_digest.hip -- index build (the compression event's tier-2 index, Sec. 4.2).
//
// Archived row u keeps (r_u, P c_u, eta_u); with the stored sketch rounded to
// bf16 the certificate needs two more row scalars (eps_u, gamma_u).  For each
// row: y_j = sum_i P[j,i] c_u[i] in fp64 with i ascending, d_j = RNE_bf16(y_j)
// in one rounding, then the upper bounds
//   eta_u >= sqrt(c^T (I - P^T P) c),  eps_u >= ||d - P c||,  gamma_u >= ||P c||
// evaluated in a fixed fp64 order and rounded toward +inf.  Not on the
// per-step path.
//
// The projection runs on the fp64 matrix cores: v_mfma_f64_16x16x4f64 adds its
// 4 products (k = 0..3) to the accumulator one after another, each with a
// single rounding, so 128 of them with i ascending give the sequential fp64
// sum bit for bit (bf16 products are exact in fp64).
//
// Bound by the matrix steps (72 cycles each on a SIMD, 66 TFLOP/s measured for a
// large product), as long as little else takes issue slots and the fp64 pipe:
// widening an operand costs both.  So a block keeps its 64 basis rows widened in
// registers, and each cache row is widened once, by the wave that loads it, into
// an LDS tile from which four waves read fp64 operands.  Two waves share a SIMD,
// each with half of the 512 dimensions: wave w takes steps 0..63 of tile t while
// wave w + 4 takes steps 64..127 of tile t - 1, continuing the accumulators w
// handed over through LDS, so one wave's side work runs under the other's matrix
// steps (128 doubles per lane in one wave spill to accumulation registers, and
// every copy back costs issue slots: 98 cycles a step).  Waves 0-3 do their side
// work (widening, ||c||^2) before their steps, waves 4-7 (digests, tail sums)
// after theirs.  The certificate's sums are sequential too: ||c||^2 runs as one
// lane per row over the 16 tiles of a 256-row group, ||y||^2 and ||d - y||^2 of
// a tile as 32 lanes of one wave, the waves in turn.  Measured at 16 x 32768 rows,
// r = 64, with the certificate: 2176 -> 793 us (43 TFLOP/s; the matrix cores are
// busy 58% of it); without its sums 730.
#include <algorithm>

#include "vkv_internal.h"

namespace vkv {

constexpr int DG_THREADS = 512;    // waves 0-3: dims 0..255, waves 4-7: dims 256..511, 16 basis rows each
constexpr int DG_CHUNK = 64;       // basis rows per pass over the block's rows
constexpr int DG_GROUP = 256;      // rows whose ||c||^2 are formed together: one per thread of waves 0-3
constexpr int DG_GTILES = DG_GROUP / 16;
constexpr int DG_MAX_GROUPS = 4;   // groups per block (one where the basis takes several chunks)
// Half a tile (16 rows, 256 dims) in LDS: element i = 4 s + k of row m at
// m DG_RS + 512 k + 8 s bytes, so the operand of step s (lane 16 k + m) and that
// of step s + 1 are one 16-byte read, eight rows of which fall into distinct banks
constexpr int DG_RS = 2048 + 16;
constexpr int DG_HALF = 16 * DG_RS;
constexpr int DG_YLD = DG_CHUNK + 1;
constexpr int DG_HAND = 4 * 64 * 4;     // doubles handed over per tile: [basis tile][lane][4]
constexpr size_t DG_LDS = 4 * DG_HALF + (DG_HAND + 2 * 16 * DG_YLD + 3 * DG_GROUP) * sizeof(double);
static_assert(DG_LDS <= 160 * 1024, "the CU's LDS");

// workgroup barrier for exchanges through LDS (global loads stay in flight)
__device__ __forceinline__ void dg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// the certificate scalars of row o of [B][T] from ||c||^2, ||y||^2 and ||d - y||^2
__device__ __forceinline__ void cert_scalars(const DigestArgs& a, int64_t o, double Nc, double Ny, double Ne) {
    const double G = CERT_G;
    const double Dm = G * (double)ru_sqrt_f32((double)a.r * Nc);
    const double sy = (double)ru_sqrt_f32(Ny);
    const double X = ((Nc - Ny) + G * (Nc + Ny)) + (2.0 * Dm) * sy;
    a.eta[o] = ru_sqrt_f32((X > 0.0 ? X : 0.0) * (1.0 + G));
    a.eps[o] = ru_f32((double)ru_sqrt_f32(Ne) * (1.0 + G) + Dm);
    a.gam[o] = ru_f32(sy * (1.0 + G) + Dm);
}

__global__ __launch_bounds__(DG_THREADS, 2) void digest_kernel(DigestArgs a, int rows) {
    extern __shared__ __align__(16) uint8_t dg_lds[];
    double* s_hand = reinterpret_cast<double*>(dg_lds + 4 * DG_HALF);
    double* s_y = s_hand + DG_HAND;                // [2][16][DG_YLD]: y, RNE(y) - y
    double* s_acc = s_y + 2 * 16 * DG_YLD;         // [256][2]: running ||y||^2, ||d - y||^2 of the group's rows
    double* s_nc = s_acc + 2 * DG_GROUP;           // [256]: ||c||^2
    const int b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave >> 2, jw = wave & 3;
    const int64_t u0 = (int64_t)blockIdx.x * rows;
    const int nrows = (int)min((int64_t)rows, a.T - u0);
    if (nrows <= 0) return;
    const int ntile = (nrows + 15) / 16;
    const uint16_t* cb = a.cache + (int64_t)b * a.cbs + u0 * a.cs;
    uint16_t* ib = a.index ? a.index + (int64_t)b * a.ibs + u0 * a.is : nullptr;
    const int off = a.with_rope ? D_ROPE : 0;
    const bool cert = a.eta != nullptr;
    const int nchunk = (a.r + DG_CHUNK - 1) / DG_CHUNK;   // (r > 0)
    uint8_t* s_t = dg_lds + half * 2 * DG_HALF;    // this half's two buffers

    // loader: wave jw of a half moves its dims of tile rows 4 jw .. 4 jw + 3, two
    // rows per load (rows past the end re-read the last one; nothing of them is stored)
    u16x8_t nx[2];
    auto load_rows = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int rr = min(16 * t + 4 * jw + 2 * e + (lane >> 5), nrows - 1);
            nx[e] = *reinterpret_cast<const u16x8_t*>(cb + (int64_t)rr * a.cs + 256 * half + 8 * (lane & 31));
        }
    };
    auto widen_rows = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            uint8_t* dst = s_t + (t & 1) * DG_HALF + (4 * jw + 2 * e + (lane >> 5)) * DG_RS + 16 * (lane & 31);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<double2*>(dst + 512 * k) =
                    make_double2(bf16_bits_f64(nx[e][k]), bf16_bits_f64(nx[e][4 + k]));
        }
    };
    // ||c||^2 (waves 0-3) of row 64 jw + lane of the current group: 32 elements
    // per tile, i ascending, loaded a tile ahead
    double nc = 0.0;
    u16x8_t cv[4];
    const uint16_t* crow = cb;
    auto nc_load = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) cv[e] = *reinterpret_cast<const u16x8_t*>(crow + 32 * i + 8 * e);
    };
    auto nc_row = [&](int grp) __attribute__((always_inline)) {
        const int rr = min(DG_GROUP * grp + 64 * jw + lane, nrows - 1);
        crow = cb + (int64_t)rr * a.cs;
        nc = 0.0;
        nc_load(0);
    };
    auto nc_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const double x = bf16_bits_f64(cv[e >> 3][e & 7]);
            nc = fma(x, x, nc);
        }
    };
    // sums of tile t (waves 4-7): lane 16 q + row continues sum q & 1 of its row over the chunk's j
    const double* ty = s_y + (kq & 1) * 16 * DG_YLD + m * DG_YLD;
    auto tail_sums = [&](int t, int ch) __attribute__((always_inline)) {
        double* slot = s_acc + (16 * (t % DG_GTILES) + m) * 2 + (kq & 1);
        double tail = ch > 0 ? *slot : 0.0;
#pragma unroll
        for (int j8 = 0; j8 < DG_CHUNK; j8 += 16) {
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = ty[j8 + e];
#pragma unroll
            for (int e = 0; e < 16; ++e) tail = fma(v[e], v[e], tail);
        }
        *slot = tail;   // (two lane pairs write the same value)
    };
    auto scalars = [&](int grp) __attribute__((always_inline)) {
        const int rr = DG_GROUP * grp + tid;
        if (tid >= DG_GROUP || rr >= nrows) return;
        cert_scalars(a, (int64_t)b * a.T + u0 + rr, s_nc[tid], s_acc[2 * tid], s_acc[2 * tid + 1]);
    };

    for (int ch = 0; ch < nchunk; ++ch) {
        const int j0 = ch * DG_CHUNK;
        const int jn = min(DG_CHUNK, a.r - j0);
        // (a wave without a basis tile multiplies zeros and contributes zeros)
        const bool active = 16 * jw < jn;
        const bool nc_on = cert && ch == 0 && half == 0;
        // basis row j0 + 16 jw + m: elements 4 s + kq of this half's 64 steps
        double P[64];
        if (active) {
            const uint16_t* pr = a.P + (int64_t)(j0 + 16 * jw + m) * D_LAT + 256 * half;
#pragma unroll
            for (int p = 0; p < 32; ++p) {
                const u16x8_t v = *reinterpret_cast<const u16x8_t*>(pr + 8 * p);
                uint64_t h[2];
                __builtin_memcpy(h, &v, 16);
                P[2 * p] = bf16_bits_f64((uint16_t)(h[0] >> (16 * kq)));
                P[2 * p + 1] = bf16_bits_f64((uint16_t)(h[1] >> (16 * kq)));
            }
        } else {
#pragma unroll
            for (int p = 0; p < 64; ++p) P[p] = 0.0;
        }
        load_rows(0);
        dg_barrier();   // the previous chunk's reads of the tiles and of s_y are done
        widen_rows(0);
        load_rows(1);
        if (nc_on) nc_row(0);
        dg_barrier();
        f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
        auto chain = [&](int t) __attribute__((always_inline)) {
            const uint8_t* pa = s_t + (t & 1) * DG_HALF + m * DG_RS + 512 * kq;
            double2 av[2][4];
            auto read_group = [&](int gi, int buf) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) av[buf][e] = *reinterpret_cast<const double2*>(pa + 16 * (4 * gi + e));
            };
            read_group(0, 0);
            // four LDS reads serve eight steps; they go out one such group
            // ahead of their use (the scheduling barriers keep them there)
#pragma unroll
            for (int gi = 0; gi < 8; ++gi) {
                if (gi + 1 < 8) read_group(gi + 1, (gi + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[gi & 1][e].x, P[8 * gi + 2 * e], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[gi & 1][e].y, P[8 * gi + 2 * e + 1], acc, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // iteration it: waves 0-3 on tile it, waves 4-7 on tile it - 1
        for (int it = 0; it <= ntile; ++it) {
            const int t = it - half;
            const bool have = t >= 0 && t < ntile;
            double* hand = s_hand + (jw * 64 + lane) * 4;
            double dev[4] = {};   // RNE(y) - y
            u16x8_t rp = u16x8_t{};
            const bool rope = have && half == 0 && ch == 0 && ib && a.with_rope && tid < 128;
            const int rope_row = 16 * t + (tid >> 3);   // the tile's branch piece: 16 rows x 128 B over 128 threads
            if (have) {
                if (half == 0) {
                    if (rope)
                        rp = *reinterpret_cast<const u16x8_t*>(cb + (int64_t)min(rope_row, nrows - 1) * a.cs + D_LAT +
                                                               8 * (tid & 7));
                    widen_rows(t + 1);
                    load_rows(t + 2);
                    if (nc_on) {
                        nc_tile();
                        if (t % DG_GTILES == DG_GTILES - 1 || t == ntile - 1) {
                            // the group's last tile: in a short last group the elements its tiles did not reach
                            for (int i = t % DG_GTILES + 1; i < DG_GTILES; ++i) {
                                nc_load(i);
                                nc_tile();
                            }
                            // (the block's last group goes to LDS after the loop: the
                            // scalars of the group before it may still be due)
                            if (t + 1 < ntile) {
                                s_nc[64 * jw + lane] = nc;
                                nc_row(t / DG_GTILES + 1);
                            }
                        } else {
                            nc_load(t % DG_GTILES + 1);
                        }
                    }
                    acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
                    chain(t);
                    // branch copy (the exact summand of every future logit)
                    if (rope && rope_row < nrows)
                        *reinterpret_cast<u16x8_t*>(ib + (int64_t)rope_row * a.is + 8 * (tid & 7)) = rp;
                } else {
                    acc = *reinterpret_cast<const f64x4_t*>(hand);
                    chain(t);
                    widen_rows(t + 1);
                    load_rows(t + 2);
                    if (cert && t > 0 && jw == (t & 3)) tail_sums(t - 1, ch);
                    // acc[i] = y of tile row 4 i + kq, basis row j0 + 16 jw + m
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int rr = 16 * t + 4 * i + kq;
                        acc[i] = active ? acc[i] : 0.0;
                        const uint16_t d = f64_to_bf16_rne(acc[i]);
                        dev[i] = (double)bf16_to_f32(d) - acc[i];
                        if (ib && active && rr < nrows) ib[(int64_t)rr * a.is + off + j0 + 16 * jw + m] = d;
                    }
                }
            }
            dg_barrier();   // the reads of s_hand and of s_y are done
            if (have) {
                if (half == 0) {
                    *reinterpret_cast<f64x4_t*>(hand) = acc;
                } else {
                    if (cert) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            s_y[(4 * i + kq) * DG_YLD + 16 * jw + m] = acc[i];
                            s_y[(16 + 4 * i + kq) * DG_YLD + 16 * jw + m] = dev[i];
                        }
                    }
                }
            }
            // the group whose last tile's sums went in above (tile it - 2)
            if (cert && ch == nchunk - 1 && it >= 2 && (it - 1) % DG_GTILES == 0) scalars((it - 2) / DG_GTILES);
            dg_barrier();   // the next tiles, s_hand and s_y are in place
        }
        // the chunk's last tile has no tile after it whose steps its sums follow
        if (cert) {
            if (wave == 4) tail_sums(ntile - 1, ch);
            if (nc_on) s_nc[64 * jw + lane] = nc;
            dg_barrier();
        }
    }
    if (cert) scalars((ntile - 1) / DG_GTILES);
}

// Short sequences without a certificate (rows appended while decoding): the
// widened basis of the kernel above costs a block 6 us before its first step,
// which few rows do not repay.  Here a chunk of 64 basis rows is staged as bf16
// and widened with the rows at each step; two streams of four waves (one 16-row
// basis tile each) take alternate 16-row tiles through the whole 512-step chain,
// each stream's next tile loading into registers beside it.  Rows and basis rows
// sit in LDS rows padded to DS_ROW bytes, so the operand reads (16 rows, one
// 16-bit element each) fall into distinct banks.
constexpr int DS_ROW = 1040;
constexpr int DS_MAX_T = 128;   // rows of a sequence up to which this form is used (launch_digest)

__global__ __launch_bounds__(DG_THREADS) void digest_short_kernel(DigestArgs a, int rows) {
    __shared__ __align__(16) uint8_t s_p[DG_CHUNK * DS_ROW];    // a chunk of basis rows
    __shared__ __align__(16) uint8_t s_c[2][2][16 * DS_ROW];    // per stream, two tiles of cache rows
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int st = wave >> 2, jw = wave & 3;   // row stream, basis tile of the chunk
    const int64_t u0 = (int64_t)blockIdx.x * rows;
    const int nrows = (int)min((int64_t)rows, a.T - u0);
    const int ntile = (nrows + 15) / 16, niter = (ntile + 1) / 2;   // stream st takes tiles 2 it + st
    const uint16_t* cb = a.cache + (int64_t)b * a.cbs + u0 * a.cs;
    uint16_t* ib = a.index + (int64_t)b * a.ibs + u0 * a.is;
    const int off = a.with_rope ? D_ROPE : 0;
    // a tile's rows 4 jw .. 4 jw + 3, one 1 KB load each (rows past the end re-read
    // the last one; nothing of them is stored)
    u32x4_t nx[4];
    auto load_tile = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            nx[q] = *reinterpret_cast<const u32x4_t*>(cb + (int64_t)min(16 * t + 4 * jw + q, nrows - 1) * a.cs + 8 * lane);
    };
    auto store_tile = [&](int it) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<u32x4_t*>(s_c[st][it & 1] + (4 * jw + q) * DS_ROW + 16 * lane) = nx[q];
    };
    load_tile(st);
    if (a.with_rope) {   // the branch copy: up to 128 rows x 128 B
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int rr = 64 * e + (tid >> 3);
            if (rr < nrows)
                *reinterpret_cast<u16x8_t*>(ib + (int64_t)rr * a.is + 8 * (tid & 7)) =
                    *reinterpret_cast<const u16x8_t*>(cb + (int64_t)rr * a.cs + D_LAT + 8 * (tid & 7));
        }
    }
    for (int j0 = 0; j0 < a.r; j0 += DG_CHUNK) {
        const int jn = min(DG_CHUNK, a.r - j0);
        const bool active = 16 * jw < jn;
        u32x4_t pr[DG_CHUNK / 8];
#pragma unroll
        for (int e = 0; e < DG_CHUNK / 8; ++e)
            pr[e] = *reinterpret_cast<const u32x4_t*>(a.P + (int64_t)min(j0 + 8 * e + wave, a.r - 1) * D_LAT + 8 * lane);
        if (j0 > 0) {
            load_tile(st);
            dg_barrier();   // the previous chunk's reads are done
        }
#pragma unroll
        for (int e = 0; e < DG_CHUNK / 8; ++e)
            *reinterpret_cast<u32x4_t*>(s_p + (8 * e + wave) * DS_ROW + 16 * lane) = pr[e];
        store_tile(0);
        dg_barrier();
        // operand rows: A = cache row (lane mod 16) of the tile, B = basis row
        // 16 jw + (lane mod 16) of the chunk; element k = lane / 16 of each step
        const uint16_t* pb = reinterpret_cast<const uint16_t*>(s_p + (16 * jw + (lane & 15)) * DS_ROW) + (lane >> 4);
        for (int it = 0; it < niter; ++it) {
            const int t = 2 * it + st;
            const bool more = it + 1 < niter;
            if (more) load_tile(t + 2);
            if (active && t < ntile) {
                const uint16_t* ca =
                    reinterpret_cast<const uint16_t*>(s_c[st][it & 1] + (lane & 15) * DS_ROW) + (lane >> 4);
                const f64x4_t acc = mfma_f64_rowdot512(ca, pb);
                // acc[i] = y of tile row 4 i + lane / 16, basis row j0 + 16 jw + lane mod 16
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int rr = 16 * t + 4 * i + (lane >> 4);
                    if (rr < nrows)
                        ib[(int64_t)rr * a.is + off + j0 + 16 * jw + (lane & 15)] = f64_to_bf16_rne(acc[i]);
                }
            }
            if (more) {
                store_tile(it + 1);
                dg_barrier();   // (the stage it fills was last read before the barrier of it - 1)
            }
        }
    }
}

// An index without a digest (r = 0): the branch copy and, with the certificate,
// eta >= ||c||.  One wave per 64 rows, without LDS, so that many share a CU: 8
// lanes per row copy its branch, then each lane runs one row's sequential sum, a
// cache line of the row (64 elements) in flight beside the one it adds.  Bound by
// the row reads: 16 x 32768 rows 134 us with the certificate (4.5 TB/s), 22
// without, 698 and 612 as a projection on no basis rows.
__global__ __launch_bounds__(64) void digest_plain_kernel(DigestArgs a) {
    const int b = blockIdx.y, lane = threadIdx.x;
    const int64_t u0 = (int64_t)blockIdx.x * 64;
    const int nrows = (int)min((int64_t)64, a.T - u0);
    const uint16_t* cb = a.cache + (int64_t)b * a.cbs + u0 * a.cs;
    if (a.index && a.with_rope) {
        uint16_t* ib = a.index + (int64_t)b * a.ibs + u0 * a.is;
        u16x8_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = *reinterpret_cast<const u16x8_t*>(cb + (int64_t)min(8 * e + (lane >> 3), nrows - 1) * a.cs + D_LAT +
                                                     8 * (lane & 7));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int rr = 8 * e + (lane >> 3);
            if (rr < nrows) *reinterpret_cast<u16x8_t*>(ib + (int64_t)rr * a.is + 8 * (lane & 7)) = v[e];
        }
    }
    if (!a.eta) return;
    const uint16_t* row = cb + (int64_t)min(lane, nrows - 1) * a.cs;
    u16x8_t x[2][8];
    auto load = [&](int p, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[buf][j] = *reinterpret_cast<const u16x8_t*>(row + 64 * p + 8 * j);
    };
    double nc = 0.0;
    auto add = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const double v = bf16_bits_f64(x[buf][j][e]);
                nc = fma(v, v, nc);
            }
    };
    load(0, 0);
#pragma unroll 1
    for (int p = 0; p < D_LAT / 64; p += 2) {
        load(p + 1, 1);
        add(0);
        if (p + 2 < D_LAT / 64) load(p + 2, 0);
        add(1);
    }
    if (lane < nrows) cert_scalars(a, (int64_t)b * a.T + u0 + lane, nc, 0.0, 0.0);
}

hipError_t launch_digest(const DigestArgs& a, hipStream_t s) {
    if (a.T <= 0) return hipSuccess;
    if (a.r == 0) {
        if (!a.eta && !(a.index && a.with_rope)) return hipSuccess;
        hipLaunchKernelGGL(digest_plain_kernel, dim3((unsigned)((a.T + 63) / 64), (unsigned)a.B), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    // Short sequences without a certificate, at r = 64 against the kernel below: one
    // row 9 and 16 us, 64 rows 14 and 31, 1000 sequences of 17 rows 50 and 81, 300
    // of 128 rows 97 and 104; at 300 of 256 rows the kernel below has caught up (a
    // form of this one 200, that one 186).  32 rows a block, one tile per stream,
    // as long as that starts no second round of blocks.
    if (!a.eta && a.T <= DS_MAX_T) {
        const int rows = a.B * ((a.T + 31) / 32) <= 256 ? 32 : DS_MAX_T;
        hipLaunchKernelGGL(digest_short_kernel, dim3((unsigned)((a.T + rows - 1) / rows), (unsigned)a.B), dim3(DG_THREADS),
                           0, s, a, rows);
        return hipGetLastError();
    }
    // Rows per block: several groups keep the widened basis in registers for
    // longer (3 of 100 us per group), one group where it takes several chunks
    // (their sums of all rows would not fit the LDS) or where blocks would be
    // fewer than two per CU; below one block per CU shorter blocks, down to four
    // tiles, since the time is then that of one block.
    const int64_t total = a.B * ((a.T + DG_GROUP - 1) / DG_GROUP);
    int64_t rows = DG_GROUP;
    if (total < 256)
        rows = std::min<int64_t>(DG_GROUP, std::max<int64_t>(64, (a.B * a.T + 256 * 16 - 1) / (256 * 16) * 16));
    else if (a.r <= DG_CHUNK)
        rows = DG_GROUP * std::min<int64_t>(DG_MAX_GROUPS, std::max<int64_t>(1, total / 512));
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&digest_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)DG_LDS);
    dim3 grid((unsigned)((a.T + rows - 1) / rows), (unsigned)a.B);
    hipLaunchKernelGGL(digest_kernel, grid, dim3(DG_THREADS), DG_LDS, s, a, (int)rows);
    return hipGetLastError();
}

// Gershgorin row sums of P P^T: rowsum[j] = sum_k |sum_i P[j,i] P[k,i]|, with
// flag[j] = 1 if any fp64 addition on the way rounded (TwoSum error != 0).
// bf16 products are exact in fp64, so flag 0 means rowsum[j] is exact.
__device__ __forceinline__ double two_sum_add(double a, double b, int* inexact) {
    const double s = a + b;
    const double bp = s - a;
    const double err = (a - (s - bp)) + (b - bp);
    if (err != 0.0) *inexact = 1;
    return s;
}

// (Block j: row j.  It returns at once where every quick sum below is inside.)
__global__ __launch_bounds__(256) void gram_rows_kernel(const uint16_t* P, int r, const double* fast, double* rowsum,
                                                        double* flag) {
    __shared__ double s_g[512];
    __shared__ int s_f[512];
    const int j = blockIdx.x;
    const int tid = threadIdx.x;
    bool inside = true;
    for (int k = tid; k < r; k += 256) inside = inside && fast[k] <= GRAM_INSIDE;
    if (__syncthreads_and(inside)) return;
    for (int k = tid; k < r; k += 256) {
        const u16x8_t* pj = reinterpret_cast<const u16x8_t*>(P + (int64_t)j * D_LAT);
        const u16x8_t* pk = reinterpret_cast<const u16x8_t*>(P + (int64_t)k * D_LAT);
        double gk = 0.0;
        int inexact = 0;
#pragma unroll 4
        for (int p = 0; p < D_LAT / 8; ++p) {
            const u16x8_t x = pj[p], y = pk[p];
#pragma unroll
            for (int e = 0; e < 8; ++e) gk = two_sum_add(gk, bf16_bits_f64(x[e]) * bf16_bits_f64(y[e]), &inexact);
        }
        s_g[k] = gk;
        s_f[k] = inexact;
    }
    __syncthreads();
    if (tid == 0) {
        double acc = 0.0;
        int inexact = 0;
        for (int k = 0; k < r; ++k) {
            acc = two_sum_add(acc, fabs(s_g[k]), &inexact);
            inexact |= s_f[k];
        }
        rowsum[j] = acc;
        flag[j] = inexact ? 1.0 : 0.0;
    }
}

// The same row sums without the exactness flags, on the matrix cores (block: 16
// rows of P; four waves share a 16-column tile, a quarter of the dimensions
// each, four tiles at a time; the sums in another order).  They decide the usual
// case, a basis well inside the bound; only a row near the bound still needs the
// sequential sums above, formed behind them without a look at the host.  38 -> 19
// us at r = 64, 2 of them the second launch; near the bound one row's build takes
// 86 us as without the quick sums (118 where the host asked for the second launch).
__global__ __launch_bounds__(1024) void gram_fast_kernel(const uint16_t* P, int r, double* rowsum) {
    __shared__ f64x4_t s_g[4][4][64];   // [column tile][quarter][lane]
    __shared__ double s_r[4][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 15, kq = lane >> 4;
    const int ct = wave >> 2, qt = wave & 3;
    const uint16_t* pa = P + (int64_t)(16 * blockIdx.x + m) * D_LAT + 128 * qt;
    double sum[4] = {};
    for (int t0 = 0; 16 * t0 < r; t0 += 4) {
        const int t = t0 + ct;
        const uint16_t* pb = P + (int64_t)min(16 * t + m, r - 1) * D_LAT + 128 * qt;
        uint64_t va[32], vb[32];   // halves of the 16-byte pieces: elements 4 s .. 4 s + 3 of step s
#pragma unroll
        for (int e = 0; e < 32; e += 2) {
            const u16x8_t x = *reinterpret_cast<const u16x8_t*>(pa + 4 * e);
            const u16x8_t y = *reinterpret_cast<const u16x8_t*>(pb + 4 * e);
            __builtin_memcpy(&va[e], &x, 16);
            __builtin_memcpy(&vb[e], &y, 16);
        }
        f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 32; ++e)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(bf16_bits_f64((uint16_t)(va[e] >> (16 * kq))),
                                                      bf16_bits_f64((uint16_t)(vb[e] >> (16 * kq))), acc, 0, 0, 0);
        s_g[ct][qt][lane] = acc;
        __syncthreads();
        if (qt == 0 && 16 * t < r) {
            acc = (s_g[ct][0][lane] + s_g[ct][1][lane]) + (s_g[ct][2][lane] + s_g[ct][3][lane]);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += fabs(acc[e]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        for (int o = 1; o < 16; o <<= 1) sum[e] += __shfl_xor(sum[e], o);
        if (qt == 0 && m == 0) s_r[ct][4 * e + kq] = sum[e];
    }
    __syncthreads();
    if (tid < 16) rowsum[16 * blockIdx.x + tid] = (s_r[0][tid] + s_r[1][tid]) + (s_r[2][tid] + s_r[3][tid]);
}

hipError_t launch_gram(const uint16_t* P, int r, double* gram, hipStream_t s) {
    hipLaunchKernelGGL(gram_fast_kernel, dim3((unsigned)(r / 16)), dim3(1024), 0, s, P, r, gram);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gram_rows_kernel, dim3((unsigned)r), dim3(256), 0, s, P, r, gram, gram + r, gram + 2 * r);
    return hipGetLastError();
}

}  // namespace vkv
