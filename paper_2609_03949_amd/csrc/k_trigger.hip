// k_trigger.hip -- the tier-1 maximum logit and the calibration statistic of
// the calibrated trigger (Sec. 4.2: Eq. (trigger), the z paragraph; Sec. 5.2).
//
// row_max_kernel: per sequence b and head h, the maximum over a row list of
// the exact full score s_h(u) = q_lat_h . c_u + q_rope_h . r_u (Sec. 3,
// Eq. (setup); the fp64 sum over the 576 dims, latent then branch, from +0)
// and the row attaining it (ties: the lower row index).  Over the tier-1
// rows it is the trigger threshold s*_h; over the whole context it is the
// causal argmax row of a calibration query.  A workgroup of 8 waves (16
// heads each) streams one range of the list through an LDS tile ring that all
// its waves read: bf16 MFMA scores in fp32 with a certified band e = 2 (n +
// n/32) 2^-23 ||q_h|| ||x_u|| (n = 576, the scan's error model), and per lane
// and head the three largest scores.  Only entries whose upper bound reaches
// the head's certified lower bound get the fp64 chain; the true maximum row
// always does.  The ranges' maxima are merged by row_merge_kernel, or in the
// outputs where the caller gives no scratch.
// Bound by the gathered row stream (1152-byte rows, 3.6 TB/s measured over a
// whole archive) and, in short ranges, by the fp64 chains at the end (about
// 12 us).  Measured: 16 x 32768 rows, 128 heads 2650 -> 169 us (one range per
// sequence before), 32 x 4608 rows 97 -> 71 us and 16 x 1280 rows 41 -> 35 us
// (candidate lists in LDS with a band and three cross-lane steps per score
// before).
//
// inflation_kernel: for each (calibration query, head), whether the causal
// argmax row is archived and outside the tier-1 set (a hard query), and then
// z_q = (s*_h - idx_h(u*)) / cert_h(u*), the inflation at which the trigger
// score reaches the tier-1 maximum.
#include "vkv_internal.h"

namespace vkv {

constexpr int RM_PAIRS = 128;         // (head slot, row) pairs a lane group can list: 4 heads x 2 in 16 lanes
constexpr int RM_KS = D_ROW / 32;     // 18 k-steps of the 576-dim score

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float sumsq8(bf16x8_t v) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bf16x2_t p = {v[2 * e], v[2 * e + 1]};
        s = __builtin_amdgcn_fdot2_f32_bf16(p, p, s, false);
    }
    return s;
}

// exact fp64 full score of row `row` for the head whose 576 query elements are
// at q in LDS (the products of two bf16 values are exact in fp64; they are added
// in dimension order from +0).  Each lane has a row of its own, so a load
// touches up to 64 lines and the address unit bounds the exact phase; with the
// query rows in LDS only the cache row's half of the loads is left.  Pieces of
// 32 dims are loaded two pieces ahead of the chain (a ring of three), so the
// memory round trips overlap the arithmetic.
__device__ __forceinline__ double full_score64(const uint16_t* q, const uint16_t* row) {
    constexpr int NP = D_ROW / 32;   // 18 pieces of 4 x 8 dims
    u16x8_t xv[3][4];
    auto load = [&](int p, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[buf][j] = *reinterpret_cast<const u16x8_t*>(row + 32 * p + 8 * j);
    };
    double acc = 0.0;
    auto chain = [&](int p, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u16x8_t qv = *reinterpret_cast<const u16x8_t*>(q + 32 * p + 8 * j);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fma((double)bf16_to_f32(qv[e]), (double)bf16_to_f32(xv[buf][j][e]), acc);
        }
    };
    static_assert(NP % 3 == 0, "pieces taken in threes");
    load(0, 0);
    load(1, 1);
    // a loop, not unrolled: a fully unrolled chain lets the compiler issue all
    // loads first and spill them
#pragma unroll 1
    for (int p = 0; p < NP; p += 3) {
        load(p + 2, 2);
        chain(p, 0);
        if (p + 3 < NP) load(p + 3, 0);
        chain(p + 1, 1);
        if (p + 4 < NP) load(p + 4, 1);
        chain(p + 2, 2);
    }
    return acc;
}

// sum over the 16 lanes of each row of the wave (DPP lane permutations)
__device__ __forceinline__ float rowsum16(float v) {
    auto perm = [](float x, auto ctrl) __attribute__((always_inline)) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    v += perm(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
    v += perm(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
    v += perm(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
    v += perm(v, std::integral_constant<int, 0x140>{});   // row_mirror
    return v;
}

// max over the 16 lanes of each row of the wave (DPP lane permutations)
__device__ __forceinline__ float rowmax16(float v) {
    auto perm = [](float x, auto ctrl) __attribute__((always_inline)) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    v = fmaxf(v, perm(v, std::integral_constant<int, 0xB1>{}));    // quad_perm [1,0,3,2]
    v = fmaxf(v, perm(v, std::integral_constant<int, 0x4E>{}));    // quad_perm [2,3,0,1]
    v = fmaxf(v, perm(v, std::integral_constant<int, 0x141>{}));   // row_half_mirror
    v = fmaxf(v, perm(v, std::integral_constant<int, 0x140>{}));   // row_mirror
    return v;
}

// (score desc, row asc): is (s1, u1) ahead of (s0, u0)?
__device__ __forceinline__ bool ahead(double s1, int64_t u1, double s0, int64_t u0) {
    return s1 > s0 || (s1 == s0 && u1 < u0);
}

// (max, lowest row) of a range merged into the output pair itself, where the
// caller gives no scratch for partials.  *argmax is the pair's lock while it
// holds RM_LOCKED: the holder compares, writes the maximum and releases by
// writing the row, all in one branch, so every wait ends.  Agent-scope atomics
// only (they act at the point all XCDs share), each completed before the next
// is issued; a maximum already above v needs no lock, as *smax only grows.
constexpr int32_t RM_LOCKED = -2;

__device__ __forceinline__ void merge_max(double* smax, int32_t* argmax, double v, int32_t u) {
    unsigned long long* sm = reinterpret_cast<unsigned long long*>(smax);
    auto current = [&]() {
        return u2d(__hip_atomic_load(sm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    bool done = false;
    while (!done) {
        if (current() > v) break;
        const int32_t old = __hip_atomic_exchange(argmax, RM_LOCKED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (old != RM_LOCKED) {
            int32_t keep = old;
            if (ahead(v, u, current(), old)) {
                // (the returned value is used: it comes back once the exchange has acted)
                unsigned long long was = __hip_atomic_exchange(sm, d2u(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" : "+v"(was) : : "memory");
                keep = u;
            }
            __hip_atomic_store(argmax, keep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            done = true;
        } else {
            __builtin_amdgcn_s_sleep(1);
        }
    }
}

// Block (hgb, b, sp): RM_WAVES waves, wave w taking heads 16 (RM_WAVES hgb +
// w) .. +15 of sequence b, over the sp-th of nsplit equal ranges of the list
// (each range yields the exact maximum of its own rows; row_merge_kernel takes
// the best of them, so the result is the same for any nsplit).  The block
// streams its range in tiles of RM_TILE rows through a two-stage LDS ring that
// all its waves read, so a row is fetched from memory once per block, not
// once per 16 heads.  Tile t + 1's 16-byte pieces are loaded into registers
// while tile t is scored and are written to the other stage after it; the row
// indices go out one tile earlier still.  Stage slot (r, p) holds piece
// p ^ (r mod 8) of tile row r, so the eight lanes that one 128-bit LDS read
// serves (eight rows, one piece) hit distinct bank groups.
constexpr int RM_WAVES = 8;
// workgroup barrier for exchanges through LDS (global loads stay in flight)
__device__ __forceinline__ void rm_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
constexpr int RM_THREADS = 64 * RM_WAVES;
constexpr int RM_TILE = 32;                                   // rows per tile
constexpr int RM_WROWS = RM_TILE / RM_WAVES;                  // tile rows each wave loads (4)
constexpr int RM_PER = (D_ROW / 8 + 15) / 16;                 // 16-byte pieces per lane (5, the last one in 8 lanes)
constexpr int RM_TAIL = D_ROW / 8 - 16 * (RM_PER - 1);
static_assert(RM_WROWS == 4, "a row per 16-lane group");
constexpr int RM_QROW = 2 * D_ROW + 16;                       // LDS bytes of a staged query row (heads in distinct banks)
static_assert(2 * RM_TILE * 2 * D_ROW <= RM_WAVES * 16 * RM_QROW, "the ring fits the query rows' room");

// LIST: a non-empty row list (else the archive, or the recent rows alone).
template <bool OFF32, bool LIST>
__global__ __launch_bounds__(RM_THREADS) void row_max_kernel(RowMaxArgs a) {
    // the tile ring; after the last tile the waves' query rows, [wave][head][RM_QROW]
    __shared__ __align__(16) uint8_t s_mem[RM_WAVES * 16 * RM_QROW];
    uint8_t (*s_x)[RM_TILE * 2 * D_ROW] = reinterpret_cast<uint8_t (*)[RM_TILE * 2 * D_ROW]>(s_mem);
    __shared__ uint8_t s_pair[RM_WAVES][4][RM_PAIRS];
    __shared__ int32_t s_id[4][RM_TILE];
    __shared__ float s_xn[2][RM_TILE];   // ||x_u||^2 of the stage's rows (fp32)
    const int HG = (a.H + 15) / 16;
    const int HGB = (HG + RM_WAVES - 1) / RM_WAVES;
    const int hgb = (int)(blockIdx.x % HGB);
    const int64_t jb = blockIdx.x / HGB;
    const int b = (int)(jb % a.B), sp = (int)(jb / a.B);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int hg = hgb * RM_WAVES + wave;
    const bool wave_on = hg < HG;   // waves past the last head group only load
    const int h0 = 16 * hg;
    const int hq = h0 + c;
    const bool hq_ok = wave_on && hq < a.H;
    const int64_t n1 = a.all_archive ? a.A : a.nrows;
    const int64_t Nall = n1 + (a.add_recent ? a.T - a.A : 0);
    const int64_t per = (Nall + a.nsplit - 1) / a.nsplit;
    const int64_t pbeg = min(Nall, (int64_t)sp * per);
    const int64_t N = min(Nall, pbeg + per);   // this block's list positions: [pbeg, N)
    const uint16_t* cb = a.cache + (int64_t)b * a.cbs;
    auto row_of = [&](int64_t p) -> int64_t {
        return p < n1 ? (a.all_archive ? p : (int64_t)a.rows[(int64_t)b * a.nrows + p]) : a.A + (p - n1);
    };
    // query fragments (A operand): head hq, dims 32 ks + 8 g; ||q_hq||^2 in fp32
    bf16x8_t qf[RM_KS];
    float qs = 0.f;
#pragma unroll
    for (int ks = 0; ks < RM_KS; ++ks) {
        const int d = 32 * ks + 8 * g;
        const int64_t hb = (int64_t)b * a.H + (hq_ok ? hq : 0);
        const uint16_t* src = d < D_LAT ? a.q_lat + hb * D_LAT + d : a.q_rope + hb * D_ROPE + (d - D_LAT);
        qf[ks] = hq_ok ? *reinterpret_cast<const bf16x8_t*>(src) : bf16x8_t{};
        qs += sumsq8(qf[ks]);
    }
    qs += __shfl_xor(qs, 16);
    qs += __shfl_xor(qs, 32);
    // per accumulator slot i: head h0 + 4 g + i; an upper bound of its ||q||
    // (the fp32 sum of 576 exact squares is within 576 * 2^-24 relative)
    // qk[i] = KE ||q|| inflated by 2^-19 (which covers the fp32 roundings of
    // qk and of the product with ||x|| below), KE = 2 (n + n/32) 2^-23
    constexpr float KE = 2.0f * (float)(D_ROW + D_ROW / 32) * 0x1p-23f;
    float qk[4], qmax = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float qub = sqrtf(__shfl(qs, 4 * g + i) * (1.0f + 0x1p-12f)) * (1.0f + 0x1p-20f);
        qk[i] = (KE * qub) * (1.0f + 0x1p-19f);
        qmax = fmaxf(qmax, qub);
    }
    // ||x||^2 up to which this lane's scores, and the partial sums on the way, stay
    // below 2^127: |sum| <= ||q|| ||x|| (0 for an infinite query)
    const float q126 = 0x1p126f / qmax;
    const float xlim = fminf(q126 * q126, 0x1.fffffep127f);
    // Per lane (tile-row class c) and head slot i: the three largest scores of
    // the rows it has seen and the rows of the first two.  The exact maximum of
    // a head is among the entries whose upper bound reaches its certified lower
    // bound M at the end; a third entry that reaches the best exact score found
    // there means that rows of its class may be missing, and then all rows of
    // that class are evaluated.
    float v1[4], v2[4], v3[4];
    int32_t r1[4], r2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v1[i] = v2[i] = v3[i] = -INFINITY;
        r1[i] = r2[i] = -1;
    }
    // the screen: a score below T[i] cannot reach the maximum (refresh below);
    // xcap is the largest finite ||x||^2 of the rows T allows for (xskip, also at
    // most xlim: rows up to it may be skipped), xm this lane's
    // (slots past the last head, whose zero scores would always reach it, and
    // those of a query that is no number, which has no maximum, pass nothing)
    bool live[4];
    float T[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        live[i] = h0 + 4 * g + i < a.H && qk[i] == qk[i];
        T[i] = live[i] ? -INFINITY : INFINITY;
    }
    float xcap = 0.f, xskip = 0.f, xm = 0.f;
    // band half-width of a score v of slot i, xb >= ||x|| of every row: e >= KE
    // ||q|| ||x|| (one rounding, inside qk's slack; the n 2^-120 term keeps e
    // away from the subnormals).  The rounding to nearest of v -+ ep moves it by
    // at most 2^-24 (|v| + ep), and ep - e >= 2^-23 (|v| + e) exceeds that, so
    // v - ep <= v - e and v + ep >= v + e without directed rounding.
    auto band = [&](int i, float v, float xb) __attribute__((always_inline)) {
        const float e = fmaf(qk[i], xb, (float)D_ROW * 0x1p-120f);
        return fmaf(fabsf(v) + e, 0x1p-22f, e);
    };
    auto norm_up = [](float x2) __attribute__((always_inline)) {   // >= ||x|| from the fp32 sum of squares
        return sqrtf(x2 * (1.0f + 0x1p-12f)) * (1.0f + 0x1p-20f);
    };

    // loader: wave w moves tile rows 4 w .. 4 w + 3, lane 16 j + l of it pieces
    // l + 16 i (i < 5, below 72) of row 4 w + j (rows past the range repeat its
    // last row; they are loaded, never scored).  A row's pieces stay in one
    // lane group, so the group also sums the row's squares once for all 8 waves
    // (the per-(row, head) band needs ||x_u||): one row index, one address and
    // one 16-lane sum per lane and tile.
    // (list positions, row indices and, with OFF32, byte offsets inside the
    // sequence's cache fit 32 bits; the bases are uniform, so the loads take
    // a scalar base and a 32-bit lane offset)
    const int32_t* rb = a.rows ? a.rows + (int64_t)b * a.nrows : nullptr;
    const int32_t n1i = (int32_t)n1, Ai = (int32_t)a.A, Nm1 = (int32_t)(N - 1);
    const int lrow = RM_WROWS * wave + g;   // this lane's tile row
    auto load_id = [&](int64_t t0) {
        const int32_t p = min((int32_t)t0 + lrow, Nm1);
        const int32_t w = p < n1i ? p : Ai + (p - n1i);
        if constexpr (!LIST) return w;
        const int32_t v = rb[min(p, n1i - 1)];
        return p < n1i ? v : w;
    };
    const uint8_t* cbb = reinterpret_cast<const uint8_t*>(cb);
    const uint32_t rs32 = (uint32_t)(2 * a.cs);   // row stride in bytes (OFF32)
    auto load_pieces = [&](u32x4_t (&xr)[RM_PER], int32_t id) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RM_PER; ++i) {
            if (i < RM_PER - 1 || c < RM_TAIL) {
                if constexpr (OFF32)
                    xr[i] = *reinterpret_cast<const u32x4_t*>(cbb + ((uint32_t)id * rs32 + 16u * (uint32_t)c) + 256 * i);
                else
                    xr[i] = *reinterpret_cast<const u32x4_t*>(cb + (int64_t)id * a.cs + 8 * (c + 16 * i));
            }
        }
    };
    auto store_pieces = [&](const u32x4_t (&xr)[RM_PER], int st) __attribute__((always_inline)) {
        float ss = 0.f;
        uint8_t* dst = s_x[st] + lrow * (2 * D_ROW) + 16 * (c ^ (lrow & 7));
#pragma unroll
        for (int i = 0; i < RM_PER; ++i) {
            if (i < RM_PER - 1 || c < RM_TAIL) {
                *reinterpret_cast<u32x4_t*>(dst + 256 * i) = xr[i];
                bf16x8_t v;
                __builtin_memcpy(&v, &xr[i], 16);
                ss += sumsq8(v);
            }
        }
        ss = rowsum16(ss);
        if (c == 0) s_xn[st][lrow] = ss;
    };

    // one 16-row half of the tile in stage st (list positions p0 ..)
    auto score_half = [&](int st, int sid, int m, int64_t p0) __attribute__((always_inline)) {
        const int rl = 16 * m + c;   // this lane's tile row
        const bool valid = p0 + c < N;
        // piece 4 ks + g sits at (4 (ks & 1) + g) ^ (c & 7) of its group of eight
        const uint8_t* xe = s_x[st] + rl * (2 * D_ROW) + 16 * (g ^ (c & 7));
        const uint8_t* xo = s_x[st] + rl * (2 * D_ROW) + 16 * ((4 + g) ^ (c & 7));
        f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < RM_KS; ++ks) {
            const bf16x8_t xv = *reinterpret_cast<const bf16x8_t*>(((ks & 1) ? xo : xe) + 128 * (ks >> 1));
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[ks], xv, acc, 0, 0, 0);
        }
        // ||x||^2 summed by the loading wave (fp32 sums of the 576 exact
        // squares in any order are within 576 * 2^-24 relative)
        const float xs = s_xn[st][rl];
        // In a long range most halves hold no row that can reach any head's
        // bound: a comparison per score and one ballot skip the rest
        bool maybe = !(xs <= xskip);
#pragma unroll
        for (int i = 0; i < 4; ++i) maybe |= acc[i] >= T[i];
        if (__ballot(maybe) == 0) return;
        const int32_t u = s_id[sid][rl];
        if (__ballot(!(xs <= xlim)) != 0) {
            // A score that is not finite says nothing, and a row whose ||x||^2 is
            // past fp32 has no band: they rank first, so that their exact score
            // decides, and such a row does not widen the bands of the others
            const bool wild = !(xs < INFINITY);
            xm = wild ? xm : fmaxf(xm, xs);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = !wild && fabsf(acc[i]) < INFINITY ? acc[i] : INFINITY;
        } else {
            xm = fmaxf(xm, xs);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = valid ? acc[i] : -INFINITY;
            const bool c1 = v > v1[i], c2 = v > v2[i];
            const float t1 = fminf(v1[i], v);
            r2[i] = c1 ? r1[i] : (c2 ? u : r2[i]);
            r1[i] = c1 ? u : r1[i];
            v1[i] = fmaxf(v1[i], v);
            const float t2 = fminf(v2[i], t1);
            v2[i] = fmaxf(v2[i], t1);
            v3[i] = fmaxf(v3[i], t2);
        }
    };
    // this lane's certified lower bound of slot i's maximum; -inf where infinite
    // scores or norms leave none (the difference is then no number)
    auto lower = [&](int i, float xb) __attribute__((always_inline)) {
        return fmaxf(v1[i] - band(i, v1[i], xb), -INFINITY);
    };
    // T from the scores so far.  With e <= ecap, v + ep <= v + 2^-22 |v| + 1.01
    // ecap, below M if v < M - 2 ecap - 2^-21 |M| (either sign of v and M); T
    // takes 3 ecap and 2^-20 |M|, which also covers its own roundings, and is
    // -inf (no screen) where M or the band is infinite.
    auto refresh = [&]() __attribute__((always_inline)) {
        xcap = rowmax16(fmaxf(xcap, xm));   // the 16 rows are the same in each lane group
        xskip = fminf(xcap, xlim);
        const float xb = norm_up(xcap);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float M = rowmax16(lower(i, xb));
            const float t = fmaxf(M - (3.0f * fmaf(qk[i], xb, (float)D_ROW * 0x1p-120f) + fabsf(M) * 0x1p-20f), -INFINITY);
            T[i] = live[i] ? t : INFINITY;
        }
    };

    const int64_t ntiles = N > pbeg ? (N - pbeg + RM_TILE - 1) / RM_TILE : 0;   // the same in every wave
    // Tile t scores while the pieces of tiles t + 1 and t + 2 and the row
    // indices of tile t + 3 are in flight; every load is unconditional (tiles
    // past the range re-read its last row), so the compiler's wait before the
    // pieces of t + 1 go to LDS leaves the younger loads in flight, and the
    // barrier waits for LDS only.  The piece buffers swap roles from tile to
    // tile, so no register copy waits for a load.
    if (ntiles > 0) {
        u32x4_t xa[RM_PER], xb[RM_PER];
        const int32_t i0 = load_id(pbeg), i1 = load_id(min(pbeg + RM_TILE, N));
        int32_t id = load_id(min(pbeg + 2 * RM_TILE, N));   // of tile t + 2
        load_pieces(xa, i0);
        load_pieces(xb, i1);
        if (c == 0) {
            s_id[0][lrow] = i0;
            s_id[1][lrow] = i1;
        }
        store_pieces(xa, 0);
        rm_lds_barrier();
        auto tile = [&](int64_t t, u32x4_t (&x1)[RM_PER], u32x4_t (&x2)[RM_PER]) __attribute__((always_inline)) {
            const int st = (int)(t & 1);
            const int64_t p0 = pbeg + RM_TILE * t;
            load_pieces(x2, id);
            if (c == 0) s_id[(t + 2) & 3][lrow] = id;   // (tile t - 2's slot)
            id = load_id(min(p0 + 3 * RM_TILE, N));
            if (wave_on) {
                score_half(st, (int)(t & 3), 0, p0);
                score_half(st, (int)(t & 3), 1, p0 + 16);
                if ((t & (t + 1)) == 0 || (t & 7) == 7) refresh();
            }
            // every wave is past tile t - 1, whose stage this refills (the barrier
            // that ended it); tile t + 1 becomes visible at the barrier below
            store_pieces(x1, st ^ 1);
            rm_lds_barrier();
        };
        for (int64_t t = 0; t < ntiles; ++t) {
            tile(t, xb, xa);
            if (++t >= ntiles) break;
            tile(t, xa, xb);
        }
    }
    if (!wave_on) return;
    // The waves are past the ring (the last tile's barrier): each lays its
    // query rows out in LDS for the exact scores.  The entries that can hold a
    // head's maximum are listed per lane group, so that the fp64 chains fill its
    // lanes.
    uint8_t* s_q = s_mem + wave * 16 * RM_QROW;
#pragma unroll
    for (int ks = 0; ks < RM_KS; ++ks) *reinterpret_cast<bf16x8_t*>(s_q + c * RM_QROW + 64 * ks + 16 * g) = qf[ks];
    double best[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int64_t arg[4] = {-1, -1, -1, -1};
    auto offer = [&](int i, double v, int64_t u) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k == i && ahead(v, u, best[k], arg[k])) {
                best[k] = v;
                arg[k] = u;
            }
    };
    auto query = [&](int i) __attribute__((always_inline)) {
        return reinterpret_cast<const uint16_t*>(s_q + (4 * g + i) * RM_QROW);
    };
    float xb;
    uint8_t* pairs = s_pair[wave][g];   // entry (lane, slot, first or second): c + 16 i + 64 second
    int npass = 0;                      // the same in the group's 16 lanes
    {
        xb = norm_up(rowmax16(fmaxf(xcap, xm)));
        auto list = [&](int i, bool pass, int second) __attribute__((always_inline)) {
            const uint32_t gm = (uint32_t)(__ballot(pass) >> (16 * g)) & 0xFFFFu;
            if (pass) pairs[npass + __popc(gm & ((1u << c) - 1u))] = (uint8_t)(c + 16 * i + 64 * second);
            npass += __popc(gm);
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool hv = live[i] && N > pbeg;
            const float M = rowmax16(lower(i, xb));
            // (not provably below M: a band that is no number reaches it)
            auto reaches = [&](float v) __attribute__((always_inline)) { return !(v + band(i, v, xb) < M); };
            list(i, hv && r1[i] >= 0 && reaches(v1[i]), 0);
            list(i, hv && r2[i] >= 0 && reaches(v2[i]), 1);
        }
    }
    __builtin_amdgcn_wave_barrier();
    int pmax = max(npass, __shfl_xor(npass, 16));
    pmax = max(pmax, __shfl_xor(pmax, 32));   // the row exchange below needs all lanes
    for (int j0 = 0; j0 < pmax; j0 += 16) {
        const int j = j0 + c;
        const bool on = j < npass;
        const int code = on ? pairs[j] : 0, i = (code >> 4) & 3, from = 16 * g + (code & 15);
        int32_t u = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t u1 = __shfl(r1[k], from), u2 = __shfl(r2[k], from);
            if (i == k) u = code >= 64 ? u2 : u1;
        }
        if (on) offer(i, full_score64(query(i), cb + (int64_t)u * a.cs), u);
    }
    // classes whose third entry reaches the best exact score: their rows are
    // dealt to the group's lanes (one class of a 576-row range: 36 rows)
    uint64_t classes = 0;   // 16 bits per slot, the same in the group's 16 lanes
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double bv = best[i];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) bv = fmax(bv, __shfl_xor(bv, o));
        const bool miss = live[i] && v3[i] > -INFINITY && !((double)(v3[i] + band(i, v3[i], xb)) < bv);
        classes |= ((__ballot(miss) >> (16 * g)) & 0xFFFFull) << (16 * i);
    }
#pragma unroll 1
    while (classes) {
        const int bit = __ffsll((unsigned long long)classes) - 1, i = bit >> 4;
        classes &= classes - 1;
#pragma unroll 1
        for (int64_t p = pbeg + (bit & 15) + 16 * c; p < N; p += 256) {
            const int64_t u = row_of(p);
            offer(i, full_score64(query(i), cb + u * a.cs), u);
        }
    }
    double mv = -INFINITY;
    int32_t mu = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int h = h0 + 4 * g + i;
        double bv = best[i];
        int64_t ba = arg[i];
        // (max, lowest row) over the 16 lanes of the group
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const double ob = __shfl_xor(bv, o);
            const int64_t oa = (int64_t)__shfl_xor((long long)ba, o);
            if (oa >= 0 && ahead(ob, oa, bv, ba)) {
                bv = ob;
                ba = oa;
            }
        }
        const int64_t hb = (int64_t)b * a.H + h;
        if (a.nsplit > 1 && !a.part_v) {
            if (c == i) {   // this lane's head for merge_max below
                mv = bv;
                mu = h < a.H ? (int32_t)ba : -1;
            }
        } else if (c == 0 && h < a.H) {
            if (a.nsplit > 1) {
                a.part_v[hb * a.nsplit + sp] = bv;
                a.part_u[hb * a.nsplit + sp] = (int32_t)ba;
            } else {
                a.smax[hb] = bv;
                a.argmax[hb] = (int32_t)ba;
            }
        }
    }
    if (a.nsplit > 1 && !a.part_v && mu >= 0) {
        const int64_t hb = (int64_t)b * a.H + h0 + 4 * g + c;
        merge_max(a.smax + hb, a.argmax + hb, mv, mu);
    }
}

// the empty maximum, before the ranges of a call without scratch are merged into it
__global__ __launch_bounds__(256) void row_init_kernel(RowMaxArgs a) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)a.B * a.H) return;
    a.smax[t] = -INFINITY;
    a.argmax[t] = -1;
}

// (max, lowest row) over the ranges of each (sequence, head)
__global__ __launch_bounds__(64) void row_merge_kernel(RowMaxArgs a) {
    const int64_t t = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (t >= (int64_t)a.B * a.H) return;
    double best = -INFINITY;
    int64_t arg = -1;
    for (int sp = 0; sp < a.nsplit; ++sp) {
        const double v = a.part_v[t * a.nsplit + sp];
        const int64_t u = a.part_u[t * a.nsplit + sp];
        if (u >= 0 && ahead(v, u, best, arg)) {
            best = v;
            arg = u;
        }
    }
    a.smax[t] = best;
    a.argmax[t] = (int32_t)arg;
}

hipError_t launch_row_max(const RowMaxArgs& a, hipStream_t s) {
    const int HG = (a.H + 15) / 16;
    const unsigned nblk = (unsigned)((HG + RM_WAVES - 1) / RM_WAVES * a.B * a.nsplit);
    const int64_t n = (int64_t)a.B * a.H;
    if (a.nsplit > 1 && !a.part_v) hipLaunchKernelGGL(row_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    const bool list = !a.all_archive && a.nrows > 0;
    // 32-bit byte offsets when every row of a sequence lies within 4 GiB of its first
    if ((a.T - 1) * a.cs * 2 + 2 * D_ROW <= (int64_t)UINT32_MAX)
        hipLaunchKernelGGL((list ? row_max_kernel<true, true> : row_max_kernel<true, false>), dim3(nblk), dim3(RM_THREADS),
                           0, s, a);
    else
        hipLaunchKernelGGL((list ? row_max_kernel<false, true> : row_max_kernel<false, false>), dim3(nblk),
                           dim3(RM_THREADS), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.nsplit <= 1 || !a.part_v) return e;
    hipLaunchKernelGGL(row_merge_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, a);
    return hipGetLastError();
}

// one thread per (calibration query b, head h)
__global__ __launch_bounds__(64) void inflation_kernel(InflArgs a) {
    const int64_t t = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (t >= (int64_t)a.B * a.H) return;
    const int b = (int)(t / a.H);
    const int32_t u = a.argmax[t];
    bool in_s = false;
    if (u >= 0 && u < a.A && a.k > 0) {
        const int32_t* sb = a.sel + (int64_t)b * a.k;
        int64_t lo = 0, hi = a.k;   // sel is ascending
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (sb[mid] < u) lo = mid + 1;
            else hi = mid;
        }
        in_s = lo < a.k && sb[lo] == u;
    }
    const bool hard = u >= 0 && u < a.A && !in_s;
    a.hard[t] = hard ? 1 : 0;
    double z = 0.0;
    if (hard) {
        const uint16_t* q = a.qt + t * a.n;
        const uint16_t* x = a.x + (int64_t)b * a.xbs + (int64_t)u * a.xs;
        // d ascending, 64 dims of both rows in flight at a time (20 us with 2-byte
        // loads, each awaited by its product)
        double acc = 0.0;
        for (int p0 = 0; p0 < a.n / 8; p0 += 8) {
            u16x8_t qv[8], xv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int p = min(p0 + j, a.n / 8 - 1);
                qv[j] = *reinterpret_cast<const u16x8_t*>(q + 8 * p);
                xv[j] = *reinterpret_cast<const u16x8_t*>(x + 8 * p);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (p0 + j >= a.n / 8) break;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc = fma((double)bf16_to_f32(qv[j][e]), (double)bf16_to_f32(xv[j][e]), acc);
            }
        }
        const float4 hs = reinterpret_cast<const float4*>(a.hsc)[t];
        const int64_t o = (int64_t)b * a.T + u;
        const double idx = acc + fma((double)hs.y, (double)a.eps[o], (double)hs.z * (double)a.gam[o]);
        const double cert = (double)hs.x * (double)a.eta[o] / sqrt((double)(D_LAT - a.r));
        const double gap = a.tier1[t] - idx;
        z = cert > 0.0 ? gap / cert : (gap > 0.0 ? INFINITY : -INFINITY);
    }
    a.zq[t] = z;
}

hipError_t launch_inflation(const InflArgs& a, hipStream_t s) {
    const int64_t n = (int64_t)a.B * a.H;
    hipLaunchKernelGGL(inflation_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace vkv
