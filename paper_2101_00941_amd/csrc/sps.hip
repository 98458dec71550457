// Single-pulse search on a dedispersed plane, for gfx950 (the paper's SPDT phase,
// section 2.2). Three kernels run in order on the caller's stream:
//   sps_stats   exact int64 moments per (DM row, stat block), then mu and sigma in
//               float64, then the per-width normalisation wmu_w = w*mu and
//               r_w = 1/(sigma*sqrt(w)), and each width's smallest window sum whose
//               S/N reaches the threshold.
//   sps_screen  per wave two DM rows and a run of tiles of 256 starts: LDS prefix sums
//               give the boxcars, an integer screen against those sums drops the cells
//               whose best S/N is below the threshold, and the rest get the float64 best
//               S/N and a 3x3 peak test on a one-sample, one-row halo. The result is a bit
//               mask of candidates per row, plus integer per-row counts.
//   sps_best    instead of it where the best plane is an output: the float64 best S/N of
//               every cell of an (8 DM rows, 256 starts) tile, then the peak test.
//   sps_emit    one work-group per DM row. The row's output offset is the sum of
//               the counts of the rows before it. A block scan of the mask ranks each
//               candidate, and the candidate is written in (dm, t) order. Its S/N and
//               width are recomputed with the same float64 operations.
// No float atomics and no cross-stream waits are involved. The only atomics are
// integer counter adds, and their sum does not depend on order. Output order comes
// from the scan, not from the atomics. The paper's section 2.2 notes that its
// streamed search stalled on atomics combined with event waits.
#pragma clang fp contract(off)

#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>

#include "aa_internal.h"
#include "dedisp_device.h"
#include "numerics.h"
#include "screen.h"
#include "xcd.h"

namespace aa {
namespace {

constexpr int kMaxWidths = 32;

struct SpsConst {
    int32_t nw;
    int32_t wmax;
    int32_t widths[kMaxWidths];
    double sqrtw[kMaxWidths];
    // decimated boxcar hierarchy: widths kfull .. nw-1 are tried only at starts t with
    // (t & smask[k]) == 0 (stride - 1); kfull = nw when the hierarchy is off
    int32_t kfull;
    int32_t smask[kMaxWidths];
};


// Inclusive prefix sum over the 64 lanes of a wave (modulo 2^32): shifts by 1, 2, 4 and
// 8 lanes inside each row of 16, then the last lane of row 0 (and of row 2) is added to
// row 1 (and 3), and the last lane of row 1 to rows 2 and 3. Lanes whose source falls
// outside the row, or rows masked off, add 0.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));
    return v;
}

// v's value in the lane that the DPP control picks, 0 where it has none or its row is masked.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xf, false));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), CTRL, ROWS, 0xf, false));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
// Sum over the 64 lanes of a wave, in every lane.
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    v += dpp_u64<0x111, 0xf>(v);
    v += dpp_u64<0x112, 0xf>(v);
    v += dpp_u64<0x114, 0xf>(v);
    v += dpp_u64<0x118, 0xf>(v);
    v += dpp_u64<0x142, 0xa>(v);
    v += dpp_u64<0x143, 0xc>(v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), 63));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// ---- statistics -------------------------------------------------------------
struct Moments {
    uint64_t n, s1, s2;
};

// The values lo .. lo + span that a clipping pass keeps; none if empty.
struct KeepRange {
    uint32_t lo, span;
    bool empty;
};

// The integers v in [0, 2^32) with |float64(v) - mu| <= lim, the difference rounded once. The
// rounded difference never decreases with v, so they are consecutive, and their ends lie
// within one of the float64 sums below (whose errors are far less than one).
__device__ __forceinline__ KeepRange keep_range(double mu, double lim) {
    auto kept = [=](double v) { return __builtin_fabs(v - mu) <= lim; };
    double a = __builtin_ceil(mu - lim) - 1.0, b = __builtin_floor(mu + lim) + 1.0;
    if (!(a >= 0.0)) a = 0.0;
    if (!(b <= 4294967295.0)) b = 4294967295.0;
    if (!kept(a)) a += 1.0;
    if (!kept(a)) a += 1.0;
    if (!kept(b)) b -= 1.0;
    if (!kept(b)) b -= 1.0;
    KeepRange r{0u, 0u, !(a <= b && kept(a) && kept(b))};
    if (!r.empty) {
        r.lo = static_cast<uint32_t>(a);
        r.span = static_cast<uint32_t>(b) - r.lo;
    }
    return r;
}

// Sums of a work-group's per-thread moments, in every thread; NARROW: the sums of a wave's n
// and s1 are below 2^32. part alternates between two buffers, so that one barrier a call is
// enough.
template <bool NARROW, int WAVES>
__device__ __forceinline__ Moments reduce_moments(Moments m, uint64_t (&part)[3][WAVES]) {
    auto wave_sum_u32 = [](uint64_t v) {
        return static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(wave_incl_scan(static_cast<uint32_t>(v))), 63));
    };
    m.n = wave_sum_u32(m.n);   // a block has less than 2^31 values
    m.s1 = NARROW ? wave_sum_u32(m.s1) : wave_sum_u64(m.s1);
    m.s2 = wave_sum_u64(m.s2);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        part[0][wave] = m.n;
        part[1][wave] = m.s1;
        part[2][wave] = m.s2;
    }
    __syncthreads();
    if constexpr (WAVES > 4) {
        m.n = wave_sum_u32(lane < WAVES ? part[0][lane] : 0);
        m.s1 = wave_sum_u64(lane < WAVES ? part[1][lane] : 0);
        m.s2 = wave_sum_u64(lane < WAVES ? part[2][lane] : 0);
    } else {
        m = Moments{0, 0, 0};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            m.n += part[0][w];
            m.s1 += part[1][w];
            m.s2 += part[2][w];
        }
    }
    return m;
}

constexpr int kHeldGroups = 16;   // 16-byte groups of a block that a thread of the statistics holds

// A thread's share of a block of n values from src on: groups of 4 values THREADS apart,
// held in registers if HELD (n <= 4 * kHeldGroups * THREADS) and read on each pass if not.
// Values past the block read as 0.
template <int THREADS, bool HELD>
struct BlockValues {
    static constexpr int kRound = 4 * THREADS;   // values of the work-group's g-th groups
    const int32_t* src;
    int64_t n;
    u32x4 held[HELD ? kHeldGroups : 1];

    __device__ __forceinline__ BlockValues(const int32_t* p, int count) : src(p), n(count) {
        if constexpr (HELD)
#pragma unroll
            for (int g = 0; g < kHeldGroups; ++g) {
                held[g] = u32x4{0u, 0u, 0u, 0u};
                if (kRound * g < n) held[g] = load(g);
            }
    }
    __device__ __forceinline__ u32x4 load(int64_t g) const {
        const int left = n - kRound * g < kRound ? static_cast<int>(n - kRound * g) : kRound;
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(src + kRound * g), 0, 4 * left, kRawBufferFlags);
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * static_cast<int>(threadIdx.x), 0, 0);
    }
    // f(group) for the thread's groups; returns how many values they hold over all threads,
    // those past the block included
    template <class F>
    __device__ __forceinline__ int64_t each(F f) const {
        if constexpr (HELD) {
#pragma unroll
            for (int g = 0; g < kHeldGroups; ++g)
                if (kRound * g < n) f(held[g]);
        } else {
#pragma unroll 4
            for (int64_t g = 0; kRound * g < n; ++g) f(load(g));
        }
        return (n + kRound - 1) / kRound * kRound;
    }
};

// mu and sigma from exact moments, with the rounding points of the definition
__device__ __forceinline__ void mu_sigma(uint64_t n, uint64_t s1, uint64_t s2, double* mu, double* sigma) {
    *mu = static_cast<double>(s1) / static_cast<double>(n);
    const unsigned __int128 num = static_cast<unsigned __int128>(n) * s2 - static_cast<unsigned __int128>(s1) * s1;
    *sigma = __builtin_sqrt(u128_to_double_rn(num) / static_cast<double>(n * n));
}

// Per (stat block j, DM row d): exact moments, optionally clipped (clip_iters rounds of
// keeping the values within clip_c * sigma of mu, recomputing exact moments over the
// kept values; a round that would keep nothing ends the clipping), then the per-width
// normalisation and each width's smallest passing window sum, one thread a width.
//
// Without clipping the plane's bytes bound it. Clipping is bound by the vector ALUs: a round
// is a range of integers (keep_range), and moments about the range's lower end, which 32 bits
// hold in a thread whenever the range spans less than 2^13, take six instructions a value
// where the float64 rule and 64-bit moments took about 25.
// 1000 x 100,000 in blocks of 8192 with three rounds: 0.12 ms (0.25 ms with a read of the
// block a pass and 64-bit sums). A block's values are held in registers, 64 a thread: with 32
// in twice the threads it took 0.15 ms, because the reductions and the divisions after each
// pass are once a wave. One block of 32,000 in each of 100 rows: 6.9 us (17.6 us with 256
// threads and one thread going through the widths); 3000 x 225,000 in blocks of 32,768 0.43 ms
// (0.46 ms), 6.2 TB/s.
template <int THREADS, bool HELD>
__global__ __launch_bounds__(THREADS) void sps_stats_kernel(const int32_t* __restrict__ dd, int64_t dd_pitch,
                                                            int64_t dd_t0, int64_t t_begin, int64_t t_end,
                                                            int32_t B, int32_t ndm, SpsConst sc,
                                                            double threshold, double clip_c, int32_t clip_iters,
                                                            double* __restrict__ norms, uint32_t* __restrict__ smin,
                                                            int32_t* __restrict__ rowcount) {
    __shared__ uint64_t part[2][3][THREADS / 64];
    const int j = blockIdx.x;
    const int d = blockIdx.y;
    const int64_t lo = t_begin + static_cast<int64_t>(j) * B;
    const int len = t_end - lo >= B ? B : static_cast<int>(t_end - lo);
    const BlockValues<THREADS, HELD> values(dd + static_cast<int64_t>(d) * dd_pitch - dd_t0 + lo, len);
    Moments m{0, 0, 0};
    values.each([&](const u32x4& x) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            m.s1 += x[q];
            m.s2 += static_cast<uint64_t>(x[q]) * x[q];
        }
    });
    m = reduce_moments<false>(m, part[0]);
    m.n = static_cast<uint64_t>(len);
    double mu, sigma;
    mu_sigma(m.n, m.s1, m.s2, &mu, &sigma);
    for (int it = 0; it < clip_iters; ++it) {
        const KeepRange r = keep_range(mu, clip_c * sigma);   // the same in every thread, as are the totals
        if (r.empty) break;
        Moments k{0, 0, 0};
        int64_t slots;
        if (HELD && r.span < (1u << 13)) {   // a thread's 64 squares stay below 2^32 in all
            uint32_t cnt = 0, a = 0, b = 0;
            slots = values.each([&](const u32x4& x) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t y = x[q] - r.lo;
                    const bool in = y <= r.span;
                    const uint32_t z = in ? y : 0u;
                    cnt += in;
                    a += z;
                    b += z * z;
                }
            });
            k = reduce_moments<true>(Moments{cnt, a, b}, part[(it + 1) & 1]);
        } else {
            slots = values.each([&](const u32x4& x) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t y = x[q] - r.lo;
                    if (y <= r.span) {
                        ++k.n;
                        k.s1 += y;
                        k.s2 += static_cast<uint64_t>(y) * y;
                    }
                }
            });
            k = reduce_moments<false>(k, part[(it + 1) & 1]);
        }
        if (r.lo == 0) k.n -= static_cast<uint64_t>(slots - len);   // the zeros past the block were counted
        if (k.n == 0) break;
        // moments about 0 from those about r.lo
        const uint64_t c = r.lo;
        m = Moments{k.n, k.s1 + k.n * c, k.s2 + 2 * c * k.s1 + k.n * c * c};
        mu_sigma(m.n, m.s1, m.s2, &mu, &sigma);
    }
    if (static_cast<int>(threadIdx.x) < sc.nw) {
        const int k = threadIdx.x;
        double* out = norms + (static_cast<int64_t>(j) * ndm + d) * (2 * sc.nw);
        const double wmu = static_cast<double>(sc.widths[k]) * mu;
        const double rw = sigma == 0.0 ? 0.0 : 1.0 / (sigma * sc.sqrtw[k]);
        out[k] = wmu;
        out[sc.nw + k] = rw;
        smin[(static_cast<int64_t>(j) * ndm + d) * sc.nw + k] = min_passing_sum(wmu, rw, threshold);
        if (j == 0 && k == 0) rowcount[d] = 0;
    }
}

// ---- detection ----------------------------------------------------------------
constexpr int kHaloRows = kSpsRows + 2;
constexpr int kHaloCols = kSpsTile + 2;

// 4-column groups of a tile's prefix sums (the starts and the widest boxcar past the last of
// them), and the row stride of a tile's prefix sums with the halo column: entry 1 of a row,
// the prefix at the tile's first start, is 16-byte aligned if the rows begin 12 bytes into
// an aligned buffer.
__host__ __device__ inline int prefix_groups(int wmax) { return (kSpsTile + wmax + 3) / 4; }
__host__ __device__ inline int prefix_row_stride(int wmax) { return 4 * (prefix_groups(wmax) + 1); }
constexpr int kPrefixHead = 12;
__host__ __device__ inline int prefix_bytes(int wmax, int rows) {
    return (kPrefixHead + rows * prefix_row_stride(wmax) * 4 + 15) / 16 * 16;
}
// LDS of a work-group of the exact detection: prefix sums of kHaloRows rows, then the
// float64 best S/N of every halo cell [kHaloRows][kHaloCols].
__host__ __device__ inline int best_lds(int wmax) { return prefix_bytes(wmax, kHaloRows) + kHaloRows * kHaloCols * 8; }

// n columns of row d of the plane from column c on as a buffer: each dword past them, or of
// a trial outside 0 .. ndm - 1, reads as 0. The arguments are the same in every lane.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const int32_t* dd, int64_t dd_pitch, int ndm, int d, int64_t c,
                                                             int n) {
    const bool in = d >= 0 && d < ndm && n > 0;
    const int32_t* src = dd + (in ? d * dd_pitch + c : 0);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(src), 0, __builtin_amdgcn_readfirstlane(in ? 4 * n : 0),
                                             kRawBufferFlags);
}
// columns from col on of a plane of dd_n columns, at most limit
__device__ __forceinline__ int columns_left(int64_t dd_n, int64_t col, int limit) {
    return dd_n - col >= limit ? limit : static_cast<int>(dd_n - col);
}
__device__ __forceinline__ u32x4 load_group(__amdgpu_buffer_rsrc_t rsrc, int u) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * u, 0, 0);
}
// Exclusive prefix sums of a wave's 256 columns (lane l: columns 4 l .. 4 l + 3) on top of
// carry, which moves on to the sum past them.
__device__ __forceinline__ u32x4 scan_group(const u32x4& x, uint32_t& carry) {
    const uint32_t a = x[0], b = a + x[1], c = b + x[2], e = c + x[3];
    const uint32_t incl = wave_incl_scan(e);
    const uint32_t base = carry + (incl - e);
    carry += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
    return u32x4{base, base + a, base + b, base + c};
}

// Prefix sums of N rows of a tile by one wave: trial dt[i] into the row at prow[i], entry j =
// sum of D[t_tile0 - 1 + i] for i < j (modulo 2^32: every window sum is exact below 2^32).
// col is the plane column of the tile's first start. The loads of all rows' first two groups
// (all there are up to a width of 256) are issued before any scan, so that their latencies
// overlap.
template <int N>
__device__ __forceinline__ void tile_prefix(const int32_t* dd, int64_t dd_pitch, int64_t dd_n, int ndm, int64_t col, int nq,
                                            const int (&dt)[N], uint32_t* const (&prow)[N], int lane) {
    u32x4 xs[N][2];
    uint32_t first[N];   // D[t_tile0 - 1], the halo column (0 before the plane's first column)
    const int n = columns_left(dd_n, col, 4 * nq);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const __amdgpu_buffer_rsrc_t rsrc = row_buffer(dd, dd_pitch, ndm, dt[i], col, n);
        const __amdgpu_buffer_rsrc_t halo = row_buffer(dd, dd_pitch, ndm, dt[i], col - 1, col > 0 ? 1 : 0);
        first[i] = __builtin_amdgcn_raw_buffer_load_b32(halo, 0, 0, 0);
        xs[i][0] = load_group(rsrc, lane);
        xs[i][1] = load_group(rsrc, 64 + lane);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t carry = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(first[i])));
        auto scan = [&](const u32x4& x, int u) {
            const u32x4 q = scan_group(x, carry);
            if (u < nq) *reinterpret_cast<u32x4*>(prow[i] + 1 + 4 * u) = q;
        };
        scan(xs[i][0], lane);
        scan(xs[i][1], 64 + lane);
#pragma unroll 1
        for (int u0 = 128; u0 < nq; u0 += 64)
            scan(load_group(row_buffer(dd, dd_pitch, ndm, dt[i], col, n), u0 + lane), u0 + lane);
        if (lane == 0) {
            prow[i][0] = 0u;
            prow[i][1 + 4 * nq] = carry;
        }
    }
}

// One row's normalisation across the lanes of a wave: lane k holds w*mu and 1/(sigma*sqrt(w))
// of width k.
struct RowNorm {
    double wmu, r;
};
__device__ __forceinline__ RowNorm load_norm(const double* nj, int d, bool valid, int nw, int lane) {
    RowNorm n{0.0, 0.0};
    if (valid && lane < nw) {
        const double* p = nj + static_cast<int64_t>(d) * (2 * nw);
        n.wmu = p[lane];
        n.r = p[nw + lane];
    }
    return n;
}
__device__ __forceinline__ double lane_value(double v, int k) {
    union { double d; int i[2]; } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readlane(u.i[0], k);
    u.i[1] = __builtin_amdgcn_readlane(u.i[1], k);
    return u.d;
}

// Best S/N over the widths of N cells of each of R rows, float64, in the oracle's order of
// operations: cell (i, c) has its prefix at pr[i][c], sits at start t[c], and row i has the
// normalisation norm[i]. All cells advance together through the widths, so that their LDS
// reads and float64 operations overlap.
template <int R, int N>
__device__ __forceinline__ void exact_best(const uint32_t* const (&pr)[R][N], const uint32_t (&t)[N],
                                           const RowNorm (&norm)[R], const SpsConst& sc, int wlane, double (&v)[R][N]) {
    uint32_t base[R][N];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int c = 0; c < N; ++c) base[i][c] = pr[i][c][0];
    for (int k = 0; k < sc.nw; ++k) {
        const int w = __builtin_amdgcn_readlane(wlane, k);
        const uint32_t sm = k >= sc.kfull ? static_cast<uint32_t>(sc.smask[k]) : 0u;   // not on this width's grid
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const double wmu = lane_value(norm[i].wmu, k), r = lane_value(norm[i].r, k);
#pragma unroll
            for (int c = 0; c < N; ++c) {
                const uint32_t s = pr[i][c][w] - base[i][c];
                const double snr = (static_cast<double>(s) - wmu) * r;
                if (k == 0 || ((t[c] & sm) == 0 && snr > v[i][c])) v[i][c] = snr;
            }
        }
    }
}

// The exact detection, for searches whose best plane is an output (and for window sums of
// 2^31 and more): float64 best S/N of every cell of a tile of 8 rows and 256 starts with a
// halo of one row and one start on each side, then the 3x3 peak test. Bound by the float64
// operations (three per cell and width): 333 trials of a 77,777-sample band 0.14 ms; with the
// row's normalisation read from the LDS for every cell and width it took 0.26 ms.
__global__ __launch_bounds__(256) void sps_best_kernel(
    const int32_t* __restrict__ dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n, int64_t t_begin,
    int64_t t_end, int64_t t_total, int32_t B, int32_t ndm, double threshold, SpsConst sc,
    const double* __restrict__ norms, int32_t* __restrict__ rowcount,
    uint32_t* __restrict__ mask, int64_t nwords, float* __restrict__ best_out, int64_t best_pitch) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int nw = sc.nw;
    const int nq = prefix_groups(sc.wmax);
    const int ps = prefix_row_stride(sc.wmax);
    uint32_t* pre = reinterpret_cast<uint32_t*>(smem + kPrefixHead);                              // [kHaloRows][ps]
    double* best = reinterpret_cast<double*>(smem + prefix_bytes(sc.wmax, kHaloRows));            // [kHaloRows][kHaloCols]
    __shared__ int32_t cnt[kSpsRows];

    // XCD-aware order: each XCD walks consecutive time tiles of a row block, which share
    // their halo columns in its L2
    const int item = xcd_remap(static_cast<int>(blockIdx.x + blockIdx.y * gridDim.x),
                               static_cast<int>(gridDim.x * gridDim.y));
    const int bx = item % static_cast<int>(gridDim.x), by = item / static_cast<int>(gridDim.x);
    const int64_t tt0 = t_begin + static_cast<int64_t>(bx) * kSpsTile;
    const int64_t tile_end = min(tt0 + kSpsTile, t_end);
    const int d0 = by * kSpsRows;
    const int j = bx / (B / kSpsTile);                // B is a multiple of kSpsTile
    const int64_t lo = max(tt0 - 1, static_cast<int64_t>(0));
    const int64_t hi = (t_total < 0 || tile_end < t_total) ? tile_end + 1 : tile_end;  // best valid in [lo, hi)
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const double* nj = norms + static_cast<int64_t>(j) * ndm * (2 * nw);
    const int wlane = lane < nw ? sc.widths[lane < kMaxWidths ? lane : 0] : 0;   // width of lane k

    // halo row r (trial d0 - 1 + r) belongs to wave r % 4
    {
        const int rows[2] = {wave, wave + 4};
        const int dt[2] = {d0 - 1 + rows[0], d0 - 1 + rows[1]};
        uint32_t* const prow[2] = {pre + rows[0] * ps, pre + rows[1] * ps};
        tile_prefix<2>(dd, dd_pitch, dd_n, ndm, tt0 - dd_t0, nq, dt, prow, lane);
        if (wave + 8 < kHaloRows) {
            const int dl[1] = {d0 - 1 + wave + 8};
            uint32_t* const pl[1] = {pre + (wave + 8) * ps};
            tile_prefix<1>(dd, dd_pitch, dd_n, ndm, tt0 - dd_t0, nq, dl, pl, lane);
        }
    }
    if (tid < kSpsRows) cnt[tid] = 0;
    __syncthreads();
    // halo row r by wave r % 4, a lane's columns lane + 64 q
    constexpr int NC = (kHaloCols + 63) / 64;
    for (int r = wave; r < kHaloRows; r += 4) {
        const int d = d0 - 1 + r;
        const bool in = d >= 0 && d < ndm;
        const RowNorm norm[1] = {load_norm(nj, d, in, nw, lane)};
        const uint32_t* pr[1][NC];
        uint32_t t[NC];
        double v[1][NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int c = min(64 * q + lane, kHaloCols - 1);
            pr[0][q] = pre + r * ps + c;
            t[q] = static_cast<uint32_t>(tt0 - 1 + c);
            v[0][q] = 0.0;
        }
        exact_best<1, NC>(pr, t, norm, sc, wlane, v);
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int c = 64 * q + lane;
            const int64_t tc = tt0 - 1 + c;
            if (c < kHaloCols) best[r * kHaloCols + c] = in && tc >= lo && tc < hi ? v[0][q] : -__builtin_huge_val();
        }
    }
    __syncthreads();
    // 3x3 peak test for the inner rows, 64 consecutive starts per wave step
    for (int item = tid; item < kSpsRows * kSpsTile; item += 256) {
        const int ri = item / kSpsTile, tc = item - ri * kSpsTile;
        const int d = d0 + ri;
        const int64_t t = tt0 + tc;
        bool ok = false;
        if (d < ndm && t < tile_end) {
            const double* m = best + (ri + 1) * kHaloCols + (tc + 1);
            const double v = m[0];
            ok = v >= threshold && v > m[-kHaloCols - 1] && v > m[-kHaloCols] && v > m[-kHaloCols + 1] &&
                 v > m[-1] && v >= m[1] && v >= m[kHaloCols - 1] && v >= m[kHaloCols] && v >= m[kHaloCols + 1];
            if (best_out) best_out[static_cast<int64_t>(d) * best_pitch + (t - t_begin)] = static_cast<float>(v);
        }
        const uint64_t bal = __ballot(ok);
        if (lane == 0 && d < ndm) {
            const int64_t w = (tt0 - t_begin) / 32 + tc / 32;
            *reinterpret_cast<uint64_t*>(mask + static_cast<int64_t>(d) * nwords + w) = bal;
            if (bal) atomicAdd(&cnt[ri], __popcll(bal));
        }
    }
    __syncthreads();
    if (tid < kSpsRows && d0 + tid < ndm && cnt[tid] > 0) atomicAdd(&rowcount[d0 + tid], cnt[tid]);
}

// The screened detection. A wave takes kRunRows adjacent rows (trials) and a run of
// consecutive tiles of 256 starts; lane l holds the four starts 4 l .. 4 l + 3 of each, so
// that a width's prefixes are one aligned 16-byte LDS read (two where the width is not a
// multiple of 4). A cell passes if some width's window sum reaches that width's smallest
// passing sum (min_passing_sum), which is exactly the float64 rule best >= threshold; only
// the cells that pass, with their 8 neighbours, are evaluated in float64 for the 3x3 peak
// decision. The launcher takes this path only when every window sum is below 2^31.
//
// Nothing is shared between waves: the prefix sums of neighbouring rows are only needed
// beside a passing cell, and are then built by the wave that has it. Up to a width of 256 a
// tile's second 256 columns are the next tile's first: their prefix sums stay in registers,
// and the columns after them are loaded while the tile is screened (STEP). Beyond that,
// each tile is built by itself.
//
// The vector ALUs bound it: 3000 trials x 225,000 starts with widths 1, 2 .. 256 take 0.68 ms
// (4 TB/s of plane). Tiles of 8 rows and 256 starts in work-groups, with a prefix for every
// halo row, an LDS read per lane, width and start and the peak test beside the screen, took
// 1.48 ms; 100 x 32,000 with 6 widths took 37.6 us against 16.8 now.
//  - The peak test runs after the run's screen, on the mask words that the lanes hold, so
//    that its registers are not live beside the screen's (with the test inside the loop over
//    tiles, spilled registers made it 2.4 ms).
//  - POW2 (widths 1, 2, 4 .. up to 256): distances are constants, two widths share one
//    three-way maximum and no width needs a branch on its alignment: 0.68 ms against 0.91 ms.
//  - Five waves per SIMD: with four 0.71 ms, with six (spilled registers) 0.85 ms.
// Past a width of 256 a work-group's LDS lets two of them on a CU at 1024 (62 KB), and a tile's
// groups are loaded one after the other; the whole search of the plane above with widths 1, 2 ..
// 1024 takes 4.09 ms (5.00 ms with the tiles of 8 rows), 100 x 32,000 34 us (55 us), seven widths
// to 1000 over 1000 x 100,000 0.62 ms (0.75 ms).
constexpr int kRunRows = 2;
constexpr int kPow2Widths = 9;   // widths 1, 2, 4 .. 256
constexpr int kCellsPerRound = 21;                       // cells of three lanes each
constexpr uint64_t kRoundMask = 0x1249249249249249ull;   // their first lanes
// LDS of one wave: the list of a row's passing cells, then prefix sums of three rows
constexpr int kListBytes = 2 * kCellsPerRound * 4 + 8;
static_assert(kListBytes % 16 == 0, "the prefix sums follow");
__host__ __device__ inline int screen_lds(int wmax) { return kListBytes + prefix_bytes(wmax, kRunRows + 1); }

// Orders a wave's LDS accesses for its lanes' reads of each other's writes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <bool STEP, bool POW2>
__global__ __launch_bounds__(256, 5) void sps_screen_kernel(
    const int32_t* __restrict__ dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n, int64_t t_begin,
    int64_t t_end, int64_t t_total, int32_t B, int32_t ndm, double threshold, SpsConst sc,
    const double* __restrict__ norms, const uint32_t* __restrict__ smin_g, int32_t* __restrict__ rowcount,
    uint32_t* __restrict__ mask, int64_t nwords, int32_t ntiles, int32_t nt, int32_t nruns) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int nw = sc.nw;
    const int nq = prefix_groups(sc.wmax);
    const int ps = prefix_row_stride(sc.wmax);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6), lane = threadIdx.x & 63;
    uint32_t* const list = reinterpret_cast<uint32_t*>(smem + wave * screen_lds(sc.wmax));
    uint8_t* const lds = smem + wave * screen_lds(sc.wmax) + kListBytes;
    uint32_t* const pre = reinterpret_cast<uint32_t*>(lds + kPrefixHead);   // three rows with halo, of a passing cell
    u32x4* const run = reinterpret_cast<u32x4*>(lds);                       // [kRunRows][nq] of the screened tile

    const int item = static_cast<int>(blockIdx.x) * 4 + wave;
    const int d0 = item / nruns * kRunRows;
    const int b0 = item % nruns * nt, b1 = min(b0 + nt, ntiles);
    if (d0 >= ndm) return;
    const int wlane = lane < nw ? sc.widths[lane < kMaxWidths ? lane : 0] : 0;   // width of lane k
    const int per_block = B / kSpsTile;                                          // B is a multiple of kSpsTile

    __amdgpu_buffer_rsrc_t rsrc[kRunRows];
    u32x4 q0[kRunRows], xn[kRunRows];   // prefix sums of the tile's first 256 columns, the next 256 columns
    uint32_t carry[kRunRows];
    {
        const int64_t col = t_begin + static_cast<int64_t>(b0) * kSpsTile - dd_t0;
        const int n = columns_left(dd_n, col, (b1 - b0 - 1) * kSpsTile + 4 * nq);
#pragma unroll
        for (int h = 0; h < kRunRows; ++h) {
            rsrc[h] = row_buffer(dd, dd_pitch, ndm, d0 + h, col, n);
            q0[h] = load_group(rsrc[h], lane);
            xn[h] = load_group(rsrc[h], 64 + lane);
            carry[h] = 0u;
        }
        if constexpr (STEP)
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) q0[h] = scan_group(q0[h], carry[h]);
    }
    uint32_t words[kRunRows] = {};   // lane 8 k + i: mask word i of the run's tile k
    // minus a width's smallest passing window sum (kNever if none): lane k of nsm, ns[k]
    int nsm[kRunRows];
    uint32_t ns[kRunRows][kPow2Widths];
    int next = b0;              // first tile past the stat block of nsm
#pragma unroll 1
    for (int b = b0; b < b1; ++b) {
        const int64_t tt0 = t_begin + static_cast<int64_t>(b) * kSpsTile;
        if (b == next) {
            const int j = b / per_block;
            next = (j + 1) * per_block;
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) {
                uint32_t v = kNever;
                if (lane < nw && d0 + h < ndm) v = smin_g[(static_cast<int64_t>(j) * ndm + d0 + h) * nw + lane];
                nsm[h] = static_cast<int>(0u - v);
                if constexpr (POW2)
#pragma unroll
                    for (int k = 0; k < kPow2Widths; ++k)
                        ns[h][k] = static_cast<uint32_t>(__builtin_amdgcn_readlane(nsm[h], k));
            }
        }
        // prefix sums of the tile
        u32x4 q1[kRunRows];
        if constexpr (STEP) {
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) {
                q1[h] = scan_group(xn[h], carry[h]);
                run[h * nq + lane] = q0[h];
                if (64 + lane < nq) run[h * nq + 64 + lane] = q1[h];
            }
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) xn[h] = load_group(rsrc[h], 64 * (b - b0 + 2) + lane);
        } else {
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) {
                carry[h] = 0u;
                if (b > b0) q0[h] = load_group(rsrc[h], 64 * (b - b0) + lane);
                q0[h] = scan_group(q0[h], carry[h]);
                run[h * nq + lane] = q0[h];
#pragma unroll 1
                for (int u0 = 64; u0 < nq; u0 += 64) {
                    const u32x4 q = scan_group(load_group(rsrc[h], 64 * (b - b0) + u0 + lane), carry[h]);
                    if (u0 + lane < nq) run[h * nq + u0 + lane] = q;
                }
            }
        }
        wave_lds_sync();
        int32_t margin[kRunRows][4];   // max over widths of (window sum - smallest passing sum)
        {
            uint32_t neg[kRunRows][4];
            const u32x4* const pr[kRunRows] = {run + lane, run + nq + lane};   // prefixes at the lane's starts
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    neg[h][q] = 0u - q0[h][q];
                    asm volatile("" : "+v"(neg[h][q]));   // keep each sum one three-way add
                    margin[h][q] = INT32_MIN;
                }
            }
            // sum - smin lies in (-2^31, 2^31): sums are below 2^31 and smin <= 2^31
            auto over = [&](int h, uint32_t n, uint32_t x, int q) { return static_cast<int32_t>(x + neg[h][q] + n); };
            if constexpr (POW2) {
                // width 2^k, k < nw: the prefixes 2^k past the lane's starts are in its own group
                // and the next one for k < 2, and whole groups at constant distances beyond; both
                // rows go together, so that their LDS reads overlap
                u32x4 y[kRunRows];
#pragma unroll
                for (int h = 0; h < kRunRows; ++h) y[h] = pr[h][1];
                auto ahead = [&](auto K, int h) -> u32x4 {
                    if constexpr (K == 0) return u32x4{q0[h][1], q0[h][2], q0[h][3], y[h][0]};
                    else if constexpr (K == 1) return u32x4{q0[h][2], q0[h][3], y[h][0], y[h][1]};
                    else if constexpr (K == 2) return y[h];
                    else return pr[h][1 << (K - 2)];
                };
                auto single = [&](auto K) {
                    if (K < sc.kfull) {
                        u32x4 x[kRunRows];
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h) x[h] = ahead(K, h);
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h)
#pragma unroll
                            for (int q = 0; q < 4; ++q) margin[h][q] = max(over(h, ns[h][K], x[h][q], q), margin[h][q]);
                    } else if (K < nw) {   // at starts that are multiples of smask + 1, a power of two, only
                        const int sm = sc.smask[K];
                        u32x4 x[kRunRows];
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h) x[h] = ahead(K, h);
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h) {
                            const int32_t m = over(h, ns[h][K], x[h][0], 0);
                            if (((4 * lane) & sm) == 0) margin[h][0] = max(m, margin[h][0]);
                            if (sm == 1) margin[h][2] = max(over(h, ns[h][K], x[h][2], 2), margin[h][2]);
                        }
                    }
                };
                auto two = [&](auto K) {
                    constexpr std::integral_constant<int, K + 1> K1{};
                    if (K1 < sc.kfull) {
                        u32x4 x0[kRunRows], x1[kRunRows];
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h) x0[h] = ahead(K, h), x1[h] = ahead(K1, h);
#pragma unroll
                        for (int h = 0; h < kRunRows; ++h)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                margin[h][q] = max(max(over(h, ns[h][K], x0[h][q], q), over(h, ns[h][K1], x1[h][q], q)),
                                                   margin[h][q]);
                    } else {
                        single(K);
                        single(K1);
                    }
                };
                two(std::integral_constant<int, 0>{});
                two(std::integral_constant<int, 2>{});
                two(std::integral_constant<int, 4>{});
                two(std::integral_constant<int, 6>{});
                single(std::integral_constant<int, 8>{});
                static_assert(kPow2Widths == 9, "the widths above");
            } else {
            auto nsmin = [&](int h, int k) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(nsm[h], k)); };
            // one width whose prefixes, entries 4 l + w .. + 3, start A entries into an aligned
            // 16 bytes (the branch on A is uniform and holds the whole update, so that nothing is
            // copied); STRIDED: a width of the decimated hierarchy, whose starts off the width's
            // grid do not count
            auto one = [&](auto A, auto STRIDED, int k, int w) {
                const uint32_t sm = STRIDED ? static_cast<uint32_t>(sc.smask[k]) : 0u;
#pragma unroll
                for (int h = 0; h < kRunRows; ++h) {
                    const u32x4 x = pr[h][w >> 2];
                    u32x4 y = x;
                    if constexpr (A != 0) y = pr[h][(w >> 2) + 1];
                    const uint32_t n = nsmin(h, k);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int32_t m = over(h, n, q + A < 4 ? x[(q + A) & 3] : y[(q + A) & 3], q);
                        if (!STRIDED || (static_cast<uint32_t>(tt0 + 4 * lane + q) & sm) == 0) margin[h][q] = max(m, margin[h][q]);
                    }
                }
            };
            auto any = [&](auto STRIDED, int k, int w) {
                switch (w & 3) {
                    case 0: one(std::integral_constant<int, 0>{}, STRIDED, k, w); break;
                    case 1: one(std::integral_constant<int, 1>{}, STRIDED, k, w); break;
                    case 2: one(std::integral_constant<int, 2>{}, STRIDED, k, w); break;
                    default: one(std::integral_constant<int, 3>{}, STRIDED, k, w);
                }
            };
#pragma unroll 1
            for (int k = 0; k < sc.kfull;) {
                const int w0 = __builtin_amdgcn_readlane(wlane, k);
                const int w1 = k + 1 < sc.kfull ? __builtin_amdgcn_readlane(wlane, k + 1) : 1;
                if (((w0 | w1) & 3) == 0) {   // two aligned widths: one three-way maximum for both
#pragma unroll
                    for (int h = 0; h < kRunRows; ++h) {
                        const u32x4 x0 = pr[h][w0 >> 2], x1 = pr[h][w1 >> 2];
                        const uint32_t n0 = nsmin(h, k), n1 = nsmin(h, k + 1);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            margin[h][q] = max(max(over(h, n0, x0[q], q), over(h, n1, x1[q], q)), margin[h][q]);
                    }
                    k += 2;
                } else {
                    any(std::false_type{}, k, w0);
                    ++k;
                }
            }
#pragma unroll 1
            for (int k = sc.kfull; k < nw; ++k) any(std::true_type{}, k, __builtin_amdgcn_readlane(wlane, k));
            }
        }
        const int nvalid = static_cast<int>(min<int64_t>(kSpsTile, t_end - tt0)) - 4 * lane;   // of the lane's starts
#pragma unroll
        for (int h = 0; h < kRunRows; ++h) {
            if (__ballot(max(max(margin[h][0], margin[h][1]), max(margin[h][2], margin[h][3])) >= 0) != 0) {
                uint32_t pass = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) pass |= static_cast<uint32_t>(margin[h][q] >= 0 && q < nvalid) << q;
                uint32_t word = pass << (4 * (lane & 7));   // lanes 8 i .. 8 i + 7: word i
                word |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(word), 1, 64));
                word |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(word), 2, 64));
                word |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(word), 4, 64));
                word = static_cast<uint32_t>(__shfl(static_cast<int>(word), 8 * (lane & 7), 64));
                if (lane >> 3 == b - b0) words[h] = word;
            }
        }
        wave_lds_sync();   // the next tile overwrites the prefix sums
        if constexpr (STEP)
#pragma unroll
            for (int h = 0; h < kRunRows; ++h) q0[h] = q1[h];
    }
    // the exact peak test of the cells that pass, in place of their bits
#pragma unroll 1
    for (int h = 0; h < kRunRows; ++h) {
        const int d = d0 + h;
        if (d >= ndm) break;
        uint32_t word = h ? words[1] : words[0];
        int found = 0;
        const uint64_t some = __ballot(word != 0);
#pragma unroll 1
        for (int k = 0; k < b1 - b0; ++k) {
            if (((some >> (8 * k)) & 0xff) == 0) continue;
            const int64_t tt0 = t_begin + static_cast<int64_t>(b0 + k) * kSpsTile;
            const int64_t tile_end = min(tt0 + kSpsTile, t_end);
            const double* nj = norms + static_cast<int64_t>((b0 + k) / per_block) * ndm * (2 * nw);
            const uint32_t nibble = static_cast<uint32_t>(__shfl(static_cast<int>(word), 8 * k + (lane >> 3), 64)) >> (4 * (lane & 7));
            if (lane >> 3 == k) word = 0;
            uint64_t pass[4];   // lanes whose start q passes
            int npass = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                pass[q] = __ballot((nibble >> q) & 1u);
                npass += __popcll(pass[q]);
            }
            const int64_t lo = max(tt0 - 1, static_cast<int64_t>(0));
            const int64_t hi = (t_total < 0 || tile_end < t_total) ? tile_end + 1 : tile_end;  // best valid in [lo, hi)
            const int dt[3] = {d - 1, d, d + 1};
            uint32_t* const prow[3] = {pre, pre + ps, pre + 2 * ps};
            const RowNorm norm[3] = {load_norm(nj, d - 1, d > 0, nw, lane), load_norm(nj, d, true, nw, lane),
                                     load_norm(nj, d + 1, d + 1 < ndm, nw, lane)};
            tile_prefix<3>(dd, dd_pitch, dd_n, ndm, tt0 - dd_t0, nq, dt, prow, lane);
            const double ninf = -__builtin_huge_val();
            // a peak at start s of the tile
            auto peaks = [&](uint64_t lanes, int s) {
                found += __popcll(lanes);
                for (; lanes; lanes &= lanes - 1) {
                    const int sl = __builtin_amdgcn_readlane(s, __ffsll(static_cast<unsigned long long>(lanes)) - 1);
                    if (lane == 8 * k + (sl >> 5)) word |= 1u << (sl & 31);
                }
            };
            if (npass <= 2 * kCellsPerRound) {
                // few cells pass: they are listed, and three lanes take one cell, one column of
                // its 3 x 3 neighbourhood each
                int below = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if ((pass[q] >> lane) & 1u) list[below + __popcll(pass[q] & ((1ull << lane) - 1))] = 4 * lane + q;
                    below += __popcll(pass[q]);
                }
                wave_lds_sync();
#pragma unroll 1
                for (int i0 = 0; i0 < npass; i0 += kCellsPerRound) {
                    const int i = lane / 3, e = lane - 3 * i;             // cell of the round, column - 1
                    const bool have = i < kCellsPerRound && i0 + i < npass;
                    const int s = have ? static_cast<int>(list[i0 + i]) : 0;
                    const int64_t tr = tt0 + s - 1 + e;
                    const uint32_t* const p0 = pre + s + e;
                    const uint32_t* const pr[3][1] = {{p0}, {p0 + ps}, {p0 + 2 * ps}};
                    const uint32_t t[1] = {static_cast<uint32_t>(tr)};
                    double v[3][1] = {};
                    exact_best<3, 1>(pr, t, norm, sc, wlane, v);
                    const bool in = tr >= lo && tr < hi;
                    const double up = in && d > 0 ? v[0][0] : ninf, mid = in ? v[1][0] : ninf;
                    const double down = in && d + 1 < ndm ? v[2][0] : ninf;
                    const double x = __shfl(mid, 3 * i + 1, 64);          // the cell's own S/N
                    const bool beside = e == 0 ? x > mid : (e == 1 ? x >= threshold : x >= mid);
                    uint64_t ok = __ballot(have && x > up && beside && x >= down);
                    ok &= ok >> 1 & ok >> 2 & kRoundMask;
                    peaks(ok, s);
                }
            } else {
                // all starts of three rows, four a lane, the halo columns in the outer lanes
                wave_lds_sync();
                double x[4];
                bool ok[4];
#pragma unroll 1
                for (int e = 0; e < 3; ++e) {
                    const int i = e == 0 ? 1 : e == 1 ? 0 : 2;            // the cells' own row first
                    const RowNorm rn[1] = {e == 0 ? norm[1] : e == 1 ? norm[0] : norm[2]};
                    const uint32_t* pr[1][4];
                    uint32_t t[4];
                    double v[1][4] = {};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        pr[0][q] = pre + i * ps + 4 * lane + q + 1;
                        t[q] = static_cast<uint32_t>(tt0 + 4 * lane + q);
                    }
                    exact_best<1, 4>(pr, t, rn, sc, wlane, v);
                    const int ch = lane < 32 ? 0 : kHaloCols - 1;
                    const uint32_t* const ph[1][1] = {{pre + i * ps + ch}};
                    const uint32_t th[1] = {static_cast<uint32_t>(tt0 - 1 + ch)};
                    double vh[1][1] = {};
                    exact_best<1, 1>(ph, th, rn, sc, wlane, vh);
                    const bool in_row = d - 1 + i >= 0 && d - 1 + i < ndm;
                    auto valid = [&](double u, int64_t tr) { return in_row && tr >= lo && tr < hi ? u : ninf; };
                    double m[6];                                          // columns 4 lane - 1 .. 4 lane + 4
#pragma unroll
                    for (int q = 0; q < 4; ++q) m[1 + q] = valid(v[0][q], tt0 + 4 * lane + q);
                    vh[0][0] = valid(vh[0][0], tt0 - 1 + ch);
                    m[0] = __shfl_up(m[4], 1, 64);
                    m[5] = __shfl_down(m[1], 1, 64);
                    if (lane == 0) m[0] = vh[0][0];
                    if (lane == 63) m[5] = vh[0][0];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (e == 0) {
                            x[q] = m[1 + q];
                            ok[q] = ((pass[q] >> lane) & 1u) != 0 && x[q] >= threshold && x[q] > m[q] && x[q] >= m[2 + q];
                        } else if (e == 1) {
                            ok[q] = ok[q] && x[q] > m[q] && x[q] > m[1 + q] && x[q] > m[2 + q];
                        } else {
                            ok[q] = ok[q] && x[q] >= m[q] && x[q] >= m[1 + q] && x[q] >= m[2 + q];
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) peaks(__ballot(ok[q]), 4 * lane + q);
            }
            wave_lds_sync();   // the next tile overwrites the prefix sums
        }
        if (lane < 8 * (b1 - b0)) mask[static_cast<int64_t>(d) * nwords + static_cast<int64_t>(b0) * (kSpsTile / 32) + lane] = word;
        if (lane == 0 && found > 0) atomicAdd(&rowcount[d], found);
    }
}

// ---- emission -------------------------------------------------------------------
// A chain of dependent loads bounds a row: its count, its mask words, its norms and samples.
// So a thread loads 64 bytes of mask at a time, the loop ends with the row's last candidate,
// and a candidate's widths are taken by the lanes of a wave, their norms loaded at once.
// 3000 rows of 225,000 starts: 29 us (58 us with a dword a thread and a load of each width's
// norms in turn); 100 rows of a 2^18-sample chunk: 8.3 us (27 us).
constexpr int kEmitList = 1024;   // candidates listed per batch in LDS
constexpr int kEmitWords = 16;    // mask words of a thread at a time
__device__ int block_excl_scan(int v, int* total, int* sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) base += sh[w];
        tot += sh[w];
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

__global__ __launch_bounds__(256) void sps_emit_kernel(
    const int32_t* __restrict__ dd, int64_t dd_pitch, int64_t dd_t0, int64_t t_begin, int32_t B,
    int32_t ndm, SpsConst sc, const double* __restrict__ norms, const int32_t* __restrict__ rowcount,
    const uint32_t* __restrict__ mask, int64_t nwords, aa_candidate_t* __restrict__ cand, int32_t cap,
    int32_t* __restrict__ count, int32_t beam_id) {
    __shared__ int sh[4];
    __shared__ int64_t red[4];
    const int d = blockIdx.x;
    // the counts of the rows before, 16 bytes a load (rowcount is 16-byte aligned)
    int64_t off = 0;
    for (int i = 4 * threadIdx.x; i < d; i += 1024) {
        if (i + 4 <= d) {
            const u32x4 c = *reinterpret_cast<const u32x4*>(rowcount + i);
            off += static_cast<int64_t>(c[0]) + c[1] + c[2] + c[3];
        } else {
            for (int e = i; e < d; ++e) off += rowcount[e];
        }
    }
    off = static_cast<int64_t>(wave_sum_u64(static_cast<uint64_t>(off)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = off;
    __syncthreads();
    off = red[0] + red[1] + red[2] + red[3];
    const int mine = rowcount[d];
    if (d == ndm - 1 && threadIdx.x == 0) *count = static_cast<int32_t>(min<int64_t>(off + mine, 0x7fffffff));
    if (mine == 0 || off >= cap) return;
    const int32_t* row = dd + static_cast<int64_t>(d) * dd_pitch - dd_t0;
    int64_t running = off;
    __shared__ int64_t tl[kEmitList];   // starts of one batch of the row's candidates, in order
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wlane = sc.widths[lane < sc.nw ? lane : 0];                                             // of width lane
    const uint32_t smlane = lane >= sc.kfull && lane < sc.nw ? static_cast<uint32_t>(sc.smask[lane]) : 0u;
    // kEmitWords consecutive mask words a thread (a row's words are a multiple of 8, 32-byte
    // aligned), until all of the row's candidates are found
    for (int64_t k0 = 0; k0 < nwords; k0 += 256 * kEmitWords) {
        const int64_t k = k0 + kEmitWords * threadIdx.x;
        const u32x4* const m = reinterpret_cast<const u32x4*>(mask + static_cast<int64_t>(d) * nwords + k);
        u32x4 words[kEmitWords / 4];
        int have = 0;
#pragma unroll
        for (int g = 0; g < kEmitWords / 4; ++g) words[g] = k + 4 * g < nwords ? m[g] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int g = 0; g < kEmitWords; ++g) have += __popc(words[g / 4][g % 4]);
        int total;
        const int excl = block_excl_scan(have, &total, sh);
        for (int b0 = 0; b0 < total; b0 += kEmitList) {
            // list the batch's starts, then one wave per candidate
            int idx = excl;
            if (have)
#pragma unroll
                for (int g = 0; g < kEmitWords; ++g)
                    for (uint32_t wv = words[g / 4][g % 4]; wv; wv &= wv - 1, ++idx)
                        if (idx >= b0 && idx < b0 + kEmitList) tl[idx - b0] = t_begin + 32 * (k + g) + (__ffs(wv) - 1);
            __syncthreads();
            const int nb = min(kEmitList, total - b0);
            for (int i = wave; i < nb && running + b0 + i < cap; i += 4) {
                const int64_t t = tl[i];
                const int jb = static_cast<int>((t - t_begin) / kSpsTile) / (B / kSpsTile);   // its stat block
                const RowNorm norm = load_norm(norms + static_cast<int64_t>(jb) * ndm * (2 * sc.nw), d, true, sc.nw, lane);
                // window sums from a wave scan: lane l holds samples c0 + 4 l .. c0 + 4 l + 3
                // of each 256-sample chunk, then lane k takes width k's sum and S/N
                uint32_t sum = 0, carry = 0;
                for (int c0 = 0; c0 < sc.wmax; c0 += 256) {
                    uint32_t x[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int ix = c0 + 4 * lane + e;
                        x[e] = ix < sc.wmax ? static_cast<uint32_t>(row[t + ix]) : 0u;
                    }
                    const uint32_t p1 = x[0] + x[1], p2 = p1 + x[2], p3 = p2 + x[3];
                    const uint32_t incl = wave_incl_scan(p3);
                    const uint32_t base = carry + (incl - p3);
                    const uint32_t pre4[4] = {base + x[0], base + p1, base + p2, base + p3};
                    const int ix = wlane - 1 - c0;               // sum of the first wlane samples
                    uint32_t sel = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t p = static_cast<uint32_t>(__shfl(static_cast<int>(pre4[e]), (ix >> 2) & 63, 64));
                        if ((ix & 3) == e) sel = p;
                    }
                    if (ix >= 0 && ix < 256) sum = sel;
                    carry += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
                }
                // the smallest best width, in the order of the detection's exact evaluation
                const double snr = (static_cast<double>(sum) - norm.wmu) * norm.r;
                const uint64_t tried = __ballot(lane < sc.nw && (static_cast<uint32_t>(t) & smlane) == 0);
                double v = lane_value(snr, 0);
                int best = 0;
                for (int q = 1; q < sc.nw; ++q) {
                    const double s = lane_value(snr, q);
                    if (((tried >> q) & 1u) && s > v) {
                        v = s;
                        best = q;
                    }
                }
                const int wbest = __builtin_amdgcn_readlane(wlane, best);
                if (lane == 0) {
                    aa_candidate_t c;
                    c.dm_idx = d;
                    c.width = wbest;
                    c.t = t;
                    c.snr = static_cast<float>(v);
                    c.beam = beam_id;
                    cand[running + b0 + i] = c;
                }
            }
            __syncthreads();
        }
        running += total;
        if (running >= cap || running - off == mine) break;
    }
}

// Tiles of a run of the screened detection: as few as still let all waves be resident at once
// (five per SIMD), at most 8 (the mask words of a row's run are one dword per lane). 3000 x
// 225,000 cells: 0.69 ms with 8, 0.78 with 4, 1.54 with 1, and 0.73 with 16 (two dwords a lane);
// 100 x 32,000 cells: 16.8 us with 2 (this rule), 17.6 with 1 or 3.
constexpr int64_t kScreenWaves = 5120;
constexpr int64_t kMaxRun = 8;

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct WorkLayout {
    size_t norms, smin, rowcount, mask, total;
    int64_t nblk, ntiles, nwords;
};

WorkLayout layout(const aa_plan_s* p, int64_t n_starts) {
    WorkLayout L{};
    L.nblk = (n_starts + p->stat_block - 1) / p->stat_block;
    L.ntiles = (n_starts + kSpsTile - 1) / kSpsTile;
    L.nwords = L.ntiles * (kSpsTile / 32);
    L.norms = 0;
    L.smin = align256(static_cast<size_t>(L.nblk) * p->ndm * 2 * p->nwidths * sizeof(double));
    L.rowcount = L.smin + align256(static_cast<size_t>(L.nblk) * p->ndm * p->nwidths * sizeof(uint32_t));
    L.mask = L.rowcount + align256(static_cast<size_t>(p->ndm) * sizeof(int32_t));
    L.total = L.mask + align256(static_cast<size_t>(p->ndm) * L.nwords * sizeof(uint32_t));
    return L;
}

}  // namespace

size_t sps_work_bytes(const aa_plan_s* p, int64_t n_starts) { return n_starts > 0 ? layout(p, n_starts).total : 0; }

int launch_single_pulse(const aa_plan_s* p, const int32_t* d_dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n,
                        int64_t t_begin, int64_t t_end, int64_t t_total, void* d_work, aa_candidate_t* d_cand,
                        int32_t cap, int32_t* d_count, float* d_best, int64_t best_pitch, hipStream_t stream,
                        int32_t beam_id) {
    const int64_t n = t_end - t_begin;
    const WorkLayout L = layout(p, n);
    uint8_t* w = static_cast<uint8_t*>(d_work);
    double* norms = reinterpret_cast<double*>(w + L.norms);
    uint32_t* smin = reinterpret_cast<uint32_t*>(w + L.smin);
    int32_t* rowcount = reinterpret_cast<int32_t*>(w + L.rowcount);
    uint32_t* mask = reinterpret_cast<uint32_t*>(w + L.mask);
    SpsConst sc{};
    sc.nw = p->nwidths;
    sc.wmax = p->wmax;
    sc.kfull = p->nwidths;
    for (int k = 0; k < p->nwidths; ++k) {
        sc.widths[k] = p->widths[k];
        sc.sqrtw[k] = p->sqrtw[k];
        int64_t stride = 1;   // smallest power of two with full_width * stride >= width
        if (p->boxcar_full_width > 0)
            while (static_cast<int64_t>(p->boxcar_full_width) * stride < p->widths[k]) stride *= 2;
        sc.smask[k] = static_cast<int32_t>(stride - 1);
        if (stride > 1 && sc.kfull == p->nwidths) sc.kfull = k;   // widths ascend: the rest are strided too
    }
    // a block of up to 64 values a thread is held in registers (more would spill); larger ones
    // are read on each pass
    const int B = p->stat_block;
    const int threads = B <= 64 * 128 ? 128 : B <= 64 * 256 ? 256 : B <= 64 * 512 ? 512 : 1024;
    const auto stats = B <= 64 * 128   ? sps_stats_kernel<128, true>
                       : B <= 64 * 256 ? sps_stats_kernel<256, true>
                       : B <= 64 * 512 ? sps_stats_kernel<512, true>
                                       : sps_stats_kernel<1024, false>;
    hipLaunchKernelGGL(stats, dim3(static_cast<unsigned>(L.nblk), static_cast<unsigned>(p->ndm)), dim3(threads),
                       0, stream, d_dd, dd_pitch, dd_t0, t_begin, t_end, B, p->ndm, sc,
                       static_cast<double>(p->threshold), static_cast<double>(p->clip_sigma),
                       p->clip_sigma > 0.0f ? p->clip_iters : 0, norms, smin, rowcount);
    AA_HIP(hipGetLastError());
    const unsigned rowblocks = static_cast<unsigned>((p->ndm + kSpsRows - 1) / kSpsRows);
    if (L.ntiles * static_cast<int64_t>(rowblocks) > 0x7fffffff)
        return fail(AA_EINVAL, "aa_single_pulse: too many detection tiles for one launch");
    // the integer screen compares window sums below 2^31
    const bool screen = !d_best && static_cast<uint64_t>(p->nchan) * 255u * static_cast<uint64_t>(p->wmax) < (1ull << 31);
    if (screen) {
        const int64_t rowpairs = (p->ndm + kRunRows - 1) / kRunRows;
        const int64_t nt = std::max<int64_t>(1, std::min<int64_t>(kMaxRun, (L.ntiles * rowpairs + kScreenWaves - 1) / kScreenWaves));
        const int64_t nruns = (L.ntiles + nt - 1) / nt;
        // widths 1, 2, 4 .. 256 (with or without the decimated hierarchy) have their own kernel:
        // 0.68 ms against 0.91 ms of the general one for 3000 x 225,000 cells, 0.13 against
        // 0.18 ms for 1000 x 100,000 with the hierarchy; past a width of 256 a tile's prefix
        // sums no longer fit two groups of 256 columns
        bool pow2 = p->nwidths <= kPow2Widths;
        for (int k = 0; k < p->nwidths; ++k) pow2 = pow2 && p->widths[k] == 1 << k;
        hipLaunchKernelGGL(pow2 ? (sps_screen_kernel<true, true>)
                                : p->wmax <= kSpsTile ? (sps_screen_kernel<true, false>) : (sps_screen_kernel<false, false>),
                           dim3(static_cast<unsigned>((nruns * rowpairs + 3) / 4)), dim3(256),
                           static_cast<size_t>(4 * screen_lds(p->wmax)), stream, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end,
                           t_total, p->stat_block, p->ndm, static_cast<double>(p->threshold), sc, norms, smin, rowcount,
                           mask, L.nwords, static_cast<int32_t>(L.ntiles), static_cast<int32_t>(nt),
                           static_cast<int32_t>(nruns));
    } else {
        hipLaunchKernelGGL(sps_best_kernel, dim3(static_cast<unsigned>(L.ntiles), rowblocks), dim3(256),
                           static_cast<size_t>(best_lds(p->wmax)), stream, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end,
                           t_total, p->stat_block, p->ndm, static_cast<double>(p->threshold), sc, norms, rowcount, mask,
                           L.nwords, d_best, best_pitch);
    }
    AA_HIP(hipGetLastError());
    hipLaunchKernelGGL(sps_emit_kernel, dim3(static_cast<unsigned>(p->ndm)), dim3(256), 0, stream, d_dd, dd_pitch,
                       dd_t0, t_begin, p->stat_block, p->ndm, sc, norms, rowcount, mask, L.nwords, d_cand, cap,
                       d_count, beam_id);
    AA_HIP(hipGetLastError());
    return AA_OK;
}

}  // namespace aa

extern "C" int aa_single_pulse_work_bytes(aa_plan_t p, int64_t n_starts, size_t* out) {
    using namespace aa;
    if (!p || !out || n_starts < 1) return fail(AA_EINVAL, "aa_single_pulse_work_bytes: bad argument");
    *out = sps_work_bytes(p, n_starts);
    return AA_OK;
}

namespace aa {
namespace {
// Argument checks shared by aa_single_pulse and aa_single_pulse_noalloc.
int check_single_pulse(const char* fn, aa_plan_t p, const int32_t* d_dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n,
                       int64_t t_begin, int64_t t_end, int64_t t_total, aa_candidate_t* d_cand, int32_t cap,
                       int32_t* d_count, float* d_best, int64_t best_pitch) {
    const std::string f(fn);
    if (!p || !d_dd || !d_count || (cap > 0 && !d_cand)) return fail(AA_EINVAL, f + ": null argument");
    if (p->device < 0) return fail(AA_EINVAL, f + ": plan was created host-only");
    if (p->nwidths > kMaxWidths) return fail(AA_EINVAL, f + ": more than 32 widths");
    if (cap < 0) return fail(AA_EINVAL, f + ": cap < 0");
    if (t_begin < 0 || t_end <= t_begin || t_begin % p->stat_block)
        return fail(AA_EINVAL, f + ": need 0 <= t_begin < t_end and t_begin a multiple of stat_block");
    if (t_total >= 0 && t_end > t_total) return fail(AA_EINVAL, f + ": t_end > t_total");
    if (dd_n < 1 || dd_n > dd_pitch) return fail(AA_EINVAL, f + ": need 1 <= dd_n <= dd_pitch");
    if (dd_t0 > (t_begin > 0 ? t_begin - 1 : t_begin)) return fail(AA_EINVAL, f + ": plane misses the left halo column");
    const int64_t right = (t_total >= 0 && t_end >= t_total) ? t_end : t_end + 1;
    if (dd_t0 + dd_n < right + p->wmax - 1) return fail(AA_EINVAL, f + ": plane too short for the right edge");
    if (d_best && best_pitch < t_end - t_begin) return fail(AA_EINVAL, f + ": best_pitch too small");
    return AA_OK;
}

// Scratch of aa_single_pulse_noalloc: one copy per GPU, alive until the process ends.
// Host code never passes `scratch` itself to a kernel (in host code the name is only a
// stand-in for the symbol): it passes the device address that hipGetSymbolAddress
// returned for the current device.
__device__ __align__(256) uint8_t scratch[AA_NOALLOC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
void* g_scratch_ptr[256] = {};

// The device address of `scratch` on the current device, looked up once per device.
int scratch_ptr(void** out) {
    int dev = 0;
    AA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 256) return fail(AA_EINVAL, "aa_single_pulse_noalloc: device index out of range");
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return hip_fail(e, "aa_single_pulse_noalloc: hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return AA_OK;
}
}  // namespace
}  // namespace aa

extern "C" int aa_single_pulse(aa_plan_t p, const int32_t* d_dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n,
                               int64_t t_begin, int64_t t_end, int64_t t_total, void* d_work, size_t work_bytes,
                               aa_candidate_t* d_cand, int32_t cap, int32_t* d_count, float* d_best,
                               int64_t best_pitch, void* stream) {
    using namespace aa;
    if (!d_work) return fail(AA_EINVAL, "aa_single_pulse: null argument");
    const int rc = check_single_pulse("aa_single_pulse", p, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end, t_total, d_cand,
                                      cap, d_count, d_best, best_pitch);
    if (rc != AA_OK) return rc;
    if (work_bytes < sps_work_bytes(p, t_end - t_begin)) return fail(AA_EINVAL, "aa_single_pulse: work buffer too small");
    if (reinterpret_cast<uintptr_t>(d_work) & 255) return fail(AA_EINVAL, "aa_single_pulse: d_work must be 256-byte aligned");
    return launch_single_pulse(p, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end, t_total, d_work, d_cand, cap, d_count,
                               d_best, best_pitch, static_cast<hipStream_t>(stream));
}

extern "C" int aa_single_pulse_noalloc(aa_plan_t p, const int32_t* d_dd, int64_t dd_pitch, int64_t dd_t0, int64_t dd_n,
                                       int64_t t_begin, int64_t t_end, int64_t t_total, aa_candidate_t* d_cand,
                                       int32_t cap, int32_t* d_count, float* d_best, int64_t best_pitch, void* stream) {
    using namespace aa;
    int rc = check_single_pulse("aa_single_pulse_noalloc", p, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end, t_total,
                                d_cand, cap, d_count, d_best, best_pitch);
    if (rc != AA_OK) return rc;
    const size_t need = sps_work_bytes(p, t_end - t_begin);
    if (need > static_cast<size_t>(AA_NOALLOC_SCRATCH_BYTES))
        return fail(AA_EINVAL, "aa_single_pulse_noalloc: the search needs " + std::to_string(need) +
                                   " bytes of scratch, more than the fixed " +
                                   std::to_string(static_cast<size_t>(AA_NOALLOC_SCRATCH_BYTES)) +
                                   "; use aa_single_pulse with a work buffer or search fewer starts per call");
    void* ptr = nullptr;
    rc = scratch_ptr(&ptr);
    if (rc != AA_OK) return rc;
    // every scratch word the kernels read is written first in the same call (moments,
    // norms, row counts cleared by the statistics kernel, every mask word by detection)
    return launch_single_pulse(p, d_dd, dd_pitch, dd_t0, dd_n, t_begin, t_end, t_total, ptr, d_cand, cap, d_count,
                               d_best, best_pitch, static_cast<hipStream_t>(stream));
}
