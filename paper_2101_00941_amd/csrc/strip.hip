// Strip kernels (layout 8): brute-force dedispersion as an exact one-hot int8 contraction on
// the matrix cores, arranged so that the matrix cores and not the step around them set the
// pace. The contraction itself (residual windows of the input against a one-hot matrix per
// channel group, partial sums on a shifted time axis t', added into the output tile at t' - e
// when a run of channels ends) is that of the layouts 4-6; tables in aa_internal.h.
//  * Sixteen waves per work-group, four per SIMD: 12 contract and 4 stage the input rows. A
//    wave that does both is slowed by its own instruction stream (address arithmetic, loads
//    that queue for the address unit): measured, such a step took 1400 cycles for 512 of
//    matrix work.
//  * A contracting wave owns one strip of 128 rows of t': row 4 R + j of the strip is row R
//    of its matrix tile j. A lane then needs, for its four tiles, one dword-aligned span of
//    each channel (2 dwords for R = 4 residuals, 3 for R = 8), and tile j's window is that
//    span shifted by the constant j bytes (v_alignbyte_b32).
//  * Rows are staged through registers and aligned to their exact start, four channels to a
//    16-byte LDS entry per dword of time, with the sign flip (XOR 0x80) done once per staged
//    dword. So the operand reads are wide LDS reads at constant offsets: no window
//    addresses, phases or sign flips remain in the matrix loop.
//  * A step is two groups of 8 channels and one barrier. The LDS ring holds two steps: in
//    step k the contracting waves run the matrix ops of step k on operands already in
//    registers and read those of step k + 1, while the staging waves store step k + 2. So a
//    step's LDS reads are waited for once, with its barrier, and not between its matrix ops.
// Measured against the 4 x 8 step kernel with 1024-sample tiles (variant 25): 4096 channels x
// 2^20 samples, 3000 trials 106 ms (230 ms; 117 T byte-adds/s), 1500 trials of a 2^17-sample
// chunk 5.8 ms (14.1 ms), 333 trials of 1001 channels x 77,777 samples 0.60 ms (0.96 ms). On the
// chunk matrix cores are busy 31% of the SIMDs' cycles, other vector instructions 38%, and 45% of
// the waves' cycles are waits. About ten vector instructions go with a matrix operation: three
// shift its window (tile 0 needs none), its share of the one-hot operand, which the four tiles
// have in common, is 1.25 (8 channels x 4 residuals) or 3.5 to 4 (4 x 8), and the other half is
// staging, flush and the loop. Launches with little to do are the step kernel's (launch_variant).
#include "dedisp_device.h"

namespace aa {
namespace {

constexpr int kContract = kStripWaves;              // contracting waves
constexpr int kStage = 4;                           // staging waves
constexpr int kThreads = 64 * (kContract + kStage);
constexpr int kAcc0 = 128;                          // LDS: accumulator rows -1 .. TILE, row 0 here
constexpr int kQuadBytes = kStripRowDwords * 16;    // four staged rows
constexpr int kGroupBytes = 2 * kQuadBytes;
constexpr int strip_ring(int tile) { return (tile + 2) * 128; }
constexpr int strip_recs(int tile) { return strip_ring(tile) + 4 * kGroupBytes; }   // 256 bytes per group

// Entry td of a quad lies at td with its low bit flipped in every other group of 8, so that
// lanes that store two entries 32 bytes apart hit all banks.
__device__ __forceinline__ int entry_at(int td) { return 16 * (td ^ ((td >> 3) & 1)); }

__device__ __forceinline__ void step_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Adds a wave's strip q of a finished run into the accumulator tile and clears its
// accumulators: register i of tile j of lane (m, h) is row 128 q + 4 (8 (i / 4) + 4 h + i % 4)
// + j of t', trial m, and goes to t = t' - e; rows outside [0, TILE) are clamped to the
// discarded rows -1 and TILE. A wave's 64 adds hit 32 banks twice each, for any e. The LDS
// takes one add instruction per 4.2 cycles (measured, and the same for stores), which hides
// the clamps of the four SIMDs: strips that lie inside the tile, added without clamps in a
// branch of their own, gained nothing (100 trials of a 2^18-sample chunk 0.158 ms, 0.149 so).
// The asm statements read the accumulators behind the compiler's back, so the wait for the
// matrix operations is stated (wait_matrix_results); beside 64 adds it costs nothing measurable
// (4096 channels x 2^20 samples, dedispersion and search 109.64 ms with and without it).
// Address and add are one block of instructions with one register between them: left to the
// compiler, the addresses of many adds were formed ahead, and the batch kernel, whose item loop
// holds a few registers more, spilled (five beams 6.2 ms, 7.8 that way).
template <int TILE>
__device__ __forceinline__ void strip_flush(i32x16 (&acc)[4], int q, int m, int h, int e, uint32_t row0) {
    const int lo = static_cast<int>(row0) + 4 * m - 128, hi = static_cast<int>(row0) + 4 * m + 128 * TILE;
    const int base = lo + 128 + 128 * (kStripRows * q + 16 * h - e);
    wait_matrix_results(acc);
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int at;
            asm volatile("v_add_u32 %0, %1, %2\n\tv_med3_i32 %0, %0, %3, %4\n\tds_add_u32 %0, %5"
                         : "=&v"(at)
                         : "n"(128 * (4 * (8 * (i >> 2) + (i & 3)) + j)), "v"(base), "v"(lo), "v"(hi), "v"(acc[j][i])
                         : "memory");
        }
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = i32x16{};
}

// The staging waves. Wave p stages quad p of the four of every step, PASSES loads of two dwords per lane and row, straight
// from the rows' byte-exact starts. Unaligned, the loads run at half of the L1 rate (16
// cycles per 512-byte load instruction, measured), but aligned ones would need three more
// vector operations per dword, and the staging waves' instruction stream is what the step
// waits for.
// EDGE: rows of the tile may start before sample 0 or run past the input's end (or row
// offsets do not fit 31 bits).
template <int TILE, int PASSES, bool EDGE>
__device__ __forceinline__ void strip_stage(const DedispArgs& A, const DmBlock& b, int blk, int64_t t0, uint8_t* lds,
                                            int p, int lane, int K) {
    constexpr int D = EDGE ? 2 : PASSES == 2 ? 4 : 3;   // steps of loads in registers, as many as fit
    const int64_t pitch = A.in_pitch;
    const uint32_t* const recs = reinterpret_cast<const uint32_t*>(A.offs) + static_cast<int64_t>(b.rec256) * 64;
    const int32_t* const rsv = A.base + static_cast<int64_t>(blk) * A.nchan_pad;
    const int group = p >> 1;                         // of the step
    int wdst[PASSES][2];
#pragma unroll
    for (int s = 0; s < PASSES; ++s)
#pragma unroll
        for (int l = 0; l < 2; ++l) wdst[s][l] = strip_ring(TILE) + (p & 1) * kQuadBytes + entry_at(128 * s + 2 * lane + l);

    // One buffer resource per step, based kStripBias bytes before its first row at the time tile; a
    // row is reached through the scalar offset, which the range check counts: channels that
    // do not exist carry an offset beyond the range and read zeros (they enter the sums as
    // -128 per channel like every zero byte, and the final correction counts them). An EDGE
    // tile takes a resource per row and keeps every load inside [0, n_in16) of it: a lane that
    // would read outside moves to the nearest dword inside, and its bytes are shifted back to
    // their places when they are written to LDS (bytes from outside only reach outputs that
    // are not stored).
    const uint8_t* sbase = EDGE ? A.in + 4 * p * pitch : A.in + t0 - kStripBias;
    int nstep = 0;             // next step to load
    // per-step tables, 64 steps at a time, lane l holding step 64 n + l
    u32x4 off_tab{};           // offsets of the quad's rows from the step's base
    uint32_t st[D][PASSES][2][4];   // dwords in flight, [stage][pass][dword][channel]
    uint32_t st_rec[D];        // record dwords in flight (waves 0 and 1: of group `p` of the step)
    int st_lo[D][4], st_hi[D][4];   // EDGE: bounds of each row's byte positions
    const __amdgpu_buffer_rsrc_t rec_rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(recs), 0, 256 * (A.nchan_pad >> 3), kRawBufferFlags);
    auto issue = [&](int s) {
        if ((nstep & 63) == 0) {
            const int c = 16 * (nstep + lane) + 4 * p;
            off_tab = c < A.nchan_pad ? *reinterpret_cast<const u32x4*>(rsv + c) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (!EDGE) off_tab[i] += static_cast<uint32_t>(kStripBias + (4 * p + i) * pitch);
                if (c + i >= A.nchan) off_tab[i] = kStripNoRow;
            }
            // wait for the tables here, so that the steps that do not load them need no wait
            asm volatile("" : "+v"(off_tab));
        }
        const int sl = nstep & 63;
        uint32_t so[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) so[i] = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(off_tab[i]), sl));
        const int voff = 8 * lane;
        if constexpr (!EDGE) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint8_t*>(sbase), 0, static_cast<int>(kStripNoRow), kRawBufferFlags);
#pragma unroll
            for (int q = 0; q < PASSES; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto x = __builtin_amdgcn_raw_buffer_load_b64(rs, voff + 512 * q, so[i], 0);
                    st[s][q][0][i] = x[0];
                    st[s][q][1][i] = x[1];
                }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool real = so[i] != kStripNoRow;
                const int64_t first = t0 + static_cast<int32_t>(so[i]);
                const int hi = real ? static_cast<int>(min(A.n_in16 - 4 - first, int64_t{1} << 20)) : 1 << 20;
                const int lo = real ? (first < 0 ? static_cast<int>(-first) : min(hi, 0)) : 0;
                st_lo[s][i] = lo;
                st_hi[s][i] = hi;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<uint8_t*>(sbase + i * pitch + (real ? first + lo : 0)), 0, real ? hi - lo + 4 : 0,
                    kRawBufferFlags);
#pragma unroll
                for (int q = 0; q < PASSES; ++q)
#pragma unroll
                    for (int l = 0; l < 2; ++l)
                        st[s][q][l][i] = __builtin_amdgcn_raw_buffer_load_b32(
                            rs, min(max(voff + 4 * (128 * q + l), lo), hi) - lo, 0, 0);
            }
        }
        st_rec[s] = __builtin_amdgcn_raw_buffer_load_b32(rec_rs, 4 * lane, 256 * (2 * nstep + (p & 1)), 0);
        ++nstep;
        sbase += 16 * pitch;
    };
    // step n from stage s into its half of the ring
    auto write = [&](int s, int n) {
        uint8_t* const dst = lds + (2 * (n & 1) + group) * kGroupBytes;
#pragma unroll
        for (int q = 0; q < PASSES; ++q)
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                u32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t v = st[s][q][l][i];
                    if constexpr (EDGE) {
                        const int want = 8 * lane + 4 * (128 * q + l);
                        const int d = want - min(max(want, st_lo[s][i]), st_hi[s][i]);
                        v = d > 0 ? (d < 4 ? v >> (8 * d) : 0u) : d < 0 ? (d > -4 ? v << (-8 * d) : 0u) : v;
                    }
                    o[i] = v ^ 0x80808080u;
                }
                *reinterpret_cast<u32x4*>(dst + wdst[q][l]) = o;
            }
        if (p < 2)
            *reinterpret_cast<uint32_t*>(lds + strip_recs(TILE) + 256 * (2 * (n & 1) + p) + 4 * lane) = st_rec[s];
    };

    // steps past the last one load rows that do not exist: zeros
#pragma unroll
    for (int s = 0; s < D; ++s) issue(s);
    write(0, 0);
    issue(0);
    write(1, 1);
    issue(1);
    step_barrier();
    auto step = [&](int s, int k) {
        step_barrier();
        write((s + 2) % D, k + 2);
        issue((s + 2) % D);
    };
    // (the loop's own waits are counted only if nothing is in flight where it is entered)
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    // whole rounds of D steps in a loop with one exit: the waits for a stage's loads are
    // counted over the loads issued after it on every path, and an exit per step would join
    // states in which fewer are. The remaining steps follow.
    int k = 0;
    for (; k + D <= K; k += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) step(s, k + s);
    }
#pragma unroll
    for (int s = 0; s < D - 1; ++s) {
        if (k + s >= K) break;
        step(s, k + s);
    }
}

// The contracting waves: strip `wave` of every run that has it.
template <int TILE, int CPS>
__device__ __forceinline__ void strip_contract(const DedispArgs& A, const DmBlock& b, uint8_t* lds, int wave, int lane,
                                               int K) {
    constexpr int NSUB = 8 / CPS;                     // matrix substeps per group
    constexpr int NE = CPS == 8 ? 2 : 3;              // entries per window
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const int m = lane & 31, h = lane >> 5;
    const uint32_t row0 = static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)(lds + kAcc0)));
    const uint32_t* const infos = reinterpret_cast<const uint32_t*>(A.offs) + static_cast<int64_t>(b.rec256) * 64 +
                                  static_cast<int64_t>(A.nchan_pad >> 3) * 64;
    // operand dwords of the step's two groups, and their records
    constexpr int NA = CPS == 8 ? 8 : 12;
    uint32_t a[2][NA], rec[2];
    const uint8_t* rsrc[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i)
        rsrc[i] = lds + strip_ring(TILE) + (CPS == 8 ? h * kQuadBytes : 8 * h) + entry_at(32 * wave + m + i);
    const uint8_t* const recp = lds + strip_recs(TILE) + 4 * lane;
    auto read = [&](int k, int gi) {
        const int place = 2 * (k & 1) + gi, off = place * kGroupBytes;
        rec[gi] = *reinterpret_cast<const uint32_t*>(recp + 256 * place);
        if constexpr (CPS == 8) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const u32x4 x = *reinterpret_cast<const u32x4*>(rsrc[i] + off);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[gi][4 * i + c] = x[c];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const u32x2 x = *reinterpret_cast<const u32x2*>(rsrc[i] + off + u * kQuadBytes);
                    a[gi][6 * u + 2 * i] = x[0];
                    a[gi][6 * u + 2 * i + 1] = x[1];
                }
        }
    };
    // infos of the steps (the low 10 bits of both groups'), lane l: step 64 n + l
    uint32_t info_tab = 0;
    auto info_of = [&](int k) {
        if ((k & 63) == 0) {
            const int g = 2 * min(k + lane, K - 1);
            info_tab = (infos[g] & 1023u) | (infos[g + 1] & 1023u) << 10;
            asm volatile("" : "+v"(info_tab));
        }
        return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(info_tab), k & 63));
    };
    auto strips = [](uint32_t info, int gi, int u) { return static_cast<int>((info >> (10 * gi + 2 + 4 * u)) & 15u) + 1; };
    auto strips_any = [&](uint32_t info, int gi) {
        return NSUB == 1 ? strips(info, gi, 0) : max(strips(info, gi, 0), strips(info, gi, 1));
    };

    i32x16 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = i32x16{};
    step_barrier();
    uint32_t info1 = info_of(0);
    read(0, 0);
    read(0, 1);
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
        const uint32_t info = info1;
        info1 = info_of(k + 1);
        step_barrier();
#pragma unroll
        for (int gi = 0; gi < 2; ++gi) {
            const uint32_t r0 = rec[gi];
#pragma unroll
            for (int u = 0; u < NSUB; ++u) {
                const bool on = wave < strips(info, gi, u);
                if (on) {
                    i32x4 B;
                    if constexpr (CPS == 8) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) B[i] = static_cast<int32_t>(1u << ((r0 >> (8 * i)) & 31u));
                    } else {
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const uint32_t r = (r0 >> (3 * (2 * u + j))) & 7u;
                            const uint32_t one = 1u << (8u * (r & 3u));
                            B[2 * j] = static_cast<int32_t>(r < 4u ? one : 0u);
                            B[2 * j + 1] = static_cast<int32_t>(r < 4u ? 0u : one);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        i32x4 w;
                        if constexpr (CPS == 8) {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                w[i] = static_cast<int32_t>(j == 0 ? a[gi][i] : __builtin_amdgcn_alignbyte(a[gi][4 + i], a[gi][i], j));
                        } else {
#pragma unroll
                            for (int i = 0; i < 2; ++i) {
                                const uint32_t x0 = a[gi][6 * u + i], x1 = a[gi][6 * u + 2 + i], x2 = a[gi][6 * u + 4 + i];
                                w[2 * i] = static_cast<int32_t>(j == 0 ? x0 : __builtin_amdgcn_alignbyte(x1, x0, j));
                                w[2 * i + 1] = static_cast<int32_t>(j == 0 ? x1 : __builtin_amdgcn_alignbyte(x2, x1, j));
                            }
                        }
                        acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, B, acc[j], 0, 0, 0);
                    }
                }
                if (u == NSUB - 1 && wave < strips_any(info1, gi)) read(k + 1, gi);
                if (on && ((info >> (10 * gi + u)) & 1u)) {
                    // the run ends here: add its strip into the accumulator tile
                    int e;
                    if constexpr (CPS == 8)
                        e = static_cast<int>(((r0 >> 5) & 7u) | ((r0 >> 10) & 0x38u) | ((r0 >> 15) & 0x1C0u) | ((r0 >> 20) & 0xE00u));
                    else
                        e = static_cast<int>((r0 >> (12 + 10 * u)) & 1023u);
                    strip_flush<TILE>(acc, wave, m, h, e, row0);
                }
            }
        }
    }
}

template <int TILE>
__device__ __forceinline__ void dedisp_strip(const DedispArgs& A, int blk, int64_t tile) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const DmBlock b = load_block(A.blocks, blk);
    const int64_t t0 = tile * TILE - b.lead;
    if (t0 + b.lead - b.span >= A.n_out) return;   // past the end of every trial
    // (opaque, so that the batch kernel's item loop does not keep per-lane values of every
    // role in registers across items)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int groups = (A.nchan + 7) / 8;
    const int K = (groups + 1) / 2;   // steps of two groups (the tables are padded)
    for (int i = tid; i < strip_ring(TILE) / 16; i += kThreads) reinterpret_cast<u32x4*>(lds)[i] = u32x4{0u, 0u, 0u, 0u};
    // the staging waves are the oldest of their SIMDs, which win issue
    if (wave >= kStage) {
        if (__builtin_amdgcn_readfirstlane(b.cps) == 8)
            strip_contract<TILE, 8>(A, b, lds, wave - kStage, lane, K);
        else
            strip_contract<TILE, 4>(A, b, lds, wave - kStage, lane, K);
    } else {
        // (b.row: staged bytes per row)
        if (t0 + b.rs_lo < 0 || t0 + b.rs_hi + kStripWideBytes > A.n_in16 || A.in_pitch > kStripMaxPitch)
            strip_stage<TILE, 3, true>(A, b, blk, t0, lds, wave, lane, K);
        else if (__builtin_amdgcn_readfirstlane(b.row) <= kStripNarrowBytes)
            strip_stage<TILE, 2, false>(A, b, blk, t0, lds, wave, lane, K);
        else
            strip_stage<TILE, 3, false>(A, b, blk, t0, lds, wave, lane, K);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();

    const int32_t corr = 128 * 8 * groups;
    const int32_t* acc_lds = reinterpret_cast<const int32_t*>(lds + kAcc0);
    // thread: trial tid % 32, 4 samples per item
    const int d = tid & 31;
    const int32_t* const skews = A.offs + static_cast<int64_t>(b.rec256) * 64 + static_cast<int64_t>(A.nchan_pad >> 3) * 64 +
                                 ((A.nchan_pad >> 3) + 63) / 64 * 64;
    const int64_t td = t0 + skews[d];
    int32_t* const orow = A.out + static_cast<int64_t>(b.first + d) * A.out_pitch;
    if (d >= b.count) return;
#pragma unroll 1
    for (int tq = tid >> 5; tq < TILE / 4; tq += kThreads / 32) {
        int32_t v[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) v[jj] = acc_lds[(4 * tq + jj) * 32 + d] + corr;
        const int64_t t = td + 4 * tq;
        if (t >= 0 && t + 4 <= A.n_out) {
            *reinterpret_cast<u32x4*>(orow + t) = u32x4{static_cast<uint32_t>(v[0]), static_cast<uint32_t>(v[1]),
                                                       static_cast<uint32_t>(v[2]), static_cast<uint32_t>(v[3])};
        } else {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                if (t + jj >= 0 && t + jj < A.n_out) orow[t + jj] = v[jj];
        }
    }
}

__global__ __launch_bounds__(kThreads, 4) void dedisp_strip_kernel(DedispArgs a) {
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    dedisp_strip<kStripTile>(a, bid % a.nblk, bid / a.nblk);
}

__global__ __launch_bounds__(kThreads, 4) void dedisp_strip_batch_kernel(const DedispArgs* __restrict__ args,
                                                                         const int64_t* __restrict__ item_begin, int nbeams,
                                                                         int64_t total, unsigned long long* counter) {
    batch_items(args, item_begin, nbeams, total, counter, [](const DedispArgs& a, int blk, int64_t tile) {
        dedisp_strip<kStripTile>(a, blk, tile);
    });
}

}  // namespace

const DedispFn kStripKernel = dedisp_strip_kernel;
const DedispBatchFn kStripBatchKernel = dedisp_strip_batch_kernel;

}  // namespace aa
