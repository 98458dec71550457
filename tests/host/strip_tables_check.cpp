// Host check of the strip variant's tables (layout 8). For every DM block, trial and channel,
// the row start, residual, run offset and skew that the kernel reads must add up to the
// shift, s[d][c] + skew[d] = rs[c] + r[d][c] + e[d], within the ranges its fields, strips,
// staged rows and LDS tile have. Host-only plan: no GPU needed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "../../paper_2101_00941_amd/csrc/aa_internal.h"

using namespace aa;

#define CHECK(x) do { if (!(x)) { printf("failed: %s (block %zu)\n", #x, bi); return 1; } } while (0)

static int run_case(int nchan, int nsamp, double ftop, double foff, double tsamp, const std::vector<double>& dms, int shape) {
    aa_plan_desc_t d{};
    d.nchan = nchan; d.nsamp = nsamp; d.f_top_mhz = ftop; d.foff_mhz = foff; d.tsamp_s = tsamp;
    d.dm = dms.data(); d.ndm = static_cast<int>(dms.size());
    int32_t widths[1] = {1};
    d.widths = widths; d.nwidths = 1; d.snr_threshold = 6.0f; d.flags = AA_PLAN_HOST_ONLY;
    aa_plan_t p = nullptr;
    if (aa_plan(&d, &p) != AA_OK) { printf("plan failed: %s\n", aa_last_error()); return 1; }
    std::vector<DmBlock> blocks; std::vector<int32_t> rs; std::vector<uint32_t> rec;
    const int tile = kStripTile;
    if (build_strip_tables(p, tile, shape, blocks, rs, rec) != AA_OK) { printf("tables failed: %s\n", aa_last_error()); return 1; }
    const int npad = strip_nchan_pad(nchan), K = npad / 8, Kinfo = (K + 63) / 64 * 64;
    int next = 0, n8 = 0;
    for (size_t bi = 0; bi < blocks.size(); ++bi) {
        const DmBlock& b = blocks[bi];
        CHECK(b.first == next && b.count >= 1 && b.count <= 32 && (b.cps == 8 || b.cps == 4) && (shape == 0 || b.cps == shape));
        next += b.count;
        n8 += b.cps == 8;
        CHECK((static_cast<size_t>(b.rec256) + K) * 64 + Kinfo + 64 <= rec.size() && (bi + 1) * npad <= rs.size());
        const uint32_t* R = &rec[static_cast<size_t>(b.rec256) * 64];
        const uint32_t* info = R + static_cast<size_t>(K) * 64;
        const int32_t* skew = reinterpret_cast<const int32_t*>(info + Kinfo);
        const int32_t* r0 = &rs[bi * npad];
        int32_t lead = skew[0], low = skew[0];
        for (int i = 0; i < b.count; ++i) {
            CHECK(skew[i] % 4 == 0);
            lead = std::max(lead, skew[i]);
            low = std::min(low, skew[i]);
        }
        CHECK(b.lead == lead && b.span == lead - low);
        const int nsub = 8 / b.cps, R_ = 32 / b.cps, subs = (nchan + 7) / 8 * nsub;
        for (int s = 0; s < subs; ++s) {
            const int k = s / nsub, u = s % nsub;
            const int strips = static_cast<int>((info[k] >> (2 + 4 * u)) & 15u) + 1;
            const int emax = static_cast<int>((info[k] >> (10 + 10 * u)) & 1023u);
            CHECK(strips <= kStripWaves && strips * kStripRows >= tile + emax && emax <= strip_spread(tile));
            CHECK(tile + emax + R_ - 1 <= b.row && b.row <= kStripWideBytes);
            int emax_seen = 0;
            for (int i = 0; i < 32; ++i) {
                int e_half[2];
                for (int h = 0; h < 2; ++h) {
                    const uint32_t v = R[64 * k + 32 * h + i];
                    e_half[h] = b.cps == 8 ? ((v >> 5) & 7) | ((v >> 10) & 0x38) | ((v >> 15) & 0x1C0) | ((v >> 20) & 0xE00)
                                           : (v >> (12 + 10 * u)) & 1023;
                }
                CHECK(e_half[0] == e_half[1] && e_half[0] <= emax && (i < b.count || e_half[0] == 0));
                emax_seen = std::max(emax_seen, e_half[0]);
                for (int j = 0; j < b.cps; ++j) {
                    const int c = s * b.cps + j;
                    const int h = b.cps == 8 ? j / 4 : j / 2;
                    const uint32_t v = R[64 * k + 32 * h + i];
                    const int r = b.cps == 8 ? static_cast<int>((v >> (8 * (j % 4))) & 31u) / 8
                                             : static_cast<int>((v >> (3 * (2 * u + j % 2))) & 7u);
                    CHECK(r < R_);
                    if (b.cps == 8) CHECK(((v >> (8 * (j % 4))) & 7u) == 0);
                    if (i >= b.count || c >= nchan) continue;
                    CHECK(r0[c] >= -kStripBias && r0[c] >= b.rs_lo && r0[c] <= b.rs_hi);
                    CHECK(p->shifts[static_cast<size_t>(b.first + i) * nchan + c] + skew[i] == r0[c] + r + e_half[0]);
                }
            }
            CHECK(emax_seen == emax);
            // a run: substeps of one strip count and one set of offsets, closed by its last flag
            const bool last = (info[k] >> u) & 1u;
            if (s + 1 == subs) CHECK(last);
            if (!last && s + 1 < subs) {
                const int k1 = (s + 1) / nsub, u1 = (s + 1) % nsub;
                CHECK(((info[k1] >> (2 + 4 * u1)) & 15u) == ((info[k] >> (2 + 4 * u)) & 15u));
                for (int l = 0; l < 64; ++l) {
                    auto e_of = [&](int kk, int uu) {
                        const uint32_t v = R[64 * kk + l];
                        return b.cps == 8 ? ((v >> 5) & 7) | ((v >> 10) & 0x38) | ((v >> 15) & 0x1C0) | ((v >> 20) & 0xE00)
                                          : (v >> (12 + 10 * uu)) & 1023;
                    };
                    CHECK(e_of(k, u) == e_of(k1, u1));
                }
            }
        }
        for (int k = (nchan + 7) / 8; k < K; ++k) CHECK((info[k] & 3u) == 0);
    }
    if (next != d.ndm) { printf("blocks do not tile the trials\n"); return 1; }
    printf("nchan %d ndm %d shape %d: %zu blocks (%d of 8 channels per op)\n", nchan, d.ndm, shape, blocks.size(), n8);
    aa_plan_destroy(p);
    return 0;
}

int main() {
    auto grid = [](int n, double step) { std::vector<double> v; for (int i = 0; i < n; ++i) v.push_back(step * i); return v; };
    int bad = 0;
    for (int shape : {0, 8, 4}) {
        bad += run_case(1, 3000, 1400.0, 1.0, 64e-6, {0.0, 10.0, 100.0}, shape);
        bad += run_case(7, 5003, 1500.0, 3.0, 64e-6, grid(5, 12.5), shape);
        bad += run_case(9, 5003, 1500.0, 3.0, 64e-6, grid(33, 1.0), shape);
        bad += run_case(48, 60000, 1200.0, 4.0, 64e-6, grid(9, 60.0), shape);      // steep: small blocks
        bad += run_case(257, 8000, 1500.0, 0.5, 64e-6, grid(65, 0.25), shape);
        bad += run_case(1001, 77777, 1450.0, 300.0 / 1001, 64e-6, grid(333, 1.0), shape);
        bad += run_case(4096, 60000, 1450.0, 300.0 / 4096, 64e-6, grid(97, 2.0), shape);
        bad += run_case(4096, 60000, 1450.0, 300.0 / 4096, 64e-6, grid(64, 1.0 / 16), shape);
    }
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}

// launch-side symbols that the plan and tuner sources refer to
namespace aa {
size_t sps_work_bytes(const aa_plan_s*, int64_t) { return 0; }
int launch_dedisperse(const aa_plan_s*, int, const uint8_t*, int64_t, int64_t, int32_t*, int64_t, hipStream_t) { return -1; }
}
extern "C" int aa_dedisperse(aa_plan_t, const uint8_t*, int64_t, int64_t, int32_t*, int64_t, void*) { return -1; }
