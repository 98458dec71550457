// Host check of launch_variant: a new plan's launches go to the step kernel where there is little
// to do and to the strip kernel elsewhere; a variant that the caller chose is used for every launch.
#include <cstdio>
#include <vector>
#include "../../paper_2101_00941_amd/csrc/aa_internal.h"

using namespace aa;

static int bad = 0;

static aa_plan_t make(int nchan, int ndm, double step, int64_t nsamp) {
    std::vector<double> dm;
    for (int i = 0; i < ndm; ++i) dm.push_back(step * i);
    aa_plan_desc_t d{};
    d.nchan = nchan; d.nsamp = nsamp; d.f_top_mhz = 1450.0; d.foff_mhz = 300.0 / nchan; d.tsamp_s = 64e-6;
    d.dm = dm.data(); d.ndm = ndm;
    int32_t widths[1] = {1};
    d.widths = widths; d.nwidths = 1; d.snr_threshold = 6.0f; d.flags = AA_PLAN_HOST_ONLY;
    aa_plan_t p = nullptr;
    if (aa_plan(&d, &p) != AA_OK) { printf("plan failed: %s\n", aa_last_error()); ++bad; }
    return p;
}

static void expect(const char* what, int got, int want) {
    if (got != want) { printf("%s: variant %d, expected %d\n", what, got, want); ++bad; }
}

static void check(int nchan, int ndm, double step, int64_t n_out, int want) {
    aa_plan_t probe = make(nchan, ndm, step, 1 << 24);
    if (!probe) return;
    aa_plan_t p = make(nchan, ndm, step, n_out + probe->maxshift);
    aa_plan_destroy(probe);
    if (!p) return;
    char what[100];
    snprintf(what, sizeof(what), "%d channels, %d trials %g apart, %lld samples", nchan, ndm, step, static_cast<long long>(n_out));
    int32_t v = -1;
    aa_plan_get_variant(p, &v);
    expect("new plan", v, kDefaultDedispVariant);
    expect(what, launch_variant(p, n_out), want);
    for (int chosen : {kDefaultDedispVariant, 17, kSmallDedispVariant}) {
        if (aa_plan_set_variant(p, chosen) != AA_OK) { printf("set_variant failed\n"); ++bad; }
        expect("chosen variant", launch_variant(p, n_out), chosen);
    }
    aa_plan_destroy(p);
}

int main() {
    const int strip = kDefaultDedispVariant, step = kSmallDedispVariant;
    expect("default is the strip kernel", kDedispVariants[strip].layout, 8);
    expect("small is a step kernel", kDedispVariants[step].layout, 4);
    // few channels, or one trial of few
    for (int64_t n : {1000, 1 << 18}) {
        check(1, 32, 1.0, n, step);
        check(4, 100, 1.0, n, step);
        check(8, 300, 1.0, n, step);
        check(16, 1, 1.0, n, step);
        check(64, 1, 1.0, n, step);
    }
    // a round less with the longer tiles
    check(64, 32, 1.0 / 16, 1 << 18, step);
    check(256, 8, 1.0 / 16, 1 << 18, step);
    check(128, 64, 1.0 / 16, 1 << 17, step);
    // everything else
    check(64, 32, 1.0, 1 << 18, strip);
    check(128, 100, 1.0, 1 << 18, strip);
    check(1001, 333, 1.0, 77777, strip);
    check(4096, 100, 1.0 / 16, 1 << 17, strip);
    check(4096, 600, 1.0 / 16, 1 << 20, strip);
    // few channels: also for launches shorter than the plan; many: no tables that are not used
    aa_plan_t p = make(16, 1, 1.0, 1 << 24);
    if (p) {
        expect("a short launch of a long plan", launch_variant(p, 5000), step);
        aa_plan_destroy(p);
    }
    p = make(4096, 100, 1.0 / 16, 1 << 20);
    if (p) {
        expect("tables of the step kernel", p->tables[step].variant, -1);
        expect("a short launch without them", launch_variant(p, 5000), strip);
        aa_plan_destroy(p);
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
