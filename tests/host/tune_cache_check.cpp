// Host check of the tuning cache: an entry counts only for the set of kernels it was timed over.
#include <cstdio>
#include <fstream>
#include <string>
#include "../../paper_2101_00941_amd/csrc/aa_internal.h"

using namespace aa;

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    const char* path = argv[1];
    double dm[2] = {0.0, 1.0};
    int32_t widths[1] = {1};
    aa_plan_desc_t d{};
    d.nchan = 16; d.nsamp = 4096; d.f_top_mhz = 1450.0; d.foff_mhz = 1.0; d.tsamp_s = 64e-6;
    d.dm = dm; d.ndm = 2; d.widths = widths; d.nwidths = 1; d.snr_threshold = 6.0f; d.flags = AA_PLAN_HOST_ONLY;
    aa_plan_t p = nullptr;
    if (aa_plan(&d, &p) != AA_OK) { printf("plan failed: %s\n", aa_last_error()); return 1; }
    int bad = 0;
    auto expect = [&](const char* what, TuneEntry e, int variant, int split) {
        if (e.variant != variant || e.split != split) {
            printf("%s: variant %d split %d, expected %d %d\n", what, e.variant, e.split, variant, split);
            ++bad;
        }
    };
    const std::string shape = tune_shape_key(p, 4096);
    expect("no file", tune_cache_read(path, p, 4096), -1, -1);
    {
        // entries of a build with other kernels: the shape alone, and another set of kernels
        std::ofstream f(path);
        f << "{\n  \"" << shape << "\": 20,\n  \"" << shape << "|split\": 1,\n  \"" << shape << "|kernels=0\": 17\n}\n";
    }
    expect("entries of other kernels", tune_cache_read(path, p, 4096), -1, -1);
    tune_cache_write(path, p, 4096, TuneEntry{20, 2});
    expect("own entry", tune_cache_read(path, p, 4096), 20, 2);
    tune_cache_write(path, p, 4096, TuneEntry{12, -1});
    expect("own entry, another variant", tune_cache_read(path, p, 4096), 12, -1);
    expect("another length", tune_cache_read(path, p, 9000), -1, -1);
    tune_cache_write(path, p, 9000, TuneEntry{3, -1});
    expect("both lengths", tune_cache_read(path, p, 4096), 12, -1);
    expect("both lengths", tune_cache_read(path, p, 9000), 3, -1);
    {
        // the other build's entries are still there for it
        std::ifstream f(path);
        const std::string text((std::istreambuf_iterator<char>(f)), std::istreambuf_iterator<char>());
        if (text.find("\"" + shape + "\": 20") == std::string::npos) { printf("entry lost:\n%s\n", text.c_str()); ++bad; }
    }
    aa_plan_destroy(p);
    if (!bad) printf("ALL OK\n");
    return bad ? 1 : 0;
}

// launch-side symbols that the plan and tuner sources refer to
namespace aa {
size_t sps_work_bytes(const aa_plan_s*, int64_t) { return 0; }
int launch_dedisperse(const aa_plan_s*, int, const uint8_t*, int64_t, int64_t, int32_t*, int64_t, hipStream_t) { return -1; }
}
extern "C" int aa_dedisperse(aa_plan_t, const uint8_t*, int64_t, int64_t, int32_t*, int64_t, void*) { return -1; }
