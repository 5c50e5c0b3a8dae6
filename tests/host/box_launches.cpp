// What the D3Q14 host runtime launches, recorded on a host without a GPU (see
// lattice_launches.cpp).  The first argument names the check.
#include "hip_stub.h"
#include "d3q14_runtime.cpp"

#include <chrono>
#include <vector>

// ------------------------------------------------------------------ recorders

struct Launch {
    int steps, zchunk;
};
static std::vector<Launch> launches;

namespace plbm3 {
hipError_t launch_step(int, int, const StepArgs&, hipStream_t) { return launches.push_back({1, 0}), hipSuccess; }
hipError_t launch_pair(int, int, int, const PairArgs& a, hipStream_t) {
    return launches.push_back({2, a.zchunk}), hipSuccess;
}
hipError_t launch_triple(int, const PairArgs& a, hipStream_t) { return launches.push_back({3, a.zchunk}), hipSuccess; }
hipError_t launch_init(int, const Geometry&, void*, const double*, const double*, const double*, const double*, double,
                       double, double, double, hipStream_t) { return hipSuccess; }
hipError_t launch_moments(int, const Geometry&, const void*, double, double, double*, double*, double*, double*,
                          hipStream_t) { return hipSuccess; }
hipError_t launch_sample(int, const Geometry&, const void*, double, double, const int64_t*, int64_t, double*,
                         hipStream_t) { return hipSuccess; }
int totals_blocks(const Geometry&) { return 1; }
hipError_t launch_totals(int, const Geometry&, const void*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_fill(void*, size_t, uint32_t, hipStream_t) { return hipSuccess; }
}

static lbm3d_config config(int nx, int ny, int nz, int storage = LBM_F32) {
    lbm3d_config c;
    std::memset(&c, 0, sizeof c);
    c.nx = nx;
    c.ny = ny;
    c.nz = nz;
    c.storage = storage;
    c.tau_n = 0.6;
    c.tau_r = 5.0;
    c.t0 = 1.0;
    c.scale = 1.0;
    return c;
}

static lbm3d_handle make(int nx, int ny, int nz, int storage = LBM_F32) {
    const lbm3d_config c = config(nx, ny, nz, storage);
    lbm3d_handle h = nullptr;
    expect(lbm3d_create(&c, &h) == LBM_OK, "create");
    static const double field = 1.0;
    expect(lbm3d_init(h, &field, nullptr, nullptr, nullptr, 1) == LBM_OK, "init");
    return h;
}

// The z ranges are searched once per box, not on every call, and over a bounded
// number of candidates.
static void ranges() {
    lbm3d_handle h = make(1, 1, 1000000);
    const auto t0 = std::chrono::steady_clock::now();
    for (int k = 0; k < 1000; ++k) expect(lbm3d_step(h, k & 1) == LBM_OK, "step");
    const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 1000;
    std::printf("a step call on a million planes: %.2f us\n", us);
    expect(us < 50.0, "host time of a step call");
    lbm3d_destroy(h);
    // the most planes: no overflow, and no long search at creation
    lbm3d_config c = config(1, 1, INT32_MAX);
    c.flags = LBM_FLAG_EXTERNAL_MEMORY;
    expect(lbm3d_create(&c, &h) == LBM_OK && h->zrange() >= 1, "a column of 2^31 - 1 planes");
    lbm3d_destroy(h);
}

// The z ranges of the two-step kernel: filled rounds, but FP32 keeps 32 planes
// where the gain is small or the ranges are long.
static void planes() {
    struct Case {
        int nx, ny, nz, storage, planes;
    };
    for (const Case& c : {Case{301, 211, 163, LBM_BF16, 24}, Case{301, 211, 163, LBM_F32, 24}, Case{192, 192, 192, LBM_F32, 48},
                          Case{130, 500, 300, LBM_F32, 150}, Case{512, 512, 512, LBM_BF16, 57}, Case{512, 512, 512, LBM_F32, 32},
                          Case{200, 160, 256, LBM_F32, 32}, Case{200, 160, 256, LBM_F16, 29}, Case{531, 498, 240, LBM_F32, 32},
                          Case{202, 436, 661, LBM_F32, 32}, Case{132, 526, 630, LBM_F32, 32}, Case{122, 213, 237, LBM_F32, 27},
                          Case{319, 203, 378, LBM_F32, 32}, Case{720, 157, 521, LBM_F32, 32}}) {
        lbm3d_handle h = make(c.nx, c.ny, c.nz, c.storage);
        expect(lbm3d_set_step_fusion(h, 2) == LBM_OK, "step fusion");
        launches.clear();
        expect(lbm3d_step(h, 2) == LBM_OK, "step");
        const bool ok = launches.size() == 1 && launches[0].steps == 2 && launches[0].zchunk == c.planes;
        if (!ok) std::printf("%d x %d x %d: %d planes\n", c.nx, c.ny, c.nz, launches.empty() ? 0 : launches[0].zchunk);
        expect(ok, "planes of a range");
        lbm3d_destroy(h);
    }
}

// The boxes that the GPU tests of three steps per launch compare with single
// steps do take three, in the calls that they make.
static void triples() {
    const int boxes[][3] = {{144, 260, 186}, {498, 109, 118}, {102, 394, 285}, {47, 800, 171}, {512, 512, 512}};
    for (auto& b : boxes) {
        lbm3d_handle h = make(b[0], b[1], b[2]);
        std::string got;
        for (int n : {3, 1, 4, 2, 5, 7}) {
            launches.clear();
            expect(lbm3d_step(h, n) == LBM_OK, "step");
            for (const Launch& l : launches) got += std::to_string(l.steps);
            got += " ";
        }
        expect(got == "3 1 22 2 32 322 ", "launches of a box that takes three steps");
        lbm3d_destroy(h);
    }
}

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "ranges") ranges();
    else if (what == "planes") planes();
    else if (what == "triples") triples();
    else expect(false, "unknown check");
    std::printf("%s: %s\n", what.c_str(), failures ? "FAILED" : "ok");
    return failures ? 1 : 0;
}
