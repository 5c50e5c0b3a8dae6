// What the D2Q8 host runtime launches, recorded on a host without a GPU: the
// runtime source is compiled in, the HIP calls and the kernel launchers are
// replaced by recorders.  The first argument names the check.
#include "hip_stub.h"
#include "lbm_runtime.cpp"

#include <functional>

// ------------------------------------------------------------------ recorders

struct Launch {
    hipStream_t stream;
    int kind;              // 0 single step, 1 fused, 2 block, 3 reduction
    int steps, end, rows, tiles;  // end: FusedEnd; rows, tiles: of a fused launch's strips
    BlockPlan plan;
    bool keep;             // a block launch that also stores the state of the step before its last
    // check records [lo, hi) it writes (or reads: reductions), and the first-stage records of a reduction
    const DD *lo, *hi, *glo, *ghi;
};
static std::vector<Launch> launches;
static std::function<double(const Launch&)> cost_us;  // what the autotuner's events report

static void note(Launch l) {
    if (cost_us) stub::clock_us += cost_us(l);
    launches.push_back(l);
}
static void records(Launch* l, const StepArgs& a, bool check) {
    l->lo = check ? a.partials + (int64_t)a.tile_base * kPartials : nullptr;
    l->hi = check ? l->lo + (int64_t)a.ntiles * kPartials : nullptr;
}

namespace plbm {
hipError_t launch_step(int, const Shape&, int mode, const StepArgs& a, int64_t, hipStream_t st) {
    Launch l{st, 0, 1, mode == kCheck ? kEndCheck : mode == kSnap ? kEndSnap : kEndPlain};
    records(&l, a, mode == kCheck);
    note(l);
    return hipSuccess;
}
hipError_t launch_fused(int, const Shape&, const StepArgs& a, int k, int end, int, int, int64_t, hipStream_t st) {
    Launch l{st, 1, k, end, a.march_rows, a.ntiles};
    records(&l, a, end == kEndCheck);
    note(l);
    return hipSuccess;
}
hipError_t launch_block(int, const BlockPlan& p, const Shape&, const BlockArgs& b, int end, hipStream_t st) {
    Launch l{st, 2, b.steps, end, 0, b.s.ntiles, p, b.prev != nullptr};
    records(&l, b.s, end == kEndCheck);
    note(l);
    return hipSuccess;
}
// first record and count of instance `d`'s tiles and groups of a kind
static void tiles_of(const InstDesc& d, int kind, int64_t* t0, int64_t* nt) {
    *t0 = kind == 2 ? d.b_tile_begin : kind ? d.p_tile_begin : d.tile_begin;
    *nt = kind == 2 ? d.b_ntiles : kind ? d.p_ntiles : d.ntiles;
}
hipError_t launch_finalize(const InstDesc* d, const int32_t*, int g0, int ngroups, RefState*, RefState*, int i0,
                           int ninst, const DD* partials, DD* gpart, double*, int fused, hipStream_t st) {
    Launch l{st, 3, 0, kEndCheck};
    int64_t a0, an, b0, bn;
    tiles_of(d[i0], fused, &a0, &an);
    tiles_of(d[i0 + ninst - 1], fused, &b0, &bn);
    l.lo = partials + a0 * kPartials;
    l.hi = partials + (b0 + bn) * kPartials;
    if (ngroups > ninst) {
        l.glo = gpart + (int64_t)g0 * kPartials;
        l.ghi = l.glo + (int64_t)ngroups * kPartials;
    }
    note(l);
    return hipSuccess;
}
hipError_t launch_moments(int, const InstDesc*, const RefState*, int, const InstDesc&, const void*, int, int, int,
                          void*, void*, void*, double, double, DD*, hipStream_t) { return hipSuccess; }
hipError_t launch_plane_moments(const InstDesc*, int, const InstDesc&, const double*, int64_t, int, void*, void*,
                                void*, double, double, DD*, hipStream_t) { return hipSuccess; }
hipError_t launch_init(int, const InitTables&, int, const InstDesc&, const RefState&, void*, void*, const double*,
                       const double*, const double*, double, double, double, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize_range(const DD*, int, DD*, DD*, hipStream_t) { return hipSuccess; }
hipError_t launch_copy_u32(uint32_t*, const uint32_t*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_set_float(float*, float, hipStream_t) { return hipSuccess; }
hipError_t launch_fill(void*, size_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t preload_fused(int, int, int, int, hipStream_t) { return hipSuccess; }
}

// ------------------------------------------------------------------ handles

static lbm_instance inst(int nx, int ny) {
    lbm_instance in;
    std::memset(&in, 0, sizeof in);
    in.nx = nx;
    in.ny = ny;
    in.tau_n = 0.6;
    in.tau_r = 5.0;
    in.cv = 1.0;
    in.t0 = 1.0;
    in.scale = 1.0;
    return in;
}

static void start(lbm_handle h, size_t n) {
    static const double field = 1.0;
    for (size_t k = 0; h && k < n; ++k)
        expect(lbm_init_device(h, (int32_t)k, &field, nullptr, nullptr) == LBM_OK, "init");
}

static lbm_handle make(const std::vector<lbm_instance>& v, int storage, int check, int flags = 0, bool init = true) {
    lbm_config c;
    std::memset(&c, 0, sizeof c);
    c.n_instances = (int32_t)v.size();
    c.storage = storage;
    c.check_interval = check;
    c.flags = flags;
    c.inst = v.data();
    lbm_handle h = nullptr;
    expect(lbm_create(&c, &h) == LBM_OK, "create");
    if (init) start(h, v.size());
    return h;
}

static bool meet(const DD* a0, const DD* a1, const DD* b0, const DD* b1) { return a0 && b0 && a0 < b1 && b0 < a1; }

// Within one call, the launches of one part's stream must not write check
// records that the other part's stream reads or writes: the streams are
// ordered at the call's beginning and end only.
static void streams() {
    const std::vector<std::vector<lbm_instance>> sets = {
        {inst(300, 200), inst(310, 150), inst(64, 64)},
        {inst(20, 20), inst(31, 9), inst(25, 33), inst(5, 7)},
        {inst(1500, 1100), inst(900, 1000)},
        {inst(3000, 3000), inst(2500, 2000), inst(700, 90)},
    };
    for (auto& v : sets)
        for (int storage : {LBM_F32, LBM_F16})
            for (int check : {2, 5, 10}) {
                lbm_handle h = make(v, storage, check);
                for (int fuse : {0, 4, 2}) {
                    if (fuse) expect(lbm_set_step_fusion(h, fuse) == LBM_OK, "step fusion");
                    // calls that end before, on and after the snapshot step of a check step
                    for (int n : {check - 1, 4 * check, check + 1, 1, 3 * check - 1}) {
                        launches.clear();
                        expect(lbm_step(h, n) == LBM_OK, "step");
                        for (auto& a : launches)
                            for (auto& b : launches)
                                if (a.stream != b.stream &&
                                    (meet(a.lo, a.hi, b.lo, b.hi) || meet(a.glo, a.ghi, b.glo, b.ghi))) {
                                    std::printf("%zu instances, storage %d, check %d, steps per launch %d, call of %d\n",
                                                v.size(), storage, check, fuse, n);
                                    expect(false, "check records of the two streams overlap");
                                    goto next;
                                }
                    }
                }
            next:
                lbm_destroy(h);
            }
}

// Strips of fused launches: by the launch's steps, whatever set the steps per
// launch (a new handle's default with short calls, a setting, the autotuner).
static void strips() {
    struct Size {
        int nx, ny, few, many;   // rows per strip below kTallSteps steps, and from there on
    };
    for (const Size& s : {Size{8192, 8192, 32, 64}, Size{8192, 8222, 32, 64}, Size{2600, 2300, 32, 32},
                          Size{837, 5577, 24, 24}, Size{1500, 1400, 16, 16}})
        for (int storage : {LBM_F16, LBM_BF16_SPLIT})
            for (int how = 0; how < 3; ++how)
                for (int k = 2; k <= fuse_max(storage); ++k) {
                    lbm_handle h = make({inst(s.nx, s.ny)}, storage, how == 0 ? 4 : -1, 0, false);
                    if (how == 1) expect(lbm_set_step_fusion(h, k) == LBM_OK, "step fusion");
                    if (how == 2) {
                        cost_us = [k](const Launch& l) { return l.kind == 1 && l.steps == k ? 1.0 * k : 10.0 * l.steps; };
                        expect(lbm_autotune(h, 4, nullptr, 0) == LBM_OK, "autotune");
                        cost_us = nullptr;
                        expect(lbm_get_step_fusion(h) == k, "tuned steps per launch");
                    }
                    start(h, 1);
                    launches.clear();
                    for (int call : {k, 4 * k, 3}) expect(lbm_step(h, call) == LBM_OK, "step");
                    double dT = 0.0;
                    expect(lbm_moments_f64(h, 0, &dT, nullptr, nullptr, 1) == LBM_OK, "moments");
                    const int tx = (int)fused_tiles_x(h->inst[0], storage);
                    int seen = 0;
                    for (const Launch& l : launches) {
                        if (l.kind != 1) continue;
                        ++seen;
                        const int rows = l.end != kEndCheck && l.steps < kTallSteps ? s.few : s.many;
                        expect(l.rows == rows, "rows of a strip");
                        const int chunks = (s.ny + s.many - 1) / s.many;
                        expect(l.tiles == tx * chunks * (rows < s.many ? 2 : 1), "strips of a launch");
                    }
                    expect(seen >= 2, "fused launches");
                    lbm_destroy(h);
                }
}

// Plans of the block kernels by the shapes of a handle's lattices.
static void plans() {
    struct Case {
        int count, nx, ny;
        BlockKind kind;
    };
    const Case cases[] = {
        // one lattice of each size class
        {1, 2, 2, kBlockWhole}, {1, 401, 3, kBlockWhole}, {1, 128, 64, kBlockPatch}, {1, 201, 201, kBlockPatch},
        {1, 999, 777, kBlockTiles}, {1, 1024, 256, kBlockTiles}, {1, 2000, 2000, kBlockTiles}, {1, 4000, 4000, kBlockNone},
        // thin lattices: windows mostly outside of them
        {1, 200000, 3, kBlockNone}, {1, 100000, 8, kBlockNone}, {1, 1000000, 2, kBlockNone}, {1, 500000, 5, kBlockNone},
        {1, 2, 1000000, kBlockNone}, {1, 3, 200000, kBlockNone}, {1, 100000, 3, kBlockNone}, {1, 100000, 2, kBlockNone},
        {1, 20000, 40, kBlockTiles}, {1, 40, 20000, kBlockTiles}, {1, 16, 60000, kBlockTiles}, {1, 8000, 100, kBlockTiles},
        // many small ones
        {2000, 20, 20, kBlockWhole}, {8000, 20, 20, kBlockWhole}, {4000, 32, 32, kBlockWhole}, {1000, 41, 25, kBlockWhole},
        {400, 401, 3, kBlockWhole}, {1500, 401, 3, kBlockWhole}, {500, 64, 32, kBlockWhole}, {300, 100, 40, kBlockTiles},
        {20000, 20, 20, kBlockNone},
    };
    for (const Case& c : cases) {
        const BlockPlan p = block_plan(std::vector<lbm_instance>((size_t)c.count, inst(c.nx, c.ny)), LBM_F32);
        if (p.kind != c.kind) {
            std::printf("%d of %d x %d: plan %d, expected %d\n", c.count, c.nx, c.ny, p.kind, c.kind);
            expect(false, "plan");
        }
    }
}

// Few steps, check steps and the state before a call's last step on handles in
// the block kernels.
static void short_runs() {
    auto kinds = [](lbm_handle h, int n) {       // kinds of a call's launches; 4: one more by a readout
        launches.clear();
        expect(lbm_step(h, n) == LBM_OK, "step");
        std::string s;
        for (const Launch& l : launches)
            if (l.kind != 3) s += std::to_string(l.kind);
        launches.clear();
        double dT = 0.0;
        expect(lbm_moments_f64(h, 0, &dT, nullptr, nullptr, 1) == LBM_OK, "moments");
        return s + (launches.empty() ? "" : "+" + std::to_string(launches[0].kind));
    };
    auto same = [](const std::string& got, const char* want, const char* what) {
        if (got != want) std::printf("%s: launched %s, expected %s\n", what, got.c_str(), want);
        expect(got == want, what);
    };
    struct Case {
        int nx, ny, storage, flags;
        const char *two, *three, *four, *seven;  // kinds launched by calls of that many steps
    };
    const int every = LBM_FLAG_ROUND_EVERY_STEP, sr = LBM_FLAG_STOCHASTIC_ROUNDING;
    const Case cases[] = {
        {128, 64, LBM_F32, 0, "2", "2", "2", "2"},          {512, 512, LBM_F32, 0, "00", "2", "2", "2"},
        {640, 640, LBM_F32, 0, "2", "2", "2", "2"},         {1000, 1000, LBM_F32, sr, "00", "2", "2", "2"},
        {1024, 1000, LBM_F16, 0, "00", "2", "2", "2"},      {1024, 1000, LBM_F16, sr, "2", "2", "2", "2"},
        {16, 20000, LBM_F32, sr, "2", "2", "2", "22"},      {1500, 1400, LBM_F32, 0, "2", "2", "2", "2"},
        {1700, 1500, LBM_F32, 0, "1+0", "1+1", "1+1", "2"}, {2048, 2048, LBM_F32, 0, "1+0", "1+1", "1+1", "2"},
        {2048, 2048, LBM_F32, sr, "2+2", "2+2", "2+2", "2"}, {2048, 2048, LBM_F16, every, "1+0", "1+1", "2", "2"},
        {1500, 1400, LBM_F16, every, "2", "2", "2", "2"},   {401, 301, LBM_F32, sr, "00", "2", "2", "2"},
        {30000, 16, LBM_F32, 0, "00", "2", "2", "2"},       {100, 3000, LBM_F16, 0, "2", "2", "2", "2"},
    };
    for (const Case& c : cases) {
        lbm_handle h = make({inst(c.nx, c.ny)}, c.storage, -1, c.flags);
        same(kinds(h, 2), c.two, "two steps");
        same(kinds(h, 3), c.three, "three steps");
        same(kinds(h, 4), c.four, "four steps");
        same(kinds(h, 7), c.seven, "seven steps");
        lbm_destroy(h);
    }
    // the state before the last step of a call of three full launches is stored
    lbm_handle big = make({inst(2048, 2048)}, LBM_F32, -1);
    same(kinds(big, 6), "2+2", "six steps");
    same(kinds(big, 20), "222+2", "20 steps");
    same(kinds(big, 21), "222", "21 steps");
    lbm_destroy(big);
    // a segment's last launches up to a check step
    for (int n : {2000, 1500, 1000, 700})
        for (int flags : {0, sr})
            for (int check : {2, 3, 5, 10, 20, 100}) {
                lbm_handle h = make({inst(n, n)}, LBM_F32, check, flags);
                launches.clear();
                expect(lbm_step(h, 2 * check) == LBM_OK, "step");
                for (const Launch& l : launches)
                    if (l.kind < 3 && l.end == kEndCheck)
                        expect(l.kind == (n == 1000 && flags ? 0 : n <= 1000 || (n == 1500 && flags && check > 3) ? 2 : 1),
                               "check launch");
                lbm_destroy(h);
            }
    // many small lattices: long launches keep the state before the last step,
    // short ones of buffers beyond the last-level cache do not
    lbm_handle h = make(std::vector<lbm_instance>(2500, inst(20, 20)), LBM_F32, -1);
    same(kinds(h, 100), "22", "100 steps of many lattices");
    same(kinds(h, 7), "22+2", "seven steps of many lattices");
    same(kinds(h, 8), "22", "eight steps of many lattices");
    lbm_destroy(h);
    // tuned to the block kernels, a handle keeps fused launches for few steps
    h = make({inst(2048, 2048)}, LBM_F32, -1, 0, false);
    cost_us = [](const Launch& l) { return l.kind == 2 ? 1.0 : l.kind == 1 ? 10.0 : 5.0 * l.steps; };
    expect(lbm_autotune(h, 4, nullptr, 0) == LBM_OK, "autotune");
    cost_us = nullptr;
    start(h, 1);
    same(kinds(h, 6), "2+2", "six steps, tuned");
    same(kinds(h, 3), "1+1", "three steps, tuned");
    lbm_destroy(h);
}

// Pinned memory of a new handle: none unless it has many check records to copy;
// none by lbm_last_check itself.
static void pinned() {
    struct Case {
        int count, check, allocs;
    };
    for (const Case& c : {Case{1, 100, 0}, Case{1, -1, 0}, Case{7, 10, 0}, Case{8, 10, 1}, Case{256, -1, 0}, Case{256, 100, 1}}) {
        const int before = stub::host_allocs;
        lbm_handle h = make(std::vector<lbm_instance>((size_t)c.count, inst(40, 30)), LBM_F32, c.check);
        expect(stub::host_allocs - before == c.allocs, "pinned allocations at creation");
        lbm_check_info info;
        expect(lbm_step(h, 100) == LBM_OK, "step");
        expect(lbm_last_check(h, 0, &info) == (c.check > 0 ? LBM_OK : LBM_ESTATE), "last check");
        expect(stub::host_allocs - before == c.allocs, "pinned allocations by lbm_last_check");
        lbm_destroy(h);
    }
}

// The forms that the GPU tests of the block kernels mean to run.
static void forms() {
    struct Case {
        int nx, ny, storage, kind, rows, waves, wx, wy, count = 1;   // 0: any
    };
    const Case cases[] = {
        {64, 16, LBM_F32, kBlockWhole, 1, 16, 0, 0}, {32, 32, LBM_F32, kBlockWhole, 1, 16, 0, 0},
        {30, 20, LBM_F32, kBlockWhole, 1, 10, 0, 0}, {41, 25, LBM_F32, kBlockWhole, 2, 9, 0, 0},
        {64, 32, LBM_F32, kBlockWhole, 2, 16, 0, 0, 600}, {20, 20, LBM_F32, kBlockWhole, 1, 7, 0, 0, 2500},
        {131, 67, LBM_BF16, kBlockPatch, 1, 16, 32, 32}, {1189, 4, LBM_F32, kBlockPatch, 1, 13, 28, 28},
        {13, 9651, LBM_F16, kBlockPatch, 1, 13, 28, 28}, {4758, 4, LBM_F32, kBlockPatch, 1, 12, 32, 24},
        {9, 16408, LBM_F32, kBlockPatch, 1, 9, 24, 24}, {401, 301, LBM_F16, kBlockTiles, 0, 0, 0, 0},
        {1500, 1400, LBM_F32, kBlockTiles, 4, 12, 0, 0},
    };
    for (const Case& c : cases) {
        const BlockPlan p = block_plan(std::vector<lbm_instance>((size_t)c.count, inst(c.nx, c.ny)), c.storage);
        const bool ok = p.kind == c.kind && (!c.rows || p.rows == c.rows) && (!c.waves || p.waves == c.waves) &&
                        p.wx == c.wx && p.wy == c.wy;
        if (!ok) std::printf("%d x %d: kind %d, rows %d, %d wavefronts, %d x %d\n", c.nx, c.ny, p.kind, p.rows, p.waves,
                             p.wx, p.wy);
        expect(ok, "form");
    }
}

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "streams") streams();
    else if (what == "strips") strips();
    else if (what == "plans") plans();
    else if (what == "short_runs") short_runs();
    else if (what == "pinned") pinned();
    else if (what == "forms") forms();
    else expect(false, "unknown check");
    std::printf("%s: %s\n", what.c_str(), failures ? "FAILED" : "ok");
    return failures ? 1 : 0;
}
