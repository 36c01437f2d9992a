// The host side of the C ABI (csrc/md_api.hip) over a model of the device, for error paths that
// a GPU must not be driven into: a HIP runtime that runs everything at once in host memory, and
// launchers that follow the control words only (rebuild flags, halt, told decisions, lists that
// overflow).  A launch that would read or write an array that is not there ends the program.
// Usage: host_model SCENARIO; exit status 0 when every check holds.
#include "../paper_1210_3450_amd/csrc/md_api.hip"

#include <cstdlib>
#include <functional>
#include <map>

namespace {
struct Model {
    std::map<const void*, size_t> size;  // live allocations
    int fail_at = -1;              // the fail_at-th allocation from now on fails (0: the next)
    bool full = false;             // every allocation fails
    hipError_t last = hipSuccess;
    int busy = 0;                  // stream queries that find the stream busy
    int dutc = 0, drop_dutc = -1;  // launches of k_dutc; the one that is lost
    hipError_t drop_error = hipSuccess;
    int build_every = 4;           // drifts between list builds
    int need = 40;                 // longest list of a build
    bool tile_overflow = false;
    double clock = 0.0;            // ms: builds without row tiles, cutting them, force passes with and without
    double build = 1.5, cut = 0.5, force_tile = 0.9, force_gather = 1.0;
} M;

int g_fail = 0;
#define CHECK(cond)                                                               \
    do {                                                                          \
        if (!(cond)) {                                                            \
            std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #cond);       \
            ++g_fail;                                                             \
        }                                                                         \
    } while (0)

void need_arrays(const Dev& d, const Params& p, const char* kernel, bool list) {
    bool ok = d.geom && d.st && d.any && d.halt && d.wave_box && d.tile_box && d.q[0] && d.q[1] && d.cnt && d.perm &&
              d.cell_cnt && d.cell_start && d.tile_sum && d.tile_pref && d.ke_part && d.pe_part && d.vir_part && d.red;
    if (p.tile) ok = ok && d.rtile && d.row_box && d.row_nt && d.row_t0 && d.cell_rt && d.rt_tmp && d.rt_rec;
    ok = ok && M.size[d.cell_cnt] >= (size_t)p.ntile * kTile * 4;
    if (p.tile) ok = ok && M.size[d.cell_rt] >= (size_t)p.ntile * kTile * 4 && M.size[d.row_nt] >= p.nrows * (size_t)4;
    if (list)
        ok = ok && d.list && p.rows * p.tpk == p.cap && M.size[d.list] >= (size_t)p.nwave * kWave * p.cap * 2;
    if (ok) return;
    std::fprintf(stderr, "%s launched on an array that is not there\n", kernel);
    std::exit(3);
}
bool off(const Dev& d) { return *d.halt || *d.any; }
}  // namespace

// ---- the runtime
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (M.full || (M.fail_at >= 0 && M.fail_at-- == 0)) return M.last = hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    M.size[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    M.size.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = M.last;
    M.last = hipSuccess;
    return e;
}
hipError_t hipStreamQuery(hipStream_t) {
    if (M.busy > 0) {
        --M.busy;
        return M.last = hipErrorNotReady;
    }
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { return p->multiProcessorCount = 256, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = reinterpret_cast<hipEvent_t>(new double(0.0)), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return delete reinterpret_cast<double*>(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return *reinterpret_cast<double*>(e) = M.clock, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    return *ms = (float)(*reinterpret_cast<double*>(b) - *reinterpret_cast<double*>(a)), hipSuccess;
}
}

// ---- the launchers
namespace mdg {
void launch_set_state(const Dev&, const Params&, const double*, const double*, int32_t, hipStream_t) {}
void launch_get_state(const Dev&, const Params&, double*, double*, int32_t, hipStream_t) {}
void launch_get_forces(const Dev&, const Params&, double*, int32_t, hipStream_t) {}
void launch_get_cells(const Dev&, const Params&, int32_t*, int32_t, hipStream_t) {}
void launch_list_counts(const Dev& d, const Params& p, int64_t*, int32_t, hipStream_t) {
    need_arrays(d, p, "k_list_counts", true);
}
void launch_list_ptr(const Dev&, int64_t, int64_t*, hipStream_t) {}
void launch_list_export(const Dev&, const Params&, const int64_t*, int32_t*, int32_t, hipStream_t) {}
void launch_mark_rebuild(const Dev& d, const Params& p, hipStream_t) {
    for (int b = 0; b < p.nbox; ++b) d.st[b].rebuild = 1;
    *d.any = 1;
}
int rowtile_blocks_per_cu(const Params&) { return 4; }
void launch_row_tiles(const Dev& d, const Params& p, hipStream_t) {
    need_arrays(d, p, "the tile cut", false);
    if (*d.any && !*d.halt) M.clock += M.cut;
}
void launch_rebuild_chain(const Dev& d, const Params& p, bool with_list, hipStream_t s) {
    need_arrays(d, p, "the rebuild chain", with_list);
    if (!*d.any || *d.halt) return;
    M.clock += M.build;
    if (p.tile) launch_row_tiles(d, p, s);
    if (p.tile && M.tile_overflow) {
        d.st[0].err |= 4;
        *d.halt = 1;
        return;
    }
    if (with_list && M.need > p.cap) {
        d.st[0].need = M.need;
        *d.halt = 1;
        return;
    }
    for (int b = 0; b < p.nbox; ++b) {
        BoxState& st = d.st[b];
        if (!st.rebuild) continue;
        st.sq ^= 1;
        st.sp ^= 1;
        st.rebuild = 0;
        if (!with_list) continue;
        st.built += 1;
        st.need = std::max(st.need, M.need);
    }
    *d.any = 0;
}
void launch_force(const Dev& d, const Params& p, int, int, hipStream_t) {
    need_arrays(d, p, "the force pass", true);
    if (p.tile) CHECK(p.tgrid >= 8);
    if (!off(d)) M.clock += p.tile ? M.force_tile : M.force_gather + 0.1 * (p.tpk - 1);
}
void launch_kick_drift(const Dev&, const Params&, hipStream_t) {}
void launch_dutc(const Dev& d, const Params& p, uint32_t seq, hipStream_t) {
    if (M.dutc++ == M.drop_dutc) {
        M.last = M.drop_error;
        return;
    }
    auto tell = [&](uint32_t code) {
        if (seq) d.told[seq & (kToldRing - 1)] = seq << 2 | code;
    };
    if (*d.halt) return tell(2);
    if (seq && *d.any) return;
    for (int b = 0; b < p.nbox; ++b) {
        BoxState& st = d.st[b];
        st.sq ^= 1;
        st.nstep += 1;
        st.rebuild = st.nstep % M.build_every == 0;
        if (st.rebuild) *d.any = 1;
        if (b == 0) tell(st.rebuild ? 1u : 0u);
    }
}
void launch_energy_reduce(const Dev& d, const Params& p, bool record, int, bool, int, hipStream_t) {
    need_arrays(d, p, "the energy sums", false);
    if (!off(d) && record) d.st[0].nseries += 1;
}
void launch_ke_partial(const Dev&, const Params&, hipStream_t) {}
void launch_vscale(const Dev&, const Params&, hipStream_t) {}
void launch_verify(const Dev&, const Params&, hipStream_t) {}
void launch_scale(const Dev&, const Params&, const double*, const double*, hipStream_t) {}
void launch_list_relayout(const Dev& d, const Params& p, const uint16_t*, int32_t, hipStream_t) {
    need_arrays(d, p, "k_list_relayout", true);
}
void launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t) { std::fill(p, p + n, v); }
void launch_bubbles(const Dev&, int32_t, int32_t, const SubGrid&, const BubbleWork&, uint8_t*, hipStream_t) {}
void launch_bubbles_scratch(const Dev&, int32_t, int32_t, const SubGrid&, unsigned char*, uint8_t*, hipStream_t) {}
hipError_t bubbles_scratch_init(int) { return hipSuccess; }
unsigned char* bubbles_scratch(int) { return nullptr; }
void bubbles_scratch_results(unsigned char*, int64_t**, int64_t**, int32_t**, NaMisc**) {}
}  // namespace mdg

namespace {
md_params params(uint32_t flags = 0) {
    md_params p{};
    p.n = 4000;
    p.box[0] = p.box[1] = p.box[2] = 20.0;
    p.rc = 2.5;
    p.skin = 0.3;
    p.dt = 0.005;
    p.mass = 1.0;
    p.flags = flags;
    return p;
}
// A context of nbox boxes with a state loaded.
md_ctx* open(const md_params& p, int nbox = 1) {
    const std::vector<md_params> b(nbox, p);
    md_ctx* c = nullptr;
    const double x = 0.0;
    CHECK(md_batch_create(b.data(), nbox, nullptr, &c) == MD_OK);
    CHECK(md_set_state(c, &x, &x) == MD_OK);
    return c;
}
int64_t steps(md_ctx* c) {
    md_stats st;
    CHECK(md_get_stats(c, &st) == MD_OK);
    return st.steps;
}

// The model itself: runs over several chunks, samples, a list that outgrows its capacity.
void plain() {
    for (int nbox : {1, 2}) {
        md_ctx* c = open(params(), nbox);
        CHECK(md_step(c, 450, 10) == MD_OK);
        CHECK(steps(c) == 450);
        int32_t n = 0;
        CHECK(md_energy_series(c, nullptr, nullptr, 0, &n) == MD_OK && n == 45);
        M.need = 300;
        CHECK(md_step(c, 50, 0) == MD_OK);
        CHECK(steps(c) == 500 && c->regrows == 1);
        M.need = 40;
        md_destroy(c);
    }
    CHECK(M.size.empty());
}

// A decision that never comes is an error, whichever drift it is and whether or not the launch
// error is still there when the host looks; never a call that reports steps it did not take.
void lost_decision() {
    for (int nbox : {1, 2})
        for (int at : {0, 1, 2, 5, 30})
            for (hipError_t e : {hipSuccess, hipErrorLaunchFailure})
                for (int busy : {0, 2})
                    for (int build_every : {4, 1000}) {
                        M.build_every = build_every;
                        md_ctx* c = open(params(), nbox);
                        CHECK(md_step(c, 3, 0) == MD_OK);
                        M.drop_dutc = M.dutc + at;
                        M.drop_error = e;
                        M.busy = busy;
                        const md_status s = md_step(c, 31, 0);
                        // with builds, the lost one may be of a drift that was left out and enqueued again
                        const bool spare = build_every == 4 && nbox == 1 && e == hipSuccess && s == MD_OK;
                        if (spare)
                            CHECK(c->steps == 34 && c->D.st[0].nstep == 34);
                        else
                            CHECK(s == MD_EHIP && c->steps == 3 && md_step(c, 1, 0) == MD_EHIP);
                        M.drop_dutc = -1;
                        M.busy = 0;
                        md_destroy(c);
                    }
}

// Memory runs out inside each call that lays arrays anew, at each of its allocations: the call says
// so, no later call launches on what is missing, and once there is memory again the context goes on.
void out_of_memory() {
    const std::function<md_status(md_ctx*)> ops[] = {
        [](md_ctx* c) { return md_rescale_box(c, 1.3); },
        [](md_ctx* c) { return md_autotune(c, nullptr); },
        [](md_ctx* c) { return M.need = 500, md_build_neighbors(c); },
        [](md_ctx* c) { return M.need = 500, md_step(c, 20, 0); },
    };
    const double x = 0.0;
    std::vector<int64_t> kp(4001);
    for (uint32_t flags : {0u, (uint32_t)MD_F_TILE_ON, (uint32_t)MD_F_HALF_LIST})
        for (const auto& op : ops)
            for (int k = 0, failed = 1; failed; ++k) {
                M.need = 40;
                md_ctx* c = open(params(flags));
                CHECK(md_step(c, 3, 0) == MD_OK);
                M.fail_at = k;
                const md_status s = op(c);
                failed = M.fail_at < 0;  // the k-th allocation was reached
                CHECK(s == (failed ? MD_ENOMEM : MD_OK));
                M.fail_at = -1;
                M.full = failed;  // nothing comes back at first
                const int32_t done = (int32_t)c->steps;
                auto only = [&](md_status t) { CHECK(t == MD_OK || t == MD_ENOMEM || t == MD_ESTATE); };
                only(md_get_neighbors(c, kp.data(), nullptr, 0, nullptr) == MD_EINVAL ? MD_OK : MD_ESTATE);
                only(md_compute_forces(c, nullptr));
                only(md_step(c, 0, 0));
                only(md_energy(c, nullptr, nullptr));
                only(md_build_cells(c));
                only(md_build_neighbors(c));
                only(md_rescale_box(c, 1.0));
                only(md_autotune(c, nullptr));
                CHECK(c->sticky == MD_OK && c->steps == done);
                M.full = false;
                CHECK(md_step(c, 10, 0) == MD_OK && c->steps == done + 10);
                CHECK(md_set_state(c, &x, &x) == MD_OK && md_step(c, 10, 0) == MD_OK);
                md_destroy(c);
            }
    CHECK(M.size.empty());
}

// Bytes of a sparse box's arrays: a context without row tiles pays nothing for them (39 words a
// tile), whichever way it came to the gather format, and the autotuner lays them when it needs them.
void tile_arrays() {
    auto bytes = [](uint32_t flags) {
        md_params p = params(flags);
        p.box[0] = p.box[1] = p.box[2] = 280.0;  // 10^6 cells
        md_ctx* c = open(p);
        size_t n = 0;
        for (const auto& a : M.size) n += a.second;
        CHECK((c->D.rt_rec != nullptr) == (flags == MD_F_TILE_ON));
        CHECK(md_step(c, 5, 0) == MD_OK && md_autotune(c, nullptr) == MD_OK && md_step(c, 5, 0) == MD_OK);
        md_destroy(c);
        return n;
    };
    const size_t tiles = bytes(MD_F_TILE_ON);
    for (uint32_t flags : {0u, (uint32_t)MD_F_TILE_OFF, (uint32_t)MD_F_HALF_LIST}) {
        CHECK(bytes(flags) < 16u * 1000000 && tiles > 150u * 1000000);
    }
}

// The autotuner where no row tile fits the staging capacity: with MD_F_TILE_ON the context is the
// gather format's by itself, and there is no candidate to time.
void autotune_without_tiles() {
    const char* cache = "host_model_tune.txt";
    std::remove(cache);
    M.tile_overflow = true;
    for (uint32_t flags : {0u, (uint32_t)MD_F_TILE_ON})
        for (const char* path : {(const char*)nullptr, cache}) {
            md_ctx* c = open(params(flags));
            CHECK(md_step(c, 5, 0) == MD_OK);
            CHECK(md_autotune(c, path) == MD_OK);
            CHECK(c->P.tpk >= 1 && c->P.tile == 0);
            CHECK(md_step(c, 5, 0) == MD_OK && steps(c) == 10);
            md_destroy(c);
        }
    std::remove(cache);
}

// Rescaling allocates only when the cells outgrow their arrays.
void rescale_in_place() {
    for (uint32_t flags : {0u, (uint32_t)MD_F_TILE_ON, (uint32_t)MD_F_HALF_LIST}) {
        md_ctx* c = open(params(flags));
        CHECK(md_step(c, 3, 0) == MD_OK);
        CHECK(md_rescale_box(c, 1.5) == MD_OK && md_step(c, 3, 0) == MD_OK);
        M.full = true;  // any allocation fails
        for (double a : {1.0, 0.9, 1.01, 1.0 / 0.9 / 1.01}) {
            CHECK(md_rescale_box(c, a) == MD_OK);
            CHECK(md_step(c, 3, 0) == MD_OK);
        }
        M.full = false;
        CHECK(md_rescale_box(c, 1.5) == MD_OK && md_step(c, 3, 0) == MD_OK);
        md_destroy(c);
    }
    CHECK(M.size.empty());
}

// The autotuner where the force pass gains 0.1 ms from row tiles and cutting them costs 0.5: one box
// cuts them with each of its builds, an ensemble whenever any box builds.
void autotune_ensemble() {
    M.build_every = 10;
    for (int nbox : {1, 2, 64}) {
        md_ctx* c = open(params(), nbox);
        CHECK(md_step(c, 40, 0) == MD_OK);  // a build every 10 steps
        CHECK(md_autotune(c, nullptr) == MD_OK);
        CHECK(c->P.tile == (nbox == 1) && c->P.tpk == 1);
        CHECK(md_step(c, 20, 0) == MD_OK && steps(c) == 60);
        md_destroy(c);
    }
}

// Staged records of FP64 row tiles: the larger capacity where most particles live in crowded cells or
// a box needs it, the smaller elsewhere; rescaling moves a context over the line and back.
void tile_capacity() {
    auto box = [](int64_t n) {
        md_params p = params(MD_F_TILE_ON);
        p.n = n;  // of 7^3 cells
        return p;
    };
    const struct {
        std::vector<int64_t> n;
        int scap;
    } cases[] = {{{8000}, kStageCap64}, {{11000}, kStageDense64}, {{8000, 8000, 11000}, kStageCap64},
                 {{8000, 8000, 16500}, kStageDense64}, {{4000, 12000, 12000}, kStageDense64}};
    for (const auto& k : cases) {
        std::vector<md_params> b;
        for (int64_t n : k.n) b.push_back(box(n));
        md_ctx* c = nullptr;
        CHECK(md_batch_create(b.data(), (int32_t)b.size(), nullptr, &c) == MD_OK);
        CHECK(c->P.scap == k.scap && c->P.tgrid >= 8);
        const double x = 0.0;
        CHECK(md_set_state(c, &x, &x) == MD_OK && md_rescale_box(c, 2.0) == MD_OK && c->P.scap == kStageCap64);
        CHECK(md_rescale_box(c, 0.5) == MD_OK && c->P.scap == k.scap);
        md_destroy(c);
    }
}
}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "plain") plain();
    else if (what == "lost_decision") lost_decision();
    else if (what == "out_of_memory") out_of_memory();
    else if (what == "tile_arrays") tile_arrays();
    else if (what == "autotune_without_tiles") autotune_without_tiles();
    else if (what == "rescale_in_place") rescale_in_place();
    else if (what == "autotune_ensemble") autotune_ensemble();
    else if (what == "tile_capacity") tile_capacity();
    else return std::fprintf(stderr, "unknown scenario\n"), 2;
    return g_fail ? 1 : 0;
}
