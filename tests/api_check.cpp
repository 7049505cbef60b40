// Host check of the calls of include/loss.h: loss_api.cpp and tables.cpp compiled against the
// stand-ins below.  "Device" memory is host memory, every copy and every index that a launch
// is given is checked against the allocations' sizes, and no kernel runs.
// Usage: api_check SCENARIO [ARGS].  Prints the scenario's result, then "ok" or what failed.
#define __align__(x) __attribute__((aligned(x)))
#define HIP_SYMBOL(x) x
#include "../paper_2301_05127_amd/csrc/loss_api.cpp"

#include <cstdarg>
#include <map>

// ---- what failed, and what was done ----------------------------------------------------
static int fails = 0;
static void check(bool ok, const char *fmt, ...)
{
    if (ok || fails++) return;
    va_list ap;
    va_start(ap, fmt);
    std::vprintf(fmt, ap);
    va_end(ap);
    std::printf("\n");
}

static std::map<char *, size_t> heap;                  // device allocations
static size_t heap_used = 0, heap_limit = ~size_t(0);
static int64_t allocations = 0, refused = -1;          // number of the allocation that fails
static int64_t bytes_h2d = 0;
static std::map<std::string, int64_t> launches;

// bytes from p to the end of its allocation; memory that is not the device's has no bound
static size_t room(const void *p)
{
    auto it = heap.upper_bound((char *)p);
    if (it == heap.begin()) return ~size_t(0);
    --it;
    return (char *)p < it->first + it->second ? size_t(it->first + it->second - (char *)p) : ~size_t(0);
}
static bool on_device(const void *p) { return room(p) != ~size_t(0); }

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    if (allocations++ == refused || n > heap_limit || heap_used > heap_limit - n) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    if (!*p) return hipErrorOutOfMemory;
    heap[(char *)*p] = n;
    heap_used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    auto it = heap.find((char *)p);
    check(it != heap.end(), "free of what was not allocated");
    if (it == heap.end()) return hipErrorInvalidValue;
    heap_used -= it->second;
    heap.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *free_mem, size_t *total)
{
    *total = std::min(heap_limit, size_t(288) << 30);
    *free_mem = *total - heap_used;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k)
{
    check(n <= room(d), "copy of %zu bytes into %zu", n, room(d));
    check(n <= room(s), "copy of %zu bytes from %zu", n, room(s));
    if (k == hipMemcpyHostToDevice) bytes_h2d += n;
    if (n <= room(d) && n <= room(s)) std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    check(n <= room(d), "fill of %zu bytes in %zu", n, room(d));
    if (n <= room(d)) std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { *p = const_cast<void *>(symbol); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)1; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)1; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = (hipGraphExec_t)1;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
}

// ---- launches ----------------------------------------------------------------------------
namespace loss {
static hipError_t count(const std::string &name)
{
    launches[name]++;
    return hipSuccess;
}
static void traces_hold(const double *traces, int64_t off, int64_t len)
{
    check(off >= 0 && (size_t)(off + len) * sizeof(double) <= room(traces), "trace samples %ld .. %ld outside the traces",
          (long)off, (long)(off + len));
}
hipError_t launch_tile(int mode, const TileArgs &a, hipStream_t)
{
    const int64_t tiles = (int64_t)a.S * a.nother * a.x.nsub * a.r.nsub;
    if (a.info) {
        check((size_t)tiles * sizeof(int2) <= room(a.info), "words of the tiles");
        launches["receivers"] = 0;
        for (int64_t t = 0; t < tiles && !fails; ++t) {
            const int plane = (int)(t / (a.x.nsub * a.r.nsub)), lr = (int)(t / a.x.nsub % a.r.nsub), lx = (int)(t % a.x.nsub);
            auto owns = [](const TileAxis &x, int l, int64_t node) {   // a piece's nodes; node N with the last one
                return node >= x.piece[l].x && (node < x.piece[l].y || (node == x.N && x.piece[l].y == x.N));
            };
            for (int k = a.info[t].x; k < a.info[t].x + a.info[t].y / 2; ++k) {
                check((size_t)(k + 1) * sizeof(RecDev) <= room(a.rec), "receiver %d of a tile", k);
                if (fails) break;
                const RecDev &r = a.rec[k];
                traces_hold(a.traces, r.trace_off, a.trace_len);
                const int64_t o = a.nother > 1 ? r.node / a.ostride : 0, in = r.node - o * a.ostride;
                check(r.shot == plane / a.nother && o == plane % a.nother && owns(a.r, lr, in / a.rstride) &&
                          owns(a.x, lx, in % a.rstride), "receiver %d in tile %ld", k, (long)t);
                check(k == a.info[t].x || r.trace_off > a.rec[k - 1].trace_off, "order of the receivers of tile %ld", (long)t);
                launches["receivers"]++;
            }
        }
    }
    launches["tiles"] = tiles;
    launches["waves"] = a.nw;
    return count("tile " + std::to_string(mode));
}
hipError_t launch_tile_z(int op, const TileZArgs &, hipStream_t) { return count("tile_z " + std::to_string(op)); }
hipError_t launch_axis_rows(int op, const AxisArgs &, hipStream_t) { return count("axis " + std::to_string(op)); }
hipError_t launch_axis_x(int op, const AxisArgs &, hipStream_t) { return count("axis " + std::to_string(op)); }
hipError_t launch_line(int, int, int, const LineArgs &, hipStream_t) { return count("line"); }
hipError_t launch_adj_junctions(int, const LineArgs &, float *, hipStream_t) { return count("adj_junctions"); }
hipError_t launch_adj_gather(int, int, const LineArgs &, const float *, hipStream_t) { return count("adj_gather"); }
hipError_t launch_adj_x(int, const LineArgs &, hipStream_t) { return count("adj_x"); }
hipError_t launch_adj_xx(const LineArgs &, const float *, float *, float, hipStream_t) { return count("adj_xx"); }
int line_xx_threads(const LineArgs &) { return 0; }
hipError_t launch_line_xx(const LineArgs &, float *, float *, hipStream_t) { return count("line_xx"); }
hipError_t launch_pml_adj_operand(float *, const float *, const float *, float, float *, const float4 *, int, int, int, int,
                                  int, int64_t, int64_t, int, hipStream_t) { return count("pml_operand"); }
hipError_t launch_el_normal_operand(float *, const float *, const float *, const float *, const float *, const float *, int,
                                    int, int64_t, int64_t, int, hipStream_t) { return count("normal_operand"); }
hipError_t launch_el_grad_accum(double *, double *, const float *const *, const float *const *, float *const *, const float *,
                                const float *, const float *, double, int, int64_t, int64_t, int, hipStream_t)
{
    return count("el_grad_accum");
}
hipError_t launch_el_grad_unpad(const double *, const double *, const double *, double *, int, int64_t, const float *,
                                const float *, const float *, int, int64_t, hipStream_t) { return count("el_grad_unpad"); }
hipError_t launch_el_grad_b(double *, const float *const *, const float *const *, double, int, int64_t, int64_t, int,
                            hipStream_t) { return count("el_grad_b"); }
hipError_t launch_inject(const SrcDev *, int, float *const *, const float *, const float *, const float *, int64_t, int64_t,
                         int64_t, const int64_t *, int, float, int, hipStream_t) { return count("inject"); }
hipError_t launch_el_grad_force(double *, const SrcDev *, int, float *const *, const float *, const float *, int64_t, int64_t,
                                int64_t, int64_t, double, const int *, hipStream_t) { return count("el_grad_force"); }
hipError_t launch_res_gather(const RecTarget *tg, int nt, const int64_t *toff, float *const *, float *, int64_t,
                             const double *res, int64_t n, float, hipStream_t)
{
    for (int t = 0; t < nt; ++t)
        for (int k = tg[t].first; k < tg[t].first + tg[t].count; ++k) traces_hold(res, toff[k] + n, 1);
    return count("res_gather");
}
hipError_t launch_record2(const RecDev *r0, int n0, float, int, const RecDev *r1, int n1, float, int, const float *const *,
                          int64_t, double *traces, const int64_t *, int, int64_t len, hipStream_t)
{
    for (int k = 0; k < n0; ++k) traces_hold(traces, r0[k].trace_off, len);
    for (int k = 0; k < n1; ++k) traces_hold(traces, r1[k].trace_off, len);
    return count("record");
}
hipError_t launch_set_step(int64_t *s, int64_t v, hipStream_t) { *s = v; return hipSuccess; }
hipError_t launch_pad_copy(const float *, float *, int, int, int64_t, int, hipStream_t) { return count("pad_copy"); }
hipError_t launch_media(const float *, const float *, const float *, float *const *, int, int, int, int64_t, double,
                        hipStream_t) { return count("media"); }
hipError_t launch_fill(float *p, int64_t n, float, hipStream_t)
{
    check((size_t)n * 4 <= room(p), "fill of %ld floats in %zu bytes", (long)n, room(p));
    return hipSuccess;
}
hipError_t launch_grad_accum(double *, const float *, const float *, float, int, int64_t, int64_t, hipStream_t)
{
    return count("grad_accum");
}
hipError_t launch_grad_unpad(const double *, double *, int, int, int64_t, const float *, const float *, int, hipStream_t)
{
    return count("grad_unpad");
}
hipError_t launch_nonfinite(const float *, int64_t, int *, hipStream_t) { return count("nonfinite"); }
hipError_t launch_energy(const EnergyArgs &, int, double *, int, double, double *, hipStream_t) { return count("energy"); }
}  // namespace loss

// ---- scenarios ---------------------------------------------------------------------------
struct Sim {
    loss_sim *s = nullptr;
    loss_desc d{};
    int64_t nodes = 0;
    loss_status status;
    Sim(int physics, const int (&n)[3], const int (&M)[3], int halo, int shots, int nt, int end_mode = 0)
    {
        d.physics = physics;
        d.ndim = physics == LOSS_ACOUSTIC ? 2 : 3;
        nodes = 1;
        for (int a = 0; a < 3; ++a) {
            d.n[a] = n[a];
            d.h[a] = 10.0;
            d.patch[a] = M[a];
            nodes *= n[a] + 1;
        }
        d.dt = 1e-3;
        d.halo = halo;
        d.end_mode = end_mode;
        d.nshots = shots;
        d.trace_len = nt;
        status = loss_create(&d, nullptr, &s);
        if (status) return;
        std::vector<float> vp(nodes, 2000.f), vs(nodes, 1000.f), rho(nodes, 1000.f);
        status = loss_set_media(s, vp.data(), physics == LOSS_ELASTIC ? vs.data() : nullptr, rho.data(), LOSS_MEM_HOST);
    }
    ~Sim() { loss_destroy(s); }
    // nrec receivers along the first row of every shot
    void receivers(int nrec)
    {
        std::vector<int32_t> idx;
        for (int i = 0; i < nrec; ++i)
            for (int v : {i % (int)(d.n[0] + 1), 0, i / (int)(d.n[0] + 1)}) idx.push_back(v);
        for (int k = 0; k < d.nshots; ++k)
            ok(loss_add_receivers(s, k, nrec, idx.data(), d.physics == LOSS_ACOUSTIC ? LOSS_F_SIGMA : LOSS_F_EV3));
    }
    void gradient(int nrec)
    {
        std::vector<double> res((size_t)d.nshots * nrec * d.trace_len, 1.0), g(3 * nodes);
        const bool el = d.physics == LOSS_ELASTIC;
        ok(loss_adjoint(s, res.data(), el ? LOSS_GRAD_LAME_RHO : LOSS_GRAD_K, g.data(), LOSS_MEM_HOST));
    }
    void ok(loss_status r) { check(r == LOSS_OK, "status %d: %s", (int)r, loss_last_error()); }
};

// receivers exchanged and their (empty) traces read between a forward run and its adjoint
static void exchanged_receivers(int physics)
{
    const int n2[3] = {40, 0, 40}, n3[3] = {20, 20, 20}, M[3] = {20, 20, 20};
    Sim sim(physics, physics == LOSS_ACOUSTIC ? n2 : n3, M, 6, 2, 4);
    sim.ok(sim.status);
    sim.receivers(100);
    sim.ok(loss_forward_ckpt(sim.s, 4, 2));
    sim.receivers(3);
    std::vector<double> t(3 * 4);
    sim.ok(loss_get_traces(sim.s, 0, t.data(), LOSS_MEM_HOST));
    sim.gradient(3);
}

// receivers on every node of some planes: each is in its tile's list, once
static void tile_receivers(int physics, const int (&n)[3], const int (&M)[3], int halo, int shots)
{
    Sim sim(physics, n, M, halo, shots, 3);
    sim.ok(sim.status);
    const int nrec = (int)std::min<int64_t>(sim.nodes, (n[0] + 1) * 40);
    std::vector<int32_t> idx;
    for (int i = nrec - 1; i >= 0; --i)
        for (int v : {i % (n[0] + 1), i * 7 % (n[1] + 1), i * 3 % (n[2] + 1)}) idx.push_back(v);
    for (int k = 0; k < shots; ++k)
        sim.ok(loss_add_receivers(sim.s, k, nrec, idx.data(), physics == LOSS_ACOUSTIC ? LOSS_F_SIGMA : LOSS_F_EV1 + 4 * (k % 2)));
    sim.ok(loss_set_shape(sim.s, 3, 0));
    sim.ok(loss_step(sim.s, 1));
    const int64_t last = launches["receivers"], want = (int64_t)nrec * (physics == LOSS_ACOUSTIC ? shots : (shots + 1) / 2);
    check(last == want, "%ld receivers in tiles, %ld given", (long)last, (long)want);
}

// the row pitch of a handle, on a device of `gib` GiB
static void pitch(int nx, int nz, int shots, int gib)
{
    heap_limit = size_t(gib) << 30;
    const int n[3] = {nx - 1, 0, nz - 1}, M[3] = {std::min(nx - 1, 64), 1, std::min(nz - 1, 64)};
    Sim sim(LOSS_ACOUSTIC, n, M, 6, shots, 0);
    sim.ok(sim.status);
    std::printf("%ld\n", sim.s ? (long)sim.s->pitch : 0);
}

// each allocation of a short run refused in turn: an error or a run without what it was for, and
// nothing left behind; prints how many runs went through
static void refusals(int physics)
{
    const int n2[3] = {40, 0, 40}, n3[3] = {20, 20, 20}, M[3] = {20, 20, 20};
    int ran = 0;
    for (int64_t k = 0;; ++k) {
        allocations = 0;
        refused = k;
        Sim sim(physics, physics == LOSS_ACOUSTIC ? n2 : n3, M, 6, 2, 4);
        loss_status r = sim.status;
        if (!r) sim.receivers(5);
        if (!r) r = loss_step(sim.s, 2);
        check(r == LOSS_OK || r == LOSS_ENOMEM, "allocation %ld: status %d", (long)k, (int)r);
        if (allocations <= k) break;
        ran += r == LOSS_OK;
    }
    refused = -1;
    std::printf("%d\n", ran);
}

// the operands that a gradient keeps for its tile passes make room for other allocations
static void operands()
{
    const int n[3] = {20, 20, 20}, M[3] = {20, 20, 20};
    Sim sim(LOSS_ELASTIC, n, M, 6, 2, 8);
    sim.ok(sim.status);
    sim.receivers(3);
    sim.ok(loss_forward_ckpt(sim.s, 8, 4));
    sim.gradient(3);
    check(sim.s->adj_el[11] != nullptr, "no operands kept");
    heap_limit = heap_used + 15 * 4 * field_elems(sim.s);     // the run below needs 18 fields more, less 4
    sim.ok(loss_forward_ckpt(sim.s, 8, 2));
}

// a second gradient, of more receivers
static void added_receivers(int physics)
{
    const int n2[3] = {40, 0, 40}, n3[3] = {20, 20, 20}, M[3] = {20, 20, 20};
    Sim sim(physics, physics == LOSS_ACOUSTIC ? n2 : n3, M, 6, 2, 4);
    sim.ok(sim.status);
    for (int nrec : {3, 100}) {
        sim.receivers(nrec);
        sim.ok(loss_forward_ckpt(sim.s, 4, 2));
        sim.gradient(nrec);
    }
}

// derivatives of host arrays: each field crosses to the device once
static void host_deriv(int physics, const int (&n)[3], const int (&M)[3], int halo, int end_mode)
{
    Sim sim(physics, n, M, halo, 2, 0, end_mode);
    sim.ok(sim.status);
    const int batch = 5;
    std::vector<float> in(batch * sim.nodes, 1.f), out(in);
    for (int axis = 0; axis < 3; axis += physics == LOSS_ACOUSTIC ? 2 : 1)
        for (int order : {1, 2, -1}) {
            bytes_h2d = 0;
            sim.ok(loss_deriv(sim.s, axis, order, in.data(), out.data(), batch, LOSS_MEM_HOST));
            check(bytes_h2d == (int64_t)in.size() * 4, "axis %d order %d: %ld bytes of %zu", axis, order, (long)bytes_h2d, in.size() * 4);
        }
    for (const auto &l : launches) std::printf("%s %ld\n", l.first.c_str(), (long)l.second);
}

// prints the schedule of a grid (0 tiles, 1 line passes), and the tiles of a pass and the waves of
// a tile when it runs as tiles
static void route(int physics, const int (&n)[3], const int (&M)[3], int halo, int shots)
{
    Sim sim(physics, n, M, halo, shots, 0);
    sim.ok(sim.status);
    int32_t schedule = -1;
    sim.ok(loss_autotune_choice(sim.s, 3, &schedule));
    sim.ok(loss_set_shape(sim.s, 3, 0));
    sim.ok(loss_step(sim.s, 1));
    std::printf("%d %ld %ld\n", (int)schedule, (long)launches["tiles"], (long)launches["waves"]);
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    auto arg = [&](int k) { return argc > k ? std::atoi(argv[k]) : 0; };
    if (what == "exchanged_receivers") exchanged_receivers(arg(2));
    else if (what == "added_receivers") added_receivers(arg(2));
    else if (what == "route" && argc == 11) {
        const int n[3] = {arg(3), arg(4), arg(5)}, M[3] = {arg(6), arg(7), arg(8)};
        route(arg(2), n, M, arg(9), arg(10));
    } else if (what == "pitch") pitch(arg(2), arg(3), arg(4), arg(5));
    else if (what == "refusals") refusals(arg(2));
    else if (what == "operands") operands();
    else if (what == "tile_receivers" && argc == 11) {
        const int n[3] = {arg(3), arg(4), arg(5)}, M[3] = {arg(6), arg(7), arg(8)};
        tile_receivers(arg(2), n, M, arg(9), arg(10));
    } else if (what == "host_deriv" && argc == 11) {
        const int n[3] = {arg(3), arg(4), arg(5)}, M[3] = {arg(6), arg(7), arg(8)};
        host_deriv(arg(2), n, M, arg(9), arg(10));
    } else check(false, "unknown scenario");
    check(heap.empty(), "%zu allocations left", heap.size());
    if (!fails) std::printf("ok\n");
    return fails ? 1 : 0;
}
