// A HIP runtime and kernel launchers that only take notes, linked with the library's
// host code (fwi_runtime.cpp) so that its order of launches, streams and waits can be
// checked without a device.  "Device" memory is host memory.  main() runs the scenario
// named by its first argument and prints what happened.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "fwi.h"
#include "fwi_internal.h"

namespace {
int g_device = 0;          // the current device
int g_stream_device = 0;   // the device of every stream but the default one
uintptr_t g_next = 0x1000;
struct Note {
    std::string what;
    hipStream_t stream;
};
std::vector<Note> g_notes;
bool g_quiet = false;      // several threads: no notes
void note(const char *what, hipStream_t st)
{
    if (!g_quiet) g_notes.push_back({what, st});
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = g_device; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t st, hipDevice_t *d)
{
    *d = st ? g_stream_device : g_device;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    memcpy(d, s, n);
    note("copy", st);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) { note("sync", st); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned)
{
    *st = reinterpret_cast<hipStream_t>(g_next += 0x10);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c)
{
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = reinterpret_cast<hipEvent_t>(g_next += 0x10);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace fwi {
void launch_step(int, int, int, bool, const Job *, const int *, int, int, int, int, int,
                 const LevelMap &, hipStream_t st) { note("step", st); }
void launch_prep_kappa(const float *, float *, int, int, int, int, int, int, int, int, int, int, int,
                       int64_t, float, hipStream_t st) { note("kappa", st); }
void launch_stage_check(const StageArgs &a, hipStream_t st)
{
    StageResult r{};
    r.vmin = 1500.f;
    r.vmax = 3000.f;
    r.bad_src = r.bad_rec = INT64_MAX;
    r.map_set = 1;
    *a.result = r;
    note("check", st);
}
void launch_stage_tables(const StageArgs &, const Job &, const JobStrides &, Job *, int *,
                         hipStream_t st) { note("tables", st); }
int nonfinite_blocks() { return 1; }
void launch_fill(float *, int64_t, float, hipStream_t st) { note("fill", st); }
void launch_zero_frames(float *, int64_t, int64_t, int, int, int, int, int, int, int, hipStream_t st)
{
    note("frames", st);
}
void launch_snapshot(const Job *, int, int64_t, int, int, int, int, const LevelMap &, hipStream_t st)
{
    note("snapshot", st);
}
void launch_gather(const Job *, const int *, int, int, int, int, const LevelMap &, hipStream_t st)
{
    note("gather", st);
}
int misfit_partials() { return 1; }
void launch_misfit(const float *, const float *, float *, int64_t, double *, double *, hipStream_t st)
{
    note("misfit", st);
}
void launch_fold(int, const Job *, int, int, int, int, int, int, int, int, int, int, float *, float *,
                 const float *, float *, hipStream_t st) { note("fold", st); }
int vstats_blocks() { return 1; }
int range_blocks() { return 1; }
void launch_vstats(const float *, int64_t, float *, int, hipStream_t st) { note("stats", st); }
void launch_nonfinite_level(const Job *, int, int, float *partial, hipStream_t st)
{
    partial[0] = 0.f;
    note("level", st);
}
void launch_assemble(const AssembleArgs &, Job *, int *, int32_t *, hipStream_t st)
{
    note("assemble", st);
}
int tb2d_width(int) { return 64; }
int tb2d_height(int) { return 64; }
void launch_step2d_tb(int, int, bool, const Job *, int, const TbLaunch &, hipStream_t st)
{
    note("tile steps", st);
}
int pipe2d_width() { return 128; }
int pipe2d_group(int) { return 12; }
void launch_step2d_pipe(int, const Job *, int, const PipeLaunch &, hipStream_t st)
{
    note("marching steps", st);
}
void launch_gather2(const Job *, int, int, int, int, int, hipStream_t) {}
void launch_trace_duplicates(const Job *, int, int, int, hipStream_t) {}
int scratch_address(void **p) { *p = nullptr; return -1; }
void launch_stream_probe(const float *, const float *, const float *, float *, int64_t, int,
                         hipStream_t) {}
void launch_tile_probe(const float *, const float *, const float *, float *, int, int, int, int, int,
                       int, hipStream_t) {}
}  // namespace fwi

namespace {
void *memory(uint64_t n) { return aligned_alloc(256, (n + 255) / 256 * 256); }

fwi_problem problem(int order)
{
    fwi_problem p{};
    p.ndim = 2;
    p.shape[0] = 30;
    p.shape[1] = 40;
    p.dx = 10.f;
    p.dt = 1e-3f;
    p.nt = 12;
    p.order = order;
    p.nsponge = 5;
    p.eta_max = -1.f;
    p.nshots = 1;
    p.nrec = 3;
    return p;
}

fwi_job *job(int order, hipStream_t st)
{
    static float data[4096];
    static int32_t pos[16];
    const fwi_problem p = problem(order);
    uint64_t n = 0;
    fwi_job *j = nullptr;
    if (fwi_job_bytes(&p, FWI_JOB_FORWARD, 4, nullptr, &n) != FWI_OK ||
        fwi_job_create(&p, FWI_JOB_FORWARD, 4, nullptr, data, data, pos, pos, nullptr, data, nullptr,
                       memory(n), n, st, &j) != FWI_OK) {
        printf("failed: %s\n", fwi_last_error());
        exit(2);
    }
    return j;
}

// What fwi_job_create does on its stream, in order.
void create()
{
    job(8, reinterpret_cast<hipStream_t>(0x10));
    for (const Note &n : g_notes) printf("%s\n", n.what.c_str());
}

// The streams that the steps of two kinds of jobs go to, where the caller's stream
// belongs to device `device` and device 0 is current.
void lanes(int device)
{
    const hipStream_t st = reinterpret_cast<hipStream_t>(0x10);
    g_stream_device = device;
    fwi_job *jobs[2] = {job(8, st), job(4, st)};
    uint64_t n = 0;
    fwi_jobs_ws_bytes(2, 4, &n);
    g_notes.clear();
    if (fwi_jobs_advance(jobs, 2, 4, memory(n), n, st) != FWI_OK) {
        printf("failed: %s\n", fwi_last_error());
        exit(2);
    }
    std::set<hipStream_t> used;
    int steps = 0;
    for (const Note &x : g_notes)
        if (x.what == "step") {
            used.insert(x.stream);
            ++steps;
        }
    printf("steps %d streams %zu caller %d\n", steps, used.size(), (int)used.count(st));
}

// The kinds of step launches of a 2-D forward of `shots` shots of 1024 x 320 cells.
void forward(int order, int shots)
{
    fwi_problem p = problem(order);
    p.shape[0] = 320;
    p.shape[1] = 1024;
    p.nsponge = 20;
    p.nshots = shots;
    p.nrec = 0;
    static float data[1 << 20];
    static int32_t pos[1 << 10];
    uint64_t n = 0;
    if (fwi_workspace_bytes(&p, FWI_MODE_FORWARD, nullptr, &n) != FWI_OK ||
        fwi_forward(&p, data, data, pos, nullptr, nullptr, memory(n), n, nullptr) != FWI_OK) {
        printf("failed: %s\n", fwi_last_error());
        exit(2);
    }
    std::set<std::string> kinds;
    for (const Note &x : g_notes)
        if (x.what.find("step") != std::string::npos) kinds.insert(x.what);
    for (const std::string &k : kinds) printf("%s\n", k.c_str());
}

// Two threads that both need the device's number of compute units first.
void threads()
{
    g_quiet = true;
    static float f[4][64];
    auto call = [] {
        int32_t zc = 0;
        if (fwi_tile_probe(f[0], f[1], f[2], f[3], 64, 64, 64, 0, 0, &zc, nullptr) != FWI_OK) exit(2);
    };
    std::thread a(call), b(call);
    a.join();
    b.join();
    printf("done\n");
}
}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "create") create();
    else if (what == "lanes") lanes(argc > 2 ? atoi(argv[2]) : 0);
    else if (what == "forward") forward(argc > 2 ? atoi(argv[2]) : 8, argc > 3 ? atoi(argv[3]) : 1);
    else if (what == "threads") threads();
    else return 3;
    return 0;
}
