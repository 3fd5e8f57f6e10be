"""The host runtime's launches, with the HIP calls replaced by a recording
stand-in (csrc/ee_runtime.cpp is included whole): the pieces in which an
allocation-free batch runs when its chosen shape takes more units than the
scratch array holds, the rows per lane of the streaming sweeps, and how a batch
is planned."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_03311_amd", "csrc")

HARNESS = r"""
#include "ee_runtime.cpp"
#include <cstdlib>
#include <map>

static int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { if (fails < 20) { printf("FAIL line %d ", __LINE__); \
  printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

static int g_cus = 256;
alignas(256) static unsigned char g_scratch[size_t(2) << 20];
static int n_device_queries;  // one per evaluation of the launch-shape model
static int n_resets, n_sweeps, n_estimates, fresh;  // fresh: the queue counter was reset since the last sweep
static std::map<std::pair<int, int>, int> seen;      // (job, trajectory) -> times run
static std::vector<ee_job*> g_jobs;

extern "C" {
hipError_t hipGetDevice(int* d) { ++n_device_queries; *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  unsigned char* p = (unsigned char*)d;
  if (p >= g_scratch && p < g_scratch + sizeof g_scratch) {
    CHECK(p + n <= g_scratch + sizeof g_scratch, "a copy of %zu bytes passes the scratch array", n);
    if (p + n <= g_scratch + sizeof g_scratch) std::memcpy(d, s, n);
  }
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "?"; }
#define STUB(name, ...) hipError_t name(__VA_ARGS__) { return hipErrorUnknown; }
STUB(hipDeviceSynchronize) STUB(hipEventCreate, hipEvent_t*) STUB(hipEventCreateWithFlags, hipEvent_t*, unsigned)
STUB(hipEventDestroy, hipEvent_t) STUB(hipEventElapsedTime, float*, hipEvent_t, hipEvent_t) STUB(hipEventQuery, hipEvent_t)
STUB(hipEventRecord, hipEvent_t, hipStream_t) STUB(hipEventSynchronize, hipEvent_t) STUB(hipFree, void*)
STUB(hipGraphAddEventRecordNode, hipGraphNode_t*, hipGraph_t, const hipGraphNode_t*, size_t, hipEvent_t)
STUB(hipGraphAddKernelNode, hipGraphNode_t*, hipGraph_t, const hipGraphNode_t*, size_t, const hipKernelNodeParams*)
STUB(hipGraphCreate, hipGraph_t*, unsigned) STUB(hipGraphDestroy, hipGraph_t) STUB(hipGraphExecDestroy, hipGraphExec_t)
STUB(hipGraphInstantiate, hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) STUB(hipGraphLaunch, hipGraphExec_t, hipStream_t)
STUB(hipHostFree, void*) STUB(hipHostMalloc, void**, size_t, unsigned) STUB(hipMalloc, void**, size_t)
STUB(hipMemcpy, void*, const void*, size_t, hipMemcpyKind)
STUB(hipOccupancyMaxActiveBlocksPerMultiprocessor, int*, const void*, int, size_t)
STUB(hipStreamCreateWithFlags, hipStream_t*, unsigned) STUB(hipStreamDestroy, hipStream_t)
STUB(hipStreamWaitEvent, hipStream_t, hipEvent_t, unsigned)

int ee_k_max_lds_bytes() { return 160 * 1024 - 256; }
size_t ee_k_scratch_bytes() { return sizeof g_scratch; }
int ee_k_scratch_ptr(void** out) { *out = g_scratch; return 0; }
int ee_k_sweep_kernel_ptr(int, const void** fn) { *fn = g_scratch; return 0; }
int ee_k_sweep_plain_ptr(const void**) { return 1; }
int ee_k_sweep_whole_ptr(const void**) { return 1; }
int ee_k_queue_reset_ptr(const void**) { return 1; }
int ee_k_estimate_plan(int, int, ee::EstLaunch*) { return 0; }
int ee_k_march_lds_bytes(int w) { return 20 * w + 32; }
int ee_k_launch_march(const ee::JobDev*, int, int, int, int, int, uint32_t, int, int, int, void*) { return 1; }
int ee_k_launch_stream(const ee::StreamArgs*, int, int, int, uint32_t, int, int, int, void*) { return 1; }
int ee_k_launch_stream_init(const ee::JobDev*, int, int, void*) { return 1; }
int ee_k_launch_zero_work(const ee::JobDev*, int, void*) { return 1; }
int ee_k_launch_queue_reset(int* q, void*) { CHECK((void*)q == g_scratch, "queue counter"); ++n_resets; fresh = 1; return 0; }
int ee_k_launch_estimate(const ee::JobDev* const* tab, int count, int max_n, void*) {
  ++n_estimates;
  CHECK(count == (int)g_jobs.size(), "estimates of %d jobs", count);
  for (int i = 0; i < count; ++i) CHECK(tab[i] == g_jobs[i]->dev_jobdev() && g_jobs[i]->d.n_traj <= max_n, "job table");
  return 0;
}
int ee_k_launch_sweep(int, const ee::JobDev* single, int, const ee::Unit* units, int n, int* q, const ee::JobDev* const* tab,
                      uint32_t flags, int, int, int grid, int block, int lds, void*) {
  ++n_sweeps;
  CHECK(single == nullptr && (void*)q == g_scratch && fresh && flags == (ee::kFlagInit | ee::kFlagProto), "arguments");
  fresh = 0;
  CHECK(n >= 1 && grid >= 1 && grid <= n && block >= 64 && block <= 1024 && lds <= ee_k_max_lds_bytes(), "shape");
  CHECK((unsigned char*)(units + n) <= g_scratch + sizeof g_scratch, "%d units pass the scratch array", n);
  for (int i = 0; i < n && fails == 0; ++i) {
    const ee::Unit& u = units[i];
    const ee_job* j = g_jobs[u.job];
    CHECK(tab[u.job] == j->dev_jobdev(), "unit %d job table", i);
    CHECK(u.count >= 1 && u.count <= u.slots && u.slots <= ee::kMaxSlots && u.j0 + u.count <= j->d.n_traj, "unit %d", i);
    CHECK(u.slots * j->L.lds_words * 4 <= lds && block / u.slots >= j->L.G, "unit %d does not fit the launch", i);
    for (int t = 0; t < u.count; ++t) seen[{u.job, u.j0 + t}] += 1;
  }
  return 0;
}
}

static ee_job* make(const ee_job_desc& d) {
  static uintptr_t arena = size_t(1) << 40;  // addresses only: nothing reads them
  size_t need = 0;
  ee_job* j = nullptr;
  if (ee_job_footprint(&d, &need) != EE_OK || ee_job_create(&d, (void*)arena, need, nullptr, &j) != EE_OK) {
    printf("FAIL create: %s\n", ee_last_error());
    exit(1);
  }
  arena += need;
  return j;
}

int main(int argc, char** argv) {
  g_cus = atoi(argv[2]);
  if (argv[1][0] == 'p') {  // pieces: dim lt lx ly n, then trajectories per job
    int total = 0;
    for (int i = 8; i < argc; ++i) {
      g_jobs.push_back(make(ee_job_desc{atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), atoi(argv[7]), 1, 1,
                                        atoi(argv[i]), 0.3, 7, 0, 0}));
      total += atoi(argv[i]);
    }
    UnitPlan up;
    plan_units(g_jobs.data(), (int)g_jobs.size(), 0, ee_launch_cfg{0, 0, 0, 1, 0}, &up);
    const size_t cap = (sizeof g_scratch - align_up(kAlign + 8 * g_jobs.size())) / sizeof(ee::Unit);
    const int pieces = (int)((up.units.size() + cap - 1) / cap);
    const ee_status s = ee_batch_run_noalloc(g_jobs.data(), (int)g_jobs.size(), 0, nullptr, nullptr);
    CHECK(s == EE_OK, "%s", ee_last_error());
    CHECK(n_sweeps == pieces && n_resets == pieces && n_estimates == 1, "%d sweeps, %d pieces", n_sweeps, pieces);
    CHECK((int)seen.size() == total, "%zu of %d trajectories", seen.size(), total);
    for (const auto& kv : seen) CHECK(kv.second == 1, "trajectory %d of job %d ran %d times", kv.first.second, kv.first.first, kv.second);
    printf("pieces %d fails %d\n", pieces, fails);
  } else if (argv[1][0] == 'q') {  // plan: block threads, LDS bytes
    const int lats[4][5] = {{2, 24, 24, 1, 2}, {3, 16, 16, 16, 2}, {2, 64, 34, 1, 3}, {2, 24, 24, 1, 3}};
    for (int i = 0; i < 60; ++i) {
      const int* l = lats[i % 4];
      g_jobs.push_back(make(ee_job_desc{l[0], l[1], l[2], l[3], l[4], 1, 10 + i % 7, 1 + i * i % 97, 0.3, 7, 0, 0}));
    }
    const ee_launch_cfg cfg{atoi(argv[3]), atoi(argv[4]), 0, 1, 0};
    n_device_queries = 0;
    UnitPlan up;
    CHECK(plan_units(g_jobs.data(), 60, 5, cfg, &up) == EE_OK, "plan");
    const int queries = n_device_queries;
    int next[60] = {0};
    double last = 1e300;
    for (size_t i = 0; i < up.units.size(); ++i) {
      const ee::Unit& u = up.units[i];
      const double cost = unit_cost(g_jobs[u.job], up.block, u.slots, 5);
      CHECK(cost <= last, "unit %zu is longer than the one before", i);
      CHECK(u.j0 == next[u.job], "unit %zu: job %d from %d, not %d", i, u.job, u.j0, next[u.job]);
      // equal ones in the order of the jobs
      if (i && cost == last) CHECK(u.job >= up.units[i - 1].job, "unit %zu out of order", i);
      next[u.job] = u.j0 + u.count;
      last = cost;
    }
    for (int i = 0; i < 60; ++i) CHECK(next[i] == g_jobs[i]->d.n_traj, "job %d ends at %d", i, next[i]);
    printf("queries %d fails %d\n", queries, fails);
  } else if (argv[1][0] == 's') {  // shape: dim lt lx ly n l n_traj flags
    ee_job* j = make(ee_job_desc{atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), atoi(argv[7]), atoi(argv[8]), 1,
                                 atoi(argv[9]), 0.3, 7, 0, (uint32_t)atoi(argv[10])});
    const Shape s = launch_shape(j->d, j->L, j->d.n_traj);
    CHECK(s.k == 1, "%d trajectories per workgroup", s.k);
    printf("block %d fails %d\n", s.block, fails);
  } else {  // rows per lane: dim lt lx ly n n_traj
    ee_job* j = make(ee_job_desc{atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), atoi(argv[7]), 1, 1, atoi(argv[8]),
                                 0.3, 7, 0, 0});
    const ee::StreamArgs a = stream_args(j);
    CHECK(a.lanes == a.slots * (j->L.G / stream_words(j)) && a.blocks == (a.lanes + 255) / 256, "lanes");
    printf("rows %d fails %d\n", (a.rows + a.slots - 1) / a.slots, fails);
  }
  return fails != 0;
}
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    (d / "r.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, "-w",
                    str(d / "r.cpp"), "-o", str(d / "r")], check=True)

    def run(*args):
        r = subprocess.run([str(d / "r"), *map(str, args)], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.endswith("fails 0\n"), r.stdout + r.stderr
        return int(r.stdout.split()[1])
    return run


# one trajectory a workgroup on 256 CUs: 136,070 units, more than the 131,040
# that the scratch array holds beside its tables
def test_noalloc_set_beyond_the_scratch_runs_in_two_pieces(runtime):
    assert runtime("pieces", 256, 2, 128, 64, 1, 2, 65535, 65535, 5000) == 2


@pytest.mark.parametrize("cus", [64, 256, 304])
@pytest.mark.parametrize("lattice", [(2, 8, 8, 1, 2), (2, 64, 64, 1, 2), (2, 40, 34, 1, 3), (3, 10, 22, 6, 2), (3, 24, 24, 24, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_noalloc_units_cover_every_trajectory_once(runtime, lattice, cus):
    for counts in ((1, 2, 17), (4000, 1, 900)):
        assert runtime("pieces", cus, *lattice, *counts) >= 1


# the first job with two rows per lane is the first of more than four row words
# per lane of the GPU (1024 per CU)
@pytest.mark.parametrize("cus", [64, 256, 304])
@pytest.mark.parametrize("lattice,per_traj", [((2, 32, 32, 1, 2), 64), ((2, 34, 24, 1, 3), 102), ((2, 16, 16, 1, 2), 32),
                                              ((2, 32, 8, 1, 2), 64), ((2, 10, 22, 1, 2), 60), ((3, 12, 32, 10, 2), 240),
                                              ((3, 6, 14, 10, 3), 360)], ids=str)
def test_rows_per_lane_of_streamed_jobs(runtime, lattice, per_traj, cus):
    n = 4 * cus * 1024 // per_traj
    assert runtime("rows", cus, *lattice, n) == 1
    assert runtime("rows", cus, *lattice, n + 1) == 2


# four lattices, interleaved: the model is evaluated once for each where it
# gives the block size, and not at all where the caller does; one more query is
# the grid's
@pytest.mark.parametrize("cfg,evaluations", [((0, 0), 4), ((0, 8192), 4), ((256, 0), 0), ((256, 8192), 0)], ids=str)
def test_plan_of_an_uneven_batch(runtime, cfg, evaluations):
    assert runtime("query", 256, *cfg) == evaluations + 1


# Microseconds per half-sweep of jobs of few trajectories over the workgroup
# sizes, one trajectory each, as measured on 256 CUs: (dim, lt, lx, ly, n,
# trajectories, l, whole-region), {threads: us}.  The runtime's own choice is
# within a quarter of the best (twice the scatter of its model).
MEASURED = [
    ((2, 116, 28, 1, 2, 1, 23, 0),
     {64: 1.73, 128: 1.16, 192: 1.13, 256: 1.73, 320: 1.71, 384: 1.71, 448: 1.38, 512: 1.44, 576: 1.22, 640: 1.22,
      704: 1.24, 768: 1.2, 832: 1.26, 896: 1.26, 960: 1.03}),
    ((3, 14, 20, 10, 3, 30, 18, 1),
     {64: 5.15, 128: 3.65, 192: 4.53, 256: 3.61, 320: 3.48, 384: 3.48, 448: 2.23, 512: 2.22, 576: 2.33, 640: 2.1,
      704: 2.25, 768: 2.25, 832: 2.26, 896: 1.94, 960: 1.94, 1024: 1.91}),
    ((2, 56, 28, 1, 3, 1, 25, 0),
     {64: 1.7, 128: 1.12, 192: 1.71, 256: 1.41, 320: 1.41, 384: 1.45, 448: 1.44, 512: 1.31, 576: 1.21, 640: 1.2,
      704: 0.91}),
    ((2, 22, 118, 1, 2, 100, 79, 0),
     {64: 1.8, 128: 1.2, 192: 1.72, 256: 1.46, 320: 1.42, 384: 1.35, 448: 1.41, 512: 1.48, 576: 1.38, 640: 1.51,
      704: 0.93}),
    ((2, 28, 68, 1, 2, 30, 43, 1),
     {64: 2.52, 128: 2.4, 192: 1.96, 256: 1.95, 320: 1.33, 384: 1.34, 448: 1.34, 512: 0.95}),
    ((3, 26, 32, 18, 2, 30, 22, 1),
     {64: 11.11, 128: 5.85, 192: 4.25, 256: 3.68, 320: 3.56, 384: 3.72, 448: 3.57, 512: 3.81, 576: 3.65, 640: 3.68,
      704: 3.18, 768: 3.19, 832: 3.14, 896: 3.17, 960: 2.58, 1024: 2.65}),
    ((2, 78, 54, 1, 3, 4, 36, 1),
     {64: 5.21, 128: 4.28, 192: 4.81, 256: 4.02, 320: 3.93, 384: 4.31, 448: 4.65, 512: 2.21, 576: 2.41, 640: 2.4,
      704: 2.5, 768: 2.59, 832: 2.41, 896: 2.35, 960: 2.22, 1024: 2.08}),
    ((2, 68, 38, 1, 2, 1, 28, 1),
     {64: 2.61, 128: 2.04, 192: 2.02, 256: 1.65, 320: 1.6, 384: 1.6, 448: 1.58, 512: 1.55, 576: 1.37, 640: 1.38,
      704: 0.97}),
    ((2, 106, 84, 1, 2, 4, 61, 1),
     {64: 6.59, 128: 4.9, 192: 4.14, 256: 4.04, 320: 3.47, 384: 3.48, 448: 3.45, 512: 4.45, 576: 4.09, 640: 2.96,
      704: 2.38, 768: 2.25, 832: 2.38, 896: 2.39, 960: 2.26, 1024: 2.37}),
    ((3, 10, 20, 8, 3, 1, 9, 0),
     {64: 2.35, 128: 1.09, 192: 1.15, 256: 1.54, 320: 1.85, 384: 1.62, 448: 1.62, 512: 1.62, 576: 1.36, 640: 1.79,
      704: 2.11, 768: 1.15}),
]


@pytest.mark.parametrize("job,us", MEASURED, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_shape_of_few_trajectories(runtime, job, us):
    dim, lt, lx, ly, n, n_traj, l, whole = job
    block = runtime("shape", 256, dim, lt, lx, ly, n, l, n_traj, 4 if whole else 0)
    assert us[block] <= 1.25 * min(us.values()), (block, us)
