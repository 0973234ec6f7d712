// The HIP calls and kernel launchers that the library's host sources need, on
// host memory, so that their allocation, admission and error paths run without
// a GPU.  Device memory is a byte budget that the test sets; the launchers
// that the tested paths reach work on the host (data movement, tile
// passes and batches leave the amplitudes alone), every other one fails.
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>

#include "kernels.h"

using namespace qsim;

namespace {

std::mutex mu;
size_t budget = SIZE_MAX, used = 0;
long mallocs = 0;
std::map<void *, size_t> blocks;
hipError_t malloc_error = hipSuccess;  // returned by every hipMalloc when set
int device = 0;
int queue_grid = 0;
uint64_t tile_launches[2] = {};  // those that read their records ahead, the others

void tile_launch(const TileArgs &a) { ++tile_launches[a.n_touch ? 0 : 1]; }

[[noreturn]] void not_here(const char *what) { fail(QS_ERR_UNSUPPORTED, std::string("no host version of ") + what); }

}  // namespace

extern "C" {

// ---- what a test sets and reads
void host_set_budget(size_t bytes) { budget = bytes; }
size_t host_used() { return used; }
long host_mallocs() { return mallocs; }
void host_set_malloc_error(int e) { malloc_error = (hipError_t)e; }
void host_set_device(int d) { device = d; }
void host_tile_launches(uint64_t *ahead, uint64_t *others)
{
    *ahead = tile_launches[0];
    *others = tile_launches[1];
    tile_launches[0] = tile_launches[1] = 0;
}
int host_queue_grid() { return queue_grid; }  // workgroups of the last batch launch

// ---- HIP
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "host runtime"; }
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *, int) { return hipErrorNotSupported; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> lk(mu);
    *p = nullptr;
    ++mallocs;
    if (malloc_error != hipSuccess)
        return malloc_error;
    if (n > budget || used > budget - n)
        return hipErrorOutOfMemory;
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    if (!*p)
        return hipErrorOutOfMemory;
    blocks[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lk(mu);
    auto it = blocks.find(p);
    if (it == blocks.end())
        return p ? hipErrorInvalidValue : hipSuccess;
    used -= it->second;
    blocks.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { return *t = 0, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

qs_status qs_run_program_noalloc(qs_state *, const qs_program *) { return QS_ERR_UNSUPPORTED; }

}  // extern "C"

// ---- kernel launchers
namespace qsim {

void launch_set_basis(void *state, qs_dtype dt, int n, uint64_t x, hipStream_t)
{
    std::memset(state, 0, (size_t)(dt == QS_C64 ? 8 : 16) << n);
    if (dt == QS_C64)
        static_cast<float *>(state)[2 * x] = 1;
    else
        static_cast<double *>(state)[2 * x] = 1;
}

void launch_logical(const void *state, qs_dtype dt, int n, const std::vector<int> &sigma, uint64_t i0, uint64_t count,
                    double *out, hipStream_t)
{
    if (device != 0)
        fail(QS_ERR_HIP, "a launch on the state's stream with another device current");
    for (uint64_t i = i0; i < i0 + count; ++i) {
        uint64_t j = 0;
        for (int q = 0; q < n; ++q)
            j |= ((i >> q) & 1) << sigma[q];
        for (int c = 0; c < 2; ++c)
            out[2 * (i - i0) + c] = dt == QS_C64 ? (double)static_cast<const float *>(state)[2 * j + c]
                                                 : static_cast<const double *>(state)[2 * j + c];
    }
}

size_t zsum_work_doubles(int n) { return n + 1; }
size_t zfold_work_doubles(uint64_t, int n) { return n + 1; }
size_t fid_work_doubles(int) { return 5; }

void launch_plain_gate(void *, qs_dtype, int, const qs_gate &, hipStream_t) { not_here("a plain gate"); }
void launch_involution(void *, qs_dtype, int, const std::vector<int> &, hipStream_t) {}
void launch_tile_f32(const TileArgs &a, uint64_t, int, int, hipStream_t) { tile_launch(a); }
void launch_tile_f64(const TileArgs &a, uint64_t, int, int, hipStream_t) { tile_launch(a); }
void launch_tile_f32_z(const TileArgs &, uint64_t, int, int, double *, hipStream_t) { not_here("a tile pass"); }
void launch_tile_f64_z(const TileArgs &, uint64_t, int, int, double *, hipStream_t) { not_here("a tile pass"); }
void launch_batch_init(void *, qs_dtype, uint64_t, const uint64_t *, int, hipStream_t) { not_here("a batch"); }
void launch_batch_f32(const BatchArgs &, int, int, int, hipStream_t) { not_here("a batch"); }
void launch_batch_f64(const BatchArgs &, int, int, int, hipStream_t) { not_here("a batch"); }
void launch_batch_reduce(const double *, const uint64_t *, const uint32_t *, int, double *, hipStream_t)
{
    not_here("a batch");
}
void launch_queue_reset(uint32_t *, uint64_t, hipStream_t) {}
void launch_batch_queue_f32(const QueueArgs &, int grid, hipStream_t) { queue_grid = grid; }
void launch_batch_queue_f64(const QueueArgs &, int grid, hipStream_t) { queue_grid = grid; }
void launch_zsum(const void *, qs_dtype, int, double *, double *, hipStream_t) { not_here("read-out sums"); }
void launch_zfold(const double *, uint64_t, int, int, const ZFoldMap &, double *, double *, hipStream_t)
{
    not_here("a folded read-out");
}
void launch_gather(const void *, qs_dtype, const uint64_t *, int64_t, double *, hipStream_t) { not_here("a gather"); }
void launch_fidelity(const void *, qs_dtype, const void *, qs_dtype, int, const std::vector<int> &, double *, double *,
                     hipStream_t)
{
    not_here("a fidelity");
}

}  // namespace qsim
