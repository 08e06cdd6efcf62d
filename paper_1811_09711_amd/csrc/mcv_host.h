// Host-side helpers shared by the C-ABI entry points: error state, problem
// validation, creation of one job's device state, and the combination of
// iterations into one estimate.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <string>

#include "mcv.h"
#include "mcv_internal.h"

namespace mcv {

// Records msg as the calling thread's last error and returns st.
mcv_status fail(mcv_status st, const std::string& msg);
const char* last_error();

#define MCV_HIP(call)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess)                                                               \
      return ::mcv::fail(MCV_E_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

mcv_status validate_problem(const mcv_problem* p);

// Device memory of the library: from the allocator installed with
// mcv_set_allocator, else hipMalloc.  Each block goes back to the allocator
// that made it.  dev_free waits for the device first (as hipFree does), so a
// caching allocator never hands out memory that queued work still reads.
hipError_t dev_alloc(void** p, size_t bytes);
void dev_free(void* p);
mcv_status set_allocator(mcv_alloc_fn alloc, mcv_free_fn release, void* ctx);

// The static work area of mcv_unweight_noalloc on `device` (noalloc.hip):
// its device address, looked up once per device with that device current,
// and its size.
mcv_status static_work_area(int device, char** out);
size_t static_work_bytes();

// Compute units of the current device.
mcv_status device_cus(int* device, int* n_cu);

// Creates one job's device state in a single device block (*block, freed with
// hipFree): problem arrays, derived constants, equidistant grids, tables,
// allocation and pass buffers, history, and the job's device record
// (j->self).  Per-unit partial buffers are carved for gmax work units when
// gmax > 0 and left null otherwise.  Synchronises `s` before returning.
mcv_status job_create(const mcv_problem* p, int gmax, int64_t n_points, int n_cu, hipStream_t s,
                      JobDev* j, void** block);

// Device bytes job_create would allocate for this problem (a valid one).
size_t job_block_bytes(const mcv_problem* p, int gmax);

// Bytes of the per-unit partial buffers of a job for G work units.
size_t partial_bytes(const JobDev& j, int G);
// Points the job's partial buffers into `base` (partial_bytes(j, G) bytes).
void carve_partials(JobDev& j, int G, char* base);

// Copies of device arrays of one job's block to the host, ordered on a stream
// and waited for.  Arrays that lie close together (carved one after another)
// are fetched by one copy.  A copy into pageable memory costs 11 to 20 us each
// and more above 64 KB (108 us for 313 KB), one into pinned memory 14 us at
// that size; so what an object reads repeatedly goes through a pinned buffer
// that it keeps, made with it if one reading takes more than kReadSmall bytes
// (making one costs 55 to 70 us, which a small job would not earn back), and
// smaller readings through the stack.
constexpr size_t kReadSmall = 16 << 10;

struct HostSeg {
  void* dst;        // null: not wanted
  const void* src;
  size_t bytes;
};

struct HostRead {
  void* pin = nullptr;
  size_t cap = 0;
  std::mutex mu;  // readers of one object on several threads share the buffer

  void reserve(size_t bytes);  // without memory: readings go straight to their places
  void release();
  mcv_status read(const HostSeg* seg, int n, hipStream_t s);
};

// Bytes of the largest single reading of a job's arrays.
size_t state_read_bytes(const JobDev& j);
// The segments of edges, alpha and the allocation (N_c and their total).
void state_segs(const JobDev& j, double* edges, double* alpha, int64_t* alloc, HostSeg (&seg)[4]);

// Inverse-variance weighted mean of history rows [first, n) (kHistStride
// doubles each), its error and chi^2/ndf; iterations with zero error are
// exact and are averaged alone.
void combine_history(const double* hist, int n, int first, mcv_summary* out);

}  // namespace mcv
