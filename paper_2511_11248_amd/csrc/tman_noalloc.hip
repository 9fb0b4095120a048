// tman_mpgemv for callers that cannot allocate device memory (code under HIP graph capture, tight serving
// loops, harnesses that forbid hipMalloc): the tickets and partial sums that tman_mpgemv takes as a caller
// workspace live in a fixed array in device memory that belongs to the library.
//
// The array's name is only a host-side stand-in for the symbol: its device address is looked up once per
// device with hipGetSymbolAddress (each GPU holds its own copy at its own address) and that pointer is what
// the kernels receive, exactly as they receive the caller's workspace in tman_mpgemv.
#include <mutex>

#include "tman_internal.h"

namespace tman {

// A call's workspace is its tickets (one per row block), then its partial sums.  Calls of different shapes share the
// array, so the partial sums of all of them start at the same byte and the tickets lie before it: a ticket is never a
// byte that another shape used for sums (with the tickets at the array's start, a shape with more row blocks found sums
// in its tickets, and its y was left unwritten).  Tickets are used when K has at least two segments, whose sums take at
// least 512 bytes per row block; the region holds the tickets of all such shapes that the sums' limit admits.
constexpr size_t kTicketRegion = (size_t)TMAN_NOALLOC_SCRATCH_BYTES / (2 * kRows * sizeof(float)) * sizeof(int32_t);
static_assert(kTicketRegion % 256 == 0, "partial sums stay aligned");
static __device__ __align__(256) unsigned char scratch[kTicketRegion + TMAN_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static void* scratch_ptr[kMaxDevices];  // device address of `scratch` on device i, once resolved

// Device address of the scratch array on the current device (resolved at the first call on that device).
static int scratch_on_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TMAN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return TMAN_ERR_LAUNCH;
        }
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return TMAN_OK;
}

}  // namespace tman

using namespace tman;

extern "C" {

int tman_noalloc_init(void) {
    void* p = nullptr;
    return scratch_on_current_device(&p);
}

int tman_mpgemv_noalloc(const tman_shape_t* shape, const void* packed, const void* lut, int32_t N, void* y,
                        void* stream) {
    int rc = check_shape(shape);
    if (rc != TMAN_OK) return rc;
    if (!packed || !lut || !y) return TMAN_ERR_NULL;
    if (N < 1 || N > TMAN_MAX_DECODE_TOKENS) return TMAN_ERR_SHAPE;
    if (!aligned16(packed) || !aligned16(lut)) return TMAN_ERR_ALIGN;
    if (tman_mpgemv_workspace_bytes(shape, N) > (size_t)TMAN_NOALLOC_SCRATCH_BYTES) return TMAN_ERR_WORKSPACE;
    void* ws = nullptr;
    rc = scratch_on_current_device(&ws);
    if (rc != TMAN_OK) return rc;
    // The tickets are zero when the library is loaded and every call returns them to zero; the partial sums are
    // written before they are read.  Nothing needs clearing between calls.
    const Layout L = make_layout(shape);
    const size_t tickets = plan_tables(L, N).ticket_bytes;  // (more than the region only when K is one segment: unused)
    if (tickets <= kTicketRegion) ws = static_cast<uint8_t*>(ws) + (kTicketRegion - tickets);
    return launch_mpgemv(L, packed, lut, N, y, ws, (hipStream_t)stream);
}

}  // extern "C"
