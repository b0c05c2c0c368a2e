// Host-side memory and read-backs of the library, shared by the triangle and
// tetrahedron handles (defined in api.hip): the process-wide stream-ordered
// cache of device blocks, the free list of pinned host blocks, and mail.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace pm {
// A block freed on a stream is handed out again only on that stream, whose
// order makes the reuse safe without a wait. block_free returns a block that
// did not come from the cache to the driver.
hipError_t block_alloc(hipStream_t s, void** p, size_t bytes);
void block_free(void* p);

// Pinned host blocks of kPinnedBytes (pinning memory is a slow driver call):
// one per handle, given back when it is destroyed. null: out of memory.
constexpr size_t kPinnedBytes = 128 * 1024;
void* pinned_take();
void pinned_give(void* p);

// Larger pinned blocks for staging a call's host arrays, taken for the call; a few
// are kept for the next one (of any handle or thread). null: out of memory.
constexpr size_t kStageBytes = 2 << 20;
void* stage_take();
void stage_give(void* p);

// Mail: a kernel at the end of the stream's work writes a few counters into
// pinned host memory and then a letter number, which the host polls: about 5 us
// from the last kernel to the host, where a copy and a stream synchronisation
// took about 15. The number's place is the last int of a pinned block.
struct Mail {
  volatile int* at = nullptr;
  int no = 0;
};
Mail mail_of(void* pinned_block);
// n ints at src to dst (in the block), then the mail's next number
void mail_send(Mail& b, const int* src, int n, int* dst, hipStream_t s);
// the number of the next letter, for a kernel that delivers by itself
void mail_next(Mail& b);
// waits for the number sent last; an error of the stream ends the wait
hipError_t mail_wait(const Mail& b, hipStream_t s);
// for kernels that deliver by themselves: threads of one work-group call it
// after their stores to host memory
__device__ __forceinline__ void mail_post(int* at, int no) {
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(at, no, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace pm
