// context.cpp - device memory of a context: the caller's allocator or the
// runtime's, and the sequence engine's workspace.
#include <hip/hip_runtime_api.h>

#include <string>

#include "runtime.h"

void* mpld_context::try_alloc(size_t bytes) {
  if (has_alloc) return alloc.alloc(bytes, alloc.user);
  void* p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();   // or the next launch's check reports it
  return nullptr;
}

void* mpld_context::dev_alloc(size_t bytes) {
  void* p = try_alloc(bytes);
  if (!p) {
    seq_give_back();
    p = try_alloc(bytes);
  }
  const std::string size = std::to_string(bytes) + " bytes";
  if (!p && has_alloc) throw mpld::NoMemory{{MPLD_E_NOMEM, "device allocator returned NULL for " + size}};
  if (!p) throw mpld::NoMemory{{MPLD_E_DEVICE, "hipMalloc: out of memory for " + size}};
  return p;
}

bool mpld_context::seq_take(size_t bytes) {
  if (seq_bytes < bytes) {
    seq_give_back();
    void* p = try_alloc(bytes);
    if (!p) return false;
    std::lock_guard<std::mutex> lk(seq_mu);
    seq_mem = p;
    seq_bytes = bytes;
  }
  std::lock_guard<std::mutex> lk(seq_mu);
  seq_used = seq_bytes >= bytes;   // (another thread's allocation may have wanted it meanwhile)
  return seq_used;
}

void mpld_context::seq_give_back() {
  std::lock_guard<std::mutex> lk(seq_mu);
  if (!seq_mem || seq_used) return;
  (void)hipStreamSynchronize(stream);   // launches on the way still use it
  dev_free(seq_mem);
  seq_mem = nullptr;
  seq_bytes = 0;
}

void mpld_context::dev_free(void* p) {
  if (!p) return;
  if (has_alloc)
    alloc.free(p, alloc.user);
  else
    (void)hipFree(p);
}
