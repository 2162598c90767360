// Device memory owned by a handle (host code only).
#pragma once
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "../../include/cvbound.h"

namespace cvb {

// Records the message of an error (cv_last_error) and returns its code.
int fail(int code, const char* fmt, ...);

#define HIPCHK(expr)                                                                            \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess) return cvb::fail(CV_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// Bytes behind every device array: the dense kernels read four neighbouring
// entries at once (gemm.hip: ld_quad), also where fewer are left.
constexpr size_t kSlack = 64;

// A handle's device arrays, dealt out of chunks (a root pass builds a handle
// per layer: an allocation and a release for each of its 33 arrays were half of
// its time), all released together.  Between begin() and flush() small uploads
// gather in one staging block and reach the device in one copy.
//
// take() hands the chunks of one sub-network of a root pass to the next, at most
// kKeep bytes of them, so that much the pass may hold beyond what its present
// sub-network needs; chunks without an array go back to the device before an
// allocation fails.
struct DevMem {
  struct Chunk {
    char* p;
    size_t size, used;
  };
  // arrays start 4 KiB apart (256 bytes apart, the smallest calls take 4 % longer:
  // 23.6 us against 22.8), staged ones 256 bytes
  static constexpr size_t kChunk = 1 << 20, kStage = 256 << 10, kAlign = 4096, kStageAlign = 256;
  static constexpr size_t kKeep = 256 << 20;
  std::vector<Chunk> chunks;
  std::vector<char> stage;  // (host) what flush() copies to sbase
  char* sbase = nullptr;
  bool staging = false, keep = false;  // keep: clear() leaves the chunks for the next arrays
  DevMem* peer = nullptr;              // whose idle chunks go too before an allocation fails
  DevMem() = default;
  DevMem(const DevMem&) = delete;
  DevMem& operator=(const DevMem&) = delete;
  ~DevMem() { release(); }
  void release() {
    for (const Chunk& c : chunks) (void)hipFree(c.p);
    chunks.clear();
  }
  // The chunks without an array, back to the device.
  void release_idle() {
    size_t n = 0;
    for (const Chunk& c : chunks) {
      if (c.used) chunks[n++] = c;
      else (void)hipFree(c.p);
    }
    chunks.resize(n);
  }
  void clear() {
    if (keep)
      for (Chunk& c : chunks) c.used = 0;
    else
      release();
    stage.clear();
    sbase = nullptr;
  }
  // o's chunks, for new arrays (o's own are gone): the smallest ones, kKeep
  // bytes in all; the others are released.
  void take(DevMem& o) {
    release();
    chunks.swap(o.chunks);
    std::sort(chunks.begin(), chunks.end(), [](const Chunk& a, const Chunk& b) { return a.size < b.size; });
    size_t kept = 0, n = 0;
    for (const Chunk& c : chunks) {
      kept += c.size;
      if (kept <= kKeep) chunks[n++] = Chunk{c.p, c.size, 0};
      else (void)hipFree(c.p);
    }
    chunks.resize(n);
  }
  template <typename T>
  int alloc(T** out, size_t count) {
    *out = nullptr;
    const size_t bytes = (std::max<size_t>(count, 1) * sizeof(T) + kSlack + kAlign - 1) & ~(kAlign - 1);
    Chunk* c = nullptr;
    for (Chunk& q : chunks)
      if (q.size - q.used >= bytes && (!c || q.size - q.used < c->size - c->used)) c = &q;
    if (!c) {
      void* p = nullptr;
      const size_t size = std::max(bytes, kChunk);
      hipError_t e = hipMalloc(&p, size);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        release_idle();
        if (peer) peer->release_idle();
        e = hipMalloc(&p, size);
      }
      if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(CV_ENOMEM, "device allocation of %zu bytes failed", count * sizeof(T));
      }
      chunks.push_back(Chunk{static_cast<char*>(p), size, 0});
      c = &chunks.back();
    }
    *out = reinterpret_cast<T*>(c->p + c->used);
    c->used += bytes;
    return CV_OK;
  }
  template <typename T>
  int upload(T** out, const T* host, size_t count, hipStream_t s) {
    (void)s;  // blocking copies: the host buffer may be a temporary
    const size_t bytes = count * sizeof(T), room = (bytes + kSlack + kStageAlign - 1) & ~(kStageAlign - 1);
    int rc;
    if (staging && host && bytes && room <= kStage / 2) {
      if (sbase && stage.size() + room > kStage && (rc = flush_stage())) return rc;
      if (!sbase && (rc = alloc(&sbase, kStage))) return rc;
      *out = reinterpret_cast<T*>(sbase + stage.size());
      stage.resize(stage.size() + room);
      std::memcpy(stage.data() + stage.size() - room, host, bytes);
      return CV_OK;
    }
    if ((rc = alloc(out, count))) return rc;
    if (count && host) HIPCHK(hipMemcpy(*out, host, bytes, hipMemcpyHostToDevice));
    return CV_OK;
  }
  void begin() { staging = true; }
  int flush() {
    staging = false;
    return flush_stage();
  }
  int flush_stage() {
    if (sbase && !stage.empty()) HIPCHK(hipMemcpy(sbase, stage.data(), stage.size(), hipMemcpyHostToDevice));
    stage.clear();
    sbase = nullptr;
    return CV_OK;
  }
};

}  // namespace cvb
