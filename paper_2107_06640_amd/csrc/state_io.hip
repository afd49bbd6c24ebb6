// Checkpoint transfers (state_io.hpp): chunks of elements go through pinned host
// memory that the kernels read and write directly, permuting and converting on
// the way, while host threads copy other chunks between it and the caller's
// array. What bounds a transfer is the host's copy of pageable memory (and the
// first touch of a fresh array's pages), so several threads share it.
#include "state_io.hpp"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <system_error>
#include <thread>
#include <vector>

#include "layout.hpp"

namespace seis {

namespace {

constexpr int kWorkers = 8;                  // host threads at most
constexpr int64_t kChunkValues = 256 * 1024;  // values of a chunk: 2 MiB

template <typename T>
__global__ __launch_bounds__(256) void k_state_in(T* Q, const int32_t* at, const double* src, int64_t e0, int64_t n, int row,
                                                  int RT) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t e = i / row;
  const int r = int(i - e * row);
  Q[qidx(at[e0 + e], r / 9, r % 9, RT)] = (T)src[i];
}

template <typename T>
__global__ __launch_bounds__(256) void k_state_out(const T* Q, const int32_t* at, double* dst, int64_t e0, int64_t n, int row,
                                                   int RT) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t e = i / row;
  const int r = int(i - e * row);
  dst[i] = (double)Q[qidx(at[e0 + e], r / 9, r % 9, RT)];
}

struct Chunk {
  int64_t e0 = 0, n = 0;  // first element, values
};

// Chunks in order over the host threads, each with two buffers and their
// events: launch(chunk, buffer) starts the kernel that uses the buffer.
template <bool READ, class Launch>
hipError_t move(StateIO& io, double* dofs, int64_t E, int row, hipStream_t s, Launch launch) {
  const int64_t per = std::max<int64_t>(1, std::min<int64_t>(E, kChunkValues / row)), chunks = (E + per - 1) / per;
  const int hw = std::max(1, (int)std::thread::hardware_concurrency());
  const int workers = (int)std::min<int64_t>(std::min(kWorkers, hw), chunks);
  const int64_t buf = per * row, need = chunks == 1 ? buf : buf * 2 * workers;
  if (io.pin_values < need) {
    state_io_free(io);
    const hipError_t st = hipHostMalloc((void**)&io.pin, need * sizeof(double), hipHostMallocDefault);
    if (st != hipSuccess) {
      io.pin = nullptr;
      return st;
    }
    io.pin_values = need;
  }
  int dev = 0;
  hipError_t st = hipGetDevice(&dev);
  if (st != hipSuccess) return st;
  std::atomic<int64_t> next{0};
  std::atomic<int> bad{hipSuccess};
  auto work = [&](int w) {
    hipEvent_t ev[2] = {nullptr, nullptr};
    Chunk in[2];
    auto ok = [&](hipError_t r) {
      if (r != hipSuccess) bad.store(r);
      return bad.load() == hipSuccess;
    };
    // wait for a buffer's kernel; a read chunk is then copied out
    auto finish = [&](int b) {
      if (!in[b].n) return true;
      const bool good = ok(hipEventSynchronize(ev[b]));
      if (READ && good) std::memcpy(dofs + in[b].e0 * row, io.pin + (2 * w + b) * buf, in[b].n * sizeof(double));
      in[b].n = 0;
      return good;
    };
    bool good = ok(hipSetDevice(dev));
    for (int b = 0; good && b < 2; ++b) good = ok(hipEventCreateWithFlags(&ev[b], hipEventDisableTiming));
    int b = 0;
    for (; good; b ^= 1) {
      good = finish(b);
      const int64_t c = next.fetch_add(1);
      if (!good || c >= chunks) break;
      in[b].e0 = c * per;
      in[b].n = std::min(per, E - in[b].e0) * row;
      double* p = io.pin + (2 * w + b) * buf;
      if (!READ) std::memcpy(p, dofs + in[b].e0 * row, in[b].n * sizeof(double));
      good = ok(launch(in[b], p)) && ok(hipEventRecord(ev[b], s));
      if (!good) in[b].n = 0;
    }
    finish(b ^ 1);
    finish(b);
    for (hipEvent_t e : ev)
      if (e) (void)hipEventDestroy(e);
  };
  std::vector<std::thread> pool;
  try {
    pool.reserve(workers);
    for (int w = 1; w < workers; ++w) pool.emplace_back(work, w);
  } catch (const std::exception&) {
    // fewer threads: the ones that run take every chunk
  }
  work(0);
  for (std::thread& t : pool) t.join();
  st = hipStreamSynchronize(s);
  return bad.load() != hipSuccess ? (hipError_t)bad.load() : st;
}

}  // namespace

void state_io_free(StateIO& io) {
  if (io.pin) (void)hipHostFree(io.pin);
  io.pin = nullptr;
  io.pin_values = 0;
}

template <typename T>
hipError_t state_write(StateIO& io, T* Q, const double* dofs, int64_t E, int B, hipStream_t s) {
  if (E <= 0) return hipSuccess;
  const int row = B * 9, RT = row_tiles(B);
  return move<false>(io, const_cast<double*>(dofs), E, row, s, [&](const Chunk& c, const double* p) {
    hipLaunchKernelGGL(k_state_in<T>, dim3((unsigned)((c.n + 255) / 256)), dim3(256), 0, s, Q, io.at, p, c.e0, c.n, row, RT);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t state_read(StateIO& io, const T* Q, double* dofs, int64_t E, int B, hipStream_t s) {
  if (E <= 0) return hipSuccess;
  const int row = B * 9, RT = row_tiles(B);
  return move<true>(io, dofs, E, row, s, [&](const Chunk& c, double* p) {
    hipLaunchKernelGGL(k_state_out<T>, dim3((unsigned)((c.n + 255) / 256)), dim3(256), 0, s, Q, io.at, p, c.e0, c.n, row, RT);
    return hipGetLastError();
  });
}

template hipError_t state_write<float>(StateIO&, float*, const double*, int64_t, int, hipStream_t);
template hipError_t state_write<double>(StateIO&, double*, const double*, int64_t, int, hipStream_t);
template hipError_t state_read<float>(StateIO&, const float*, double*, int64_t, int, hipStream_t);
template hipError_t state_read<double>(StateIO&, const double*, double*, int64_t, int, hipStream_t);

}  // namespace seis
