// A workgroup of a HIP kernel as host threads: enough of the language for kernels whose blocks
// share data through LDS, barriers and the wave sums of dfdg_device.h.  One block runs at a
// time; a thread that returns leaves its barriers, as an ended wave does.
#pragma once
#include <algorithm>
#include <barrier>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <thread>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __shared__ static  // one block at a time: kept from block to block, like LDS contents
#define __launch_bounds__(...)
using std::isfinite;
using std::max;
using std::min;

struct emu_dim { int x; };
struct emu_wave {
  std::barrier<> bar{64};
  int word[64];
};
inline emu_dim gridDim, blockDim, blockIdx;
inline thread_local emu_dim threadIdx;
inline thread_local emu_wave* emu_my_wave;
inline std::unique_ptr<std::barrier<>> emu_block_bar;

struct double2 { double x, y; };
struct float2 { float x, y; };

inline void __syncthreads() { emu_block_bar->arrive_and_wait(); }

inline int emu_lane(int x, int from) {  // lane `from`'s x (-1: none, 0)
  emu_wave& w = *emu_my_wave;
  w.word[threadIdx.x & 63] = x;
  w.bar.arrive_and_wait();
  const int v = from >= 0 ? w.word[from] : 0;
  w.bar.arrive_and_wait();
  return v;
}
// row shifts right within 16 lanes (0x110 + n), the last lane of a row to the next row (0x142)
// and of the lower half to the upper (0x143); rows outside the mask keep `old`
inline int emu_update_dpp(int old, int x, int ctrl, int rows, int, bool) {
  const int l = threadIdx.x & 63, row = l >> 4;
  int from = -1;
  if (ctrl > 0x110 && ctrl < 0x120) from = (l & 15) >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
  else if (ctrl == 0x142) from = row > 0 ? row * 16 - 1 : -1;
  else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
  const int v = emu_lane(x, from);
  return ((rows >> row) & 1) && from >= 0 ? v : old;
}
inline int emu_readlane(int x, int lane) { return emu_lane(x, lane); }
inline double __shfl_xor(double x, int off, int) {
  int w[2];
  std::memcpy(w, &x, 8);
  for (int& v : w) v = emu_lane(v, (threadIdx.x & 63) ^ off);
  std::memcpy(&x, w, 8);
  return x;
}
#define __builtin_amdgcn_update_dpp emu_update_dpp
#define __builtin_amdgcn_readlane emu_readlane
inline int __double2loint(double x) { int64_t b; std::memcpy(&b, &x, 8); return (int)(uint32_t)b; }
inline int __double2hiint(double x) { int64_t b; std::memcpy(&b, &x, 8); return (int)(b >> 32); }
inline double __hiloint2double(int hi, int lo) {
  const int64_t b = ((int64_t)hi << 32) | (uint32_t)lo;
  double x;
  std::memcpy(&x, &b, 8);
  return x;
}

// Runs body(thread) on the threads of block `block` of a grid.
template <typename F>
inline void emu_block(int block, int grid, int threads, F body) {
  gridDim.x = grid;
  blockDim.x = threads;
  blockIdx.x = block;
  emu_block_bar = std::make_unique<std::barrier<>>(threads);
  std::vector<std::unique_ptr<emu_wave>> waves;
  for (int w = 0; w < threads / 64; ++w) waves.push_back(std::make_unique<emu_wave>());
  std::vector<std::thread> th;
  for (int t = 0; t < threads; ++t)
    th.emplace_back([&, t] {
      threadIdx.x = t;
      emu_my_wave = waves[t / 64].get();
      body(t);
      emu_my_wave->bar.arrive_and_drop();
      emu_block_bar->arrive_and_drop();
    });
  for (auto& x : th) x.join();
}
