// Shared definitions of the gfx950 spectrum-slicing library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <mutex>
#include <stdexcept>
#include <string>

#include "sislice.h"

namespace sislice {

// Errors inside the library are C++ exceptions carrying a status; every C entry
// point catches them and returns the status.
struct Error : std::runtime_error {
  sislice_status status;
  Error(sislice_status s, const std::string& what) : std::runtime_error(what), status(s) {}
};

#define SL_HIP(call)                                                                      \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess)                                                                 \
      throw ::sislice::Error(SISLICE_ERR_HIP, std::string(#call) + ": " +                 \
                                                  hipGetErrorString(e_));                 \
  } while (0)

#define SL_CHECK_ARG(cond, msg)                                                           \
  do {                                                                                    \
    if (!(cond)) throw ::sislice::Error(SISLICE_ERR_ARG, msg);                            \
  } while (0)

#define SL_LAUNCH_CHECK() SL_HIP(hipGetLastError())

typedef double d4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4_f64 on gfx950, one wavefront: D(16x16) += A(16x4) * B(4x16).
// Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator element r
// of lane l is D[l / 16 + 4 r][l % 16] (rows interleaved by 4; measured on the
// device with random operands).
__device__ __forceinline__ d4 mfma16x16x4(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// p, known to be in global memory.  The compiler takes a pointer read from a table in memory
// to be generic, and a generic (flat) access counts as an access to LDS as well: every wait
// for LDS then waits for all such loads and stores, so none can be in flight across a
// barrier or an exchange through LDS.  p is the same in every lane.
template <typename T>
__device__ __forceinline__ T* global_ptr(T* p) {
  const auto u = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return (T*)(__attribute__((address_space(1))) T*)((unsigned long long)hi << 32 | lo);
}

// Bunch-Kaufman pivot threshold alpha = (1 + sqrt(17)) / 8 (Bunch & Kaufman 1977).
constexpr double kBkAlpha = 0.6403882032022076;

// Per-shift factorization state kept in device memory, so that a fixed sequence
// of launches can advance panels whose width depends on the pivots chosen.
struct FactorState {
  int32_t k0;        // first column of the panel factored last
  int32_t kb;        // columns factored by that panel
  int32_t done;      // 1 once every column is factored
  int32_t npanel;    // panels factored so far
  int64_t neg, zero, pos;  // inertia of D accumulated over the pivots
  int32_t jstart;    // columns of the current panel accepted by the pivot-free path
  int32_t whole;     // panels accepted whole by it so far
  // Whole panels' updates may wait for later panels (their columns so far, else 0): the next
  // panel's columns have them, the columns after it do not.  Their W stays in columns
  // 0 .. pend - 1 of the workspace; the next panel's goes behind it.
  int32_t pend;
  // the update after the panel: columns u_c0 .. u_c1 - 1 by the u_kb columns of L from
  // u_k0 and of W from u_w0 of the workspace
  int32_t u_k0, u_kb, u_w0, u_c0, u_c1;
};

// Largest panel width the factorization kernels are built for.
constexpr int kMaxNb = 64;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace sislice
