// What csrc/lookahead.hpp needs of HIP, on the host: the threads of a launch are fibers that a test
// schedules one at a time, so that an order which is rare on the GPU can be chosen.
#pragma once

#include <cstddef>
#include <cstdint>

#define __device__
#define __host__
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct dim { uint32_t x; };
extern dim threadIdx, blockIdx, blockDim, gridDim;
template <typename T> inline T min(T a, T b) { return b < a ? b : a; }
void __syncthreads();                            // the fiber waits for the other fibers of its block
int __shfl_up(int value, int delta, int width);
uint32_t atomicAdd(uint32_t* at, uint32_t value);
