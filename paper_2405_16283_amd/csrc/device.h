// Device-side helpers shared by the kernel files: storage types and conversions, addressing of tile
// grids, and the matrix-core wrappers for fp32.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tn {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef unsigned short bf16_t;  // storage of a bf16 value

// Tiles lie in global memory; said so, their loads are not counted among the LDS and scalar ones.
#define TN_GLOBAL __attribute__((address_space(1)))

__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }
// round to nearest, ties to even: the hardware conversion of gfx950 (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
// two values at once, the first in the low half
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}
template <typename T> __device__ __forceinline__ float ld(const T* p);
template <> __device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p) { return bf2f(*p); }
// four neighbouring elements (p aligned to four of them)
__device__ __forceinline__ f32x4 ld4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 ld4(const bf16_t* p) {
  const uint2 u = *(const uint2*)p;
  return (f32x4){__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                 __uint_as_float(u.y & 0xFFFF0000u)};
}
template <typename T> __device__ __forceinline__ void st(T* p, float v);
template <> __device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st<bf16_t>(bf16_t* p, float v) { *p = f2bf(v); }
__device__ __forceinline__ void st4(float* p, f32x4 v) { *(f32x4*)p = v; }
__device__ __forceinline__ void st4(bf16_t* p, f32x4 v) { *(uint2*)p = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3])); }

// fp32 product on the matrix cores, D[16,16] += A[16,4] B[4,16]: lane (n = lane & 15, g = lane >> 4) gives
// A[n][g] and B[g][n] and holds D[4g + i][n] in element i.  256 flop per clock and compute unit, twice what
// unpacked vector FMAs reach, with the same fp32 products and sums.
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <typename T>
__device__ __forceinline__ const T* tile_elem(void* const* tiles, int nc, int t_rows, int t_cols, int row, int col) {
  const int rt = row / t_rows, ct = col / t_cols;
  return (const T*)tiles[rt * nc + ct] + (size_t)(row - rt * t_rows) * t_cols + (col - ct * t_cols);
}

// The same for a grid of transposed tiles: tile (rt, ct) holds [its columns, its rows]; the last
// row tile may be shorter, which changes its pitch.
template <typename T>
__device__ __forceinline__ const T* tile_elem_t(void* const* tiles, int nc, int t_rows, int t_cols, int total_rows,
                                                int row, int col) {
  const int rt = row / t_rows, ct = col / t_cols;
  const int pitch = min(t_rows, total_rows - rt * t_rows);
  return (const T*)tiles[rt * nc + ct] + (size_t)(col - ct * t_cols) * pitch + (row - rt * t_rows);
}

// 16 bytes per lane from global memory straight into LDS at lds_addr + imm + 16 * lane.  In assembly, so that the compiler does
// not wait for them: kernels keep several in flight across barriers and count them themselves.  (M0 has to be written one
// instruction ahead of the load that uses it.)
typedef __attribute__((address_space(3))) void* lptr_t;
typedef __attribute__((ext_vector_type(4))) uint32_t rsrc_t;
// from a 32-bit byte offset per lane and a uniform one
__device__ __forceinline__ void load_lds(uint32_t voff, rsrc_t r, uint32_t soff, uint32_t lds_addr, int imm) {
  asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               ::"v"(voff), "s"(r), "s"(soff), "s"(lds_addr), "n"(imm) : "memory", "scc");
}
__device__ __forceinline__ void load_lds(uint64_t addr, uint32_t lds_addr, int imm) {
  asm volatile("s_add_u32 m0, %1, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds_addr), "n"(imm) : "memory", "scc");
}
__device__ __forceinline__ void load_lds(const void* addr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds_addr) : "memory");
}
// Reads of the (read-only, wavefront-uniform) operand tables through the scalar unit, so that
// they are counted by lgkmcnt and never force a wait on the vector loads in flight.
__device__ __forceinline__ const void* sload_ptr(const void* const* addr) {
  const void* v;
  asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(addr) : "memory");
  return v;
}
__device__ __forceinline__ int sload_int(const int* addr) {
  int v;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(addr) : "memory");
  return v;
}

// Workgroups are handed to the 8 XCDs round-robin in launch order, and each XCD has its own L2.
// This turns the launch position into a position in which each XCD gets a contiguous run of
// (vertex, tile) pairs, so that the workgroups sharing an L2 work on neighbouring tiles -- the
// tiles of one vertex and of vertices with the same A row block -- instead of every XCD
// streaming every operand.
__device__ __forceinline__ void xcd_remap(int& bx, int& by) {
  const int gx = gridDim.x, total = gx * gridDim.y;
  const int n = blockIdx.x + gx * blockIdx.y;
  const int xcd = n & 7, slot = n >> 3;
  const int q = total >> 3, r = total & 7;
  const int v = xcd * q + min(xcd, r) + slot;
  by = v / gx;
  bx = v - by * gx;
}

}  // namespace
}  // namespace tn
