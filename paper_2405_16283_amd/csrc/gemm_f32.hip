// Tile products with fp32 products on the matrix cores (MFMA 16x16x4): fp32 graphs, and the bf16 products
// whose layout or shape the bf16 kernels do not take (A stored transposed, B stored [K, N], tiles whose K is no
// multiple of 8).  Any shape and any of the layouts of the GEMM vertex are served.
//
// One workgroup = 32x32 elements of the output; its four wavefronts form the same 32x32 each over a quarter of
// K (32-deep pieces of the K tiles, dealt out in turn) and add up through LDS.  Operands go from memory straight
// into the registers that feed the MFMAs: lane (n = lane & 15, g = lane >> 4) reads four neighbours along K of row
// n, elements 4g .. 4g + 3 of a 16-deep slab, and MFMA c of the slab takes element c of every lane, so K is summed
// in a permuted but fixed order.  No LDS and no barrier on the way, three pieces in flight per wavefront.
//
// Why: tile products of fp32 graphs are many and small (64x64 to 256x256 with K of 64 to 2752), and a launch
// seldom holds more than a few, so what bounds them is the wait for memory along a serial K loop and the number of
// workgroups, not the L1 traffic of a small tile (8 flop per byte; L1 delivers enough for the 256 flop per clock
// and CU of the fp32 MFMA).  Against 64x64 tiles staged through LDS for vector FMAs, per launch: 64x64 tiles with K
// of 256 and 688, 40 -> 7 us; 256x256 tiles with K of 1024 and 2752, two or three of them to a launch, 172 -> 20 us.
#include "device.h"
#include "kernels.h"

namespace tn {
namespace {

constexpr int kTile = kGemmF32Tile;  // 32: output rows and columns of a workgroup
constexpr int kDeep = 32;            // elements along K of a piece
constexpr int kWaves = 4;
constexpr int kPitch = kTile + 4;    // floats per row of a partial in LDS
static_assert(kTile == 32, "two 16-row MFMA tiles per side");

typedef f32x4 Frag[2][2];  // [16-deep slab][16-row tile]

// Tiles lie in global memory; said so, their loads are not counted among the LDS and scalar ones.
#define TN_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ f32x4 ldg4(const TN_GLOBAL float* p) { return *(const TN_GLOBAL f32x4*)p; }
__device__ __forceinline__ f32x4 ldg4(const TN_GLOBAL bf16_t* p) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 u = *(const TN_GLOBAL u32x2*)p;
  return (f32x4){__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u), __uint_as_float(u[1] << 16),
                 __uint_as_float(u[1] & 0xFFFF0000u)};
}
__device__ __forceinline__ float ldg(const TN_GLOBAL float* p) { return *p; }
__device__ __forceinline__ float ldg(const TN_GLOBAL bf16_t* p) { return bf2f(*p); }

// What a workgroup multiplies: image[X, Y] = sum over k of x_k[., K_k] y_k[., K_k]^T.  The image is C, or its
// transpose (the sides exchanged) where C is stored transposed.
struct Sides {
  void* const* px;
  void* const* py;
  const int* ks;
  int nk, X, Y, x0, y0, w, n, g;
};

// One side of the product in the K tile at hand.  KC: tiles are stored [rows, K], else [K, rows].
template <typename T, bool KC>
struct Side {
  const TN_GLOBAL T* p;
  int rows, K, r[2], g;
  uint32_t off[2];  // bytes from a piece's first element along K to this lane's, for both 16-row tiles (a tile is below 4 GiB)
  __device__ __forceinline__ Side(int rows_, int r0, int n, int g_) : p(nullptr), rows(rows_), K(0), g(g_) {
#pragma unroll
    for (int i = 0; i < 2; ++i) r[i] = min(r0 + 16 * i + n, rows - 1);  // rows past the end: any row, they are not stored
  }
  __device__ __forceinline__ void open(const void* tile, int K_) {
    p = (const TN_GLOBAL T*)tile;
    K = K_;
#pragma unroll
    for (int i = 0; i < 2; ++i) off[i] = ((uint32_t)r[i] * (KC ? (uint32_t)K : 1u) + 4u * g * (KC ? 1u : (uint32_t)rows)) * (uint32_t)sizeof(T);
  }
  // a piece all of whose elements exist along K
  __device__ __forceinline__ void load(int k0, Frag& f) const {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if constexpr (KC) {
          f[j][i] = ldg4((const TN_GLOBAL T*)((const TN_GLOBAL char*)(p + k0 + 16 * j) + off[i]));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            f[j][i][e] = ldg((const TN_GLOBAL T*)((const TN_GLOBAL char*)(p + (size_t)(k0 + 16 * j + e) * rows) + off[i]));
        }
      }
  }
  // the last piece of a K tile, and rows that are not aligned to four elements
  __device__ __forceinline__ void load_ragged(int k0, Frag& f) const {
    if (KC && (K & 3) == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f[j][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
          if (k0 + 16 * j + 4 * g < K) f[j][i] = ldg4((const TN_GLOBAL T*)((const TN_GLOBAL char*)(p + k0 + 16 * j) + off[i]));
        }
      return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = k0 + 16 * j + 4 * g + e;
          f[j][i][e] = k < K ? ldg(KC ? p + (size_t)r[i] * K + k : p + (size_t)k * rows + r[i]) : 0.f;
        }
  }
};

// lane (n, g) of the result holds rows 16 i + n and columns 16 j + 4 g .. + 3 of the image
__device__ __forceinline__ void multiply(const Frag& x, const Frag& y, f32x4 (&acc)[2][2]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(y[s][j][c], x[s][i][c], acc[i][j]);
}

template <typename T, bool XK, bool YK>
__device__ __forceinline__ void product(const Sides& s, f32x4 (&acc)[2][2]) {
  // whole pieces of a K tile; none where rows stored along K are not aligned to four elements
  auto pieces = [](int K) { return ((XK || YK) && (K & 3)) ? 0 : K / kDeep; };
  Side<T, XK> x(s.X, s.x0, s.n, s.g);
  Side<T, YK> y(s.Y, s.y0, s.n, s.g);
  int total = 0;
  for (int q = 0; q < s.nk; ++q) total += pieces(s.ks[q]);
  const int mine = (total - s.w + kWaves - 1) / kWaves;  // this wavefront's pieces: w, w + 4, ...
  int kt = -1, left = 0, at = s.w;  // `at`: the next one, counted from the first of the `left` pieces of K tile kt
  Frag fx[3], fy[3];
  auto fetch = [&](int b) {
    if (at >= left) {
      int K = 0;
      do {
        at -= left;
        K = s.ks[++kt];
        left = pieces(K);
      } while (at >= left);
      x.open(s.px[kt], K);
      y.open(s.py[kt], K);
    }
    x.load(at * kDeep, fx[b]);
    y.load(at * kDeep, fy[b]);
    at += kWaves;
  };
  if (mine >= 3) {  // three pieces in flight
    fetch(0);
    fetch(1);
    fetch(2);
    int left_over = mine;
    for (; left_over >= 6; left_over -= 3) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        multiply(fx[b], fy[b], acc);
        fetch(b);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    multiply(fx[0], fy[0], acc);
    if (left_over > 3) fetch(0);
    multiply(fx[1], fy[1], acc);
    if (left_over > 4) fetch(1);
    multiply(fx[2], fy[2], acc);
    if (left_over > 3) multiply(fx[0], fy[0], acc);
    if (left_over > 4) multiply(fx[1], fy[1], acc);
  } else if (mine > 0) {
    fetch(0);
    if (mine > 1) fetch(1);
    multiply(fx[0], fy[0], acc);
    if (mine > 1) multiply(fx[1], fy[1], acc);
  }
  // what the whole pieces leave of each K tile
  for (int q = 0, turn = 0; q < s.nk; ++q) {
    const int K = s.ks[q];
    for (int k0 = pieces(K) * kDeep; k0 < K; k0 += kDeep, ++turn) {
      if (turn % kWaves != s.w) continue;
      x.open(s.px[q], K);
      y.open(s.py[q], K);
      x.load_ragged(k0, fx[0]);
      y.load_ragged(k0, fy[0]);
      multiply(fx[0], fy[0], acc);
    }
  }
}

// The four partials of the workgroup added up: thread t receives columns 4 (t % 8) .. + 3 of row t / 8.
__device__ __forceinline__ f32x4 add_up(const f32x4 (&acc)[2][2], float (*part)[kTile][kPitch], int w, int n, int g) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) *(f32x4*)&part[w][16 * i + n][16 * j + 4 * g] = acc[i][j];
  __syncthreads();
  const int r = threadIdx.x >> 3, c = (threadIdx.x & 7) * 4;
  const f32x4 v = (*(const f32x4*)&part[0][r][c] + *(const f32x4*)&part[1][r][c]) +
                  (*(const f32x4*)&part[2][r][c] + *(const f32x4*)&part[3][r][c]);
  __syncthreads();
  return v;
}

template <typename T>
__global__ void __launch_bounds__(64 * kWaves, sizeof(T) == 4 ? 3 : 2) gemm_f32_kernel(DeviceTables t, Batch b) {
  __shared__ __attribute__((aligned(16))) float part[kWaves][kTile][kPitch];
  int bx, by;
  xcd_remap(bx, by);
  const OpDesc& d = t.descs[b.at(by)];
  if (bx >= d.nblocks) return;
  const int nk = d.p.nk, lane = threadIdx.x & 63;
  const bool tc = d.p.trans_c != 0;
  void* const* const A = t.ptrs + d.ptr0;
  Sides s;
  s.ks = t.aux + d.aux0;
  s.nk = nk;
  s.X = tc ? d.cols : d.rows;
  s.Y = tc ? d.rows : d.cols;
  const bool a_k = d.p.trans_a == 0, b_k = d.trans_b != 0;
  const bool xk = tc ? b_k : a_k, yk = tc ? a_k : b_k;
  const int across = (s.Y + kTile - 1) / kTile;
  s.x0 = bx / across * kTile;
  s.y0 = bx % across * kTile;
  s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  s.n = lane & 15;
  s.g = lane >> 4;
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, gate = v;
  const int passes = d.p.mode == 2 ? 2 : 1;  // mode 2: the gate product, then the up product
  for (int pass = 0; pass < passes; ++pass) {
    void* const* const Bt = A + (1 + pass) * nk;
    s.px = tc ? Bt : A;
    s.py = tc ? A : Bt;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (xk && yk) product<T, true, true>(s, acc);
    else if (xk) product<T, true, false>(s, acc);
    else if (yk) product<T, false, true>(s, acc);
    else product<T, false, false>(s, acc);
    gate = v;
    v = add_up(acc, part, s.w, s.n, s.g);
  }
  const int row = s.x0 + (threadIdx.x >> 3), col = s.y0 + (threadIdx.x & 7) * 4;
  if (row >= s.X || col >= s.Y) return;
  if (d.p.mode == 2) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gate[e] / (1.f + __expf(-gate[e])) * v[e];
  }
  const size_t at = (size_t)row * s.Y + col;
  const T* const R = d.p.mode == 1 ? (const T*)A[2 * nk] + at : nullptr;  // the residual operand
  T* const out = (T*)d.out + at;
  if ((s.Y & 3) == 0) {
    if (R) v += ld4(R);
    st4(out, v);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < s.Y) st(out + e, R ? v[e] + ld(R + e) : v[e]);
  }
}

}  // namespace

hipError_t launch_gemm_f32(int dtype, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t s) {
  const dim3 grid((unsigned)max_blocks, (unsigned)b.n), wg(64 * kWaves);
  if (dtype == TN_BF16) hipLaunchKernelGGL(gemm_f32_kernel<bf16_t>, grid, wg, 0, s, t, b);
  else hipLaunchKernelGGL(gemm_f32_kernel<float>, grid, wg, 0, s, t, b);
  return hipGetLastError();
}

}  // namespace tn
