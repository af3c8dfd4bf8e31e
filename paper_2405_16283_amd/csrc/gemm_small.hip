// Tile products that are small, thin or fp32.
//
// gemm_small_kernel with fp32 products (MFMA 16x16x4): fp32 graphs, and the bf16 products whose layout the bf16
// kernels do not take (A stored transposed, B stored [K, N], tiles whose K is no multiple of 8); any shape and any
// layout of the GEMM vertex.  With bf16 products (MFMA 16x16x32): bf16 products of which a 128x128 workgroup would
// be mostly empty.  gemm_rows_kernel: single rows, those of many vertices at once.
//
// One workgroup = 32x32 elements of the output; its four wavefronts form the same 32x32 each over a quarter of
// K (pieces of 128 bytes per row, dealt out in turn) and add up through LDS.  Operands go from memory straight
// into the registers that feed the MFMAs: lane (n = lane & 15, g = lane >> 4) reads 16 bytes along K of row n, and
// K is summed in a permuted but fixed order.  No LDS and no barrier on the way, three pieces in flight per wavefront.
//
// Why: these products are many and small (fp32 graphs: 64x64 to 256x256 with K of 64 to 2752; decode steps: one row;
// adapters: 16 rows or columns), and a launch seldom holds more than a few, so what bounds them is the wait for
// memory along a serial K loop and the number of workgroups, not the L1 traffic of a small tile.  (With many
// workgroups L1 is the bound: 53-65 TFLOP/s in fp32, of 157, and 150 in bf16.)  Per launch, before -> after:
// fp32, 64x64 tiles staged through LDS for vector FMAs: 64x64 with K of 256 and 688, 40 -> 7 us; 256x256 with K of 1024
// and 2752, two or three to a launch, 172 -> 20 us.  bf16, 128x128 tiles: 32 products of 512x16, K 4096, 59 -> 28 us;
// 8 of 16x512, K 16384, 223 -> 53 us; 32 single rows against 24 tiles of 512, K 4096, 486 -> 47 us.
#include "device.h"
#include "kernels.h"

namespace tn {
namespace {

constexpr int kTile = kGemmSmallTile;  // 32: output rows and columns of a workgroup
constexpr int kWaves = 4;
constexpr int kPitch = kTile + 4;  // floats per row of a partial in LDS
static_assert(kTile == 32, "two 16-row MFMA tiles per side");

__device__ __forceinline__ f32x4 ldg4(const TN_GLOBAL float* p) { return *(const TN_GLOBAL f32x4*)p; }
__device__ __forceinline__ f32x4 ldg4(const TN_GLOBAL bf16_t* p) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 u = *(const TN_GLOBAL u32x2*)p;
  return (f32x4){__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u), __uint_as_float(u[1] << 16),
                 __uint_as_float(u[1] & 0xFFFF0000u)};
}
__device__ __forceinline__ float ldg(const TN_GLOBAL float* p) { return *p; }
__device__ __forceinline__ float ldg(const TN_GLOBAL bf16_t* p) { return bf2f(*p); }

// The two kinds of products.  A piece is what a wavefront takes at once along K: two slabs, of which a lane
// (n = lane & 15, g = lane >> 4) holds W neighbours, elements W g .. W g + W - 1, of row n.
// lane (n, g) of the result holds rows 16 i + n and columns 16 j + 4 g .. + 3 of the image.
template <typename T>
struct Fp32Products {  // element c of every lane goes to MFMA c of a slab
  static constexpr int W = 4;
  typedef f32x4 Vec;
  static __device__ __forceinline__ Vec wide(const TN_GLOBAL T* p) { return ldg4(p); }
  static __device__ __forceinline__ Vec zero() { return (f32x4){0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ void multiply(const Vec (&x)[2][2], const Vec (&y)[2][2], f32x4 (&acc)[2][2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f32(y[s][j][c], x[s][i][c], acc[i][j]);
  }
};
struct Bf16Products {
  static constexpr int W = 8;
  typedef bf16x8 Vec;
  static __device__ __forceinline__ Vec wide(const TN_GLOBAL bf16_t* p) { return *(const TN_GLOBAL bf16x8*)p; }
  static __device__ __forceinline__ Vec zero() { return __builtin_bit_cast(bf16x8, (f32x4){0.f, 0.f, 0.f, 0.f}); }
  static __device__ __forceinline__ void multiply(const Vec (&x)[2][2], const Vec (&y)[2][2], f32x4 (&acc)[2][2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[s][j], x[s][i], acc[i][j], 0, 0, 0);
  }
};

// What a workgroup multiplies: image[X, Y] = sum over k of x_k[., K_k] y_k[., K_k]^T.  The image is C, or its
// transpose (the sides exchanged) where C is stored transposed.
struct Sides {
  void* const* px;
  void* const* py;
  const int* ks;
  int nk, X, Y, x0, y0, w, n, g;
};

// One side of the product in the K tile at hand.  KC: tiles are stored [rows, K], else [K, rows] (fp32 products only).
template <typename T, typename P, bool KC>
struct Side {
  static constexpr int W = P::W;
  typedef typename P::Vec Vec;
  void* const* tiles;
  const TN_GLOBAL T* p = nullptr;  // the workgroup's first row of the tile
  int rows, r0, K = 0, r[2], g;    // r: rows from there
  uint32_t off[2];  // bytes from a piece's first element along K in the first row to this lane's, for both 16-row tiles
  __device__ __forceinline__ Side(void* const* tiles_, int rows_, int r0_, int n, int g_) : tiles(tiles_), rows(rows_), r0(r0_), g(g_) {
#pragma unroll
    for (int i = 0; i < 2; ++i) r[i] = min(16 * i + n, rows - 1 - r0);  // rows past the end: any row, they are not stored
  }
  // Whether `off` holds the way from the workgroup's first row to its last (a tile of any size is fine as long as 32 of its
  // rows, or what a lane skips along K of [K, rows], stay below 4 GiB).
  __device__ __forceinline__ bool reaches(int K_) const {
    const uint64_t elems = KC ? (uint64_t)kTile * (uint32_t)K_ : (uint64_t)(4 * W) * (uint32_t)rows;
    return elems * sizeof(T) <= 0xFFFFFFFFull;
  }
  __device__ __forceinline__ void open(int kt, int K_, int) {
    K = K_;
    p = (const TN_GLOBAL T*)tiles[kt] + (KC ? (size_t)r0 * K : (size_t)r0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      off[i] = ((uint32_t)r[i] * (KC ? (uint32_t)K : 1u) + (uint32_t)(W * g) * (KC ? 1u : (uint32_t)rows)) * (uint32_t)sizeof(T);
  }
  __device__ __forceinline__ const TN_GLOBAL T* at(const TN_GLOBAL T* base, int i) const {
    return (const TN_GLOBAL T*)((const TN_GLOBAL char*)base + off[i]);
  }
  // a piece all of whose elements exist along K
  __device__ __forceinline__ void load(int k0, Vec (&f)[2][2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if constexpr (KC) {
          f[j][i] = P::wide(at(p + k0 + 4 * W * j, i));
        } else {
#pragma unroll
          for (int e = 0; e < W; ++e) f[j][i][e] = ldg(at(p + (size_t)(k0 + 4 * W * j + e) * rows, i));
        }
      }
  }
  // the last piece of a K tile, and rows that are not aligned to a whole vector or too long for `off`
  __device__ __forceinline__ void load_ragged(int k0, Vec (&f)[2][2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = k0 + 4 * W * j + W * g;
        f[j][i] = P::zero();
        if (KC && K % W == 0) {
          if (k < K) f[j][i] = P::wide(p + (size_t)r[i] * K + k);
        } else if constexpr (W == 4) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e < K) f[j][i][e] = ldg(KC ? p + (size_t)r[i] * K + k + e : p + (size_t)(k + e) * rows + r[i]);
        }
      }
  }
};

template <typename P, typename SX, typename SY>
__device__ __forceinline__ void product(const Sides& s, SX x, SY y, bool vectors, f32x4 (&acc)[2][2]) {
  constexpr int DEEP = 8 * P::W;  // elements along K of a piece
  // whole pieces of a K tile; none where rows stored along K are not aligned to a vector or the tile is too wide
  auto pieces = [&](int K) { return (vectors && K % P::W) || !x.reaches(K) || !y.reaches(K) ? 0 : K / DEEP; };
  int total = 0;
  for (int q = 0; q < s.nk; ++q) total += pieces(s.ks[q]);
  const int mine = (total - s.w + kWaves - 1) / kWaves;  // this wavefront's pieces: w, w + 4, ...
  int kt = -1, left = 0, at = s.w;  // `at`: the next one, counted from the first of the `left` pieces of K tile kt
  typename P::Vec fx[3][2][2], fy[3][2][2];
  auto fetch = [&](int b) {
    if (at >= left) {
      int K = 0;
      do {
        at -= left;
        K = s.ks[++kt];
        left = pieces(K);
      } while (at >= left);
      x.open(kt, K, s.nk);
      y.open(kt, K, s.nk);
    }
    x.load(at * DEEP, fx[b]);
    y.load(at * DEEP, fy[b]);
    at += kWaves;
  };
  auto multiply = [&](int b) { P::multiply(fx[b], fy[b], acc); };
  if (mine >= 3) {  // three pieces in flight
    fetch(0);
    fetch(1);
    fetch(2);
    int left_over = mine;
    for (; left_over >= 6; left_over -= 3) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        multiply(b);
        fetch(b);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    multiply(0);
    if (left_over > 3) fetch(0);
    multiply(1);
    if (left_over > 4) fetch(1);
    multiply(2);
    if (left_over > 3) multiply(0);
    if (left_over > 4) multiply(1);
  } else if (mine > 0) {
    fetch(0);
    if (mine > 1) fetch(1);
    multiply(0);
    if (mine > 1) multiply(1);
  }
  // what the whole pieces leave of each K tile
  for (int q = 0, turn = 0; q < s.nk; ++q) {
    const int K = s.ks[q];
    for (int k0 = pieces(K) * DEEP; k0 < K; k0 += DEEP, ++turn) {
      if (turn % kWaves != s.w) continue;
      x.open(q, K, s.nk);
      y.open(q, K, s.nk);
      x.load_ragged(k0, fx[0]);
      y.load_ragged(k0, fy[0]);
      multiply(0);
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

// B16: bf16 products (both sides stored along K, every K a multiple of 8), else fp32 products
template <typename T, bool B16>
__global__ void __launch_bounds__(64 * kWaves, sizeof(T) == 4 || B16 ? 3 : 2) gemm_small_kernel(DeviceTables t, Batch b) {
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
    if constexpr (B16) {
      typedef Side<T, Bf16Products, true> K;
      product<Bf16Products>(s, K(s.px, s.X, s.x0, s.n, s.g), K(s.py, s.Y, s.y0, s.n, s.g), true, acc);
    } else {
      typedef Fp32Products<T> P;
      typedef Side<T, P, true> K;
      typedef Side<T, P, false> R;
      if (xk && yk) product<P>(s, K(s.px, s.X, s.x0, s.n, s.g), K(s.py, s.Y, s.y0, s.n, s.g), true, acc);
      else if (xk) product<P>(s, K(s.px, s.X, s.x0, s.n, s.g), R(s.py, s.Y, s.y0, s.n, s.g), true, acc);
      else if (yk) product<P>(s, R(s.px, s.X, s.x0, s.n, s.g), K(s.py, s.Y, s.y0, s.n, s.g), true, acc);
      else product<P>(s, R(s.px, s.X, s.x0, s.n, s.g), R(s.py, s.Y, s.y0, s.n, s.g), false, acc);
    }
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

// Single rows of different vertices against the same B tiles (decode steps): the rows of a group of vertices are the
// 32 rows of one image, so that B comes from memory once for all of them.
// The batch: n groups; idx[0 .. n] where each group starts, then the vertices' descriptor indices.
template <typename T, typename P>
struct RowsSide {  // row r of the image: the A tiles of vertex r of the group
  static constexpr int W = P::W;
  typedef typename P::Vec Vec;
  typedef const TN_GLOBAL T* Ptr;
  typedef const TN_GLOBAL uint64_t* Table;  // operand addresses
  Table tiles[2];
  Ptr p[2], next[2];  // this K tile's, and the following one's fetched ahead
  int kt = -2, K = 0, g;
  __device__ __forceinline__ RowsSide(const DeviceTables& t, const Batch& b, int first, int count, int n, int g_) : g(g_) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const OpDesc& d = t.descs[b.base + b.idx[b.n + 1 + first + min(16 * i + n, count - 1)]];
      tiles[i] = (Table)(t.ptrs + d.ptr0);
    }
  }
  __device__ __forceinline__ bool reaches(int) const { return true; }
  __device__ __forceinline__ void open(int kt_, int K_, int nk) {
    if (kt_ == kt + 1) {
      p[0] = next[0];
      p[1] = next[1];
    } else {
      p[0] = (Ptr)tiles[0][kt_];
      p[1] = (Ptr)tiles[1][kt_];
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0) here, so that the other branch has nothing to wait for
    }
    next[0] = (Ptr)tiles[0][min(kt_ + 1, nk - 1)];
    next[1] = (Ptr)tiles[1][min(kt_ + 1, nk - 1)];
    kt = kt_;
    K = K_;
  }
  __device__ __forceinline__ void load(int k0, Vec (&f)[2][2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) f[j][i] = P::wide(p[i] + k0 + 4 * W * j + W * g);
  }
  __device__ __forceinline__ void load_ragged(int k0, Vec (&f)[2][2]) const {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f[j][i] = P::zero();
        if (k0 + 4 * W * j + W * g < K) f[j][i] = P::wide(p[i] + k0 + 4 * W * j + W * g);
      }
  }
};

template <typename T, typename P>
__global__ void __launch_bounds__(64 * kWaves, 3) gemm_rows_kernel(DeviceTables t, Batch b) {
  __shared__ __attribute__((aligned(16))) float part[kWaves][kTile][kPitch];
  int bx, by;
  xcd_remap(bx, by);
  const int first = b.idx[by], count = b.idx[by + 1] - first;
  const OpDesc& d = t.descs[b.base + b.idx[b.n + 1 + first]];  // what the group has in common
  if (bx >= d.nblocks) return;
  const int nk = d.p.nk, lane = threadIdx.x & 63;
  Sides s;
  s.ks = t.aux + d.aux0;
  s.nk = nk;
  s.X = count;
  s.Y = d.cols;
  s.x0 = 0;
  s.y0 = bx * kTile;
  s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  s.n = lane & 15;
  s.g = lane >> 4;
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, gate = v;
  const int passes = d.p.mode == 2 ? 2 : 1;
  for (int pass = 0; pass < passes; ++pass) {
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    product<P>(s, RowsSide<T, P>(t, b, first, count, s.n, s.g),
               Side<T, P, true>(t.ptrs + d.ptr0 + (1 + pass) * nk, s.Y, s.y0, s.n, s.g), true, acc);
    gate = v;
    v = add_up(acc, part, s.w, s.n, s.g);
  }
  const int row = threadIdx.x >> 3, col = s.y0 + (threadIdx.x & 7) * 4;
  if (row >= count || col >= s.Y) return;
  if (d.p.mode == 2) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gate[e] / (1.f + __expf(-gate[e])) * v[e];
  }
  const OpDesc& own = t.descs[b.base + b.idx[b.n + 1 + first + row]];
  const T* const R = d.p.mode == 1 ? (const T*)t.ptrs[own.ptr0 + 2 * nk] + col : nullptr;  // the residual operand
  T* const out = (T*)own.out + col;
  if (col + 3 < s.Y) {
    if (R) v += ld4(R);
    st4(out, v);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < s.Y) st(out + e, R ? v[e] + ld(R + e) : v[e]);
  }
}

}  // namespace

hipError_t launch_gemm_small(bool bf16_products, int dtype, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t s) {
  const dim3 grid((unsigned)max_blocks, (unsigned)b.n), wg(64 * kWaves);
  if (bf16_products) hipLaunchKernelGGL((gemm_small_kernel<bf16_t, true>), grid, wg, 0, s, t, b);
  else if (dtype == TN_BF16) hipLaunchKernelGGL((gemm_small_kernel<bf16_t, false>), grid, wg, 0, s, t, b);
  else hipLaunchKernelGGL((gemm_small_kernel<float, false>), grid, wg, 0, s, t, b);
  return hipGetLastError();
}

hipError_t launch_gemm_rows(int dtype, const DeviceTables& t, uint32_t base, const RowVertex* rows, int n, int32_t max_blocks,
                            hipStream_t s) {
  Batch b;
  b.base = base;
  for (int at = 0; at < n;) {
    // as many groups of up to kTile vertices with one key as the list holds: a start per group, the last one's
    // end, and the vertices
    uint16_t start[kMaxBatch + 1];
    int groups = 0, taken = 0;
    start[0] = 0;
    while (at + taken < n) {
      int c = 1;
      while (c < kTile && at + taken + c < n && rows[at + taken + c].key == rows[at + taken].key) ++c;
      if (groups + 2 + taken + c > kMaxBatch) break;
      taken += c;
      start[++groups] = (uint16_t)taken;
    }
    b.n = groups;
    for (int k = 0; k <= groups; ++k) b.idx[k] = start[k];
    for (int k = 0; k < taken; ++k) b.idx[groups + 1 + k] = (uint16_t)(rows[at + k].desc - base);
    const dim3 grid((unsigned)max_blocks, (unsigned)groups), wg(64 * kWaves);
    if (dtype == TN_BF16) hipLaunchKernelGGL((gemm_rows_kernel<bf16_t, Bf16Products>), grid, wg, 0, s, t, b);
    else hipLaunchKernelGGL((gemm_rows_kernel<float, Fp32Products<float>>), grid, wg, 0, s, t, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    at += taken;
  }
  return hipSuccess;
}

}  // namespace tn
