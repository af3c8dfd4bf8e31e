// Tile products that are small, thin or fp32.
//
// gemm_small_kernel with fp32 products (MFMA 16x16x4): fp32 graphs, and the bf16 products whose layout the bf16
// kernels do not take (A stored transposed, B stored [K, N], tiles whose K is no multiple of 8); any shape and any
// layout of the GEMM vertex.  With bf16 products (MFMA 16x16x32): bf16 products of which a 128x128 workgroup would
// be mostly empty.  gemm_rows_kernel: single rows, those of many vertices at once.
//
// One workgroup = 32x32 elements of the output; its four wavefronts form the same 32x32 each over a quarter of
// K (pieces of 128 bytes per row, dealt out in turn) and add up through LDS.  K is summed in a permuted but fixed order.
// Where both operands are stored along K, pieces come by `buffer_load ... lds` into a ring of the wavefront's own in LDS (no barrier),
// three of them in flight, eight lanes to a row; fragments are read from there (how much LDS that is: gemm_small_stages).  Other
// layouts, and tiles whose rows are not aligned, go from memory straight into the registers that feed the MFMAs: lane (n = lane & 15, g = lane >> 4) reads 16 bytes
// along K of row n.  That way a load instruction touches 16 rows out of order, and a wavefront spends more time on issuing its
// eight loads per piece than on its 32 MFMAs.
//
// Why: these products are many and small (fp32 graphs: 64x64 to 256x256 with K of 64 to 2752; decode steps: one row;
// adapters: 16 rows or columns), and a launch seldom holds more than a few, so what bounds them is one workgroup's walk along K,
// the way to its first operands (about 4 us with launch and end) and the number of workgroups.  Per launch, straight into
// registers -> by way of LDS: 256x256 in fp32 with K of 1024, one to four of them, 11.5 -> 9.7 us, twelve 28.9 -> 26.2 (61 TFLOP/s); with K of
// 2560 22.6 -> 19.1 and 66.4 -> 54.8 (73, of 157); 64x64 with K of 256 5.7 -> 5.4, with 704 in tiles of 64 9.5 -> 9.8 (every piece
// lies in another tile).  bf16: 32 products of 512x16, K 4096, 30 -> 18 us; 8 of 16x512, K 16384, 52 -> 24.
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace tn {
namespace {

constexpr int kTile = kGemmSmallTile;  // 32: output rows and columns of a workgroup
constexpr int kWaves = kGemmSmallWaves, kStages = kGemmSmallStages, kTableTiles = kGemmRowsTable;
// F: fragments of 16 rows or columns per side of a workgroup's tile; floats per row of a partial in LDS, bytes of a piece and of a ring
constexpr int pitch(int f) { return 16 * f + 4; }
constexpr int piece_bytes(int f) { return 2 * 16 * f * 128; }
constexpr int partials_bytes(int f) { return kWaves * 16 * f * pitch(f) * 4; }
// (the partials take the place of the rings)
constexpr int ring_bytes(int f, int stages) { return std::max(kWaves * stages * piece_bytes(f), partials_bytes(f)); }
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

__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
// The first 64 entries of a table, one per lane.  Read where it is needed, each would be a wait of its own in the walk along K: 64x64
// products with 11 tiles of 64 along K spent more time on these than on their products.
struct LaneTable {
  uint32_t lo, hi;
  __device__ __forceinline__ uint64_t address(void* const* t, int q) const {
    if (q >= 64) return uniform((uint64_t)t[q]);
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, q) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)lo, q);
  }
  __device__ __forceinline__ int size(const int* t, int q) const {
    return q >= 64 ? __builtin_amdgcn_readfirstlane(t[q]) : __builtin_amdgcn_readlane((int)lo, q);
  }
};
__device__ __forceinline__ LaneTable read_addresses(void* const* t, int n) {
  const uint64_t a = (uint64_t)t[min((int)(threadIdx.x & 63), n - 1)];
  return {(uint32_t)a, (uint32_t)(a >> 32)};
}
__device__ __forceinline__ LaneTable read_sizes(const int* t, int n) { return {(uint32_t)t[min((int)(threadIdx.x & 63), n - 1)], 0}; }

// The two kinds of products.  A piece is what a wavefront takes at once along K: two slabs, of which a lane
// (n = lane & 15, g = lane >> 4) holds W neighbours, elements W g .. W g + W - 1, of row n.
// lane (n, g) of the result holds rows 16 i + n and columns 16 j + 4 g .. + 3 of the image.
template <typename T>
struct Fp32Products {  // element c of every lane goes to MFMA c of a slab
  static constexpr int W = 4;
  typedef f32x4 Vec;
  static __device__ __forceinline__ Vec wide(const TN_GLOBAL T* p) { return ldg4(p); }
  static __device__ __forceinline__ Vec zero() { return (f32x4){0.f, 0.f, 0.f, 0.f}; }
  template <int F>
  static __device__ __forceinline__ void multiply(const Vec (&x)[2][F], const Vec (&y)[2][F], f32x4 (&acc)[F][F]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j) acc[i][j] = mfma_f32(y[s][j][c], x[s][i][c], acc[i][j]);
  }
};
struct Bf16Products {
  static constexpr int W = 8;
  typedef bf16x8 Vec;
  static __device__ __forceinline__ Vec wide(const TN_GLOBAL bf16_t* p) { return *(const TN_GLOBAL bf16x8*)p; }
  static __device__ __forceinline__ Vec zero() { return __builtin_bit_cast(bf16x8, (f32x4){0.f, 0.f, 0.f, 0.f}); }
  template <int F>
  static __device__ __forceinline__ void multiply(const Vec (&x)[2][F], const Vec (&y)[2][F], f32x4 (&acc)[F][F]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[s][j], x[s][i], acc[i][j], 0, 0, 0);
  }
};

// What a workgroup multiplies: image[X, Y] = sum over k of x_k[., K_k] y_k[., K_k]^T.  The image is C, or its
// transpose (the sides exchanged) where C is stored transposed.
struct Sides {
  void* const* px;
  void* const* py;
  const int* ks;
  int nk, X, Y, x0, y0, w, n, g, stages;
  LaneTable sizes;
  __device__ __forceinline__ int size(int q) const { return sizes.size(ks, q); }
};

// One side of the product in the K tile at hand.  KC: tiles are stored [rows, K], else [K, rows] (fp32 products only).
template <typename T, typename P, bool KC, int F>
struct Side {
  static constexpr int W = P::W;
  typedef typename P::Vec Vec;
  void* const* tiles;
  const TN_GLOBAL T* p = nullptr;  // the workgroup's first row of the tile
  int rows, r0, K = 0, r[F], g;    // r: rows from there
  uint32_t off[F];  // bytes from a piece's first element along K in the first row to this lane's, for the 16-row tiles
  LaneTable at_lane;  // addresses of the tiles
  __device__ __forceinline__ Side(void* const* tiles_, int nk, int rows_, int r0_, int n, int g_)
      : tiles(tiles_), rows(rows_), r0(r0_), g(g_), at_lane(read_addresses(tiles_, nk)) {
#pragma unroll
    for (int i = 0; i < F; ++i) r[i] = min(16 * i + n, rows - 1 - r0);  // rows past the end: any row, they are not stored
  }
  // Whether `off` holds the way from the workgroup's first row to its last (a tile of any size is fine as long as 32 of its
  // rows, or what a lane skips along K of [K, rows], stay below 4 GiB).
  __device__ __forceinline__ bool reaches(int K_) const {
    const uint64_t elems = KC ? (uint64_t)kTile * (uint32_t)K_ : (uint64_t)(4 * W) * (uint32_t)rows;
    return elems * sizeof(T) <= 0xFFFFFFFFull;
  }
  __device__ __forceinline__ void open(int kt, int K_, int) {
    K = K_;
    p = (const TN_GLOBAL T*)at_lane.address(tiles, kt) + (KC ? (size_t)r0 * K : (size_t)r0);
#pragma unroll
    for (int i = 0; i < F; ++i)
      off[i] = ((uint32_t)r[i] * (KC ? (uint32_t)K : 1u) + (uint32_t)(W * g) * (KC ? 1u : (uint32_t)rows)) * (uint32_t)sizeof(T);
  }
  __device__ __forceinline__ const TN_GLOBAL T* at(const TN_GLOBAL T* base, int i) const {
    return (const TN_GLOBAL T*)((const TN_GLOBAL char*)base + off[i]);
  }
  // a piece all of whose elements exist along K
  __device__ __forceinline__ void load(int k0, Vec (&f)[2][F]) const {
#pragma unroll
    for (int i = 0; i < F; ++i)
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
  // The same by way of LDS (KC only): what `load_staged` issues for the piece `bytes` along K, eight rows to an instruction.
  uint32_t lane_off[2 * F] = {};
  rsrc_t rsrc = {0, 0, 0, 0};
  __device__ __forceinline__ void open_staged(int kt, int K_) {
    const uint64_t a = uniform(at_lane.address(tiles, kt) + (uint64_t)r0 * (uint64_t)K_ * sizeof(T));
    rsrc = (rsrc_t){(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, 0xFFFFFFF0u, 0x00020000u};
    if (K_ == K) return;
    K = K_;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 2 * F; ++i)
      lane_off[i] = (uint32_t)min(8 * i + (lane >> 3), rows - 1 - r0) * (uint32_t)K * (uint32_t)sizeof(T) + (((lane & 7) ^ (lane >> 3)) * 16);
  }
  __device__ __forceinline__ void load_staged(int i, uint32_t bytes, uint32_t lds_addr, int imm) const {
    load_lds(lane_off[i], rsrc, bytes, lds_addr, imm + i * 1024);
  }
  // the last piece of a K tile, and rows that are not aligned to a whole vector or too long for `off`
  __device__ __forceinline__ void load_ragged(int k0, Vec (&f)[2][F]) const {
#pragma unroll
    for (int i = 0; i < F; ++i)
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

template <typename P, bool STAGED, int F, typename SX, typename SY>
__device__ __forceinline__ void product(const Sides& s, SX x, SY y, bool vectors, f32x4 (&acc)[F][F], char* lds) {
  constexpr int kPieceBytes = piece_bytes(F), LOADS = 4 * F;  // (of a stage of the ring; load instructions)
  constexpr int DEEP = 8 * P::W;  // elements along K of a piece
  // whole pieces of a K tile; none where rows stored along K are not aligned to a vector or the tile is too wide
  auto pieces = [&](int K) { return (vectors && K % P::W) || !x.reaches(K) || !y.reaches(K) ? 0 : K / DEEP; };
  int total = 0;
  for (int q = 0; q < s.nk; ++q) total += pieces(s.size(q));
  const int mine = __builtin_amdgcn_readfirstlane((total - s.w + kWaves - 1) / kWaves);  // this wavefront's pieces: w, w + 4, ...
  int kt = -1, left = 0, at = s.w;  // `at`: the next one, counted from the first of the `left` pieces of K tile kt
  // goes on to the K tile that holds piece `at`; true if that is another one
  auto seek = [&](int& K) {
    if (__builtin_amdgcn_readfirstlane(at < left)) return false;
    do {
      at -= left;
      K = s.size(++kt);
      left = pieces(K);
    } while (__builtin_amdgcn_readfirstlane(at >= left));
    return true;
  };
  typename P::Vec fx[STAGED ? 1 : 3][2][F], fy[STAGED ? 1 : 3][2][F];
  auto multiply = [&](int b) __attribute__((always_inline)) { P::template multiply<F>(fx[b], fy[b], acc); };
  if constexpr (STAGED) {
    const uint32_t ring = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lptr_t)lds + s.w * s.stages * kPieceBytes);
    const char* const mem = lds + s.w * s.stages * kPieceBytes;
    uint32_t put = 0, get = 0;  // stages, in bytes
    int issued = 0;
    uint32_t bytes = 0;  // the next piece's place along K
    auto load = [&](int q) __attribute__((always_inline)) {
      if (q < 2 * F) x.load_staged(q, bytes, ring + put, 0);
      else y.load_staged(q - 2 * F, bytes, ring + put, kPieceBytes / 2);
    };
    auto find = [&]() {
      int K = 0;
      if (seek(K)) {
        x.open_staged(kt, K);
        y.open_staged(kt, K);
      }
      bytes = __builtin_amdgcn_readfirstlane(at * 128);
    };
    auto next = [&]() {
      put = put + kPieceBytes == kStages * kPieceBytes ? 0 : put + kPieceBytes;
      at += kWaves;
      ++issued;
    };
    auto load_next = [&]() __attribute__((always_inline)) {
      find();
#pragma unroll
      for (int q = 0; q < LOADS; ++q) load(q);
      next();
    };
#pragma clang loop unroll(disable)
    for (int q = 0; q < kStages - 1 && q < mine; ++q) load_next();
    // One piece: its fragments are read, and behind them the loads of the piece three on are issued, into the stage of the one
    // before.  (Taking these in turn with the MFMAs of the piece before, with two sets of registers, needs several
    // copies of the loop, whose instructions come cold: 256x256 with K of 2560 took 18.8 us against 19.1, 64x64 with K of 704 10.3 against 9.8.)
#pragma clang loop unroll(disable)
    for (int done = 0; done < mine; ++done) {
      const int behind = issued - done - 1;  // pieces behind this one that may be on their way
      if (behind >= 2) __builtin_amdgcn_s_waitcnt(0x0070 | ((2 * LOADS) & 15) | (((2 * LOADS) >> 4) << 14));  // vmcnt(2 LOADS)
      else if (behind == 1) __builtin_amdgcn_s_waitcnt(0x0070 | LOADS);
      else __builtin_amdgcn_s_waitcnt(0x0070);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int q = 0; q < 4 * F; ++q) {  // rows 16 i + n, 16-byte piece 4 j + g
        const int i = (q >> 1) % F, j = q / (2 * F);
        const char* const p = mem + get + (q & 1) * (kPieceBytes / 2) + (16 * i + s.n) * 128 + (((4 * j + s.g) ^ (s.n & 7)) * 16);
        if (q & 1) fy[0][j][i] = *(const typename P::Vec*)p;
        else fx[0][j][i] = *(const typename P::Vec*)p;
      }
      __builtin_amdgcn_sched_barrier(0);
      if (issued < mine) load_next();
      __builtin_amdgcn_sched_barrier(0);
      get = get + kPieceBytes == kStages * kPieceBytes ? 0 : get + kPieceBytes;
      multiply(0);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    auto fetch = [&](int b) {
      int K = 0;
      if (seek(K)) {
        x.open(kt, K, s.nk);
        y.open(kt, K, s.nk);
      }
      x.load(at * DEEP, fx[b]);
      y.load(at * DEEP, fy[b]);
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
  }
  // what the whole pieces leave of each K tile
  for (int q = 0, turn = 0; q < s.nk; ++q) {
    const int K = s.size(q);
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

// The four partials of the workgroup added up: thread t < 64 F F receives columns 4 (t % 4F) .. + 3 of row t / 4F.
template <int F>
__device__ __forceinline__ f32x4 add_up(const f32x4 (&acc)[F][F], char* lds, int w, int n, int g) {
  float (*const part)[16 * F][pitch(F)] = (float (*)[16 * F][pitch(F)])lds;
  __syncthreads();  // the rings are read to the end
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) *(f32x4*)&part[w][16 * i + n][16 * j + 4 * g] = acc[i][j];
  __syncthreads();
  const int t = threadIdx.x & (64 * F * F - 1), r = t / (4 * F), c = t % (4 * F) * 4;
  const f32x4 v = (*(const f32x4*)&part[0][r][c] + *(const f32x4*)&part[1][r][c]) +
                  (*(const f32x4*)&part[2][r][c] + *(const f32x4*)&part[3][r][c]);
  __syncthreads();
  return v;
}

// B16: bf16 products (both sides stored along K, every K a multiple of 8), else fp32 products
template <typename T, bool B16, int F>
__global__ void __launch_bounds__(64 * kWaves) gemm_small_kernel(DeviceTables t, Batch b) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int bx, by;
  xcd_remap(bx, by);
  const OpDesc& d = t.descs[b.at(by)];
  const int nk = __builtin_amdgcn_readfirstlane(d.p.nk), lane = threadIdx.x & 63;
  // (told to be uniform: the compiler does not see it, and staged loads take their descriptors from scalar registers)
  const int rows = __builtin_amdgcn_readfirstlane(d.rows), cols = __builtin_amdgcn_readfirstlane(d.cols), mode = __builtin_amdgcn_readfirstlane(d.p.mode);
  const bool tc = __builtin_amdgcn_readfirstlane(d.p.trans_c) != 0;
  void* const* const A = t.ptrs + __builtin_amdgcn_readfirstlane(d.ptr0);
  Sides s;
  s.ks = t.aux + __builtin_amdgcn_readfirstlane(d.aux0);
  s.nk = nk;
  s.stages = b.stages;
  s.sizes = read_sizes(s.ks, nk);
  s.X = tc ? cols : rows;
  s.Y = tc ? rows : cols;
  const bool a_k = __builtin_amdgcn_readfirstlane(d.p.trans_a) == 0, b_k = __builtin_amdgcn_readfirstlane(d.trans_b) != 0;
  const bool xk = tc ? b_k : a_k, yk = tc ? a_k : b_k;
  constexpr int TILE = 16 * F;
  const int across = (s.Y + TILE - 1) / TILE;
  if (bx >= (s.X + TILE - 1) / TILE * across) return;
  s.x0 = bx / across * TILE;
  s.y0 = bx % across * TILE;
  s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  s.n = lane & 15;
  s.g = lane >> 4;
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, gate = v;
  const int passes = mode == 2 ? 2 : 1;  // mode 2: the gate product, then the up product
  for (int pass = 0; pass < passes; ++pass) {
    void* const* const Bt = A + (1 + pass) * nk;
    s.px = tc ? Bt : A;
    s.py = tc ? A : Bt;
    f32x4 acc[F][F];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if constexpr (B16) {
      typedef Side<T, Bf16Products, true, F> K;
      product<Bf16Products, true, F>(s, K(s.px, nk, s.X, s.x0, s.n, s.g), K(s.py, nk, s.Y, s.y0, s.n, s.g), true, acc, lds);
    } else {
      typedef Fp32Products<T> P;
      typedef Side<T, P, true, F> K;
      typedef Side<T, P, false, F> R;
      if (xk && yk) product<P, sizeof(T) == 4, F>(s, K(s.px, nk, s.X, s.x0, s.n, s.g), K(s.py, nk, s.Y, s.y0, s.n, s.g), true, acc, lds);
      else if (xk) product<P, false, F>(s, K(s.px, nk, s.X, s.x0, s.n, s.g), R(s.py, nk, s.Y, s.y0, s.n, s.g), true, acc, lds);
      else if (yk) product<P, false, F>(s, R(s.px, nk, s.X, s.x0, s.n, s.g), K(s.py, nk, s.Y, s.y0, s.n, s.g), true, acc, lds);
      else product<P, false, F>(s, R(s.px, nk, s.X, s.x0, s.n, s.g), R(s.py, nk, s.Y, s.y0, s.n, s.g), false, acc, lds);
    }
    gate = v;
    v = add_up(acc, lds, s.w, s.n, s.g);
  }
  if (threadIdx.x >= 64 * F * F) return;
  const int row = s.x0 + threadIdx.x / (4 * F), col = s.y0 + threadIdx.x % (4 * F) * 4;
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
  const uint64_t* table = nullptr;  // addresses of the image's rows in the first K tiles, in LDS
  uint64_t lane_at[4];              // this lane's place in piece 0 of the K tile at hand, for each of four loads
  __device__ __forceinline__ void open_staged(int kt_, int) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) lane_at[i] = table[kt_ * kTile + 8 * i + (lane >> 3)] + (((lane & 7) ^ (lane >> 3)) * 16);
  }
  __device__ __forceinline__ void load_staged(int i, uint32_t bytes, uint32_t lds_addr, int imm) const {
    load_lds(lane_at[i] + bytes, lds_addr, imm + i * 1024);
  }
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
__global__ void __launch_bounds__(64 * kWaves) gemm_rows_kernel(DeviceTables t, Batch b) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  int bx, by;
  xcd_remap(bx, by);
  const int first = b.idx[by], count = b.idx[by + 1] - first;
  const OpDesc& d = t.descs[b.base + b.idx[b.n + 1 + first]];  // what the group has in common
  if (bx >= d.nblocks) return;
  const int nk = __builtin_amdgcn_readfirstlane(d.p.nk), lane = threadIdx.x & 63;
  Sides s;
  s.ks = t.aux + __builtin_amdgcn_readfirstlane(d.aux0);
  s.nk = nk;
  s.stages = b.stages;
  s.sizes = read_sizes(s.ks, nk);
  s.X = count;
  s.Y = __builtin_amdgcn_readfirstlane(d.cols);
  s.x0 = 0;
  s.y0 = bx * kTile;
  s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  s.n = lane & 15;
  s.g = lane >> 4;
  RowsSide<T, P> x(t, b, first, count, s.n, s.g);
  uint64_t* const table = (uint64_t*)(lds + ring_bytes(2, b.stages));
  if (nk <= kTableTiles) {
    for (int q = threadIdx.x; q < kTile * nk; q += 64 * kWaves) {
      const OpDesc& o = t.descs[b.base + b.idx[b.n + 1 + first + min(q % kTile, count - 1)]];
      table[q] = (uint64_t)t.ptrs[o.ptr0 + q / kTile];
    }
    x.table = table;
    __syncthreads();
  }
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, gate = v;
  const int passes = __builtin_amdgcn_readfirstlane(d.p.mode) == 2 ? 2 : 1;
  for (int pass = 0; pass < passes; ++pass) {
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const Side<T, P, true, 2> y(t.ptrs + __builtin_amdgcn_readfirstlane(d.ptr0) + (1 + pass) * nk, nk, s.Y, s.y0, s.n, s.g);
    if (nk <= kTableTiles) product<P, true, 2>(s, x, y, true, acc, lds);
    else product<P, false, 2>(s, x, y, true, acc, lds);
    gate = v;
    v = add_up(acc, lds, s.w, s.n, s.g);
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

#define TN_LAUNCH_SMALL(KERNEL, LDS)                                                                                              \
  do {                                                                                                                            \
    static std::atomic<uint64_t> allowed{0};                                                                                      \
    if (const hipError_t e = allow_lds(allowed, (const void*)KERNEL, LDS(kStages)); e != hipSuccess) return e;                    \
    hipLaunchKernelGGL(KERNEL, grid, wg, LDS(b.stages), s, t, b);                                                                 \
  } while (0)

hipError_t launch_gemm_small(bool bf16_products, int dtype, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t s) {
  // 32x32 tiles that leave half of the CUs without one are cut into 16x16 tiles: a quarter of the products each, half of the
  // loads, and the same bits.  fp32, 64x64 with K of 256 5.4 -> 4.5 us, with 704 9.8 -> 7.3; 256x256 with K of 2560, one of them 19.1 -> 11.1, two
  // (128 workgroups) 18.9 -> 14.1, four 18.9 -> 26.2.
  const bool tiny = !bf16_products && dtype == TN_F32 && (int64_t)max_blocks * b.n <= 128;
  const dim3 grid((unsigned)max_blocks * (tiny ? 4 : 1), (unsigned)b.n), wg(64 * kWaves);
  auto lds = [](int stages) { return ring_bytes(2, stages); };
  auto lds_tiny = [](int stages) { return ring_bytes(1, stages); };
  if (bf16_products) TN_LAUNCH_SMALL((gemm_small_kernel<bf16_t, true, 2>), lds);
  else if (dtype == TN_BF16) TN_LAUNCH_SMALL((gemm_small_kernel<bf16_t, false, 2>), lds);
  else if (tiny) TN_LAUNCH_SMALL((gemm_small_kernel<float, false, 1>), lds_tiny);
  else TN_LAUNCH_SMALL((gemm_small_kernel<float, false, 2>), lds);
  return hipGetLastError();
}

hipError_t launch_gemm_rows(int dtype, const DeviceTables& t, uint32_t base, const RowVertex* rows, int n, int32_t max_blocks,
                            hipStream_t s) {
  Batch b;
  b.base = base;
  b.stages = 0;
  for (int k = 0; k < n; ++k) b.stages = std::max(b.stages, rows[k].stages);
  auto lds = [](int stages) { return ring_bytes(2, stages) + kTableTiles * kTile * 8; };
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
    if (dtype == TN_BF16) TN_LAUNCH_SMALL((gemm_rows_kernel<bf16_t, Bf16Products>), lds);
    else TN_LAUNCH_SMALL((gemm_rows_kernel<float, Fp32Products<float>>), lds);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    at += taken;
  }
  return hipSuccess;
}

#undef TN_LAUNCH_SMALL

}  // namespace tn
