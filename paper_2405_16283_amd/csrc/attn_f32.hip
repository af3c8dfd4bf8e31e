// Attention forward and reverse with fp32 products on the matrix cores (MFMA 16x16x4): fp32 graphs, and
// bf16 graphs whose tiling the bf16 kernels in kernels.hip do not take (key tiles that are no multiple of
// 64 rows, heads that straddle column tiles).  Any tile grid the executor admits is served.
//
// One workgroup = one head x 64 rows of its own side (queries; keys in the dK and dV forms); a wavefront
// owns 16 of them and a lane (n = lane & 15, g = lane >> 4) row n of those 16.  The other side comes
// through LDS as fp32, 64 rows at a time.  Scores are formed transposed, S^T = K Q^T, so that a lane holds
// the scores of its own row against rows 4g + i of a 16-row tile -- which is the B operand of the second
// product if step c of its four MFMAs takes the rows 4g + c: probabilities never leave their registers.
//
// Bound: the matrix cores (256 flop per clock and CU in fp32, 157 TFLOP/s); 64 keys cost a wavefront 256
// MFMAs of 32 cycles at head size 128 against 64 KiB of LDS reads, a quarter of what LDS delivers in that time.
// The kernels these replace ran one query row per thread on the vector ALUs with every operand read from
// memory.  Per launch, before -> after: fp32, 16 heads of 64, 1024 positions in blocks of 512, 5.6 ms -> 58 us;
// fp32 reverse, 3 heads of 64, 160 positions, 2.8 ms -> 17 us (latency: a handful of workgroups); bf16, 32 heads
// of 128, 347 queries against 1371 keys, 6.6 ms -> 0.10 ms.  (Reverse pass with the own rows by
// way of LDS and all loads up to the first chunk issued before any is waited for: 18.1 -> 17.8 us, not kept.)
#include "device.h"
#include "kernels.h"

namespace tn {
namespace {

constexpr int kRows = 64;  // rows of a workgroup's own side, and rows of the other side per round

// One side's tile grid, seen from one head.
template <typename T, int HD>
struct Side {
  void* const* t;
  int nc, trows, tc, rows;
  int c0;       // first column of the head
  bool whole;   // the head lies inside one column tile: ct, cin name it
  int ct, cin;
  __device__ Side(void* const* tiles, int nc_, int trows_, int tc_, int rows_, int h)
      : t(tiles), nc(nc_), trows(trows_), tc(tc_), rows(rows_), c0(h * HD), whole(tc_ % HD == 0), ct(c0 / tc_), cin(c0 - ct * tc_) {}
  // columns c..c+3 of the head in row `row`
  __device__ f32x4 at(int row, int c) const {
    if (whole) {
      const int rt = row / trows;
      return ld4((const T*)t[rt * nc + ct] + (size_t)(row - rt * trows) * tc + cin + c);
    }
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ld(tile_elem<T>(t, nc, trows, tc, row, c0 + c + i));
    return v;
  }
  // the same where the tiles hold the transpose
  __device__ f32x4 at_t(int row, int c) const {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ld(tile_elem_t<T>(t, nc, trows, tc, rows, row, c0 + c + i));
    return v;
  }
};

constexpr int kPieces(int hd) { return kRows * hd / 4 / 256; }  // pieces of four elements per thread and chunk

// Rows row0 .. row0 + 63 into registers: piece p = i * 256 + tid is columns 4 (p % (HD / 4)) .. of row p / (HD / 4).
// Rows past the end are zero.
// (pieces I0 .. I0 + N - 1 only.)
template <typename T, int HD, int I0 = 0, int N = kPieces(HD)>
__device__ __forceinline__ void load_chunk(const Side<T, HD>& s, bool transposed, int row0, f32x4 (&v)[N]) {
  const int rt0 = row0 / s.trows, rin0 = row0 - rt0 * s.trows, n = min(kRows, s.rows - row0);
  const bool plain = s.whole && !transposed && rin0 + n <= s.trows;  // one tile: the address is linear in the row
  const T* base = plain ? (const T*)s.t[rt0 * s.nc + s.ct] + (size_t)rin0 * s.tc + s.cin : nullptr;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = (I0 + i) * 256 + threadIdx.x, r = p / (HD / 4), c = (p % (HD / 4)) * 4;
    v[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (r < n) v[i] = plain ? ld4(base + (size_t)r * s.tc + c) : transposed ? s.at_t(row0 + r, c) : s.at(row0 + r, c);
  }
}
template <int HD, int I0 = 0, int N = kPieces(HD)>
__device__ __forceinline__ void store_chunk(float (*buf)[HD + 4], const f32x4 (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = (I0 + i) * 256 + threadIdx.x;
    *(f32x4*)&buf[p / (HD / 4)][(p % (HD / 4)) * 4] = v[i];
  }
}

// The 64-row chunk of V as V^T[HD][64]: piece p is keys 4 (p % 16) .. of head column p / 16.
template <typename T, int HD, int I0 = 0, int N = kPieces(HD)>
__device__ __forceinline__ void load_chunk_vt(const Side<T, HD>& s, bool transposed, int row0, f32x4 (&v)[N]) {
  const int rt0 = row0 / s.trows, rin0 = row0 - rt0 * s.trows, n = min(kRows, s.rows - row0);
  const int pitch = min(s.trows, s.rows - rt0 * s.trows);
  const bool linear = s.whole && transposed && rin0 + n <= s.trows;  // one tile: the address is linear in the key and the column
  const bool plain = linear && pitch % 4 == 0 && rin0 % 4 == 0;
  const T* base = linear ? (const T*)s.t[rt0 * s.nc + s.ct] + (size_t)s.cin * pitch + rin0 : nullptr;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = (I0 + i) * 256 + threadIdx.x, c = p / 16, k = (p % 16) * 4;
    v[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (plain) {  // n is a multiple of 4 here: the tile's rows are
      if (k < n) v[i] = ld4(base + (size_t)c * pitch + k);
    } else if (linear) {  // (347 keys: with the tile looked up for every element 132 us a launch, so 103)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < n) v[i][e] = ld(base + (size_t)c * pitch + k + e);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < n)
          v[i][e] = ld(transposed ? tile_elem_t<T>(s.t, s.nc, s.trows, s.tc, s.rows, row0 + k + e, s.c0 + c)
                                  : tile_elem<T>(s.t, s.nc, s.trows, s.tc, row0 + k + e, s.c0 + c));
    }
  }
}

template <int HD, int I0 = 0, int N = kPieces(HD)>
__device__ __forceinline__ void store_chunk_vt(float (*buf)[kRows + 4], const f32x4 (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = (I0 + i) * 256 + threadIdx.x;
    *(f32x4*)&buf[p / 16][(p % 16) * 4] = v[i];
  }
}

// A row's sum leaves out what the causal mask hides from it.  The matrix cores multiply that by a weight of zero, which
// is the same as long as it is finite.  Chunks the diagonal crosses are looked through for infinities and NaN in LDS;
// a workgroup that finds some forms its rows again, each summed over what it sees, sixteen lanes to a row (`*_by_rows`: many
// times slower, and outside the loops on the matrix cores, whose registers and order of instructions it must not cost
// anything: inside them, and with the look between loads and stores, it took 2 % of a decode program).
template <int ROWS, int COLS, int PITCH>
__device__ __forceinline__ bool not_finite(const float (*buf)[PITCH]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < ROWS * COLS / 4 / 256; ++i) {
    const int p = i * 256 + threadIdx.x;
    const f32x4 v = *(const f32x4*)&buf[p / (COLS / 4)][p % (COLS / 4) * 4];
#pragma unroll
    for (int e = 0; e < 4; ++e) z = fmaf(v[e], 0.f, z);
  }
  return !(z == 0.f);
}

// whether any lane of the workgroup says so, once its chunks in LDS are done with
__device__ __forceinline__ bool any_wave(bool mine, char* lds) {
  const int wave = __ballot(mine) != 0;
  int* const said = (int*)lds;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) said[threadIdx.x >> 6] = wave;
  __syncthreads();
  return __builtin_expect((said[0] | said[1] | said[2] | said[3]) != 0, 0);
}

__device__ __forceinline__ float dot4(f32x4 a, f32x4 b) { return fmaf(a[0], b[0], fmaf(a[1], b[1], fmaf(a[2], b[2], a[3] * b[3]))); }
__device__ __forceinline__ float row_sum(float v) {  // over the sixteen lanes of a row
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <typename T, int HD>
__device__ __forceinline__ void attn_by_rows(DeviceTables t, const OpDesc& d) {
  const int* ax = t.aux + d.aux0;
  const int tq = ax[0], tk = ax[1], tc = ax[2], q_rows = ax[3], kv_rows = ax[4], nc = d.p.n_col_tiles, gw = nc * tc;
  const int qblocks = (q_rows + kRows - 1) / kRows, h = blockIdx.x / qblocks, qb = blockIdx.x % qblocks;
  void* const* Qt = t.ptrs + d.ptr0;
  void* const* Kt = Qt + d.p.n_q_tiles * nc;
  const Side<T, HD> Q(Qt, nc, tq, tc, q_rows, h), K(Kt, nc, tk, tc, kv_rows, h), V(Kt + d.p.n_kv_tiles * nc, nc, tk, tc, kv_rows, h);
  constexpr int C = HD / 64;  // pieces of four columns per lane: c0, c0 + 64
  const int c0 = (threadIdx.x & 15) * 4;
#pragma unroll 1
  for (int row = qb * kRows + (threadIdx.x >> 4); row < min(Q.rows, (qb + 1) * kRows); row += 16) {
    f32x4 q[C], o[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      q[i] = Q.at(row, c0 + 64 * i) * d.p.scale;
      o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    float m = -INFINITY, l = 0.f;
    const int seen = min(K.rows, d.p.q_pos0 + row - d.p.k_pos0 + 1);
#pragma unroll 1
    for (int k = 0; k < seen; ++k) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < C; ++i) s += dot4(q[i], K.at(k, c0 + 64 * i));
      s = row_sum(s);
      const float mn = fmaxf(m, s), ms = mn == -INFINITY ? 0.f : mn;
      const float alpha = __expf(m - ms), p = __expf(s - ms);
      m = mn;
      l = l * alpha + p;
#pragma unroll
      for (int i = 0; i < C; ++i) o[i] = o[i] * alpha + (d.p.v_trans ? V.at_t(k, c0 + 64 * i) : V.at(k, c0 + 64 * i)) * p;
    }
    float* out = (float*)d.out + (size_t)row * d.cols;
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) out[h * HD + c0 + 64 * i + e] = o[i][e];
    if (c0 == 0) {
      out[gw + h] = m;
      out[gw + gw / HD + h] = l;
    }
  }
}

// aux: [rows per Q tile, rows per K/V tile, columns per tile, q rows, kv rows]
template <typename T, int HD>
__global__ void __launch_bounds__(256, 2) attn_f32_kernel(DeviceTables t, Batch b) {
  const OpDesc& d = t.descs[b.at(blockIdx.y)];
  if ((int)blockIdx.x >= d.nblocks) return;
  const int* ax = t.aux + d.aux0;
  const int tq = ax[0], tk = ax[1], tc = ax[2], q_rows = ax[3], kv_rows = ax[4];
  const int nc = d.p.n_col_tiles, gw = nc * tc, hpg = gw / HD;
  const int qblocks = (q_rows + kRows - 1) / kRows;
  const int h = blockIdx.x / qblocks, qb = blockIdx.x % qblocks;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
  void* const* Qt = t.ptrs + d.ptr0;
  void* const* Kt = Qt + d.p.n_q_tiles * nc;
  void* const* Vt = Kt + d.p.n_kv_tiles * nc;
  const Side<T, HD> Q(Qt, nc, tq, tc, q_rows, h), K(Kt, nc, tk, tc, kv_rows, h), V(Vt, nc, tk, tc, kv_rows, h);
  const bool v_trans = d.p.v_trans != 0;
  const int causal = d.p.causal, k_pos0 = d.p.k_pos0;

  extern __shared__ __attribute__((aligned(16))) char lds[];
  float(*const ks)[HD + 4] = (float(*)[HD + 4])lds;                                   // K chunk [64][HD], padded
  float(*const vs)[kRows + 4] = (float(*)[kRows + 4])(lds + sizeof(float) * kRows * (HD + 4));  // V^T chunk [HD][64], padded
  bool odd = false;  // a chunk on the diagonal whose V is not finite

  const int row = qb * kRows + w * 16 + n, qpos = d.p.q_pos0 + row;
  const int wpos0 = d.p.q_pos0 + qb * kRows + w * 16;  // first position of the wavefront
  f32x4 q[HD / 16];
#pragma unroll
  for (int j = 0; j < HD / 16; ++j) q[j] = Q.at(min(row, q_rows - 1), 16 * j + 4 * g) * d.p.scale;
  f32x4 o[HD / 16];
#pragma unroll
  for (int j = 0; j < HD / 16; ++j) o[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;

  int end = kv_rows;  // keys above the diagonal of this workgroup's rows contribute nothing
  if (causal) end = min(kv_rows, d.p.q_pos0 + qb * kRows + kRows - k_pos0);
  // head size 64 has the registers to fetch the next chunk while one is multiplied; at 128 the second
  // workgroup of the compute unit covers the wait instead
  constexpr bool kAhead = HD == 64;
  constexpr int P = kAhead ? kPieces(HD) : kPieces(HD) / 2;
  f32x4 kn[P], vn[P];
  if (kAhead && end > 0) {
    load_chunk<T, HD, 0, P>(K, false, 0, kn);
    load_chunk_vt<T, HD, 0, P>(V, v_trans, 0, vn);
  }
  for (int kv0 = 0; kv0 < end; kv0 += kRows) {
    __syncthreads();  // everybody is done with the chunk before
    if constexpr (!kAhead) {
      load_chunk<T, HD, 0, P>(K, false, kv0, kn);
      load_chunk_vt<T, HD, 0, P>(V, v_trans, kv0, vn);
    }
    store_chunk<HD, 0, P>(ks, kn);
    store_chunk_vt<HD, 0, P>(vs, vn);
    if constexpr (!kAhead) {
      load_chunk<T, HD, P, P>(K, false, kv0, kn);
      load_chunk_vt<T, HD, P, P>(V, v_trans, kv0, vn);
      store_chunk<HD, P, P>(ks, kn);
      store_chunk_vt<HD, P, P>(vs, vn);
    }
    __syncthreads();
    if (kAhead && kv0 + kRows < end) {
      load_chunk<T, HD, 0, P>(K, false, kv0 + kRows, kn);
      load_chunk_vt<T, HD, 0, P>(V, v_trans, kv0 + kRows, vn);
    }
    if (causal && k_pos0 + kv0 + kRows - 1 > d.p.q_pos0 + qb * kRows && not_finite<HD, kRows>(vs)) odd = true;
    f32x4 s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < HD / 16; ++j) {
      f32x4 a[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = *(const f32x4*)&ks[16 * k + n][16 * j + 4 * g];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = mfma_f32(a[k][c], q[j][c], s[k]);
      if (j & 1) __builtin_amdgcn_sched_barrier(0);  // no more than two steps' fragments at a time: registers
    }
    // element i of s[k]: key kv0 + 16 k + 4 g + i
    float mx = -INFINITY;
    const bool mask = kv0 + kRows > kv_rows || (causal && k_pos0 + kv0 + kRows - 1 > wpos0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kv = kv0 + 16 * k + 4 * g + i;
        if (mask && (kv >= kv_rows || (causal && k_pos0 + kv > qpos))) s[k][i] = -INFINITY;
        mx = fmaxf(mx, s[k][i]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), ms = mn == -INFINITY ? 0.f : mn;  // nothing visible yet: every weight is exp(-inf)
    const float alpha = __expf(m - ms);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[k][i] = __expf(s[k][i] - ms);
        l += s[k][i];
      }
#pragma unroll
    for (int j = 0; j < HD / 16; ++j) o[j] *= alpha;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < HD / 16; j += 4) {
        f32x4 a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = *(const f32x4*)&vs[16 * (j + e) + n][16 * k + 4 * g];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[j + e] = mfma_f32(a[e][c], s[k][c], o[j + e]);
        if (j & 4) __builtin_amdgcn_sched_barrier(0);
      }
  }
  if (causal && any_wave(odd, lds)) return attn_by_rows<T, HD>(t, d);
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (row >= q_rows) return;
  float* out = (float*)d.out + (size_t)row * d.cols;
#pragma unroll
  for (int j = 0; j < HD / 16; ++j) {
    float* o4 = out + h * HD + 16 * j + 4 * g;
    if ((d.cols & 3) == 0) {  // rows of the partial are 16-byte aligned
      st4(o4, o[j]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) o4[i] = o[j][i];
    }
  }
  if (g == 0) {
    out[gw + h] = m;
    out[gw + hpg + h] = l;
  }
}

template <typename T, int HD, int MODE, typename Stat>
__device__ __forceinline__ void attn_bwd_by_rows(const OpDesc& d, const Side<T, HD>& Q, const Side<T, HD>& K, const Side<T, HD>& V,
                                                 const Side<T, HD>& D, int rb, int h, int gw, Stat stat) {
  constexpr int C = HD / 64;
  const Side<T, HD>&own = MODE == 1 ? Q : K, &other = MODE == 1 ? K : Q;
  const int c0 = (threadIdx.x & 15) * 4;
  auto v_at = [&](int r, int c) { return d.p.v_trans ? V.at_t(r, c) : V.at(r, c); };
#pragma unroll 1
  for (int row = rb * kRows + (threadIdx.x >> 4); row < min(own.rows, (rb + 1) * kRows); row += 16) {
    f32x4 m1[C], m2[C], acc[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      m1[i] = own.at(row, c0 + 64 * i);
      m2[i] = MODE == 1 ? D.at(row, c0 + 64 * i) : v_at(row, c0 + 64 * i);
      acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const int begin = MODE == 1 ? 0 : max(0, d.p.k_pos0 + row - d.p.q_pos0);
    const int end = MODE == 1 ? min(K.rows, d.p.q_pos0 + row - d.p.k_pos0 + 1) : Q.rows;
#pragma unroll 1
    for (int o = begin; o < end; ++o) {
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int i = 0; i < C; ++i) {
        s += dot4(m1[i], other.at(o, c0 + 64 * i));
        if (MODE != 3) dp += dot4(m2[i], MODE == 1 ? v_at(o, c0 + 64 * i) : D.at(o, c0 + 64 * i));
      }
      const int q = MODE == 1 ? row : o;
      float p = __expf(row_sum(s) * d.p.scale - stat(q, 0));
      if (MODE != 3) p *= (row_sum(dp) - stat(q, 1)) * d.p.scale;
#pragma unroll
      for (int i = 0; i < C; ++i) acc[i] += (MODE == 3 ? D.at(o, c0 + 64 * i) : other.at(o, c0 + 64 * i)) * p;
    }
    T* out = (T*)d.out + (size_t)row * gw + h * HD + c0;
#pragma unroll
    for (int i = 0; i < C; ++i) st4(out + 64 * i, acc[i]);
  }
}

// Reverse pass.  Modes 0 (statistics) and 1 (dQ): the workgroup's own rows are queries, keys come in
// chunks.  Modes 2 (dK) and 3 (dV): its own rows are keys, queries and their statistics come in chunks.
// Scores are formed again from Q and K; p = exp(scale q.k - lse).
template <typename T, int HD, int MODE>
__device__ __forceinline__ void attn_bwd_f32_body(const DeviceTables& t, const OpDesc& d, char* lds) {
  const int* ax = t.aux + d.aux0;
  const int tq = ax[0], tk = ax[1], tc = ax[2], q_rows = ax[3], kv_rows = ax[4];
  const int nc = d.p.n_col_tiles, gw = nc * tc, hpg = gw / HD, nq = d.p.n_q_tiles, nkv = d.p.n_kv_tiles;
  void* const* Qt = t.ptrs + d.ptr0;
  void* const* Kt = Qt + nq * nc;
  void* const* Vt = Kt + nkv * nc;
  void* const* Dt = Vt + nkv * nc;  // dO tiles
  void* const* St = Dt + nq * nc;   // statistics, one tensor per Q row tile (modes 1..3)
  const int my_rows = MODE <= 1 ? q_rows : kv_rows, o_rows = MODE <= 1 ? kv_rows : q_rows;
  const int rblocks = (my_rows + kRows - 1) / kRows;
  const int h = blockIdx.x / rblocks, rb = blockIdx.x % rblocks;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
  const Side<T, HD> Q(Qt, nc, tq, tc, q_rows, h), K(Kt, nc, tk, tc, kv_rows, h), V(Vt, nc, tk, tc, kv_rows, h),
      D(Dt, nc, tq, tc, q_rows, h);
  const bool v_trans = d.p.v_trans != 0;
  const int causal = d.p.causal;
  const float scale = d.p.scale;
  auto stat = [&](int r, int which) -> float {  // which 0: lse, 1: D
    const int rt = r / tq;
    return ((const float*)St[rt])[(size_t)(r - rt * tq) * (2 * hpg) + which * hpg + h];
  };
  float(*const x1)[HD + 4] = (float(*)[HD + 4])lds;                                             // K, or Q
  float(*const x2)[HD + 4] = (float(*)[HD + 4])(lds + sizeof(float) * kRows * (HD + 4));        // V, or dO
  float(*const xs)[2] = (float(*)[2])(lds + 2 * sizeof(float) * kRows * (HD + 4));              // statistics of the queries
  bool odd = false;  // a chunk on the diagonal that is not finite

  const int row = rb * kRows + w * 16 + n, rc = min(row, my_rows - 1);
  const int pos = (MODE <= 1 ? d.p.q_pos0 : d.p.k_pos0) + row;
  f32x4 m1[HD / 16], m2[HD / 16], acc[HD / 16];  // this lane's own row: Q and dO, or K and V
#pragma unroll
  for (int j = 0; j < HD / 16; ++j) {
    m1[j] = MODE <= 1 ? Q.at(rc, 16 * j + 4 * g) : K.at(rc, 16 * j + 4 * g);
    if (MODE <= 1) m2[j] = D.at(rc, 16 * j + 4 * g);
    if (MODE == 2) m2[j] = v_trans ? V.at_t(rc, 16 * j + 4 * g) : V.at(rc, 16 * j + 4 * g);
    acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const float lse = MODE == 1 ? stat(rc, 0) : 0.f, Dr = MODE == 1 ? stat(rc, 1) : 0.f;
  float mrun = -INFINITY, l = 0.f, dsum = 0.f;  // mode 0: this lane's share of the keys
  int begin = 0, end = o_rows;
  if (causal && MODE <= 1) end = min(kv_rows, d.p.q_pos0 + rb * kRows + kRows - d.p.k_pos0);
  if (causal && MODE >= 2) begin = max(0, d.p.k_pos0 + rb * kRows - d.p.q_pos0);

  for (int r0 = begin; r0 < end; r0 += kRows) {
    f32x4 v1[kPieces(HD)], v2[kPieces(HD)];
    load_chunk<T, HD>(MODE <= 1 ? K : Q, false, r0, v1);
    load_chunk<T, HD>(MODE <= 1 ? V : D, MODE <= 1 && v_trans, r0, v2);
    float sv = 0.f;
    if (MODE >= 2 && threadIdx.x < 2 * kRows) sv = stat(min(r0 + (int)threadIdx.x / 2, q_rows - 1), threadIdx.x & 1);
    __syncthreads();  // everybody is done with the chunk before
    store_chunk<HD>(x1, v1);
    store_chunk<HD>(x2, v2);
    if (MODE >= 2 && threadIdx.x < 2 * kRows) xs[threadIdx.x / 2][threadIdx.x & 1] = sv;
    __syncthreads();
    // some row of the workgroup and some row of the chunk do not see each other
    if (MODE != 0 && causal && (MODE == 1 ? d.p.k_pos0 + r0 + kRows - 1 > d.p.q_pos0 + rb * kRows
                                          : d.p.k_pos0 + rb * kRows + kRows - 1 > d.p.q_pos0 + r0) &&
        not_finite<kRows, HD>(MODE == 3 ? x2 : x1))
      odd = true;
#pragma unroll 1
    for (int k = 0; k < 4; k += 2) {  // two 16-row tiles of the other side at a time
      f32x4 s[2], dp[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) s[e] = dp[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < HD / 16; ++j) {
        f32x4 a[2], a2[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          a[e] = *(const f32x4*)&x1[16 * (k + e) + n][16 * j + 4 * g];
          if (MODE != 3) a2[e] = *(const f32x4*)&x2[16 * (k + e) + n][16 * j + 4 * g];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            s[e] = mfma_f32(a[e][c], m1[j][c], s[e]);
            if (MODE != 3) dp[e] = mfma_f32(a2[e][c], m2[j][c], dp[e]);
          }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        // element i: row r0 + 16 (k + e) + 4 g + i of the other side
        f32x4 wgt;
        float mx = mrun;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int lr = 16 * (k + e) + 4 * g + i, o = r0 + lr;
          bool ok = o < o_rows;
          if (causal) ok = ok && (MODE <= 1 ? d.p.k_pos0 + o <= pos : pos <= d.p.q_pos0 + o);
          const float z = s[e][i] * scale;
          if (MODE == 0) {
            s[e][i] = ok ? z : -INFINITY;
            if (!ok) dp[e][i] = 0.f;
            mx = fmaxf(mx, s[e][i]);
          } else {
            float p = __expf(z - (MODE == 1 ? lse : xs[lr][0]));
            if (MODE == 1) p *= (dp[e][i] - Dr) * scale;
            if (MODE == 2) p *= (dp[e][i] - xs[lr][1]) * scale;
            wgt[i] = ok ? p : 0.f;
          }
        }
        if (MODE == 0) {
          const float ms = mx == -INFINITY ? 0.f : mx, alpha = __expf(mrun - ms);
          l *= alpha;
          dsum *= alpha;
          mrun = mx;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p = __expf(s[e][i] - ms);
            l += p;
            dsum = fmaf(p, dp[e][i], dsum);
          }
          continue;
        }
        // acc^T[column, own row] += X^T[column, other row] wgt[other row, own row]; X: K, Q or dO
        float(*const xt)[HD + 4] = MODE == 3 ? x2 : x1;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int j = 0; j < HD / 16; ++j) acc[j] = mfma_f32(xt[16 * (k + e) + 4 * g + c][16 * j + n], wgt[c], acc[j]);
      }
    }
  }
  if (MODE == 0) {
    // the four lanes of a query saw different keys: merge their states
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float m2_ = __shfl_xor(mrun, off, 64), l2 = __shfl_xor(l, off, 64), d2 = __shfl_xor(dsum, off, 64);
      const float mn = fmaxf(mrun, m2_), ms = mn == -INFINITY ? 0.f : mn;
      const float w1 = __expf(mrun - ms), w2 = __expf(m2_ - ms);
      l = l * w1 + l2 * w2;
      dsum = dsum * w1 + d2 * w2;
      mrun = mn;
    }
    if (row < my_rows && g == 0) {
      float* out = (float*)d.out + (size_t)row * (2 * hpg);
      out[h] = mrun + __logf(l);
      out[hpg + h] = dsum / l;
    }
    return;
  }
  if (causal && any_wave(odd, lds)) return attn_bwd_by_rows<T, HD, MODE>(d, Q, K, V, D, rb, h, gw, stat);
  if (row >= my_rows) return;
  T* out = (T*)d.out + (size_t)row * gw + h * HD;
#pragma unroll
  for (int j = 0; j < HD / 16; ++j) st4(out + 16 * j + 4 * g, acc[j]);
}

template <typename T, int HD>
__global__ void __launch_bounds__(256, 2) attn_bwd_f32_kernel(DeviceTables t, Batch b) {
  const OpDesc& d = t.descs[b.at(blockIdx.y)];
  if ((int)blockIdx.x >= d.nblocks) return;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  switch (d.p.mode) {
    case 0: attn_bwd_f32_body<T, HD, 0>(t, d, lds); break;
    case 1: attn_bwd_f32_body<T, HD, 1>(t, d, lds); break;
    case 2: attn_bwd_f32_body<T, HD, 2>(t, d, lds); break;
    default: attn_bwd_f32_body<T, HD, 3>(t, d, lds); break;
  }
}

constexpr int fwd_lds(int hd) { return 4 * (kRows * (hd + 4) + hd * (kRows + 4)); }
constexpr int bwd_lds(int hd) { return 4 * (2 * kRows * (hd + 4) + 2 * kRows); }

template <auto kernel>
hipError_t launch(int lds, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t s) {
  static std::atomic<uint64_t> allowed{0};
  if (const hipError_t e = allow_lds(allowed, (const void*)kernel, lds); e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3((unsigned)max_blocks, (unsigned)b.n), dim3(256), lds, s, t, b);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_f32(bool reverse, int dtype, int head_dim, const DeviceTables& t, const Batch& b, int32_t max_blocks,
                           hipStream_t s) {
  const bool bf = dtype == TN_BF16;
  if (head_dim != 64 && head_dim != 128) return hipErrorInvalidValue;
#define TN_PICK(kernel, lds)                                                                                  \
  (head_dim == 64 ? (bf ? launch<kernel<bf16_t, 64>>(lds(64), t, b, max_blocks, s)                            \
                        : launch<kernel<float, 64>>(lds(64), t, b, max_blocks, s))                            \
                  : (bf ? launch<kernel<bf16_t, 128>>(lds(128), t, b, max_blocks, s)                          \
                        : launch<kernel<float, 128>>(lds(128), t, b, max_blocks, s)))
  return reverse ? TN_PICK(attn_bwd_f32_kernel, bwd_lds) : TN_PICK(attn_f32_kernel, fwd_lds);
#undef TN_PICK
}

}  // namespace tn
