// Tile products in bf16 on the matrix cores, C[M,N] = sum_k A_k[M,K_k] * B_k[N,K_k]^T, fp32 accumulation, bf16 store, for
// outputs of more than a few thousand elements (smaller and thinner ones: gemm_small.hip).
//
// What bounds them.  A launch that fills the chip with random operands runs at the power limit, so that what counts is the energy
// of an operation as much as the cycles it takes.  Measured in registers alone (256 workgroups of four wavefronts, N(0, 1)
// operands): MFMA 32x32x16 1.79 GHz and 1860 TFLOP/s, MFMA 16x16x32, which moves half as many accumulators per product, 2.03 GHz
// and 2070, and 2130 when neighbouring instructions share an operand both ways (rows of tiles walked to and fro).  Hence:
//   - MFMA 16x16x32 (the sums come out bit by bit as those of 32x32x16);
//   - four wavefronts, one per SIMD, with 128x128 of the 256x256 tile each: eight with 128x64 read half as much again from LDS;
//   - K in chunks of 64, so that the eight lanes of a row fetch a whole 128-byte line once (counted: 256 workgroups with K of 4096 read
//     1074 MB into LDS, their operands and no more); of a chunk of 32 a line is two, half of it used by each;
//   - one wavefront per SIMD has nothing beside it to hide its other instructions, so these are placed one by one into
//     the 16 cycles of an MFMA, and the position in LDS of a load is set ahead of the MFMA before it.
// The loop of the 256x256 form takes 2250 cycles per chunk, 2048 of them MFMAs, at 1.72 GHz (256 workgroups, K of 4096 and 8192: 174 and
// 319 thousand cycles); what does not depend on K, the first operands and the stores, takes 30 thousand.  Against the kernel it replaced
// (32x32x16, eight wavefronts, K in steps of 32), launches of 512x512 vertices one behind the other, when it came: 4096 x 12288 with
// K of 4096 367 -> 327 us, 4096 x 4096 133 -> 119, with K of 11008 315 -> 276, 8192 x 8192 x 8192 877 -> 762.  With the present epilogue, twelve
// launches in a row: 289, 100, 242 and 743 us (1480 TFLOP/s).
//
// Operands lie in LDS in regions of 128 rows x 64 of K (16 KiB), a ring of them that `buffer_load ... lds` fills directly, 64 lanes
// x 16 bytes per instruction, unpadded: piece c of row r lies at position c ^ (r & 7) of its row, so that the 16 lanes
// of a fragment read fall on different banks.  A resource begins at the workgroup's first row, found in 64 bits: tiles of any size are
// fine as long as 256 of their rows stay below 4 GiB.  Rows past the edge of a ragged tile are clamped (their products are never
// stored); past the end of K a lane's offset lies outside the buffer resource and zeros arrive, in both operands.  Chunks are
// taken two at a time, an odd one is followed by zeros.
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace tn {
namespace {

constexpr int kChunk = 64;               // of K
constexpr int kRegionRows = 128;
constexpr uint32_t kRegionBytes = kRegionRows * kChunk * 2;
constexpr int kPieceLoads = 4;           // load instructions per wavefront and region
constexpr uint32_t kNoOffset = 0xFFFFFFFFu;  // outside every buffer resource: the lane's bytes in LDS become zero

// The accumulators stay in the accumulation registers and each is updated in place: left to itself the compiler gives the
// result other registers than the summand, and the 256 of a wavefront do not fit twice.  It does not know that these
// are MFMAs, so whatever else reads accumulators comes after mfma_drain(), through which they pass.
__device__ __forceinline__ void mfma(f32x4& c, bf16x8 x, bf16x8 y) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
}
__device__ __forceinline__ void mfma_then_load(f32x4& c, bf16x8 x, bf16x8 y, uint32_t voff, rsrc_t r, uint32_t soff, uint32_t lds_addr,
                                               int imm) {
  asm volatile("s_add_u32 m0, %6, %7\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\tbuffer_load_dwordx4 %3, %4, %5 offen lds"
               : "+a"(c) : "v"(x), "v"(y), "v"(voff), "s"(r), "s"(soff), "s"(lds_addr), "n"(imm) : "memory", "scc");
}
template <int N, int M>
__device__ __forceinline__ void mfma_drain(f32x4 (&acc)[N][M]) {
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < M; ++j) asm volatile("" : "+a"(acc[i][j]));  // behind the wait: volatile statements keep their order
}

// all LDS operations of this wavefront done and at most N (0..63) of its loads on their way
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}
__device__ __forceinline__ void barrier() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// What a workgroup works on.  The output is stored along Q: C[P][Q] with P = rows of A and Q = rows of B, or, transposed, with
// the two exchanged; MFMAs take their first operand from Q, so that a lane holds four neighbouring elements of one P row.
struct Job {
  int P, Q, p0, q0, nk;
  bool gated;
  const void* const* tiles_p;
  const void* const* tiles_q;
  const int* ksz;
};

// Loads: the sequence of a workgroup's chunks along K, and the offsets of this lane's pieces.
// HP, HQ: regions per chunk and operand.  In a tile of two regions each, a region holds 64 of the 128 rows of either wavefront.
template <int HP, int HQ>
struct Source {
  uint32_t off_p[HP][kPieceLoads], off_q[HQ][kPieceLoads];
  rsrc_t rp, rq, rq2;
  uint32_t at;  // bytes along K
  int kt, k0, K;

  __device__ __forceinline__ static rsrc_t resource(const void* p) {
    return (rsrc_t){(uint32_t)(uintptr_t)p, (uint32_t)((uintptr_t)p >> 32) & 0xFFFFu, 0xFFFFFFF0u, 0x00020000u};
  }
  // a tile's resource, from the workgroup's first row on
  __device__ __forceinline__ rsrc_t tile(const void* const* p, int row0) const {
    return resource((const char*)sload_ptr(p) + (uint64_t)(uint32_t)row0 * (uint32_t)K * 2u);
  }
  // (lane goes through an empty asm statement: rows and columns are not to be kept in registers between two calls)
  __device__ __forceinline__ void set_offsets(const Job& j, int w, int lane) {
    asm volatile("" : "+v"(lane));
    const int lr = lane >> 3, lcol = ((lane & 7) ^ lr) * 8;
#pragma unroll
    for (int i = 0; i < kPieceLoads; ++i) {
      const int rr = i * 32 + w * 8 + lr;  // row of the region
#pragma unroll
      for (int h = 0; h < HP; ++h) {
        const int row = HP == 1 ? rr : (rr >> 6) * 128 + h * 64 + (rr & 63);
        off_p[h][i] = ((uint32_t)min(row, j.P - 1 - j.p0) * (uint32_t)K + (uint32_t)lcol) * 2u;
      }
#pragma unroll
      for (int h = 0; h < HQ; ++h) {
        const int row = HQ == 1 ? rr : (rr >> 6) * 128 + h * 64 + (rr & 63);
        // gated: 32 rows of the gate tile, then the 32 rows of the up tile for the same outputs, and so on
        off_q[h][i] = ((uint32_t)min(j.gated ? (row >> 6) * 32 + (row & 31) : row, j.Q - 1 - j.q0) * (uint32_t)K + (uint32_t)lcol) * 2u;
      }
    }
  }
  __device__ __forceinline__ void cut_offsets(int lane) {  // the chunk reaches past K: zeros behind it
    asm volatile("" : "+v"(lane));
    const bool in = ((lane & 7) ^ (lane >> 3)) * 8 < K - k0;
#pragma unroll
    for (int i = 0; i < kPieceLoads; ++i) {
#pragma unroll
      for (int h = 0; h < HP; ++h) off_p[h][i] = in ? off_p[h][i] : kNoOffset;
#pragma unroll
      for (int h = 0; h < HQ; ++h) off_q[h][i] = in ? off_q[h][i] : kNoOffset;
    }
  }
  __device__ __forceinline__ void start(const Job& j, int w, int lane) {
    kt = k0 = 0;
    at = 0;
    K = sload_int(j.ksz);
    rp = tile(j.tiles_p, j.p0);
    rq = tile(j.tiles_q, j.q0);
    rq2 = j.gated ? tile(j.tiles_q + j.nk, j.q0) : rq;
    set_offsets(j, w, lane);
    if (K < kChunk) cut_offsets(lane);
  }
  __device__ __forceinline__ void advance(const Job& j, int w, int lane) {
    k0 += kChunk;
    at += 2 * kChunk;
    if (k0 + kChunk <= K) return;
    if (k0 >= K && kt + 1 < j.nk) {
      ++kt;
      k0 = 0;
      at = 0;
      const int before = K;
      K = sload_int(j.ksz + kt);
      rp = tile(j.tiles_p + kt, j.p0);
      rq = tile(j.tiles_q + kt, j.q0);
      rq2 = j.gated ? tile(j.tiles_q + j.nk + kt, j.q0) : rq;
      if (K != before || K % kChunk) set_offsets(j, w, lane);
    }
    if (k0 + kChunk > K) cut_offsets(lane);
  }
};

// Finds the workgroup's job; false if it has none (ragged vertices of a launch take fewer workgroups than its largest).
__device__ __forceinline__ bool find_job(const DeviceTables& t, const Batch& b, int bp, int bq, Job& j, const OpDesc*& desc) {
  int bx, by;
  xcd_remap(bx, by);
  const OpDesc& d = t.descs[b.at(by)];
  desc = &d;
  const bool tc = d.p.trans_c != 0;
  j.nk = d.p.nk;
  j.gated = d.p.mode == 2;
  j.P = tc ? d.cols : d.rows;
  j.Q = tc ? d.rows : d.cols;
  const int q_out = j.gated ? bq / 2 : bq;  // output columns per workgroup
  const int nq = (j.Q + q_out - 1) / q_out;
  if (bx >= ((j.P + bp - 1) / bp) * nq) return false;
  j.p0 = (bx / nq) * bp;
  j.q0 = (bx % nq) * q_out;
  j.tiles_p = t.ptrs + __builtin_amdgcn_readfirstlane(d.ptr0 + (tc ? j.nk : 0));
  j.tiles_q = t.ptrs + __builtin_amdgcn_readfirstlane(d.ptr0 + (tc ? 0 : j.nk));
  j.ksz = t.aux + __builtin_amdgcn_readfirstlane(d.aux0);
  return true;
}

__device__ __forceinline__ int count_chunks(const Job& j) {  // an even number
  int n = 0;
  for (int k = 0; k < j.nk; ++k) n += (j.ksz[k] + kChunk - 1) / kChunk;
  return (n + 1) & ~1;
}

// Stores a wavefront's TQ x TP accumulator tiles of 16x16 as bf16.  They go through LDS of the wavefront's own, 32 P rows at a time, so that a
// store instruction writes whole runs of a row, 16 bytes per lane.  They lie there in fp32, straight from their
// registers, whatever becomes of them then: a wavefront with 256 accumulators has no others to turn them over in.  Those of the 128x128 form
// are rounded before, where nothing is left to be done to them (LDS is what bounds its epilogue).
// Against bf16 rows in LDS for every form, which left the 256x256 form 152 bytes of scratch, and element by element stores of 16 bytes
// per lane where rows are not aligned: 512x512 with K of 1024, 300 of them, 173 -> 158 us; with K of 504, 100 of them, 52 -> 46;
// 347x512 with K of 4096 stored transposed, 32 of them, 61 -> 56; 96x100 with K of 512, 300 of them, 20 -> 15.
// MODE 1: a [P, Q] bf16 tensor R is added before the rounding.  MODE 2: silu(gate) * up, every 32 gates are followed by their 32 ups.
constexpr int epilogue_pitch(int tq) { return tq * 64 + 16; }  // bytes
constexpr int epilogue_bytes(int tq) { return 32 * epilogue_pitch(tq); }
constexpr int kRounded = 3;  // a MODE
// V columns per lane (1: any row length; else rows of C are aligned to V elements)
template <int MODE, int TQ, int V>
__device__ __forceinline__ void store_rows(const char* st, bf16_t* C, int P, int Q, int prow0, int qcol0, int lane, const bf16_t* R) {
  constexpr int QW = MODE == 2 ? 8 * TQ : 16 * TQ;  // columns of the wavefront's piece
  constexpr int LPR = QW / V < 64 ? QW / V : 64, RPI = 64 / LPR;  // lanes per row, rows per store instruction
  typedef float vec __attribute__((ext_vector_type(V)));
  typedef bf16_t half_vec __attribute__((ext_vector_type(V)));
#pragma clang loop unroll_count(4)
  for (int n = 0; n < 32 / RPI; ++n) {
    const int r = n * RPI + lane / LPR, row = prow0 + r;
    const char* const from = st + r * epilogue_pitch(TQ);
#pragma unroll
    for (int half = 0; half < QW / (LPR * V); ++half) {
      const int cin = (half * LPR + lane % LPR) * V, c = qcol0 + cin;
      const size_t at = (size_t)row * Q + c;
      half_vec out;
      if constexpr (MODE == kRounded) {
        out = *(const half_vec*)(from + 2 * cin);
      } else {
        const float* const x = (const float*)from + (MODE == 2 ? (cin >> 5) * 64 + (cin & 31) : cin);
        vec v = *(const vec*)x, u = v;
        if constexpr (MODE == 2) u = *(const vec*)(x + 32);
        if constexpr (MODE == 1) {
          if (row < P && c < Q) {
            const half_vec res = *(const half_vec*)(R + at);
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] += bf2f(res[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < V; ++k) {
          if constexpr (MODE == 2) v[k] = v[k] / (1.f + __expf(-v[k])) * u[k];
          out[k] = f2bf(v[k]);
        }
      }
      if (row < P && c < Q) *(half_vec*)(C + at) = out;
    }
  }
}
template <int MODE, int TQ, int TP, int V>
__device__ __forceinline__ void store_tiles(const f32x4 (&acc)[TQ][TP], char* st, bf16_t* C, int P, int Q, int prow0, int qcol0, int lane,
                                            const bf16_t* R) {
  constexpr int PITCH = epilogue_pitch(TQ);
  char* const to = st + (lane & 15) * PITCH + (lane >> 4) * (MODE == kRounded ? 8 : 16);
#pragma unroll
  for (int h = 0; h < TP / 2; ++h) {
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int i = 0; i < TQ; ++i) {
        const f32x4 v = acc[i][2 * h + jj];
        if constexpr (MODE == kRounded) *(uint2*)(to + 16 * jj * PITCH + 32 * i) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
        else *(f32x4*)(to + 16 * jj * PITCH + 64 * i) = v;
      }
    store_rows<MODE, TQ, V>(st, C, P, Q, prow0 + 32 * h, qcol0, lane, R);
  }
}
// wp, wq: the wavefront's place in the tile
template <int TQ, int TP>
__device__ __forceinline__ void finish(const f32x4 (&acc)[TQ][TP], char* lds, const DeviceTables& t, const OpDesc& d, const Job& j, int w,
                                       int wp, int wq, int lane) {
  __syncthreads();  // nobody reads the regions any more
  char* const st = lds + w * epilogue_bytes(TQ);
  bf16_t* const C = (bf16_t*)d.out;
  const int p = j.p0 + wp * 16 * TP, q = j.q0 + wq * (j.gated ? 8 * TQ : 16 * TQ);
  const int mode = __builtin_amdgcn_readfirstlane(d.p.mode);
  const bf16_t* const R = mode == 1 ? (const bf16_t*)sload_ptr(t.ptrs + __builtin_amdgcn_readfirstlane(d.ptr0 + 2 * j.nk)) : nullptr;
  // (modes outermost: what a short product takes is the way of its instructions from memory as much as anything, and those that are
  // run lie next to each other)
  auto store = [&](auto v) __attribute__((always_inline)) {
    constexpr int V = decltype(v)::value;
    if (mode == 0) store_tiles<TQ == 4 ? kRounded : 0, TQ, TP, V>(acc, st, C, j.P, j.Q, p, q, lane, R);
    else if (mode == 1) store_tiles<1, TQ, TP, V>(acc, st, C, j.P, j.Q, p, q, lane, R);
    else store_tiles<2, TQ, TP, V>(acc, st, C, j.P, j.Q, p, q, lane, R);
  };
  if ((j.Q & 7) == 0) store(std::integral_constant<int, 8>());
  else if ((j.Q & 3) == 0) store(std::integral_constant<int, 4>());
  else store(std::integral_constant<int, 1>());
}

// ---------------------------------------------------------------------------------------------
// 256x256 per workgroup.  A chunk is multiplied in four quarters, 64x64 of the wavefront's tile over 64 of K; halves of the operands stay
// in registers for the two quarters that need them, and each quarter reads the one region that a later one needs:
//   even chunks: P0 Q0, P0 Q1, P1 Q1, P1 Q0, reading Q1, P1, then P0 and Q1 of the next chunk;
//   odd chunks:  P0 Q1, P0 Q0, P1 Q0, P1 Q1, reading Q0, P1, then P0 and Q0 of the next chunk.
// So the regions of a chunk are read, and loaded, in the order P0 Q0 Q1 P1 or P0 Q1 Q0 P1, and with a ring of eight
// a load has seven quarters, 3600 cycles, to arrive.  One barrier per quarter publishes the region to be read and
// frees the one read in the quarter before.
// ---------------------------------------------------------------------------------------------
constexpr int kRing256 = 8;
constexpr uint32_t kLds256 = kRing256 * kRegionBytes;

__global__ void __launch_bounds__(256, 1) gemm_bf16_256_kernel(DeviceTables t, Batch b) {
  constexpr int NS = kRing256;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  Job job;
  const OpDesc* desc;
  if (!find_job(t, b, 256, 256, job, desc)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wp = w >> 1, wq = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  f32x4 acc[8][8];  // [q][p]
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const int total = 4 * count_chunks(job);  // regions
  Source<2, 2> src;
  src.start(job, w, lane);
  const uint32_t ldsw = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lptr_t)lds + w * 1024);
  uint32_t dst = ldsw;  // where the next region goes
  int issued = 0;       // regions whose loads have been issued
  // operand and half of the region at position POS (0..3) of an even or odd chunk
#define TN_IS_P(POS) ((POS) == 0 || (POS) == 3)
#define TN_HALF(ODD, POS) ((POS) == 0 ? 0 : (POS) == 3 ? 1 : (((POS) == 2) != (ODD)) ? 1 : 0)
  // the arguments of the load of piece I of that region
#define TN_PIECE(ODD, POS, I)                                                                                     \
  (TN_IS_P(POS) ? src.off_p[TN_HALF(ODD, POS)][I] : src.off_q[TN_HALF(ODD, POS)][I]),                             \
      (TN_IS_P(POS) ? src.rp : ((I) & 1) ? src.rq2 : src.rq), src.at, dst, (I) * 4096
#define TN_LOAD_REGION(ODD, POS)          \
  do {                                    \
    load_lds(TN_PIECE(ODD, POS, 0));      \
    load_lds(TN_PIECE(ODD, POS, 1));      \
    load_lds(TN_PIECE(ODD, POS, 2));      \
    load_lds(TN_PIECE(ODD, POS, 3));      \
  } while (0)
#define TN_NEXT_REGION(POS)                                                               \
  do {                                                                                    \
    dst = dst + kRegionBytes == ldsw + NS * kRegionBytes ? ldsw : dst + kRegionBytes;     \
    ++issued;                                                                             \
    if ((POS) == 3) src.advance(job, w, lane);                                            \
  } while (0)
  // fragments: 16 rows of the wavefront's 64 in a region, piece 4 s + g of their K
  uint32_t col[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) col[s] = l16 * 128 + (((4 * s + g) ^ (l16 & 7)) * 16);
  const uint32_t base_p = wp * 64 * 128, base_q = wq * 64 * 128;
  uint32_t get = 0;                 // the region to be read next
  bf16x8 fp[2][4][2], fq[2][4][2];  // [half][fragment][slab]
#define TN_READ(DST, BASE, F, S) DST[F][S] = *(const bf16x8*)(lds + get + BASE + col[S] + (F) * 2048)
#define TN_READ_REGION(DST, BASE)                                                                                 \
  do {                                                                                                            \
    _Pragma("unroll") for (int s_ = 0; s_ < 2; ++s_)                                                              \
        _Pragma("unroll") for (int f_ = 0; f_ < 4; ++f_) TN_READ(DST, BASE, f_, s_);                              \
    get = get + kRegionBytes == NS * kRegionBytes ? 0 : get + kRegionBytes;                                       \
  } while (0)

  if (total > 0) {
    // fill the ring (two chunks), read the first two regions, and refill the first
#define TN_FIRST(R)                                 \
  TN_LOAD_REGION((((R) >> 2) & 1) != 0, (R) & 3);   \
  TN_NEXT_REGION((R) & 3);
    TN_FIRST(0) TN_FIRST(1) TN_FIRST(2) TN_FIRST(3) TN_FIRST(4) TN_FIRST(5) TN_FIRST(6) TN_FIRST(7)
#undef TN_FIRST
    wait_loads<kPieceLoads * (NS - 2)>();
    barrier();
    TN_READ_REGION(fp[0], base_p);
    TN_READ_REGION(fq[0], base_q);
    wait_loads<kPieceLoads * (NS - 2)>();
    barrier();
    if (issued < total) {
      TN_LOAD_REGION(false, 0);
      TN_NEXT_REGION(0);
    }
    int done = 2;  // regions read
    // One quarter; reads region `done`, loads region done + NS - 1, which is at position LPOS of an (odd: LODD) chunk.  STEADY: there is
    // such a region.  Four loads and eight reads between 32 MFMAs.
#define TN_QUARTER(HP, HQ, RD, BASE, LODD, LPOS)                                                                  \
  do {                                                                                                            \
    const int behind_ = issued - done - 1; /* regions behind the one to be read that may be on their way */       \
    if (STEADY || behind_ >= NS - 2) wait_loads<kPieceLoads * (NS - 2)>();                                        \
    else if (behind_ >= 4) wait_loads<kPieceLoads * 4>();                                                         \
    else if (behind_ >= 2) wait_loads<kPieceLoads * 2>();                                                         \
    else wait_loads<0>();                                                                                         \
    barrier();                                                                                                    \
    const bool more_ = STEADY || issued < total;                                                                  \
    if (!STEADY && more_) TN_LOAD_REGION(LODD, LPOS);                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                                            \
    _Pragma("unroll") for (int n_ = 0; n_ < 32; ++n_) {                                                           \
      const int s_ = n_ >> 4, i_ = (n_ >> 2) & 3, j_ = (i_ & 1) ? 3 - (n_ & 3) : (n_ & 3);                        \
      f32x4& c_ = acc[4 * (HQ) + i_][4 * (HP) + j_];                                                              \
      if (STEADY && n_ == 3) mfma_then_load(c_, fq[HQ][i_][s_], fp[HP][j_][s_], TN_PIECE(LODD, LPOS, 0));         \
      else if (STEADY && n_ == 11) mfma_then_load(c_, fq[HQ][i_][s_], fp[HP][j_][s_], TN_PIECE(LODD, LPOS, 1));   \
      else if (STEADY && n_ == 19) mfma_then_load(c_, fq[HQ][i_][s_], fp[HP][j_][s_], TN_PIECE(LODD, LPOS, 2));   \
      else if (STEADY && n_ == 27) mfma_then_load(c_, fq[HQ][i_][s_], fp[HP][j_][s_], TN_PIECE(LODD, LPOS, 3));   \
      else mfma(c_, fq[HQ][i_][s_], fp[HP][j_][s_]);                                                              \
      __builtin_amdgcn_sched_barrier(0);                                                                          \
      if (n_ < 16 && !(n_ & 1)) TN_READ(RD, BASE, (n_ >> 1) & 3, n_ >> 3);                                        \
      __builtin_amdgcn_sched_barrier(0);                                                                          \
    }                                                                                                             \
    get = get + kRegionBytes == NS * kRegionBytes ? 0 : get + kRegionBytes;                                       \
    ++done;                                                                                                       \
    if (more_) TN_NEXT_REGION(LPOS);                                                                              \
  } while (0)
    static_assert(NS == 8, "the positions below: region done + 7, one place further on in the same or the next chunk");
    auto two_chunks = [&](auto steady) __attribute__((always_inline)) {
      constexpr bool STEADY = decltype(steady)::value;
      TN_QUARTER(0, 0, fq[1], base_q, false, 1);
      TN_QUARTER(0, 1, fp[1], base_p, false, 2);
      TN_QUARTER(1, 1, fp[0], base_p, false, 3);
      TN_QUARTER(1, 0, fq[1], base_q, true, 0);
      TN_QUARTER(0, 1, fq[0], base_q, true, 1);
      TN_QUARTER(0, 0, fp[1], base_p, true, 2);
      TN_QUARTER(1, 0, fp[0], base_p, true, 3);
      TN_QUARTER(1, 1, fq[0], base_q, false, 0);
    };
    // (the loops end in the wait: where paths meet, the compiler moves accumulators)
    int r = 0;
    if (8 + NS < total)
      for (;;) {
        two_chunks(std::integral_constant<bool, true>());
        r += 8;
        if (r + 8 + NS < total) continue;
        mfma_drain(acc);
        break;
      }
    for (;;) {
      two_chunks(std::integral_constant<bool, false>());
      r += 8;
      if (r < total) continue;
      mfma_drain(acc);
      break;
    }
  }
#undef TN_QUARTER
#undef TN_READ_REGION
#undef TN_READ
#undef TN_NEXT_REGION
#undef TN_LOAD_REGION
#undef TN_PIECE
#undef TN_HALF
#undef TN_IS_P
  static_assert(4 * epilogue_bytes(8) <= (int)kLds256, "the rows of the epilogue fit the ring");
  finish<8, 8>(acc, lds, t, *desc, job, w, wp, wq, lane);
}

// ---------------------------------------------------------------------------------------------
// 128x128 per workgroup: every wavefront has 64x64.  A chunk's fragments are read while the chunk before is multiplied, into a second
// set of registers, with one barrier per chunk and a ring of NC chunks.  96 KiB go through LDS per chunk and 512 cycles of MFMAs: twice
// the bytes per product of the larger form.
// NC = 4: 128 KiB, one workgroup per CU, for launches of at most 256 workgroups: loads have three chunks to arrive, 680 cycles
// each (256 workgroups, K of 4096 and 8192: 60 and 103 thousand cycles).  (320 rows x 4096 with K of 11008, 96 workgroups: 65 to 68 us; the
// register-staged 128x128 kernel it replaced 93.)
// NC = 2: 64 KiB, two workgroups per CU hide each other's waits, 580 cycles per chunk, for larger launches (1371 x 4096 with K of 11008, 352
// workgroups: 138 us, 153 with NC = 4; 688 workgroups with K of 2048: 57 and 67; but 96 workgroups with K of 11008: 100 and 65).
// A form with 256x128 per workgroup measured within 3 % of NC = 2 wherever that is the fastest and is not kept.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kChunkBytes = 2 * kRegionBytes;  // P region, then the Q region

template <int NC>
__global__ void __launch_bounds__(256, NC == 2 ? 2 : 1) gemm_bf16_128_kernel(DeviceTables t, Batch b) {
  constexpr int LOADS = 2 * kPieceLoads, READS = 16;
  constexpr uint32_t CB = kChunkBytes;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  Job job;
  const OpDesc* desc;
  if (!find_job(t, b, 128, 128, job, desc)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wp = w >> 1, wq = w & 1;
  const int l16 = lane & 15, g = lane >> 4;
  f32x4 acc[4][4];  // [q][p]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const int total = count_chunks(job);
  Source<1, 1> src;
  src.start(job, w, lane);
  const uint32_t ldsw = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lptr_t)lds + w * 1024);
  uint32_t dst = ldsw;  // where the next chunk goes
  int issued = 0;       // chunks whose loads have been issued
  // load I of a chunk: four pieces of each region
#define TN_PIECE(I)                                                                 \
  ((I) < 4 ? src.off_p[0][(I) & 3] : src.off_q[0][(I) & 3]),                        \
      ((I) < 4 ? src.rp : ((I) & 1) ? src.rq2 : src.rq), src.at, dst, (I) * 4096
  auto next_chunk = [&]() __attribute__((always_inline)) {
    dst = dst + CB == ldsw + NC * CB ? ldsw : dst + CB;
    ++issued;
    src.advance(job, w, lane);
  };
  auto load_chunk = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) load_lds(TN_PIECE(i));
  };
  uint32_t col[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) col[s] = l16 * 128 + (((4 * s + g) ^ (l16 & 7)) * 16);
  const uint32_t base_p = wp * 64 * 128, base_q = kRegionBytes + wq * 64 * 128;
  uint32_t get = 0;  // the chunk to be read next
  bf16x8 xp[4][2], xq[4][2], yp[4][2], yq[4][2];  // [fragment][slab]
  auto read = [&](bf16x8 (&p)[4][2], bf16x8 (&q)[4][2], int r) __attribute__((always_inline)) {  // in the order in which they are multiplied
    const int s = r >> 3, f = r & 3;
    if (r & 4) p[f][s] = *(const bf16x8*)(lds + get + base_p + col[s] + f * 2048);
    else q[f][s] = *(const bf16x8*)(lds + get + base_q + col[s] + f * 2048);
  };
  auto next_get = [&]() __attribute__((always_inline)) { get = get + CB == NC * CB ? 0 : get + CB; };

  if (total > 0) {
    // (one copy of it: what a short product takes is the way of its instructions from memory as much as that of its operands.  128x128
    // with K of 128, 256 and 1024 of them 7.5 -> 6.4 and 18.5 -> 14.9 us against the unrolled form and element stores)
#pragma clang loop unroll(disable)
    for (int c = 0; c < NC && c < total; ++c) {
      load_chunk();
      next_chunk();
    }
    if (total >= NC) wait_loads<LOADS * (NC - 1)>();
    else wait_loads<0>();
    barrier();
#pragma unroll
    for (int r = 0; r < READS; ++r) read(xp, xq, r);
    next_get();
    int done = 1;  // chunks read
    // multiplies a chunk from (ap, aq), reads the next one into (np, nq) and, STEADY, loads the one NC chunks on
    auto chunk = [&](auto steady, bf16x8 (&ap)[4][2], bf16x8 (&aq)[4][2], bf16x8 (&np)[4][2], bf16x8 (&nq)[4][2])
                     __attribute__((always_inline)) {
      constexpr bool STEADY = decltype(steady)::value;
      const int behind = issued - done - 1;  // chunks behind the one to be read that may be on their way
      if (STEADY || behind >= NC - 2) wait_loads<LOADS * (NC - 2)>();
      else if (NC > 3 && behind >= 1) wait_loads<LOADS>();
      else wait_loads<0>();
      barrier();
      const bool more = STEADY || issued < total;
      if (!STEADY && more) load_chunk();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < 32; ++n) {  // 16 reads and eight loads between 32 MFMAs
        const int s = n >> 4, i = (n >> 2) & 3, j = (i & 1) ? 3 - (n & 3) : (n & 3);
        if (STEADY && (n & 3) == 1) mfma_then_load(acc[i][j], aq[i][s], ap[j][s], TN_PIECE(n >> 2));
        else mfma(acc[i][j], aq[i][s], ap[j][s]);
        __builtin_amdgcn_sched_barrier(0);
        if (!(n & 1)) read(np, nq, n >> 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      next_get();
      ++done;
      if (more) next_chunk();
    };
    int c = 0;
    if (2 + NC <= total)
      for (;;) {
        chunk(std::integral_constant<bool, true>(), xp, xq, yp, yq);
        chunk(std::integral_constant<bool, true>(), yp, yq, xp, xq);
        c += 2;
        if (c + 2 + NC <= total) continue;
        mfma_drain(acc);
        break;
      }
    for (;;) {  // (at least two chunks are left: the ring holds as many)
      chunk(std::integral_constant<bool, false>(), xp, xq, yp, yq);
      chunk(std::integral_constant<bool, false>(), yp, yq, xp, xq);
      c += 2;
      if (c < total) continue;
      mfma_drain(acc);
      break;
    }
  }
#undef TN_PIECE
  static_assert(4 * epilogue_bytes(4) <= (int)(NC * CB), "the rows of the epilogue fit the ring");
  finish<4, 4>(acc, lds, t, *desc, job, w, wp, wq, lane);
}

}  // namespace

hipError_t launch_gemm_bf16(int form, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t s) {
  const dim3 grid((unsigned)max_blocks, (unsigned)b.n), wg(256);
#define TN_LAUNCH_GEMM(KERNEL, LDS)                                                                                             \
  do {                                                                                                                          \
    static std::atomic<uint64_t> allowed{0};                                                                                    \
    if (const hipError_t e = allow_lds(allowed, (const void*)KERNEL, (LDS)); e != hipSuccess) return e;                         \
    hipLaunchKernelGGL(KERNEL, grid, wg, (LDS), s, t, b);                                                                       \
  } while (0)
  switch (form) {
    case LC_GEMM_BF16: TN_LAUNCH_GEMM(gemm_bf16_256_kernel, kLds256); break;
    case LC_GEMM_BF16_128: TN_LAUNCH_GEMM(gemm_bf16_128_kernel<4>, 4 * kChunkBytes); break;
    case LC_GEMM_BF16_PAIRED: TN_LAUNCH_GEMM(gemm_bf16_128_kernel<2>, 2 * kChunkBytes); break;
    default: return hipErrorInvalidValue;
  }
#undef TN_LAUNCH_GEMM
  return hipGetLastError();
}

}  // namespace tn
