// Interface between the executor (host) and the gfx950 task kernels.
//
// Every kernel is *grouped*: one launch serves a batch of ready memgraph vertices of the same
// launch class.  Because a memgraph fixes the GPU location of every tensor before execution
// (Section 5, first paragraph), the per-vertex operand tables can be built once, at executor
// creation, and stay in device memory; a launch only names the vertices it covers.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "turnip.h"

namespace tn {

// One kernel-call vertex, as the kernels see it.
struct OpDesc {
  void* out;        // device address of the output tensor
  uint32_t ptr0;    // index of the first operand address in the pointer table
  uint32_t aux0;    // index of the first auxiliary integer (meaning depends on the kind)
  int32_t rows, cols;  // output shape
  int32_t n_in;
  int32_t nblocks;  // workgroups this vertex needs in its launch class
  int32_t dtype;    // storage type of its non-statistics operands (TN_F32 / TN_BF16)
  int32_t trans_b;  // gemm: B tiles are stored [cols, K]
  tn_op_params p;
};

// Lets `kernel` be launched with `bytes` of dynamic LDS on the current GPU, where that is more than 64 KiB: a GPU is told of it
// once per kernel (done: a bit for each GPU).
inline hipError_t allow_lds(std::atomic<uint64_t>& done, const void* kernel, int bytes) {
  int dev = -1;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Launch classes: vertices of one class can share a launch.
enum LaunchClass {
  LC_GEMM_F32 = 0,   // GEMM with fp32 products, any layout, fp32 or bf16 storage
  LC_GEMM_BF16_SMALL,  // MFMA bf16 GEMM for small or thin products, B tiles stored [cols, K], 32x32 tile per workgroup
  LC_GEMM_ROWS,      // single-row products, either type (see launch_gemm_rows)
  LC_GEMM_BF16_128,  // MFMA bf16 GEMM, B tiles stored [cols, K], 128x128 tile per workgroup
  LC_GEMM_BF16,      // the same for outputs of at least 256x256: 256x256 or 128x128 per workgroup
  LC_RMS_STAT,
  LC_RMS_APPLY,
  LC_ROPE,
  LC_ATTN_F32,       // attention block with fp32 products (fp32 storage, or shapes the bf16 kernel does not take)
  LC_ATTN_BF16,      // MFMA attention block
  LC_ATTN_COMBINE,
  LC_SILU_MUL,
  LC_ADD,
  LC_SILU_BWD,
  LC_RMS_BWD_STAT,
  LC_RMS_BWD_APPLY,
  LC_ATTN_BWD,       // attention backward with fp32 products (statistics, dQ, dK, dV)
  LC_ATTN_BWD_BF16,  // MFMA attention backward: statistics; the next three values are its dQ, dK and dV forms
  LC_ATTN_BWD_BF16_DQ,
  LC_ATTN_BWD_BF16_DK,
  LC_ATTN_BWD_BF16_DV,
  LC_TRANSPOSE,
  LC_ZERO,           // clears a tensor: the start of a sum's output
  LC_SOFTMAX_STAT,   // row maximum and sum of exponentials over the score tiles of a row block
  LC_SOFTMAX_APPLY,  // probabilities of one score tile
  LC_COUNT,
  // Not a class of its own for grouping: 128x128 tiles with two workgroups per CU, a form for launches of either of the two above.
  LC_GEMM_BF16_PAIRED
};

// Vertices per launch.  The list travels in the kernel arguments (4 KiB at most), as 16-bit
// offsets from the smallest descriptor index of the group.
constexpr int kMaxBatch = 1920;
constexpr uint32_t kMaxBatchSpan = 65535;  // largest descriptor index distance inside one group

struct Batch {
  int32_t n;
  uint32_t base;            // smallest descriptor index of the group
  int32_t stages;           // products of gemm_small.hip: pieces along K that a wavefront holds in LDS
  uint16_t idx[kMaxBatch];  // descriptor index minus base
  __host__ __device__ uint32_t at(uint32_t i) const { return base + idx[i]; }
};

struct DeviceTables {
  const OpDesc* descs;
  void* const* ptrs;
  const int32_t* aux;
  const double* rope_theta;  // base^(-2i/head_dim), i < head_dim/2, for the graph's rotary vertices
};

// A group of tensor copies between GPU memory and pinned (device-visible) host memory, moved by
// one kernel launch: offloads, reloads, loads and stores of the memgraph.  The copy routine of
// the runtime spends a launch and a gap per tensor, which at tile sizes of a few hundred KiB
// leaves half of the host link idle.
constexpr int kMaxCopies = 128;
constexpr int kCopyThreads = 1024;
constexpr int kCopyLoads = 2;  // 16-byte loads in flight per lane
constexpr uint32_t kCopyBlockBytes = kCopyLoads * 16 * kCopyThreads;  // bytes one workgroup moves per step: 32 KiB
constexpr int kDefaultCopyWorkgroups = 8;
constexpr int kDeviceCopyThreads = 512;  // copies that stay inside GPU memory
constexpr int kDeviceCopyPieces = 1024;  // workgroups per tensor at most
struct CopyItem {
  const void* src;
  void* dst;
  uint32_t bytes;
  uint32_t first_block;  // index of its first 32 KiB piece among the pieces of the group
};
struct CopyBatch {
  int32_t n;
  int32_t total_blocks;
  CopyItem it[kMaxCopies];
};
// max_workgroups <= 0 selects kDefaultCopyWorkgroups
hipError_t launch_copies(const CopyBatch& b, int max_workgroups, hipStream_t stream);
// every source and destination in memory of this GPU, 16-byte aligned
hipError_t launch_device_copies(const CopyBatch& b, hipStream_t stream);

// A region of GPU memory that exists from the moment the library is loaded until the process ends,
// for callers that want the operand tables of a run somewhere nobody has to allocate.  Each GPU
// holds its own copy of the region at its own address; *ptr receives the address on the current
// device (looked up once per device).  Contents are whatever the last user left there.
constexpr size_t kStaticTableBytes = 8u << 20;
hipError_t static_table_region(void** ptr);

// Workgroups a vertex needs in the given class (host side, used to fill OpDesc::nblocks).
int32_t blocks_for(int cls, const OpDesc& d, const int32_t* aux);

// Enqueues one grouped launch on `stream`.  All vertices of the batch share the class, the storage
// type and (for attention) the head size.  max_blocks = largest nblocks in the batch.
hipError_t launch_batch(int cls, int dtype, int head_dim, const DeviceTables& t, const Batch& b,
                        int32_t max_blocks, hipStream_t stream);

// The three forms of bf16 tile products: gemm_bf16.hip.  The bits of a product do not depend on the form.
inline int32_t gemm_blocks(int tile, const OpDesc& d) {  // workgroups for output tiles of tile x tile
  const int q = d.p.mode == 2 ? tile / 2 : tile;         // gate and up products take half a tile's columns each
  return (int32_t)(((int64_t)d.rows + tile - 1) / tile * (((int64_t)d.cols + q - 1) / q));
}
constexpr int32_t kGemmBf16MaxK = (1 << 23) - 8;  // their offsets from a workgroup's first row hold 256 rows of a tile that is no deeper
hipError_t launch_gemm_bf16(int form, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t stream);

// LC_GEMM_F32 and LC_GEMM_BF16_SMALL: gemm_small.hip.
constexpr int kGemmSmallTile = 32;  // output rows and columns per workgroup
constexpr int kGemmSmallWaves = 4;  // wavefronts per workgroup, which share its pieces along K
constexpr int kGemmSmallStages = 4; // pieces of a wavefront in LDS, at most
constexpr int kGemmRowsTable = 64;  // LC_GEMM_ROWS: K tiles whose addresses are held in LDS
// The stages a vertex of these classes or of LC_GEMM_ROWS uses (ksz: the depths of its K tiles); a launch takes its largest.  What a
// short product has no use for would only keep other workgroups off the CU: fp32, 64 of 256x256 with K of 128 53 -> 36 us; bf16, 256 of 64x64
// with K of 256 14.1 -> 8.4; single rows, 4 against each of 64 B tiles of 512 with K of 512 20.8 -> 14.4; rows not aligned to four elements
// (no stages), 64 of 128x128 with K of 1022 110 -> 96.
// The layouts that go by registers hold no stages but are given their room: two workgroups on a CU push one another's
// lines out of L1 (fp32, B stored [K, N], 192 of 64x64 with K of 704 26.8 us, 33.4 without the room; 64 of 256x256 with K of 1024 147 and 132).
inline int32_t gemm_small_stages(int cls, const OpDesc& d, const int32_t* ksz) {
  const bool b16 = cls == LC_GEMM_BF16_SMALL || (cls == LC_GEMM_ROWS && d.dtype == TN_BF16);
  if (cls == LC_GEMM_ROWS ? d.p.nk > kGemmRowsTable : !b16 && d.dtype != TN_F32) return 0;
  const int vec = b16 ? 8 : 4;
  const bool vectors = b16 || !d.p.trans_a || d.trans_b;  // as `pieces` in `product` counts them
  int64_t pieces = 0;
  for (int k = 0; k < d.p.nk; ++k) pieces += vectors && ksz[k] % vec ? 0 : ksz[k] / (8 * vec);
  return (int32_t)(pieces < kGemmSmallWaves * kGemmSmallStages ? (pieces + kGemmSmallWaves - 1) / kGemmSmallWaves : kGemmSmallStages);
}
hipError_t launch_gemm_small(bool bf16_products, int dtype, const DeviceTables& t, const Batch& b, int32_t max_blocks, hipStream_t stream);

// LC_GEMM_ROWS: products of a single row whose B tiles are stored [cols, K], with rows along K aligned to 16 bytes.
// Vertices with one key multiply the same B tiles; those that stand next to each other in the list are formed
// together, B read once.  (A row's bits do not depend on its company.)  base: the smallest descriptor index of the list.
struct RowVertex {
  int32_t key;
  uint32_t desc;
  int32_t stages;
};
hipError_t launch_gemm_rows(int dtype, const DeviceTables& t, uint32_t base, const RowVertex* rows, int n, int32_t max_blocks,
                            hipStream_t stream);

// LC_ATTN_F32 (reverse == false) and LC_ATTN_BWD: attn_f32.hip.
hipError_t launch_attn_f32(bool reverse, int dtype, int head_dim, const DeviceTables& t, const Batch& b, int32_t max_blocks,
                           hipStream_t stream);

}  // namespace tn
