// Argument records and launch factories of the gfx950 kernel library (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <cstdint>
#include <vector>

namespace psc {

struct GemmArgs {           // C (M x N) = alpha * A (M x K) * B (K x N), row-major, leading dims
  const void *A;
  const void *B;
  void *C;
  int64_t lda, ldb, ldc;    // in elements
  int32_t M, N, K;
  float alpha;
  int32_t tiles_n;          // filled by make_gemm
  int32_t pad;
  // a launch of several kernels (group_launch), here and in the records below: block b of the
  // grid runs block map[b] % 65536 of kernel map[b] / 65536 of the list; map = nullptr otherwise
  const uint32_t *map;
  const GemmArgs *list;
};

struct SoftmaxArgs {        // Y (R x C) = row-softmax(X)
  const void *X;
  void *Y;
  int64_t ldx, ldy;
  int32_t R, C;
  const uint32_t *map;
  const SoftmaxArgs *list;
};

struct TransArgs {          // B (C x R) = A (R x C)^T
  const void *A;
  void *B;
  int64_t lda, ldb;
  int32_t R, C;
  const uint32_t *map;
  const TransArgs *list;
};

struct AddArgs {            // Cp (R x C) = A + B
  const void *A;
  const void *B;
  void *Cp;
  int64_t lda, ldb, ldc;
  int32_t R, C;
  uint32_t inv, unused;     // inv: 2^32 over the units of a row (make_add)
  const uint32_t *map;
  const AddArgs *list;
};

// A prepared kernel launch: hipLaunchKernel(func, grid, block, {args}, shmem, stream).
struct Launch {
  const void *func = nullptr;
  dim3 grid, block;
  unsigned shmem = 0;
  bool empty = false;       // nothing to compute (an empty operand): skip the launch
  int tile = 0;             // GEMM tile configuration used
  int kind = -1;            // psc_kind of a kernel of the DAG, -1 for marks and fills
  alignas(16) unsigned char args[96];
};

// dtype codes: 0 = f32, 1 = bf16
bool make_gemm(Launch &L, GemmArgs a, int ab_dtype, int c_dtype, int tile);
bool make_softmax(Launch &L, SoftmaxArgs a, int in_dtype, int out_dtype);
bool make_transpose(Launch &L, TransArgs a, int dtype, int tile = 0);
bool make_add(Launch &L, AddArgs a, int in_dtype, int out_dtype);
int gemm_num_tiles();

// Whether a launch may run together with others of the same kernel function: not one that is
// empty, that fills the GPU several times over by itself, or whose block order needs its grid.
bool groupable(const Launch &L);
// Bytes of the table a launch of these kernels needs in device memory (16-byte multiple), its
// host image, and the launch itself, with the table at `dev` (16-byte aligned).  All members have
// one kernel function.
size_t group_table_bytes(const std::vector<Launch> &members);
Launch group_launch(const std::vector<Launch> &members, void *host_image, void *dev);
// The tile for a launch of several GEMMs whose tile is automatic: `tile` is what one of them
// takes alone.  Only tiles that sum K in the same order are considered, so the results do not
// depend on what a kernel is launched with.  gemm_sum_order: equal for tiles of one order.
int gemm_group_tile(const std::vector<GemmArgs> &args, int tile);
int gemm_sum_order(int tile);
// One-thread kernel that stores the device wall clock (wall_clock64) to *slot.
void make_mark(Launch &L, uint64_t *slot);
// Fills bytes / 4 32-bit words at p with values uniform in [-1, 1) from a hash of (index, seed):
// one FP32 value per word, or (bf16) two bfloat16 values.  Timing operands for the autotuner
// (the matrix cores' power, and with it the clock, depends on the data).
void make_fill(Launch &L, void *p, int64_t bytes, int bf16, uint32_t seed);
// The tile cache keeps two choices per shape: for a launch of one kernel and for one of several.
enum class TileUse { alone, shared, both };
void tile_cache_set(int M, int N, int K, int ab, int c, int tile, TileUse use);  // tile 0: none
int tile_cache_get(int M, int N, int K, int ab, int c, TileUse use);             // alone or shared
void tile_cache_clear();
size_t tile_cache_size();
std::vector<std::array<int, 7>> tile_cache_entries();  // (M, N, K, operand dtype, output dtype, alone, shared)
int gemm_auto_tile(int M, int N, int K, int dtype);

}  // namespace psc
