// Standalone gfx950 kernels of the DAG (one tile function call per block; the tile functions live
// in tiles.hpp) and the launch factories that pick a kernel instance for a problem and fill a
// Launch record that the runtime passes to hipLaunchKernel.
#include <array>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "tiles.hpp"

namespace psc {

// Tile choices measured by the autotuner or set by the user, keyed by (M, N, K, operand dtype,
// output dtype).  The choice for a launch of one kernel, which the automatic choice of make_gemm
// consults first, is kept apart from the one for a launch of several: kernels that share a launch
// fill the GPU together, with tiles that leave most of it idle under one of them (1024 x 64 x 1024
// BF16, sixteen to a launch: tile 6, alone 7.8 us on sixteen blocks against 3.8 us).
namespace {
std::mutex g_tile_mu;
struct TileChoice {
  int alone = 0, shared = 0;  // 0 = none
};
std::map<std::tuple<int, int, int, int, int>, TileChoice> g_tile_cache;
}  // namespace

void tile_cache_set(int M, int N, int K, int ab, int c, int tile, TileUse use) {
  std::lock_guard<std::mutex> lk(g_tile_mu);
  TileChoice &t = g_tile_cache[{M, N, K, ab, c}];
  tile = std::max(tile, 0);
  if (use != TileUse::shared) t.alone = tile;
  if (use != TileUse::alone) t.shared = tile;
  if (!t.alone && !t.shared) g_tile_cache.erase({M, N, K, ab, c});
}

int tile_cache_get(int M, int N, int K, int ab, int c, TileUse use) {
  std::lock_guard<std::mutex> lk(g_tile_mu);
  auto it = g_tile_cache.find({M, N, K, ab, c});
  if (it == g_tile_cache.end()) return 0;
  return use == TileUse::shared ? it->second.shared : it->second.alone;
}

void tile_cache_clear() {
  std::lock_guard<std::mutex> lk(g_tile_mu);
  g_tile_cache.clear();
}

size_t tile_cache_size() {
  std::lock_guard<std::mutex> lk(g_tile_mu);
  return g_tile_cache.size();
}

std::vector<std::array<int, 7>> tile_cache_entries() {
  std::lock_guard<std::mutex> lk(g_tile_mu);
  std::vector<std::array<int, 7>> out;
  for (const auto &kv : g_tile_cache) {
    const auto &k = kv.first;
    out.push_back({std::get<0>(k), std::get<1>(k), std::get<2>(k), std::get<3>(k), std::get<4>(k), kv.second.alone,
                   kv.second.shared});
  }
  return out;
}

// ---------------------------------------------------------------------------------------------
// Standalone kernels: one tile function call per 256-thread block.  A launch of several kernels
// (group_launch) finds its block's kernel in the table: two scalar loads, one after the other,
// before the block starts (~1 us, paid once per launch instead of a dispatch per kernel).
// A launch of one kernel reads its whole record before it looks at `map`: left to itself the compiler
// reads `map` first and the rest behind the branch, a memory round trip more for every launch.
// Measured: 64 x 64 x 64 FP32 2.98 -> 2.8 us, 512 x 64 x 512 BF16 2.96 -> 2.8 us (2.72, 2.73 without
// the table).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void read_all(GemmArgs &p) {
  asm volatile("" : "+s"(p.A), "+s"(p.B), "+s"(p.C), "+s"(p.lda), "+s"(p.ldb), "+s"(p.ldc), "+s"(p.M), "+s"(p.N),
               "+s"(p.K), "+s"(p.alpha), "+s"(p.tiles_n));
}
__device__ __forceinline__ void read_all(SoftmaxArgs &p) {
  asm volatile("" : "+s"(p.X), "+s"(p.Y), "+s"(p.ldx), "+s"(p.ldy), "+s"(p.R), "+s"(p.C));
}
__device__ __forceinline__ void read_all(TransArgs &p) {
  asm volatile("" : "+s"(p.A), "+s"(p.B), "+s"(p.lda), "+s"(p.ldb), "+s"(p.R), "+s"(p.C));
}
__device__ __forceinline__ void read_all(AddArgs &p) {
  asm volatile("" : "+s"(p.A), "+s"(p.B), "+s"(p.Cp), "+s"(p.lda), "+s"(p.ldb), "+s"(p.ldc), "+s"(p.R), "+s"(p.C),
               "+s"(p.inv));
}

#define PSC_CONSTANT __attribute__((address_space(4)))
template <typename Args>
__device__ __forceinline__ int member_block(Args &p, int b) {
  static_assert(sizeof(Args) % 8 == 0, "copied as 8-byte words");
  read_all(p);
  if (!p.map) return b;
  // the table does not change while a kernel runs: constant memory, read by scalar loads
  const uint32_t m = ((const PSC_CONSTANT uint32_t *)p.map)[b];
  const auto *rec = (const PSC_CONSTANT uint64_t *)(p.list + (m >> 16));
  uint64_t w[sizeof(Args) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(Args) / 8; ++i) w[i] = rec[i];
  __builtin_memcpy(&p, w, sizeof(Args));
  return int(m & 0xffffu);
}

template <int BM, int BN, int BK, int WM, int WN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_f32_smem<BM, BN, BK>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_f32_tile<BM, BN, BK, WM, WN, OUT_BF16>(p, bid, smem);
}

template <int BM, int BN, int BK, int WM, int WN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_bf16_smem<BM, BN, BK>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_bf16_tile<BM, BN, BK, WM, WN, OUT_BF16>(p, bid, smem);
}

template <int TM, int TN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_f32_splitk_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_f32_splitk_smem<TM, TN>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_f32_splitk_tile<TM, TN, OUT_BF16>(p, bid, smem);
}

template <int TM, int TN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_bf16_splitk_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_bf16_splitk_smem<TM, TN>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_bf16_splitk_tile<TM, TN, OUT_BF16>(p, bid, smem);
}

template <int TM, int TN, int D, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_bf16_deep_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_bf16_deep_smem<TM, TN, D>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_bf16_deep_tile<TM, TN, D, OUT_BF16>(p, bid, smem);
}

template <bool OUT_BF16>
__global__ __launch_bounds__(512) void gemm_bf16_big_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_bf16_big_smem()];
  // 4-row groups of tiles per XCD (measured 1-3% faster than plain rows at 4096^3 and 8192^3)
  gemm_bf16_big_tile<OUT_BF16>(p, group_tile(xcd_tile(blockIdx.x, gridDim.x), gridDim.x / p.tiles_n, p.tiles_n, 4), smem);
}

template <int WN, bool OUT_BF16>
__global__ __launch_bounds__(128 * WN) void gemm_bf16_w4_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_bf16_w4_smem()];
  gemm_bf16_w4_tile<WN, OUT_BF16>(p, group_tile(xcd_tile(blockIdx.x, gridDim.x), gridDim.x / p.tiles_n, p.tiles_n, 4), smem);
}

template <int FN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_f32_direct_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_direct_smem<FN, false>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_direct_tile<FN, false, OUT_BF16>(p, bid, smem);
}

template <int FN, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_bf16_direct_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[gemm_direct_smem<FN, true>()];
  const int bid = member_block(p, xcd_tile(blockIdx.x, gridDim.x));
  gemm_direct_tile<FN, true, OUT_BF16>(p, bid, smem);
}

template <int NV, bool IN_BF16, bool OUT_BF16, bool NT = false, int CW = 4>
__global__ __launch_bounds__(256) void softmax_kernel(SoftmaxArgs p) {
  const int row = member_block(p, blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row < p.R) softmax_row<NV, IN_BF16, OUT_BF16, NT, CW, true>(p, row);
}

template <typename T, bool NT>
__global__ __launch_bounds__(256) void transpose_vec_kernel(TransArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[64 * 65 * sizeof(T)];
  const int bid = member_block(p, blockIdx.x);
  transpose_tile_vec<T, NT>(p, bid, smem);
}

template <typename T, int TR, int TC, bool NT>
__global__ __launch_bounds__(256) void transpose_rc_kernel(TransArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[transpose_rc_smem<TR, TC, T>()];
  const int bid = member_block(p, blockIdx.x);
  transpose_rc_tile<T, TR, TC, NT>(p, bid, smem);
}

template <bool IN_BF16, bool OUT_BF16, bool NT = false>
__global__ __launch_bounds__(256) void add_vec_kernel(AddArgs p) {
  const int bid = member_block(p, blockIdx.x);
  add_block<IN_BF16, OUT_BF16, NT>(p, bid);
}

// ---------------------------------------------------------------------------------------------
// Launch factories
// ---------------------------------------------------------------------------------------------
namespace {

// Softmax and transpose launches whose output is at least this large (bytes, the size of the
// last-level cache) read and write with streaming hints: neither operand would stay cached for a
// consumer.
constexpr int64_t kStreamBytes = int64_t(256) << 20;

template <typename Args>
void set_args(Launch &L, const Args &a) {
  static_assert(sizeof(Args) <= sizeof(L.args), "argument struct too large");
  memcpy(L.args, &a, sizeof(Args));
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct TileCfg {
  int bm, bn;
  bool splitk;  // K split across the block's four wavefronts
};
// 1..5: large tiles; 6..12: K split over the wavefronts, operands through LDS; 13..15: K split
// over the wavefronts, operands read directly into matrix-core registers (16-row tiles);
// 16: 256 x 256 BF16 tile, eight wavefronts, 512 threads (for FP32 operands it means tile 1);
// 17..19: BF16 K split over the wavefronts with each wavefront's K share loaded at once (16 x 16
// and 16 x 32 with four 64-deep chunks in flight, 32 x 32 with two); for FP32 operands they mean
// the staged split-K tiles of the same shape (12, 10, 9).

// GEMM tile configurations (index = psc_kernel_params.tile; 0 = automatic)
constexpr TileCfg kTiles[] = {{0, 0, false},     {128, 128, false}, {64, 64, false},  {32, 32, false},
                              {128, 64, false},  {64, 128, false},  {64, 64, true},   {32, 64, true},
                              {64, 32, true},    {32, 32, true},    {16, 32, true},   {32, 16, true},
                              {16, 16, true},    {16, 16, true},    {16, 32, true},   {16, 64, true},
                              {256, 256, false}, {16, 16, true},    {16, 32, true},   {32, 32, true},
                              {256, 256, false}, {256, 256, false}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

#define PSC_VO(KERNEL, ...) \
  (obf ? (const void *)&KERNEL<__VA_ARGS__, true> : (const void *)&KERNEL<__VA_ARGS__, false>)

const void *gemm_fn(int ab_dtype, int tile, bool obf) {
  if (ab_dtype == 0) {
    switch (tile) {
      case 1: return PSC_VO(gemm_f32_kernel, 128, 128, 16, 64, 64);
      case 2: return PSC_VO(gemm_f32_kernel, 64, 64, 16, 32, 32);
      case 3: return PSC_VO(gemm_f32_kernel, 32, 32, 32, 16, 16);
      case 4: return PSC_VO(gemm_f32_kernel, 128, 64, 16, 64, 32);
      case 5: return PSC_VO(gemm_f32_kernel, 64, 128, 16, 32, 64);
      case 6: return PSC_VO(gemm_f32_splitk_kernel, 64, 64);
      case 7: return PSC_VO(gemm_f32_splitk_kernel, 32, 64);
      case 8: return PSC_VO(gemm_f32_splitk_kernel, 64, 32);
      case 9: return PSC_VO(gemm_f32_splitk_kernel, 32, 32);
      case 10: return PSC_VO(gemm_f32_splitk_kernel, 16, 32);
      case 11: return PSC_VO(gemm_f32_splitk_kernel, 32, 16);
      case 12: return PSC_VO(gemm_f32_splitk_kernel, 16, 16);
      case 13: return PSC_VO(gemm_f32_direct_kernel, 1);
      case 14: return PSC_VO(gemm_f32_direct_kernel, 2);
      case 15: return PSC_VO(gemm_f32_direct_kernel, 4);
    }
  } else {
    switch (tile) {
      case 1: return PSC_VO(gemm_bf16_kernel, 128, 128, 64, 64, 64);
      case 2: return PSC_VO(gemm_bf16_kernel, 64, 64, 64, 32, 32);
      case 3: return PSC_VO(gemm_bf16_kernel, 32, 32, 64, 16, 16);
      case 4: return PSC_VO(gemm_bf16_kernel, 128, 64, 64, 64, 32);
      case 5: return PSC_VO(gemm_bf16_kernel, 64, 128, 64, 32, 64);
      case 6: return PSC_VO(gemm_bf16_splitk_kernel, 64, 64);
      case 7: return PSC_VO(gemm_bf16_splitk_kernel, 32, 64);
      case 8: return PSC_VO(gemm_bf16_splitk_kernel, 64, 32);
      case 9: return PSC_VO(gemm_bf16_splitk_kernel, 32, 32);
      case 10: return PSC_VO(gemm_bf16_splitk_kernel, 16, 32);
      case 11: return PSC_VO(gemm_bf16_splitk_kernel, 32, 16);
      case 12: return PSC_VO(gemm_bf16_splitk_kernel, 16, 16);
      case 13: return PSC_VO(gemm_bf16_direct_kernel, 1);
      case 14: return PSC_VO(gemm_bf16_direct_kernel, 2);
      case 15: return PSC_VO(gemm_bf16_direct_kernel, 4);
      case 16: return obf ? (const void *)&gemm_bf16_big_kernel<true> : (const void *)&gemm_bf16_big_kernel<false>;
      case 17: return PSC_VO(gemm_bf16_deep_kernel, 16, 16, 4);
      case 18: return PSC_VO(gemm_bf16_deep_kernel, 16, 32, 4);
      case 19: return PSC_VO(gemm_bf16_deep_kernel, 32, 32, 2);
      case 20: return obf ? (const void *)&gemm_bf16_w4_kernel<2, true> : (const void *)&gemm_bf16_w4_kernel<2, false>;
      case 21: return obf ? (const void *)&gemm_bf16_w4_kernel<4, true> : (const void *)&gemm_bf16_w4_kernel<4, false>;
    }
  }
  return nullptr;
}
#undef PSC_VO

int64_t tiles_of(int t, int M, int N) {
  return int64_t((M + kTiles[t].bm - 1) / kTiles[t].bm) * ((N + kTiles[t].bn - 1) / kTiles[t].bn);
}

}  // namespace

int gemm_num_tiles() { return kNumTiles; }

// (external linkage: the AQL dispatcher finds kernels by the name of their host handle)
__global__ __launch_bounds__(64) void mark_kernel(uint64_t *slot) {
  if (threadIdx.x == 0) *slot = wall_clock64();
}

void make_mark(Launch &L, uint64_t *slot) {
  L = Launch{};
  L.func = reinterpret_cast<const void *>(&mark_kernel);
  L.grid = dim3(1, 1, 1);
  L.block = dim3(64, 1, 1);
  std::memcpy(L.args, &slot, sizeof(slot));
}

namespace {
struct FillArgs {
  uint32_t *p;
  int64_t words;
  int32_t bf16;
  uint32_t seed;
};
// 32-bit integer mix (xor-shift-multiply rounds); only its spread matters here
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16; x *= 0x7feb352du;
  x ^= x >> 15; x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}
__global__ __launch_bounds__(256) void fill_kernel(FillArgs a) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < a.words; i += int64_t(gridDim.x) * 256) {
    const uint32_t h = mix32(uint32_t(i) ^ mix32(uint32_t(i >> 32) + a.seed));
    const float lo = float(h & 0xffffu) * (1.0f / 32768.0f) - 1.0f, hi = float(h >> 16) * (1.0f / 32768.0f) - 1.0f;
    a.p[i] = a.bf16 ? uint32_t(f32_to_bf16(lo)) | (uint32_t(f32_to_bf16(hi)) << 16) : __float_as_uint(lo);
  }
}
}  // namespace

void make_fill(Launch &L, void *p, int64_t bytes, int bf16, uint32_t seed) {
  L = Launch{};
  const FillArgs a{static_cast<uint32_t *>(p), bytes / 4, bf16, seed};
  L.func = reinterpret_cast<const void *>(&fill_kernel);
  L.grid = dim3(unsigned(std::min<int64_t>(4096, std::max<int64_t>(1, (a.words + 255) / 256))), 1, 1);
  L.block = dim3(256, 1, 1);
  L.empty = a.words == 0;
  std::memcpy(L.args, &a, sizeof(a));
}

namespace {
constexpr int kStaged[] = {1, 4, 5, 2}, kSplit[] = {6, 7, 8, 9, 10, 11, 12};

// A tile at least twice as wide (or high) as the matrix works mostly on padding.
bool wasteful(int t, int M, int N) { return kTiles[t].bm >= 2 * std::max(M, 16) || kTiles[t].bn >= 2 * std::max(N, 16); }
}  // namespace

int gemm_auto_tile(int M, int N, int K, int dtype) {
  // BF16 shapes of whole 256 x 256 tiles that fill the chip: the four-wavefront tile with direct
  // global-to-LDS copies (the launch factory still checks alignment).  Otherwise, enough output tiles to fill the chip: the
  // large-tile kernels; else the split-K kernels, which run four wavefronts per tile along K: the
  // largest tile that still yields >= 256 blocks (>= 128 when K is long), else the smallest tile.
  if (dtype == 1 && M % 256 == 0 && N % 256 == 0 && K % 64 == 0 && K > 0 && tiles_of(20, M, N) >= 256) return 20;
  for (int t : kStaged)
    if (tiles_of(t, M, N) >= 256 && (!wasteful(t, M, N) || t == 2)) return t;
  const int64_t want = K >= 256 ? 128 : 256;
  for (int t : kSplit)
    if (tiles_of(t, M, N) >= want) return t;
  return 12;
}

int gemm_sum_order(int tile) {
  // 1-5 walk K in steps of one matrix-core depth; 6-12 deal 64-deep (FP32: 32-deep) chunks to the
  // wavefronts in turn and add the four sums in order; the others each have an order of their own
  return tile >= 1 && tile <= 5 ? 1 : tile >= 6 && tile <= 12 ? 6 : tile;
}

int gemm_group_tile(const std::vector<GemmArgs> &args, int tile) {
  // The largest tile of the same order that still yields kGroupBlocks blocks over all kernels and is
  // not wasteful for those that hold more than an eighth of them: one short instance of a batch does
  // not set the tile of the long ones (lengths 1 and eight times 512, FP32: 0.535 ms, and 0.580 when
  // it does; eight times 1 and of 512: 0.564 and 0.679).
  constexpr int64_t kGroupBlocks = 384;
  auto fits = [&](int t) {
    int64_t n = 0, waste = 0;
    for (const GemmArgs &a : args) {
      const int64_t b = tiles_of(t, a.M, a.N);
      n += b;
      if (wasteful(t, a.M, a.N)) waste += b;
    }
    return n >= kGroupBlocks && 8 * waste <= n;
  };
  if (gemm_sum_order(tile) == 1) {
    for (int t : kStaged)
      if (fits(t)) return t;
    return 2;
  }
  if (gemm_sum_order(tile) == 6) {
    for (int t : kSplit)
      if (fits(t)) return t;
    return 12;
  }
  return tile;
}

namespace {
size_t args_size(int kind) {
  return kind == 0 ? sizeof(GemmArgs) : kind == 1 ? sizeof(TransArgs) : kind == 2 ? sizeof(SoftmaxArgs) : sizeof(AddArgs);
}
size_t up16(size_t n) { return (n + 15) & ~size_t(15); }

template <typename Args>
void point_at(Launch &L, const uint32_t *map, const void *list) {
  Args a;
  std::memcpy(&a, L.args, sizeof(a));
  a.map = map;
  a.list = static_cast<const Args *>(list);
  std::memcpy(L.args, &a, sizeof(a));
}
}  // namespace

bool groupable(const Launch &L) {
  return L.kind >= 0 && !L.empty && L.grid.x < 2048 && !(L.kind == 0 && (L.tile == 16 || L.tile >= 20));
}

size_t group_table_bytes(const std::vector<Launch> &m) {
  size_t blocks = 0;
  for (const Launch &L : m) blocks += L.grid.x;
  return up16(m.size() * args_size(m[0].kind)) + up16(4 * blocks);
}

Launch group_launch(const std::vector<Launch> &m, void *host_image, void *dev) {
  const size_t as = args_size(m[0].kind), map_off = up16(m.size() * as);
  auto *list = static_cast<unsigned char *>(host_image);
  auto *map = reinterpret_cast<uint32_t *>(list + map_off);
  size_t b = 0;
  for (size_t i = 0; i < m.size(); ++i) {
    std::memcpy(list + i * as, m[i].args, as);
    for (uint32_t t = 0; t < m[i].grid.x; ++t) map[b++] = uint32_t(i) << 16 | t;
  }
  Launch L = m[0];
  L.grid = dim3(unsigned(b), 1, 1);
  const auto *dmap = reinterpret_cast<const uint32_t *>(static_cast<const unsigned char *>(dev) + map_off);
  switch (L.kind) {
    case 0: point_at<GemmArgs>(L, dmap, dev); break;
    case 1: point_at<TransArgs>(L, dmap, dev); break;
    case 2: point_at<SoftmaxArgs>(L, dmap, dev); break;
    default: point_at<AddArgs>(L, dmap, dev); break;
  }
  return L;
}

bool make_gemm(Launch &L, GemmArgs a, int ab_dtype, int c_dtype, int tile) {
  if (tile <= 0 || tile >= kNumTiles) tile = tile_cache_get(a.M, a.N, a.K, ab_dtype, c_dtype, TileUse::alone);
  if (tile <= 0 || tile >= kNumTiles) tile = gemm_auto_tile(a.M, a.N, a.K, ab_dtype);
  if ((tile == 16 || tile >= 20) && ab_dtype == 0) tile = 1;  // the 256 x 256 tiles exist for BF16 only
  if (ab_dtype == 0 && tile >= 17 && tile <= 19) tile = tile == 17 ? 12 : tile == 18 ? 10 : 9;  // BF16 only
  if (tile == 16 || tile >= 20) {  // whole tiles, aligned operands only
    const bool fits = a.M % 256 == 0 && a.N % 256 == 0 && a.K % 64 == 0 && a.K > 0 && aligned16(a.A) &&
                      aligned16(a.B) && a.lda % 8 == 0 && a.ldb % 8 == 0;
    if (!fits) tile = 4;
  }
  const int bm = kTiles[tile].bm, bn = kTiles[tile].bn;
  a.tiles_n = (a.N + bn - 1) / bn;
  const int tiles_m = (a.M + bm - 1) / bm;
  const bool obf = c_dtype == 1;
  const void *fn = gemm_fn(ab_dtype, tile, obf);
  if (!fn) return false;
  L.func = fn;
  L.grid = dim3(unsigned(int64_t(tiles_m) * a.tiles_n), 1, 1);
  L.block = dim3(tile == 16 || tile == 21 ? 512 : 256, 1, 1);  // four wavefronts, eight for tiles 16 and 21
  L.shmem = 0;
  L.empty = a.M == 0 || a.N == 0;
  L.tile = tile;
  L.kind = 0;
  set_args(L, a);
  return true;
}

bool make_softmax(Launch &L, SoftmaxArgs a, int in_dtype, int out_dtype) {
  const bool ib = in_dtype == 1, ob = out_dtype == 1;
  int nv = 0;
  if (a.C <= 256) nv = 1;
  else if (a.C <= 512) nv = 2;
  else if (a.C <= 1024) nv = 4;
  else if (a.C <= 2048) nv = 8;
  const bool nt = nv > 0 && int64_t(a.R) * a.C * (ob ? 2 : 4) >= kStreamBytes;
// (NV register quads per lane, streaming hint, chunk width of bf16 input)
#define PSC_SMS(NV, NT, W)                                                                          \
  (ib ? (ob ? (const void *)&softmax_kernel<NV, true, true, NT, W> : (const void *)&softmax_kernel<NV, true, false, NT, W>) \
      : (ob ? (const void *)&softmax_kernel<NV, false, true, NT> : (const void *)&softmax_kernel<NV, false, false, NT>))
#define PSC_SM(NV, W) (nt ? PSC_SMS(NV, true, W) : PSC_SMS(NV, false, W))
  switch (nv) {
    case 1: L.func = PSC_SM(1, 4); break;   // (no eight-wide chunks for rows of at most 256)
    case 2: L.func = PSC_SM(2, 8); break;
    case 4: L.func = PSC_SM(4, 8); break;
    case 8: L.func = PSC_SM(8, 8); break;
    default: L.func = PSC_SMS(0, false, 4); break;
  }
#undef PSC_SM
#undef PSC_SMS
  L.grid = dim3(unsigned((a.R + 3) / 4), 1, 1);
  L.block = dim3(256, 1, 1);
  L.shmem = 0;
  L.empty = a.R == 0 || a.C == 0;
  L.kind = 2;
  set_args(L, a);
  return true;
}

#define PSC_TRC(T, TR, TC) (nt ? (const void *)&transpose_rc_kernel<T, TR, TC, true> : (const void *)&transpose_rc_kernel<T, TR, TC, false>)

// tile: 1 64 x 64, 2 64 x 128, 3 128 x 64, 4 64 x 256 (rows x columns of the input).  Automatic (0),
// 64 x 64 below kStreamBytes; from there, measured (us):
//   - streaming hints only where every row of B starts on a cache line; elsewhere the lines shared
//     by two tiles go to memory in pieces: 9001 x 9003 FP32 in 128 x 64 tiles 215 with, 190 without;
//     13001 x 12003 BF16 288 / 211; 8192 x 8193 FP32 98 / 103; 16384^2 FP32 382 / 396
//   - with them 64 x 256 (16384^2 FP32 382, 64 x 128 399, 128 x 64 404, 64 x 64 409), but not for
//     matrices narrower than that, whose tiles would lie mostly outside (900000 x 100 FP32: 64 x 256
//     169, 64 x 128 143, 64 x 64 175; 4500000 x 15: 515, 216, 102)
//   - without them 128 x 64 (9001 x 9003 FP32 190, the others 207 to 219; 100 x 900000 139 / 235 to
//     242), but not for matrices of few rows (15 x 4500000: 294, 64 x 64 101)
bool make_transpose(Launch &L, TransArgs a, int dtype, int tile) {
  const int es = dtype == 1 ? 2 : 4;
  const bool large = int64_t(a.R) * a.C * es >= kStreamBytes;
  const bool nt = large && reinterpret_cast<uintptr_t>(a.B) % 128 == 0 && a.ldb * es % 128 == 0;
  if (tile < 1 || tile > 4) tile = !large ? 1 : nt ? (a.C >= 256 ? 4 : a.C > 64 ? 2 : 1) : a.R > 64 ? 3 : 1;
  int tr = 64, tcl = 64;
  if (tile == 1)
    L.func = dtype == 1 ? (nt ? (const void *)&transpose_vec_kernel<uint16_t, true> : (const void *)&transpose_vec_kernel<uint16_t, false>)
                        : (nt ? (const void *)&transpose_vec_kernel<float, true> : (const void *)&transpose_vec_kernel<float, false>);
  else if (tile == 2)
    L.func = dtype == 1 ? PSC_TRC(uint16_t, 64, 128) : PSC_TRC(float, 64, 128), tcl = 128;
  else if (tile == 4)
    L.func = dtype == 1 ? PSC_TRC(uint16_t, 64, 256) : PSC_TRC(float, 64, 256), tcl = 256;
  else
    L.func = dtype == 1 ? PSC_TRC(uint16_t, 128, 64) : PSC_TRC(float, 128, 64), tr = 128;
  L.tile = tile;
  L.grid = dim3(unsigned(int64_t((a.R + tr - 1) / tr) * ((a.C + tcl - 1) / tcl)), 1, 1);
  L.block = dim3(256, 1, 1);
  L.shmem = 0;
  L.empty = a.R == 0 || a.C == 0;
  L.kind = 1;
  set_args(L, a);
  return true;
}

bool make_add(Launch &L, AddArgs a, int in_dtype, int out_dtype) {
  const bool ib = in_dtype == 1, ob = out_dtype == 1;
  // plain loads and stores: streaming hints measured slower for the two-input add
  L.func = ib ? (ob ? (const void *)&add_vec_kernel<true, true> : (const void *)&add_vec_kernel<true, false>)
              : (ob ? (const void *)&add_vec_kernel<false, true> : (const void *)&add_vec_kernel<false, false>);
  const int64_t units = add_units(a.C);
  a.inv = units > 1 ? uint32_t((int64_t(1) << 32) / units) : ~0u;
  L.grid = dim3(unsigned((units * a.R + 255) / 256), 1, 1);
  L.block = dim3(256, 1, 1);
  L.shmem = 0;
  L.empty = a.R == 0 || a.C == 0;
  L.kind = 3;
  set_args(L, a);
  return true;
}

}  // namespace psc
