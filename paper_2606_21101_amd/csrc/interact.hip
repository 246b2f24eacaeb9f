// Layers of the interaction modules, for gfx950: a GEMM and the run of
// non-GEMM operators after it in one kernel.
//
// §IV-D fuses every run of neighbouring non-GEMM operators of a model's
// interaction modules into one kernel.  After each GEMM of a DCNv2 cross layer
// the run is  x_next = x0 * (y + b) + x  (a broadcast add, a multiply, an
// add); after each GEMM of the MLP it is  h = max(0, z + c).  Here the run is
// the epilogue of the GEMM itself, on the sums in registers, so y and z never
// reach memory.  A one-thread marker kernel records the device wall clock, to
// time when each module's first operator starts (Algorithm 2's measurement,
// §V).
#include <type_traits>

#include "dpi_internal.h"

namespace dpi {
namespace {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// out[m][n] = epilogue(sum_k x[m][k] w[n][k]), fp32 throughout (fp32 matrix
// instructions, fp32 sums).  A block of four waves takes a tile of 2*WT rows
// by 2*WT columns, a wave WT by WT.  Both operands are contiguous along k: K
// blocks of kBk columns of both go through registers, kAhead of them in
// flight, into one of two LDS buffers, one barrier per K block.  Which k a lane
// feeds a matrix instruction is free as long as both operands agree, so lane
// group h takes k = 4h .. 4h + 3 of a chunk with one 16-byte LDS read and feeds
// one of them to each of four instructions.  LDS rows are padded to 36 dwords:
// 16 lanes' reads then cover all 64 banks once.  The weights are the
// instruction's row operand, so a lane's registers hold four consecutive
// columns of an output row, stored (and the epilogue's operands loaded) 16
// bytes at a time.
// The bound is the fp32 matrix rate (157 TFLOP/s) for large batches and the
// trips to memory along K for small ones: with one K block in flight a
// layer's block waited about 0.8 us per K block.
// Three cross layers of dim 416 and an MLP 1024-512-256, both on two streams:
// 4,096 samples 190 -> 146 us (13.2 GFLOP), 16,384 samples 504 -> 449 us (118
// TFLOP/s), 64 samples 182 -> 55 us, against a library GEMM and an element-wise
// kernel per layer.  One K block in flight: 159, 491 and 68 us; three, with an
// exit inside the unrolled rounds (the first step of a round then waits for
// every load): 151, 464 and 68 us; tiles of 128 by 128: 249, 548 and 192 us.
// Reads go through buffer descriptors of the tile's own rows: rows past the
// matrix read as zeros, and so do columns past K (offset kOut, past any
// descriptor).
// ---------------------------------------------------------------------------
constexpr int kBk = 32;
constexpr int kLdRow = kBk + 4;
constexpr uint32_t kOut = 0xfffffff0u;
// Tiles of 64 by 64 (half the reads per multiplication) from this many of them
// on, six per CU; below it tiles of 32 by 32, which fill the chip and have a
// shorter chain.  The workload above, 32 against 64: 4,096 samples (256 to 1024
// tiles a layer) 143 against 148 us, 1,000 samples 67 against 91, 16,384 samples
// (1024 to 4096 tiles) 499 against 464.
constexpr int64_t kTiles64 = 1536;
// Up to this many tiles of 32 by 32, one per CU, a layer is a chain of its own
// multiplications: two sums (even and odd chunks) halve that chain and its
// rounding error (64 samples: 54.7 -> 51.6 us, error of the MLP against 64 bits 6.1e-07 -> 4.3e-07).  Where more
// tiles share a CU they cost 5 % (4,096 samples 146 -> 159 us).
constexpr int64_t kTilesTwo = 256;
constexpr int kAhead = 3;   // K blocks in flight per tile
constexpr int64_t kMaxLayerBlocks = 1 << 20;   // a larger grid loops over its tiles

template <int WT> struct Mfma;
template <> struct Mfma<32> {
  typedef float16_t acc_t;
  static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<16> {
  typedef float4_t acc_t;
  static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

typedef int int2_t __attribute__((ext_vector_type(2)));
typedef int int4_t __attribute__((ext_vector_type(4)));

// One operand's tile of 32 * N rows: a thread stages 4 columns of N of them per K block.
template <int N, int VW>
struct Operand {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t row0;   // byte offset of the thread's first row, from the tile's first

  __device__ __forceinline__ void init(const float* base, int64_t first, int64_t rows_left, int32_t K, int tid) {
    const int rows = (int)(rows_left < 32 * N ? rows_left : 32 * N);
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + first * K), (short)0, rows * K * 4, 0x00020000);
    row0 = (uint32_t)(tid / 8) * (uint32_t)K * 4u;
  }
  // columns k .. k + 3, VW (which divides K) at a time; no branch: loads under one are waited for where it ends
  __device__ __forceinline__ void load(int4_t (&v)[N], int32_t k, int32_t K) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t o = row0 + 32u * i * (uint32_t)K * 4u + (uint32_t)k * 4u;
      if constexpr (VW == 4) {
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(k < K ? o : kOut), 0, 0);
      } else if constexpr (VW == 2) {
        const int2_t lo = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(k < K ? o : kOut), 0, 0);
        const int2_t hi = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(k + 2 < K ? o + 8u : kOut), 0, 0);
        v[i] = int4_t{lo[0], lo[1], hi[0], hi[1]};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[i][j] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(k + j < K ? o + 4u * j : kOut), 0, 0);
      }
    }
  }
  static __device__ __forceinline__ void store(const int4_t (&v)[N], float* lds, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      *reinterpret_cast<int4_t*>(lds + (tid / 8 + 32 * i) * kLdRow + (tid & 7) * 4) = v[i];
  }
};

// Every wave's LDS accesses before it are done; global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One lane's columns n .. n + 3 (and, at WT = 32, n + 8 .., n + 16 .., n + 24 ..) of row m.
template <int WT, bool CROSS>
__device__ __forceinline__ void store_tile(const LayerArgs& a, const typename Mfma<WT>::acc_t& acc, int64_t m,
                                           int32_t n_first) {
  if (m >= a.M) return;
  const int32_t N = a.N;
#pragma unroll
  for (int q = 0; q < (int)sizeof(acc) / 16; ++q) {
    const int32_t n = n_first + q * 8;
    const int64_t o = m * N + n;
    if (N % 4 == 0) {
      if (n < N) {
        const float4_t bb = *reinterpret_cast<const float4_t*>(a.bias + n);
        float4_t res;
        if constexpr (CROSS) {
          const float4_t c0 = *reinterpret_cast<const float4_t*>(a.x0 + o);
          const float4_t xx = *reinterpret_cast<const float4_t*>(a.x + o);
#pragma unroll
          for (int i = 0; i < 4; ++i) res[i] = c0[i] * (acc[4 * q + i] + bb[i]) + xx[i];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) res[i] = fmaxf(acc[4 * q + i] + bb[i], 0.f);
        }
        *reinterpret_cast<float4_t*>(a.out + o) = res;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (n + i < N) {
          const float y = acc[4 * q + i] + a.bias[n + i];
          a.out[o + i] = CROSS ? a.x0[o + i] * y + a.x[o + i] : fmaxf(y, 0.f);
        }
      }
    }
  }
}

template <int WT, int VW, bool CROSS, bool TWO>
__global__ __launch_bounds__(kBlockThreads) void layer_kernel(const LayerArgs a) {
  constexpr int BT = 2 * WT;
  constexpr int NS = BT / 32;               // rows a thread stages, per operand
  constexpr int CH = WT == 32 ? 8 : 16;     // columns of a chunk: 4 per lane group
  constexpr int D = kAhead;
  __shared__ float lds[2][2][BT * kLdRow];
  const int tid = threadIdx.x, lane = tid & (kWaveSize - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int wm = (wave >> 1) * WT, wn = (wave & 1) * WT;
  const int r = lane % WT, h = lane / WT;
  const int32_t K = a.K, N = a.N;
  const int64_t M = a.M;
  const int64_t tn = (N + BT - 1) / BT, tiles = (M + BT - 1) / BT * tn;
  const int32_t blocks_k = (K + kBk - 1) / kBk;
  const int kcol = (tid & 7) * 4;
  for (int64_t blk = blockIdx.x; blk < tiles; blk += gridDim.x) {
    // workgroups go round-robin over 8 XCDs: XCD x takes a contiguous range of
    // tiles, so that a row tile of x is read into one L2
    const int64_t xcd = blk & 7, lo = tiles >> 3, rem = tiles & 7;
    const int64_t tile = xcd * lo + (xcd < rem ? xcd : rem) + (blk >> 3);
    const int64_t m0 = tile / tn * BT;
    const int32_t n0 = (int32_t)(tile % tn) * BT;
    Operand<NS, VW> ox, ow;
    ox.init(a.x, m0, M - m0, K, tid);
    ow.init(a.w, n0, N - n0, K, tid);
    typename Mfma<WT>::acc_t acc = {}, acc2 = {};   // acc2: odd chunks' sums (TWO)
    int4_t vx[D][NS], vw[D][NS];   // the K blocks in flight
#pragma unroll
    for (int d = 0; d < D; ++d) {
      ox.load(vx[d], kcol + d * kBk, K);
      ow.load(vw[d], kcol + d * kBk, K);
    }
    lds_barrier();   // the tile before this one is done with the buffers
    int32_t kb = 0;
    const auto step = [&](int4_t (&px)[NS], int4_t (&pw)[NS]) {   // K block kb, staged in px and pw
      float* const bx = lds[kb & 1][0];
      float* const bw = lds[kb & 1][1];
      // one barrier per K block: this buffer's readers of two blocks ago passed the last one
      ox.store(px, bx, tid);
      ow.store(pw, bw, tid);
      ox.load(px, kcol + (kb + D) * kBk, K);
      ow.load(pw, kcol + (kb + D) * kBk, K);
      lds_barrier();
#pragma unroll
      for (int c = 0; c < kBk; c += CH) {
        const float4_t fx = *reinterpret_cast<const float4_t*>(bx + (wm + r) * kLdRow + 4 * h + c);
        const float4_t fw = *reinterpret_cast<const float4_t*>(bw + (wn + r) * kLdRow + 4 * h + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (!TWO || c / CH % 2 == 0)
            acc = Mfma<WT>::mul(fw[j], fx[j], acc);
          else
            acc2 = Mfma<WT>::mul(fw[j], fx[j], acc2);
        }
      }
      ++kb;
    };
    // whole rounds, then the rest: an exit inside a round would make its first step wait for every load
    for (int32_t n = blocks_k / D; n > 0; --n) {
#pragma unroll
      for (int d = 0; d < D; ++d) step(vx[d], vw[d]);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (kb < blocks_k) step(vx[d], vw[d]);
    if (TWO) acc += acc2;
    store_tile<WT, CROSS>(a, acc, m0 + wm + r, n0 + wn + h * 4);
  }
}

__global__ void mark_kernel(uint64_t* slot) {
  if (threadIdx.x == 0) *slot = (uint64_t)wall_clock64();
}

}  // namespace

template <int WT, bool TWO, bool CROSS>
static void launch_tiles(const LayerArgs& a, int64_t tiles, hipStream_t s) {
  const dim3 grid((unsigned)std::min(tiles, kMaxLayerBlocks)), block(kBlockThreads);
  if (a.K % 4 == 0)
    hipLaunchKernelGGL((layer_kernel<WT, 4, CROSS, TWO>), grid, block, 0, s, a);
  else if (a.K % 2 == 0)
    hipLaunchKernelGGL((layer_kernel<WT, 2, CROSS, TWO>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((layer_kernel<WT, 1, CROSS, TWO>), grid, block, 0, s, a);
}

hipError_t launch_layer(const LayerArgs& a, hipStream_t s) {
  const auto tiles = [&](int64_t bt) { return (a.M + bt - 1) / bt * ((a.N + bt - 1) / bt); };
  const auto launch = [&](auto cross) {
    if (tiles(64) >= kTiles64)
      launch_tiles<32, false, decltype(cross)::value>(a, tiles(64), s);
    else if (tiles(32) > kTilesTwo)
      launch_tiles<16, false, decltype(cross)::value>(a, tiles(32), s);
    else
      launch_tiles<16, true, decltype(cross)::value>(a, tiles(32), s);
  };
  if (a.x0)
    launch(std::true_type());
  else
    launch(std::false_type());
  return hipGetLastError();
}

hipError_t launch_mark(uint64_t* slot, hipStream_t s) {
  hipLaunchKernelGGL(mark_kernel, dim3(1), dim3(kWaveSize), 0, s, slot);
  return hipGetLastError();
}

}  // namespace dpi
