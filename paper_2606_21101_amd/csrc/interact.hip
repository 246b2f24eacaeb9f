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
// instructions, fp32 sums).  Four waves take a tile of 2*WT rows by 2*WT
// columns, a wave WT by WT.  Both operands are contiguous along k: K blocks of
// kBk columns of both go through registers, D of them in flight, into one of
// two LDS buffers, one barrier per K block.  Which k a lane feeds a matrix
// instruction is free as long as both operands agree, so lane group h takes
// k = 4h .. 4h + 3 of a chunk with one 16-byte LDS read and feeds one of them
// to each of four instructions.  LDS rows are padded to 36 dwords: 16 lanes'
// reads then cover all 64 banks once.  The weights are the instruction's row
// operand, so a lane's registers hold four consecutive columns of an output
// row, stored (and the epilogue's operands loaded) 16 bytes at a time.
// The bound is the fp32 matrix rate (157 TFLOP/s) for large batches and the
// trips to memory along K for small ones: with one K block in flight a
// layer's block waited about 0.8 us per K block.  A block may hold KS groups of
// four waves that share a tile's K blocks and add their sums at the end, and a
// tile of 32 by 32 may keep two sums (even and odd chunks): shorter chains, and
// rounding errors that shrink with them.
// Against a library GEMM and an element-wise kernel per layer, cross network and
// MLP on two streams: three cross layers of dim 416 and an MLP 1024-512-256, 64
// samples 176 -> 72 us, 4,096 samples 182 -> 134 (13.2 GFLOP), 16,384 samples
// 504 -> 449; two of dim 1664 and the same MLP, 64 samples 147 -> 64, 2,048 297
// -> 317, 8,192 1036 -> 1032; one of dim 12800 and an MLP 1024-512, 64 samples
// 2845 -> 301, 512 2872 -> 1574, 2,048 5799 -> 6251.  Slower stay about two tiles
// a CU at depth (512 samples, one of dim 1664 and an MLP 4096-4096: 223 -> 249,
// where two blocks a CU hide less than the library does) and a few columns of a
// very deep layer (16 samples, 65,536 to 8: one block holds all of K).
// Reads go through buffer descriptors of the tile's own rows: rows past the
// matrix read as zeros, and so do columns past K (offset kOut, past any
// descriptor).
// ---------------------------------------------------------------------------
constexpr int kBk = 32;
constexpr int kLdRow = kBk + 4;
constexpr uint32_t kOut = 0xfffffff0u;
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

// How rows of K columns are read: 16 bytes at a time (K % 4 == 0), 8 bytes
// (K % 2 == 0), 16 bytes at any 4-byte address with the last piece shifted back
// into the row (odd K), or single columns (K of 1 and 3).  8-byte pieces of an
// even K beat shifted ones (9,000 samples, 390 by 390: 34.2 and 38.2 us); single
// columns of an odd one do not (1,024 samples, a cross layer of dim 1663 and an
// MLP layer of 1023: 233 us, 123 shifted).
enum ReadWidth { kQuads, kPairs, kShifted, kSingles };

// One operand's tile of 32 * N rows: a thread stages 4 columns of N of them per K block.
template <int N, ReadWidth RW>
struct Operand {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t row0;   // byte offset of the thread's first row, from the tile's first

  __device__ __forceinline__ void init(const float* base, int64_t first, int64_t rows_left, int32_t K, int tid) {
    const int rows = (int)(rows_left < 32 * N ? rows_left : 32 * N);
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + first * K), (short)0, rows * K * 4, 0x00020000);
    row0 = (uint32_t)(tid / 8) * (uint32_t)K * 4u;
  }
  // columns k .. k + 3; no branch: loads under one are waited for where it ends
  __device__ __forceinline__ void load(int4_t (&v)[N], int32_t k, int32_t K) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t row = row0 + 32u * i * (uint32_t)K * 4u;
      const uint32_t o = row + (uint32_t)k * 4u;
      if constexpr (RW == kQuads) {
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(k < K ? o : kOut), 0, 0);
      } else if constexpr (RW == kPairs) {
        const int2_t lo = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(k < K ? o : kOut), 0, 0);
        const int2_t hi = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(k + 2 < K ? o + 8u : kOut), 0, 0);
        v[i] = int4_t{lo[0], lo[1], hi[0], hi[1]};
      } else if constexpr (RW == kShifted) {
        const uint32_t last = row + (uint32_t)(K - 4) * 4u;
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(k < K ? (k < K - 4 ? o : last) : kOut), 0, 0);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[i][j] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(k + j < K ? o + 4u * j : kOut), 0, 0);
      }
    }
  }
  static __device__ __forceinline__ void store(const int4_t (&v)[N], float* lds, int tid, int32_t k, int32_t K) {
    const int32_t past = k + 4 - K;   // kShifted, 1 to 3: this many columns of the piece lie before k
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int4_t x = v[i];
      if (RW == kShifted && past > 0 && past < 4) {
        x[0] = past == 1 ? v[i][1] : past == 2 ? v[i][2] : v[i][3];
        x[1] = past == 1 ? v[i][2] : past == 2 ? v[i][3] : 0;
        x[2] = past == 1 ? v[i][3] : 0;
        x[3] = 0;
      }
      *reinterpret_cast<int4_t*>(lds + (tid / 8 + 32 * i) * kLdRow + (tid & 7) * 4) = x;
    }
  }
};

// Every wave's LDS accesses before it are done; global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length

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
    if (n + 4 <= N) {
      const float4_t bb = *reinterpret_cast<const float4_any*>(a.bias + n);
      float4_t res;
      if constexpr (CROSS) {
        const float4_t c0 = *reinterpret_cast<const float4_any*>(a.x0 + o);
        const float4_t xx = *reinterpret_cast<const float4_any*>(a.x + o);
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = c0[i] * (acc[4 * q + i] + bb[i]) + xx[i];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = fmaxf(acc[4 * q + i] + bb[i], 0.f);
      }
      *reinterpret_cast<float4_any*>(a.out + o) = res;
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (n + i < N) {
          const float y = acc[4 * q + i] + a.bias[n + i];
          a.out[o + i] = CROSS ? a.x0[o + i] * y + a.x[o + i] : fmaxf(y, 0.f);
        }
      }
    }
  }
}

// SUMS: a wave's sums, of even and odd chunks where two.  KS: groups of four waves; group s takes K blocks s, s + KS,
// ...  D: K blocks in flight per group.
template <int WT, int SUMS, int KS, int D, ReadWidth RW, bool CROSS>
__global__ __launch_bounds__(kBlockThreads * KS) void layer_kernel(const LayerArgs a) {
  constexpr int BT = 2 * WT;
  constexpr int NS = BT / 32;               // rows a thread stages, per operand
  constexpr int CH = WT == 32 ? 8 : 16;     // columns of a chunk: 4 per lane group
  constexpr int NACC = sizeof(typename Mfma<WT>::acc_t) / sizeof(float);
  constexpr int kTile = BT * kLdRow;        // an operand's K block in LDS
  constexpr int kStep = kBk * KS;
  // The forms for deep K and for many tiles take tiles row by row within groups of 512 columns, so that an XCD's tiles
  // in flight share their rows of both operands in its L2 (4,096 by 4,096 of K 4096: 1170 us with rows of tiles across
  // all columns, now 1020; 8,192 samples, 1664 by 1664: 354 and 343).  Few K blocks do not pay for the divisions.
  constexpr bool kGrouped = WT == 32 || (SUMS == 2 && KS != 2);
  constexpr int kCols = 512 / BT;
  constexpr bool kEarly = WT == 32 && KS == 2;
  __shared__ float lds_all[KS * 4 * kTile];
  const int tid = threadIdx.x % kBlockThreads, lane = tid & (kWaveSize - 1);
  const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kBlockThreads);
  float* const lds = lds_all + group * 4 * kTile;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
  const int wm = (wave >> 1) * WT, wn = (wave & 1) * WT;
  const int r = lane % WT, h = lane / WT;
  const int32_t K = a.K, N = a.N;
  const int64_t M = a.M;
  const int32_t tm = (int32_t)((M + BT - 1) / BT), tn = (N + BT - 1) / BT;
  const int64_t tiles = (int64_t)tm * tn;
  const int32_t blocks_k = (K + kStep - 1) / kStep;   // of every group; those past K read zeros
  const int kcol = (tid & 7) * 4 + group * kBk;
  for (int64_t blk = blockIdx.x; blk < tiles; blk += gridDim.x) {
    // workgroups go round-robin over 8 XCDs: XCD x takes a contiguous range of
    // tiles, so that a row tile of x is read into one L2
    const int64_t xcd = blk & 7, lo = tiles >> 3, rem = tiles & 7;
    const int64_t tile = xcd * lo + (xcd < rem ? xcd : rem) + (blk >> 3);
    int64_t m0;
    int32_t n0;
    if constexpr (kGrouped) {
      const int32_t group_n = (int32_t)(tile / ((int64_t)tm * kCols)) * kCols;
      const int32_t in_group = (int32_t)(tile - (int64_t)tm * group_n), group_w = min(kCols, tn - group_n);
      m0 = (int64_t)(in_group / group_w) * BT;
      n0 = (group_n + in_group % group_w) * BT;
    } else {
      m0 = tile / tn * BT;
      n0 = (int32_t)(tile % tn) * BT;
    }
    Operand<NS, RW> ox, ow;
    ox.init(a.x, m0, M - m0, K, tid);
    ow.init(a.w, n0, N - n0, K, tid);
    typename Mfma<WT>::acc_t acc = {}, acc2 = {};
    int4_t vx[D][NS], vw[D][NS];   // the K blocks in flight
#pragma unroll
    for (int d = 0; d < D; ++d) {
      ox.load(vx[d], kcol + d * kStep, K);
      ow.load(vw[d], kcol + d * kStep, K);
    }
    lds_barrier();   // the tile before this one is done with the buffers
    int32_t kb = 0;
    // K block b of the group from px and pw to its buffer, and block b + D on its way
    const auto stage = [&](int4_t (&px)[NS], int4_t (&pw)[NS], int32_t b) {
      float* const bx = lds + (b & 1) * (2 * kTile);
      ox.store(px, bx, tid, kcol + b * kStep, K);
      ow.store(pw, bx + kTile, tid, kcol + b * kStep, K);
      ox.load(px, kcol + (b + D) * kStep, K);
      ow.load(pw, kcol + (b + D) * kStep, K);
    };
    const auto multiply = [&](const float4_t fx, const float4_t fw, int c) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (SUMS == 1 || c / CH % 2 == 0)
          acc = Mfma<WT>::mul(fw[j], fx[j], acc);
        else
          acc2 = Mfma<WT>::mul(fw[j], fx[j], acc2);
      }
    };
    const auto frag = [&](const float* buf, int row, int c) {   // this lane's columns of chunk c
      return *reinterpret_cast<const float4_t*>(buf + (row + r) * kLdRow + 4 * h + c);
    };
    const auto step = [&](int4_t (&px)[NS], int4_t (&pw)[NS]) {
      const float* const bx = lds + (kb & 1) * (2 * kTile);
      const float* const bw = bx + kTile;
      if constexpr (!kEarly) {
        // one barrier per K block: this buffer's readers of two blocks ago passed the last one
        stage(px, pw, kb);
        lds_barrier();
#pragma unroll
        for (int c = 0; c < kBk; c += CH) multiply(frag(bx, wm, c), frag(bw, wn, c), c);
      } else {
        // block kb is in its buffer and px, pw hold the next one, which goes to the other buffer (its readers have
        // passed this barrier) among the multiplications: with two blocks of four waves a CU nothing else covers that
        lds_barrier();
        float4_t fx = frag(bx, wm, 0), fw = frag(bw, wn, 0);
#pragma unroll
        for (int c = 0; c < kBk; c += CH) {
          const float4_t cx = fx, cw = fw;
          if (c + CH < kBk) fx = frag(bx, wm, c + CH), fw = frag(bw, wn, c + CH);
          if (c == kBk / 2) stage(px, pw, kb + 1);
          __builtin_amdgcn_sched_barrier(0);
          multiply(cx, cw, c);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      ++kb;
    };
    if constexpr (kEarly) {
      // block 0 to its buffer; the registers move on by one block
      static_assert(D == 2, "two blocks in registers");
      stage(vx[0], vw[0], 0);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int4_t x = vx[0][i], w = vw[0][i];
        vx[0][i] = vx[1][i], vw[0][i] = vw[1][i];
        vx[1][i] = x, vw[1][i] = w;
      }
    }
    // whole rounds, then the rest: an exit inside a round would make its first step wait for every load
    for (int32_t n = blocks_k / D; n > 0; --n) {
#pragma unroll
      for (int d = 0; d < D; ++d) step(vx[d], vw[d]);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (kb < blocks_k) step(vx[d], vw[d]);
    if (SUMS == 2) acc += acc2;
    if constexpr (KS > 1) {
      // group 0 adds the others' sums, in their order
      static_assert((KS - 1) * NACC * kBlockThreads <= KS * 4 * kTile, "sums fit the operands' buffers");
      lds_barrier();
      if (group > 0) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) lds_all[((group - 1) * NACC + i) * kBlockThreads + tid] = acc[i];
      }
      lds_barrier();
      if (group > 0) continue;
#pragma unroll
      for (int g = 0; g < KS - 1; ++g)
#pragma unroll
        for (int i = 0; i < NACC; ++i) acc[i] += lds_all[(g * NACC + i) * kBlockThreads + tid];
    }
    store_tile<WT, CROSS>(a, acc, m0 + wm + r, n0 + wn + h * 4);
  }
}

__global__ void mark_kernel(uint64_t* slot) {
  if (threadIdx.x == 0) *slot = (uint64_t)wall_clock64();
}

}  // namespace

template <int WT, int SUMS, int KS, int D, bool CROSS>
static void launch_tiles(const LayerArgs& a, hipStream_t s) {
  const int64_t bt = 2 * WT, tiles = (a.M + bt - 1) / bt * ((a.N + bt - 1) / bt);
  const dim3 grid((unsigned)std::min(tiles, kMaxLayerBlocks)), block(kBlockThreads * KS);
  if (a.K % 4 == 0)
    hipLaunchKernelGGL((layer_kernel<WT, SUMS, KS, D, kQuads, CROSS>), grid, block, 0, s, a);
  else if (a.K % 2 == 0)
    hipLaunchKernelGGL((layer_kernel<WT, SUMS, KS, D, kPairs, CROSS>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((layer_kernel<WT, SUMS, KS, D, kShifted, CROSS>), grid, block, 0, s, a);
}

// Which tiles, and how a tile's K is shared (one layer by itself unless said
// otherwise, us).  Tiles of 64 by 64 read half as much per multiplication, tiles
// of 32 by 32 fill the chip's 256 CUs more evenly and have a shorter chain.
// Deep K: the larger ones where their rounds over the chip, four times as long,
// are at most 1.25 times the smaller ones': 512 samples, 4096 columns of K 4096
// (512 and 2048 tiles) 148 against 166; 2,048 samples, 1664 by 1664 (832, 3328)
// 108 and 112; 256 samples (104, 416) 35 and 21.  Otherwise from 1536 of them on:
// the head above, 16,384 samples (1024 to 4096 tiles) 464 against 499, 4,096
// samples (256 to 1024) 148 against 143.  Deep is from K 1536 on: in the head of
// 8,192 samples the layer of K 1024 costs 1 to 5 % more in any of the deep forms.
// Groups of waves: 64 by 64 with at most two tiles a CU, where four waves a block
// wait for each other: 512 samples, 4096 by 4096 148, two groups 130; 1,024
// samples, 1664 by 1664 59.9 and 55.4.  32 by 32 with at most one a CU: 64
// samples, 512 columns of K 1024 9.6 with two sums, two groups 8.2, four 8.1;
// 1664 by 1664 14.3, 11.9, 11.2; 416 by 416 5.3, 5.0, 5.6.
// Two sums cost nothing at depth (2,048 samples, 1664 by 1664: 112 either way)
// and halve the chain that the rounding error grows with.
hipError_t launch_layer(const LayerArgs& a, hipStream_t s) {
  constexpr int64_t kCus = 256;
  const auto tiles = [&](int64_t bt) { return (a.M + bt - 1) / bt * ((a.N + bt - 1) / bt); };
  const int64_t tiles32 = tiles(32), rounds64 = (tiles(64) + kCus - 1) / kCus, rounds32 = (tiles32 + kCus - 1) / kCus;
  const bool deep = a.K >= 1536;
  const auto launch = [&](auto cross) {
    constexpr bool CROSS = decltype(cross)::value;
    if (a.K < 4 && a.K % 2 != 0) {
      const dim3 grid((unsigned)std::min(tiles32, kMaxLayerBlocks)), block(kBlockThreads);
      hipLaunchKernelGGL((layer_kernel<16, 1, 1, 3, kSingles, CROSS>), grid, block, 0, s, a);
    } else if (deep ? 16 * rounds64 <= 5 * rounds32 : tiles(64) >= 6 * kCus) {
      if (deep && rounds64 <= 2)
        launch_tiles<32, 1, 2, 2, CROSS>(a, s);
      else
        launch_tiles<32, 1, 1, 3, CROSS>(a, s);
    } else if (tiles32 <= kCus) {
      if (deep)
        launch_tiles<16, 2, 4, 2, CROSS>(a, s);
      else
        launch_tiles<16, 2, 2, 3, CROSS>(a, s);
    } else if (deep) {
      launch_tiles<16, 2, 1, 3, CROSS>(a, s);
    } else {
      launch_tiles<16, 1, 1, 3, CROSS>(a, s);
    }
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
