// Second-order factorization-machine term over the pooled field block, for
// gfx950 (MI355X).
//
// DeepFM's explicit interaction holds, besides GEMMs, element-wise squares,
// subtractions and reduce-sums; §IV-D fuses such neighbouring non-GEMM
// operators into one kernel whose threads fill the output element by element
// with contiguous reads.  For sample b of a [B, row_stride] block holding T
// fields of dim D:
//   out[b] = 1/2 * sum_c ((sum_t e[t][c])^2 - sum_t e[t][c]^2).
// One wave per sample.  Fast path (fields of 16 to 1024 bytes, all of them
// 4-byte aligned): the wave is split into field slots of LPR lanes; lane k of a
// slot reads 16-byte piece k of every G-th field row, so a load instruction
// covers G consecutive field rows of the sample (contiguous in memory); the
// per-lane sums and sums of squares are then combined across slots by a fixed
// xor butterfly and reduced over the columns.  Otherwise lanes take columns.
// fp32 accumulation in a fixed order: deterministic.
// The bound is HBM for wide blocks and the exchanges between lanes for narrow
// ones.  With all columns exchanged at every step of the butterfly and four
// rows a round whatever the fields, 26 fields of dim 8 fp16, 16,384 samples,
// took 18.9 us and 4 fields of dim 10 fp16, 65,536 samples, 58.4; now 6.8 and
// 11.4 (by columns; 20.0 by pieces).  26 fields of dim 16 fp32: 8.9 -> 5.1.
#include "dpi_internal.h"

namespace dpi {
namespace {

typedef int raw16_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

typedef const __attribute__((address_space(4))) FmArgs* FA;

template <typename T> struct Epl;
template <> struct Epl<float> { static constexpr int value = 4; };
template <> struct Epl<_Float16> { static constexpr int value = 8; };

__device__ __forceinline__ void unpack16(const raw16_t r, float* v, float) {
  const float4_t f = __builtin_bit_cast(float4_t, r);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = f[i];
}
__device__ __forceinline__ void unpack16(const raw16_t r, float* v, _Float16) {
  const half8_t h = __builtin_bit_cast(half8_t, r);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)h[i];
}

// Sum over groups of N neighbouring lanes.
template <int N>
__device__ __forceinline__ float lanes_sum(float v) {
#pragma unroll
  for (int m = 1; m < N; m <<= 1) v += __shfl_xor(v, m, kWaveSize);
  return v;
}

// Sums of v[0 .. N) over the lanes k, k + LPR, ...: each step adds the partner's
// half of the columns this lane keeps (all, once one is left), so the sums are
// those of an xor butterfly with a third of its exchanges or less.  Lane k of
// slot g ends with columns [c, c + HELD), g = holder_slot(c).
template <int N, int LPR>
__device__ __forceinline__ void slot_sums(float* v, int lane) {
  if constexpr (LPR < kWaveSize) {
    if constexpr (N > 1) {
      const bool up = (lane & LPR) != 0;
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const float keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
        v[i] = keep + __shfl_xor(send, LPR, kWaveSize);
      }
      slot_sums<N / 2, LPR * 2>(v, lane);
    } else {
      v[0] += __shfl_xor(v[0], LPR, kWaveSize);
      slot_sums<1, LPR * 2>(v, lane);
    }
  }
}

// The least slot that holds column c: bit j of the slot chose the half at step j.
template <int N, int HELD>
constexpr int holder_slot(int c) {
  int slot = 0;
  for (int half = N / 2, bit = 1; half >= HELD; half /= 2, bit *= 2)
    if (c & half) slot |= bit;
  return slot;
}

// The sample's row is read through a buffer descriptor of its own T * dim
// elements: field rows past T read as zeros, so every load of a round is issued
// without a branch and a wave waits once per round of U * G fields.  (With the
// last, partial round in a loop of single loads most slots of 26 fields of dim
// 64 fp16 made three dependent trips: 16,384 samples took 13.9 us, without
// them 12.3, and 10.4 with the sums over slots as below, 5.2 TB/s.)
// RAGGED: fields that are no multiple of 16 bytes; the last piece is shifted
// back into the field and the columns it shares with the piece before drop out.
// U: field rows in flight per lane.
template <typename TIN, int LPR, bool RAGGED, int U>
__device__ __forceinline__ float fm_fast(FA a, const char* row, int lane) {
  constexpr int EPL = Epl<TIN>::value;
  constexpr int G = kWaveSize / LPR;
  const int g = lane / LPR, k = lane % LPR;
  const int T = a->T;
  const int32_t field_bytes = a->dim * (int)sizeof(TIN);
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), (short)0, T * field_bytes, 0x00020000);
  const int32_t piece = RAGGED ? min(k * 16, field_bytes - 16) : k * 16;
  const int skip = RAGGED ? (k * 16 - piece) / (int)sizeof(TIN) : 0;
  float s[EPL], q[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) s[i] = q[i] = 0.f;
  // a lane without a piece stays at an offset past any row (U * G steps of at most 1024 bytes wrap no offset:
  // T * 1024 + 2^31 < 2^32)
  uint32_t off = k * 16 < field_bytes ? (uint32_t)(g * field_bytes + piece) : 0x80000000u;
  const uint32_t step = (uint32_t)(G * field_bytes);
  for (int t = 0; t < T; t += U * G) {
    raw16_t raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      raw[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + u * step), 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v[EPL];
      unpack16(raw[u], v, TIN());
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        if (RAGGED && i < skip) v[i] = 0.f;
        s[i] += v[i];
        q[i] += v[i] * v[i];
      }
    }
    off += U * step;
  }
  // Sum over the slots (fields t = g mod G): a butterfly whose lanes keep half
  // of their columns at each step while they hold more than one, so that slot g
  // ends with HELD of the EPL columns.
  constexpr int HELD = EPL / G > 0 ? EPL / G : 1;
  slot_sums<EPL, LPR>(s, lane);
  slot_sums<EPL, LPR>(q, lane);
#pragma unroll
  for (int i = 0; i < HELD; ++i) s[i] = s[i] * s[i] - q[i];
  // slot 0 adds its columns, in their order, then its lanes
  float y = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i)
    y += G == 1 ? s[i] : __shfl(s[i % HELD], k + LPR * holder_slot<EPL, HELD>(i), kWaveSize);
  return lanes_sum<LPR>(y);
}

template <typename TIN>
__device__ __forceinline__ float fm_general(FA a, const TIN* row, int lane) {
  float y = 0.f;
  for (int c = lane; c < a->dim; c += kWaveSize) {
    float s = 0.f, q = 0.f;
    for (int t = 0; t < a->T; ++t) {
      const float v = (float)row[(int64_t)t * a->dim + c];
      s += v;
      q += v * v;
    }
    y += s * s - q;
  }
  return lanes_sum<kWaveSize>(y);
}

// As many rows in flight as the fields of one round need: loads past the last field cost their adds.
template <typename TIN, int LPR, bool RAGGED>
__device__ __forceinline__ float fm_rounds(FA a, const char* row, int lane) {
  constexpr int G = kWaveSize / LPR;
  if (a->T <= G) return fm_fast<TIN, LPR, RAGGED, 1>(a, row, lane);
  if (a->T <= 2 * G) return fm_fast<TIN, LPR, RAGGED, 2>(a, row, lane);
  return fm_fast<TIN, LPR, RAGGED, 4>(a, row, lane);
}

template <typename TIN>
__global__ __launch_bounds__(kBlockThreads) void fm_kernel(const FmArgs args) {
  (void)args;
  const FA a = (FA)__builtin_amdgcn_kernarg_segment_ptr();
  const int lane = threadIdx.x & (kWaveSize - 1);
  const int64_t b = (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
  if (b >= a->B) return;
  const TIN* row = reinterpret_cast<const TIN*>(a->emb) + b * a->row_stride;
  float y;
  const char* const bytes = reinterpret_cast<const char*>(row);
  const bool ragged = a->dim * sizeof(TIN) % 16 != 0;
  switch (a->lpr_log) {
#define DPI_FM_CASE(L, LPR) \
  case L:                   \
    y = ragged ? fm_rounds<TIN, LPR, true>(a, bytes, lane) : fm_rounds<TIN, LPR, false>(a, bytes, lane); \
    break;
    DPI_FM_CASE(0, 1) DPI_FM_CASE(1, 2) DPI_FM_CASE(2, 4) DPI_FM_CASE(3, 8) DPI_FM_CASE(4, 16)
    DPI_FM_CASE(5, 32) DPI_FM_CASE(6, 64)
#undef DPI_FM_CASE
    default:
      y = fm_general<TIN>(a, row, lane);
  }
  if (lane == 0) a->out[b] = 0.5f * y;
}

}  // namespace

hipError_t launch_fm(const FmArgs& a, hipStream_t s) {
  const int64_t blocks = (a.B + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks <= 0) return hipSuccess;
  if (a.f16)
    hipLaunchKernelGGL(fm_kernel<_Float16>, dim3((unsigned)blocks), dim3(kBlockThreads), 0, s, a);
  else
    hipLaunchKernelGGL(fm_kernel<float>, dim3((unsigned)blocks), dim3(kBlockThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace dpi
