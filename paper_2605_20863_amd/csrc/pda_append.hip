// HIP kernel that appends one decode step's new keys and values to the paged
// KV cache on MI355X (gfx950).
//
// Every rollout decode step (the paper's Sec. 2.2) produces one token per
// live sequence; its key and value go into the sequence's paged cache (the
// vLLM block layout the paper cites in Sec. 8) before attention reads it.
// Token t of sequence b lands in block block_table[b, t / 16], slot t % 16:
// a row of the token-major K tile [16][D] and a column of the dim-major V tile
// [D][16].
//
// fp8 (OCP E4M3) caches keep one scale per (block, KV head) tile and per K / V
// at max(amax / 448, 2^-126) over the tokens written to the tile so far, so a
// full tile ends with the per-tile amax scale. A token whose amax exceeds
// 448 * scale raises the scale to its own amax / 448 and re-encodes the tile's
// earlier codes (decoded value * old / new); otherwise only the new token is
// encoded. Slot 0 always starts a fresh scale. Every step that decides a code
// is float32 with one rounding per operation (correctly rounded division), and
// E4M3 encoding rounds to nearest even after clamping to +-448.

#include "pda_internal.h"

#include <stdint.h>

namespace pda {
namespace {

constexpr float kE4M3Max = 448.f;
constexpr float kMinScale = 0x1p-126f;
constexpr int kAppendWaves = 4;  // waves per workgroup
// Workgroups in a row of the grid. A launch has below 2^32 threads in x, which
// one row of a workgroup per 2 pairs would reach at 2^25 (sequence, KV head)
// pairs; the entry takes up to 2^31 - 1.
constexpr uint32_t kAppendRow = 1u << 22;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// The same in memory at any address: an fp8 cache may start at any byte, and the
// device's unaligned accesses are as wide as its aligned ones.
typedef u32x4 __attribute__((aligned(1))) u32x4_any;
typedef uint32_t __attribute__((aligned(1))) u32_any;

__device__ __forceinline__ int lane() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

// float32 -> E4M3 code: clamp to +-448, then the hardware conversion (round
// to nearest even).
__device__ __forceinline__ uint8_t enc_e4m3(float z) {
  z = fminf(fmaxf(z, -kE4M3Max), kE4M3Max);
  return (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(z, z, 0, false) & 0xFF);
}

__device__ __forceinline__ float dec_e4m3(uint8_t c) { return __builtin_amdgcn_cvt_f32_fp8((int)c, 0); }

// f32 -> bf16 bits, round to nearest even (NaN stays a quiet NaN).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Four codes of a word under another scale: enc(dec(c) * old / s) for codes
// first .. below `end`, the others as they are.
__device__ __forceinline__ uint32_t reencode4(uint32_t w, int first, int end, float old, float s) {
  uint32_t r = w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t c = enc_e4m3(__fdiv_rn(dec_e4m3((uint8_t)(w >> (8 * i))) * old, s));
    if (first + i < end) r = (r & ~(0xFFu << (8 * i))) | (c << (8 * i));
  }
  return r;
}

// A token raised the scale of an fp8 tile: its earlier tokens 0 .. o - 1 are
// re-encoded, 16 codes a lane at a time, all of a lane's loads before its
// stores. Only codes of earlier tokens are written.
template <int D>
__device__ __forceinline__ void reencode_tile(uint8_t* tile, bool is_v, int o, float old, float s) {
  constexpr int N = D / 64;  // 16-byte pieces of a whole tile per lane
  u32x4 x[N];
  // K: piece p holds 16 dims of token 16 p / D. V: dim row p, tokens 0 .. 15.
  // None at slot 0 (with V's rows loaded and divided there for nothing, slot 0 took
  // 4.7 us per call for 8 sequences x 4 heads and 9.8 for 512 x 8; now 2.8 and 5.5).
  const int pieces = is_v ? (o > 0 ? D : 0) : o * (D / 16);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int p = lane() + 64 * n;
    if (p < pieces) x[n] = *reinterpret_cast<const u32x4_any*>(tile + 16 * p);
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int p = lane() + 64 * n;
    if (p >= pieces) continue;
    u32x4 y;
#pragma unroll
    for (int w = 0; w < 4; ++w) y[w] = reencode4(x[n][w], 4 * w, is_v ? o : 16, old, s);
    if (!is_v) {
      *reinterpret_cast<u32x4_any*>(tile + 16 * p) = y;
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (4 * w + 4 <= o) {
          *reinterpret_cast<u32_any*>(tile + 16 * p + 4 * w) = y[w];
        } else {
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (4 * w + i < o) tile[16 * p + 4 * w + i] = (uint8_t)(y[w] >> (8 * i));
        }
      }
    }
  }
}

// One wave per (sequence, KV head, K or V). Bound by its chain of round trips:
// position, block id, (fp8) old scale, and for a token that raises the scale
// the tile's codes; the new values load beside the position. In large batches
// by the V columns, which touch every line of their tiles: lane l owns dims l
// and l + 64 there (neighbouring lanes on neighbouring lines; 2 l and 2 l + 1
// took 7.5 us where this takes 6.6), and dims 2 l and 2 l + 1 of a K row.
// Measured in a HIP graph, us per call, against one wave per pair that
// re-encoded byte by byte (an empty kernel takes 1.75): bf16, D = 128, 8
// sequences x 4 heads 2.7 -> 2.1, 512 x 8 6.9 -> 6.6; fp8 8 x 4 3.7 -> 3.3,
// 64 x 8 8.0 -> 4.7, 512 x 8 10.3 -> 8.5 (averages over the 16 slots of a block).
template <KvType KV, int D>
__global__ __launch_bounds__(64 * kAppendWaves) void append_kernel(AppendArgs a) {
  const uint32_t w = (blockIdx.y * kAppendRow + blockIdx.x) * kAppendWaves + (threadIdx.x >> 6);  // below 2^32
  if (w >= 2u * (uint32_t)a.B * (uint32_t)a.Hkv) return;
  const int pair = (int)(w >> 1);
  const bool is_v = __builtin_amdgcn_readfirstlane(w & 1);
  const int b = pair / a.Hkv, h = pair - b * a.Hkv;
  constexpr int E = D / 64;  // elements per lane
  const int d0 = is_v ? lane() : E * lane(), dstep = is_v ? 64 : 1;  // dims d0 + e * dstep
  const int64_t src = (int64_t)pair * D + d0;
  const void* in = is_v ? a.v_new : a.k_new;
  const int t = a.positions[b];
  uint32_t raw[E];  // loaded beside the position; converted once the block id is on its way
  if (a.new_bf16) {
#pragma unroll
    for (int e = 0; e < E; ++e) raw[e] = (uint32_t)static_cast<const uint16_t*>(in)[src + e * dstep] << 16;
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) raw[e] = static_cast<const uint32_t*>(in)[src + e * dstep];
  }
  if (t < 0) return;
  if (t >= kBlockSize * a.max_blocks) {
    if (lane() == 0) atomicOr(a.status, kStatusLenClamped);
    return;
  }
  const int p = a.block_table[(int64_t)b * a.max_blocks + t / kBlockSize];
  if ((unsigned)p >= (uint64_t)a.num_blocks) {
    if (lane() == 0) atomicOr(a.status, kStatusBadBlock);
    return;
  }
  const int o = t % kBlockSize;
  const int64_t tile = (int64_t)p * a.Hkv + h;
  float x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) x[e] = __builtin_bit_cast(float, raw[e]);

  // element e of this lane's dims: in the K tile [16][D] at row o, in the V tile [D][16] at column o
  void* cache = is_v ? a.v_cache : a.k_cache;
  const int64_t at = tile * kBlockSize * D + (is_v ? d0 * kBlockSize + o : o * D + d0);
  const int step = is_v ? 64 * kBlockSize : 1;
  if constexpr (KV == KvType::F32) {
#pragma unroll
    for (int e = 0; e < E; ++e) static_cast<float*>(cache)[at + e * step] = x[e];
  } else if constexpr (KV == KvType::BF16) {
#pragma unroll
    for (int e = 0; e < E; ++e) static_cast<uint16_t*>(cache)[at + e * step] = to_bf16(x[e]);
  } else {
    uint8_t* cb = static_cast<uint8_t*>(cache);
    float* sp = a.kv_scales + (is_v ? a.num_blocks * a.Hkv : 0) + tile;
    const float old = o > 0 ? *sp : 0.f;
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) m = fmaxf(m, fabsf(x[e]));
    const float amax = wave_max(m);
    float s = old;
    if (!(o > 0 && old > 0.f && amax <= kE4M3Max * old)) {
      s = fmaxf(__fdiv_rn(amax, kE4M3Max), kMinScale);
      reencode_tile<D>(cb + tile * kBlockSize * D, is_v, o, old, s);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) cb[at + e * step] = enc_e4m3(__fdiv_rn(x[e], s));
    if (lane() == 0) *sp = s;
  }
}

template <KvType KV>
void* append_for_d(int D) {
  return D == 64 ? reinterpret_cast<void*>(&append_kernel<KV, 64>) : reinterpret_cast<void*>(&append_kernel<KV, 128>);
}

}  // namespace

hipError_t launch_append(const AppendArgs& a, KvType kv, hipStream_t s) {
  const int64_t waves = 2 * (int64_t)a.B * a.Hkv;
  if (waves == 0) return hipSuccess;
  void* fn = kv == KvType::F32 ? append_for_d<KvType::F32>(a.D)
             : kv == KvType::BF16 ? append_for_d<KvType::BF16>(a.D)
                                  : append_for_d<KvType::FP8>(a.D);
  AppendArgs args = a;
  void* params[] = {&args};
  const int64_t wgs = (waves + kAppendWaves - 1) / kAppendWaves;
  const int64_t rows = (wgs + kAppendRow - 1) / kAppendRow;
  return hipLaunchKernel(fn, dim3((unsigned)(rows > 1 ? kAppendRow : wgs), (unsigned)rows), dim3(64 * kAppendWaves),
                         params, 0, s);
}

}  // namespace pda
