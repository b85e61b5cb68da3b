// One launch from the packed weight to the product of a few tokens.  A call that brings a packed weight and no prepared
// copy of it otherwise runs the stream-order pre-pass over the weight and then the tiled kernel; at up to a few dozen
// tokens the pre-pass is the longer of the two and its output is read once.  Here a block decodes the weight of its 32 or 16
// out-features into LDS as the operand of the matrix instructions and multiplies it with up to 64 tokens; a second form, further
// down, takes 64 out-features and 128 tokens.
//
// What bounds it: latency.  768 -> 1000 at 4:8 and 8 tokens is 1.3 MB, under 1 us of HBM time; what takes time is one
// round trip to memory, decoding 16 weights per lane and pass (the 2:4 operand in registers, the dense one with a 2-byte LDS write
// per kept value), and a serial chain of K / 64 steps.  So a block is small (768 out-features are 24 of them per 64 tokens), all
// four waves decode, the loads of two spans of 256 reduction positions are in flight in registers while a third is multiplied, and a
// span has one barrier; in blocks of 16 or 32 tokens four spans, those that there are, share one (launch_level).  No load of a span is
// under a condition of its own, which would make the span wait for the next one's.  With such conditions, and with 2-byte writes
// everywhere: 197 tokens x 768 -> 768 at 1:4 5.4 us, now 4.9; 32 x 2048 -> 1024 at 4:8 10.4 and 8.7; 16 x 4096 -> 32768 at 4:8 75.7 and 54.8.
// Which products it takes is decided in nm_spmm.hip (direct_form).  In a graph, pre-pass and product, and here: 768 -> 1000 at 4:8 and 8
// tokens 8.1 and 3.7 us, 16 x 3072 -> 16384 at 4:16, where the weight's 100 MB are read and written once more, 41.7 and 19.2.
//
// Two summation orders, so that a product is the same bytes whichever kernel of its route computes it:
//   PACKED = false  the tiled kernel's (nm_spmm.hip): the sum starts from the bias; the dense instruction takes the
//                   positions of a 64-wide step as 0 .. 31 and 32 .. 63
//   PACKED = true   the few-token kernel's (nm_fewtok.hip): the bias is added last; the dense instruction takes the even
//                   and the odd runs of 8 positions
#include "nm_launch.h"
#include "nm_mma.h"

#include <algorithm>
#include <type_traits>

namespace nm {
namespace {

constexpr int kSteps = 4;  // 64-wide steps per span.  Of a block: TOKS tokens, 64, 32 or 16, ROWS out-features, 32 or 16

struct DirectArgs {
  const bf16_t* values;
  const uint32_t* indices;
  const bf16_t* X;
  const float* bias;  // nullable
  void* Y;
  int64_t ldx, ldy;
  int32_t O, K, T;
  int32_t out_bf16, pieces;  // pieces: rows of Y are made of aligned runs of four outputs
  int32_t rows16;            // rows of Y in whole aligned 16-byte pieces
  int32_t again;             // a sum that ended as NaN is computed again by the definition, as the ragged form of the tiled kernel has it
};

// The 2:4 operand of 16 weights into its 16 bytes of LDS; returns its selectors, four bits per run.  A run of four owns two 16-bit
// slots, its first kept value in the first one and a second one in the second, free slots zero.  v: the kept values in pairs, fields:
// their positions.  Put together in registers, but for 1:16, whose one value is cheaper as a 2-byte write over the zeros.
template <int N, int M>
__device__ __forceinline__ uint32_t put_sparse_piece(unsigned char* at, const uint32_t* v, uint32_t fields) {
  u32x4_t piece = u32x4_t{0, 0, 0, 0};
  uint32_t sel = 0;
  if constexpr (M == 4) {  // 1:4: a value per run, always in its first slot
    piece = u32x4_t{v[0] & 0xFFFFu, v[0] >> 16, v[1] & 0xFFFFu, v[1] >> 16};
    const uint32_t four = fields & 0xFFu, pairs = (four | (four << 4)) & 0x0F0Fu;
    sel = (pairs | (pairs << 2)) & 0x3333u;
  } else if constexpr (M == 8) {  // two groups of two runs
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if constexpr (N == 1) {
        const uint32_t pos = (fields >> (3 * g)) & 7u, value = (v[0] >> (16 * g)) & 0xFFFFu;
        piece[2 * g] = pos & 4u ? 0u : value;
        piece[2 * g + 1] = pos & 4u ? value : 0u;
        sel |= (pos & 3u) << (8 * g + (pos & 4u));
      } else {
        const uint32_t p0 = (fields >> (6 * g)) & 7u, p1 = (fields >> (6 * g + 3)) & 7u;
        const bool upper = p0 & 4u, same = ((p0 ^ p1) & 4u) == 0;
        const uint32_t first = v[g] & 0xFFFFu, second = v[g] >> 16;
        piece[2 * g] = same ? (upper ? 0u : v[g]) : (upper ? second : first);
        piece[2 * g + 1] = same ? (upper ? v[g] : 0u) : (upper ? first : second);
        sel |= ((p0 & 3u) << (p0 & 4u) | (p1 & 3u) << ((p1 & 4u) + (same ? 2u : 0u))) << (8 * g);
      }
    }
  } else {  // one group of four runs
    const uint32_t p0 = fields & 15u;
    if constexpr (N == 1) {
      *reinterpret_cast<u32x4_t*>(at) = piece;
      *reinterpret_cast<uint16_t*>(at + (p0 & 12u)) = (uint16_t)v[0];
      return (p0 & 3u) << (p0 & 12u);
    } else {
      const uint32_t p1 = (fields >> 4) & 15u, first = v[0] & 0xFFFFu;
      const bool same = ((p0 ^ p1) & 12u) == 0;
      const uint32_t second = same ? v[0] & 0xFFFF0000u : v[0] >> 16;
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) piece[r] = ((p0 >> 2) == r ? first : 0u) | ((p1 >> 2) == r ? second : 0u);
      sel = (p0 & 3u) << (p0 & 12u) | (p1 & 3u) << ((p1 & 12u) + (same ? 2u : 0u));
    }
  }
  *reinterpret_cast<u32x4_t*>(at) = piece;
  return sel;
}

template <int N, int M, int TOKS, int ROWS>
struct DirectCfg {
  static constexpr int X_STEP = TOKS * 128, X_SPAN = kSteps * X_STEP;  // bytes of the activations of a step, of a span
  static constexpr int SETS = TOKS == 64 ? 2 : 4;      // spans in flight
  static constexpr bool SPARSE = N <= 2 && N < M;
  static constexpr int B = log2_of(M);
  static constexpr int VPC = 16 / M * N;               // kept values of 16 weights
  static constexpr int BITS = VPC * B;                 // their index fields
  static constexpr int WORDS = 32 % BITS == 0 ? 1 : 2;  // 32-bit words those may lie in
  static constexpr int A_ROWB = SPARSE ? 64 : 128;     // bytes of a weight row per step
  static constexpr int A_STEP = ROWS * A_ROWB;
  static constexpr int CHUNKS = ROWS / 16;             // 16-weight chunks of a lane per span
  static constexpr int S_STEP = SPARSE ? 256 : 0;      // a selector word per pair of rows and lane group
  static constexpr int SPAN = X_SPAN + kSteps * (A_STEP + S_STEP);
  static constexpr int LDS_BYTES = SETS * SPAN;
  static constexpr int VW = (VPC + 1) / 2;             // registers of a chunk's values
  // Word of a row's index stream in which the fields of a chunk begin; `in`: the chunk does not lie past K (else the span's first one's).
  static constexpr int64_t field_word(int span, int chunk, bool in) { return (int64_t)(span * 16 + (in ? chunk : 0)) * BITS >> 5; }
  static_assert(BITS <= 32 && LDS_BYTES <= 160 * 1024, "chunk fields and LDS budget");
};

// What a lane brings of a span: the packed form of its 16-weight chunks and TOKS / 8 16-byte pieces of X.
template <int N, int M, int TOKS, int ROWS>
struct DirectLoads {
  using C = DirectCfg<N, M, TOKS, ROWS>;
  uint32_t v[C::CHUNKS][C::VW], f[C::CHUNKS][C::WORDS];
  u32x4_t x[TOKS / 8];
};

template <int N, int M, int TOKS, int ROWS, bool PACKED>
__global__ void __launch_bounds__(256) nm_direct_kernel(const DirectArgs a) {
  using C = DirectCfg<N, M, TOKS, ROWS>;
  using Loads = DirectLoads<N, M, TOKS, ROWS>;
  static_assert(ROWS == 32 || (ROWS == 16 && TOKS == 16), "blocks");
  constexpr int kXStep = C::X_STEP, kXSpan = C::X_SPAN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kb = lane >> 4;
  const int o0 = (int)blockIdx.x * ROWS, t0 = (int)blockIdx.y * TOKS;
  const int nk = (a.K + 63) >> 6, spans = (nk + kSteps - 1) / kSteps;  // a last step may be short (K % 16 == 0)
  const int64_t nf = (int64_t)a.K / M * N;
  const int64_t nw = (nf * C::B + 31) / 32;

  // a lane's chunks are tid and tid + 256 of the span's rows x 16, its pieces of X tid + 256 i of TOKS rows x 32; rows past the
  // last out-feature or token re-read the last one (never stored)
  const int chunk = tid & 15;
  const bf16_t* v_at[C::CHUNKS];
  const uint32_t* f_at[C::CHUNKS];
  const bf16_t* x_at[TOKS / 8];
#pragma unroll
  for (int u = 0; u < C::CHUNKS; ++u) {
    const int o = o0 + (tid >> 4) + 16 * u;
    const int64_t row = o < a.O ? o : a.O - 1;
    v_at[u] = a.values + row * nf + chunk * C::VPC;
    f_at[u] = a.indices + row * nw;
  }
#pragma unroll
  for (int i = 0; i < TOKS / 8; ++i) {
    const int t = t0 + (tid >> 5) + 8 * i;
    x_at[i] = a.X + (int64_t)(t < a.T ? t : a.T - 1) * a.ldx + (tid & 31) * 8;
  }
  // No load carries a condition: the compiler then counts them, and a span waits for its own loads and not for the next one's too.
  // What lies past K is fetched from the span's first positions instead and cleared on its way into LDS.
  auto fetch = [&](Loads& d, int span) {
    const int k_left = a.K - span * 256;
    const bool in = chunk * 16 < k_left;
#pragma unroll
    for (int u = 0; u < C::CHUNKS; ++u) {
      const bf16_t* src = v_at[u] + (int64_t)span * (16 * C::VPC) - (in ? 0 : chunk * C::VPC);
      if constexpr (C::VPC % 8 == 0) {
        const uint4 q = *reinterpret_cast<const uint4*>(src);
        d.v[u][0] = q.x; d.v[u][1] = q.y; d.v[u][2] = q.z; d.v[u][3] = q.w;
      } else if constexpr (C::VPC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < C::VW; i += 2) {
          const uint2 q = *reinterpret_cast<const uint2*>(src + 2 * i);
          d.v[u][i] = q.x; d.v[u][i + 1] = q.y;
        }
      } else if constexpr (C::VPC % 2 == 0) {
#pragma unroll
        for (int i = 0; i < C::VW; ++i) d.v[u][i] = *reinterpret_cast<const uint32_t*>(src + 2 * i);
      } else {
        d.v[u][0] = src[0];
      }
      const int64_t word = C::field_word(span, chunk, in);
      d.f[u][0] = f_at[u][word];
      if constexpr (C::WORDS == 2) d.f[u][1] = f_at[u][word + 1 < nw ? word + 1 : word];
    }
    const int back = (tid & 31) * 8 < k_left ? 0 : (tid & 31) * 8;
#pragma unroll
    for (int i = 0; i < TOKS / 8; ++i) d.x[i] = *reinterpret_cast<const u32x4_t*>(x_at[i] + (int64_t)span * 256 - back);
  };
  // the same into the span's LDS buffer, the weight decoded.  16-byte pieces of a row are XOR-swizzled with the row.
  auto put = [&](Loads& d, int span, unsigned char* buf) {
    const int k_left = a.K - span * 256;
    if (k_left < 256) {  // the last span
      if (chunk * 16 >= k_left)
#pragma unroll
        for (int u = 0; u < C::CHUNKS; ++u)
#pragma unroll
          for (int i = 0; i < C::VW; ++i) d.v[u][i] = 0;
      if ((tid & 31) * 8 >= k_left)
#pragma unroll
        for (int i = 0; i < TOKS / 8; ++i) d.x[i] = u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < C::CHUNKS; ++u) {
      const int row = (tid >> 4) + 16 * u, step = chunk >> 2, c = chunk & 3;
      // (at six bits a chunk, where a span ends inside a word, sixteen chunks are three words: every span starts on one)
      const uint32_t shift = ((uint32_t)chunk * C::BITS) & 31;
      uint32_t fields = d.f[u][0] >> shift;
      if constexpr (C::WORDS == 2) fields = __builtin_amdgcn_alignbit(d.f[u][1], d.f[u][0], shift);
      unsigned char* at = buf + kXSpan + step * C::A_STEP + row * C::A_ROWB;
      if constexpr (C::SPARSE) {
        const uint32_t sel = put_sparse_piece<N, M>(at + (c ^ ((row >> 1) & 3)) * 16, d.v[u], fields);
        *reinterpret_cast<uint16_t*>(buf + kXSpan + kSteps * C::A_STEP + step * C::S_STEP + (row & 15) * 16 + c * 4 +
                                     (row >> 4) * 2) = (uint16_t)sel;
      } else {
        const int key = row & 7;
        *reinterpret_cast<u32x4_t*>(at + ((2 * c) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
        *reinterpret_cast<u32x4_t*>(at + ((2 * c + 1) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < C::VPC; ++j) {
          const uint32_t pos = (uint32_t)(j / N * M) + ((fields >> (C::B * j)) & (uint32_t)(M - 1));
          *reinterpret_cast<uint16_t*>(at + (((2 * c + (pos >> 3)) ^ key) * 16) + (pos & 7) * 2) =
              (uint16_t)(d.v[u][j / 2] >> (16 * (j & 1)));
        }
      }
    }
#pragma unroll
    for (int i = 0; i < TOKS / 8; ++i) {
      const int row = (tid >> 5) + 8 * i, p = tid & 31;
      *reinterpret_cast<u32x4_t*>(buf + (p >> 3) * kXStep + row * 128 + (((p & 7) ^ (row & 7)) * 16)) = d.x[i];
    }
  };

  f32x4_t acc[2];
  // a lane holds out-features o_lane + 16 i .. + 3 of token r16 of its wave's 16; in blocks of 16 or 32 tokens a wave holds one
  // block of 16 out-features (acc[0]) of the tokens `wave_t`, the lower one in the even waves
  const int half = ROWS == 32 ? wave & 1 : 0, wave_t = ROWS == 32 ? wave >> 1 : wave;
  const int o_lane = o0 + kb * 4;
  auto bias_of = [&](int i) {
    f32x4_t b = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (a.bias != nullptr)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (o_lane + 16 * i + e < a.O) b[e] = a.bias[o_lane + 16 * i + e];
    return b;
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) acc[i] = PACKED ? f32x4_t{0.f, 0.f, 0.f, 0.f} : bias_of(TOKS == 64 ? i : half);

  auto multiply = [&](const unsigned char* buf, int span) {
    const int steps = nk - span * kSteps < kSteps ? nk - span * kSteps : kSteps;
    if (t0 + wave * 16 >= a.T) return;  // (wave-uniform: no token of this wave is stored)
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
      if (st >= steps) break;
      const unsigned char* x = buf + st * kXStep + (wave * 16 + r16) * 128;
      const unsigned char* w = buf + kXSpan + st * C::A_STEP + r16 * C::A_ROWB;
      const int xk = r16 & 7;
      if constexpr (C::SPARSE) {
        const int at = (kb ^ ((r16 >> 1) & 3)) * 16;
        const u32x4_t a0 = *reinterpret_cast<const u32x4_t*>(w + at);
        const u32x4_t a1 = *reinterpret_cast<const u32x4_t*>(w + 16 * C::A_ROWB + at);
        const int sel = (int)*reinterpret_cast<const uint32_t*>(buf + kXSpan + kSteps * C::A_STEP + st * C::S_STEP + r16 * 16 + kb * 4);
        const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(x + ((kb ^ xk) * 16));
        const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(x + (((4 + kb) ^ xk) * 16));
        const u32x8_t b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc[0] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, a0), __builtin_bit_cast(bf16x16_t, b), acc[0], sel, 0, 0);
        acc[1] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, a1), __builtin_bit_cast(bf16x16_t, b), acc[1], sel, 0, 1);
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int at = ((PACKED ? 2 * kb + h : 4 * h + kb) ^ xk) * 16;
          const u32x4_t a0 = *reinterpret_cast<const u32x4_t*>(w + at);
          const u32x4_t a1 = *reinterpret_cast<const u32x4_t*>(w + 16 * C::A_ROWB + at);
          const u32x4_t b = *reinterpret_cast<const u32x4_t*>(x + at);
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a0), __builtin_bit_cast(bf16x8_t, b), acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a1), __builtin_bit_cast(bf16x8_t, b), acc[1], 0, 0, 0);
        }
      }
    }
  };

  // The same for one block of out-features, in the same order.
  auto multiply_block = [&](const unsigned char* buf, int span) {
    const unsigned char* x = buf + (wave_t * 16 + r16) * 128;
    const unsigned char* w = buf + kXSpan + (half * 16 + r16) * C::A_ROWB;
    const int xk = r16 & 7;
    auto one = [&](int st) {
      if constexpr (C::SPARSE) {
        const u32x4_t a0 = *reinterpret_cast<const u32x4_t*>(w + st * C::A_STEP + (kb ^ ((r16 >> 1) & 3)) * 16);
        const uint32_t sel = *reinterpret_cast<const uint32_t*>(buf + kXSpan + kSteps * C::A_STEP + st * C::S_STEP + r16 * 16 + kb * 4);
        const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(x + st * kXStep + ((kb ^ xk) * 16));
        const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(x + st * kXStep + (((4 + kb) ^ xk) * 16));
        const u32x8_t b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc[0] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, a0), __builtin_bit_cast(bf16x16_t, b), acc[0],
                                                           (int)(sel >> (16 * half)), 0, 0);
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int at = ((PACKED ? 2 * kb + h : 4 * h + kb) ^ xk) * 16;
          const u32x4_t a0 = *reinterpret_cast<const u32x4_t*>(w + st * C::A_STEP + at);
          const u32x4_t b = *reinterpret_cast<const u32x4_t*>(x + st * kXStep + at);
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a0), __builtin_bit_cast(bf16x8_t, b), acc[0], 0, 0, 0);
        }
      }
    };
    const int steps = nk - span * kSteps;
    if (steps >= kSteps) {
#pragma unroll
      for (int st = 0; st < kSteps; ++st) one(st);
    } else {
      for (int st = 0; st < steps; ++st) one(st);
    }
  };

  if constexpr (TOKS == 64) {
    // Two register sets and two LDS buffers.  A buffer is written again two spans later: between the two lies a barrier
    // that every wave reaches only after it has multiplied the first.  A single span goes by itself: the loads of a second one,
    // unused, took 0.2 to 0.4 us.
    Loads even, odd;
    fetch(even, 0);
    if (spans == 1) {
      put(even, 0, smem);
      __syncthreads();
      multiply(smem, 0);
    } else {
      fetch(odd, 1);
      int span = 0;
      for (; span + 3 < spans; span += 2) {
        put(even, span, smem);
        fetch(even, span + 2);
        __syncthreads();
        multiply(smem, span);
        put(odd, span + 1, smem + C::SPAN);
        fetch(odd, span + 3);
        __syncthreads();
        multiply(smem + C::SPAN, span + 1);
      }
      if (span + 2 < spans) {  // three are left
        put(even, span, smem);
        fetch(even, span + 2);
        __syncthreads();
        multiply(smem, span);
        put(odd, span + 1, smem + C::SPAN);
        __syncthreads();
        multiply(smem + C::SPAN, span + 1);
        span += 2;
      }
      put(even, span, smem);
      __syncthreads();
      multiply(smem, span);
      if (span + 1 < spans) {
        put(odd, span + 1, smem + C::SPAN);
        __syncthreads();
        multiply(smem + C::SPAN, span + 1);
      }
    }
  } else {
    // Four spans at a time, all their loads in flight together and one barrier for them.
    Loads d[4];
    const bool stored = wave_t * 16 < TOKS && t0 + wave_t * 16 < a.T;  // some token of this wave's 16 is
    auto fetch_four = [&](int first) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (first + u < spans) fetch(d[u], first + u);
    };
    fetch_four(0);
    for (int first = 0; first < spans; first += 4) {
      if (first) __syncthreads();  // the four before have been multiplied
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (first + u < spans) put(d[u], first + u, smem + u * C::SPAN);
      fetch_four(first + 4);
      __syncthreads();
      if (stored) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (first + u < spans) multiply_block(smem + u * C::SPAN, first + u);
      }
    }
    if (!stored) return;
  }

  const int t = t0 + (TOKS == 64 ? wave : wave_t) * 16 + r16;
  if (t >= a.T) return;
#pragma unroll
  for (int i = 0; i < (TOKS == 64 ? 2 : 1); ++i) {
    const int o = o_lane + 16 * (TOKS == 64 ? i : half);
    if (o >= a.O) continue;
    f32x4_t y = PACKED ? acc[i] + bias_of(TOKS == 64 ? i : half) : acc[i];
    if (a.again) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (__builtin_isnan(y[e]) && o + e < a.O)
          y[e] = gather_output(a.values, a.indices, a.K, N, M, a.X + t * a.ldx, a.bias, o + e);
    }
    const uint32_t p[2] = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    if (a.out_bf16) {
      bf16_t* dst = reinterpret_cast<bf16_t*>(a.Y) + t * a.ldy + o;
      if (a.pieces) *reinterpret_cast<uint2*>(dst) = make_uint2(p[0], p[1]);
      else
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (o + e < a.O) dst[e] = (bf16_t)(p[e >> 1] >> (16 * (e & 1)));
    } else {
      float* dst = reinterpret_cast<float*>(a.Y) + t * a.ldy + o;
      if (a.pieces) *reinterpret_cast<f32x4_t*>(dst) = y;
      else
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (o + e < a.O) dst[e] = y[e];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The same for more tokens: blocks of 64 out-features x 128 tokens on eight waves, in the tiled kernel's summation order.
// Against the pre-pass and the tiled kernel it saves a launch (about 4 us) and the weight's way through memory, and it decodes the
// weight once per 128 tokens: it wins while its blocks are one round or two on the chip and the reduction is not long (the choice is
// nm_spmm.hip's).  A whole call in a graph, the two launches and here: 1576 x 1024 -> 1024 at 2:8 10.7 and 8.4 us, 788 x 768 -> 2304 at 1:8 10.8
// and 6.9, 6304 x 256 -> 256 at 1:8 6.7 and 4.3, 1579 x 1000 -> 1001 in fp32 12.6 and 11.2; 2048 tokens x 3072 -> 768, which stays with the
// two, would lose.
// What bounds it: a span of 128 reduction positions brings 40 KB into a unit, 0.4 us at the 100 GB/s that a unit gets, and
// moves 137 KB through its LDS; it takes 0.5 us at 1:16 and 0.59 at 2:8 (LDS busy for 0.37 of a unit's cycles, matrix pipes for 0.1).  So the loads of two spans are in flight, the lanes decode in
// registers, and two whole spans at a time run without conditions.  Slower, 1576 x 1024 -> 1024 on the card where this took 8.9: 2-byte LDS
// writes per kept value (9.4), four waves of 64 x 32 (12.0), half the waves bringing and half multiplying (10.3), activations straight
// from memory into the operand registers (12.8: rows 2 KB apart share the first-level cache's lines).
// ---------------------------------------------------------------------------------------------
template <int N, int M>
struct WideCfg {
  static constexpr int ROWS = 64, TOKS = 128, STEPS = 2;   // of a block; 64-wide steps per span
  static constexpr int NW = 8, NT = NW * 64;
  static constexpr int WO = 2, WT = 4;                     // waves along out-features, along tokens
  static constexpr int OT = ROWS / 16 / WO, TT = TOKS / 16 / WT;
  static constexpr bool SPARSE = N <= 2 && N < M;
  static constexpr int B = log2_of(M);
  static constexpr int VPC = 16 / M * N;
  static constexpr int BITS = VPC * B;
  static constexpr int WORDS = 32 % BITS == 0 ? 1 : 2;
  static constexpr int VW = (VPC + 1) / 2;
  static constexpr int PIECES = TOKS * STEPS * 8 / NT;     // of X, per lane and span; of the weight a chunk of 16
  static constexpr int X_STEP = TOKS * 128, X_SPAN = STEPS * X_STEP;
  static constexpr int A_ROWB = SPARSE ? 64 : 128;
  static constexpr int A_STEP = ROWS * A_ROWB, S_STEP = SPARSE ? ROWS * 8 : 0;
  static constexpr int SPAN = X_SPAN + STEPS * (A_STEP + S_STEP);
  static constexpr int LDS_BYTES = 2 * SPAN;
  // A span's index fields begin on a word of the row's stream, or ODD_BITS into one where the span is an odd one.
  static constexpr int SPAN_BITS = 8 * BITS, ODD_BITS = SPAN_BITS % 32;
  // The word in which the fields of a chunk begin; `in`: the chunk does not lie past K (else the row's first one).
  static constexpr int64_t field_word(int span, int begin, int chunk, bool in) {
    return in ? ((int64_t)span * SPAN_BITS >> 5) + ((begin + chunk * BITS) >> 5) : 0;
  }
  static_assert(NT == ROWS * STEPS * 4 && NW * wave_tile_slice_bytes<OT, 4>() <= LDS_BYTES && LDS_BYTES <= 160 * 1024, "LDS budget");
};

template <int N, int M>
struct WideLoads {
  using C = WideCfg<N, M>;
  uint32_t v[C::VW], f[C::WORDS];
  u32x4_t x[C::PIECES];
};

template <int N, int M, bool WHOLE>
__global__ void __launch_bounds__(512) nm_direct_wide_kernel(const DirectArgs a) {
  using C = WideCfg<N, M>;
  using Loads = WideLoads<N, M>;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kb = lane >> 4;
  const int wo = wave % C::WO, wt = wave / C::WO;
  const int o0 = (int)blockIdx.x * C::ROWS, t0 = (int)blockIdx.y * C::TOKS;
  const int nk = (a.K + 63) >> 6, spans = (nk + C::STEPS - 1) / C::STEPS;
  const int64_t nf = (int64_t)a.K / M * N;
  const int64_t nw = (nf * C::B + 31) / 32;

  // Where a lane's chunk and pieces of span 0 lie; rows past the last out-feature or token re-read the last one (never stored).
  // A span ends on a word of the index stream or in the middle of one: `begin` is where in its first word it begins.
  const int row = tid >> 3, chunk = tid & 7;
  const int64_t o_row = o0 + row < a.O ? o0 + row : a.O - 1;
  const bf16_t* const v_at = a.values + o_row * nf + chunk * C::VPC;
  const uint32_t* const f_at = a.indices + o_row * nw;
  uint32_t x_off[C::PIECES];
  const unsigned char* x_base = reinterpret_cast<const unsigned char*>(a.X + (int64_t)t0 * a.ldx);
#pragma unroll
  for (int i = 0; i < C::PIECES; ++i) {
    int t = (tid >> 4) + C::NT / 16 * i;
    if (t0 + t >= a.T) t = a.T - 1 - t0;
    x_off[i] = (uint32_t)t * (uint32_t)(a.ldx * 2) + (uint32_t)(tid & 15) * 16;
  }
  auto load_run = [](const bf16_t* src, auto count, uint32_t* out) {  // `count` values at an address aligned to them
    constexpr int n = decltype(count)::value;
    if constexpr (n % 8 == 0) {
#pragma unroll
      for (int i = 0; i < n / 2; i += 4) {
        const uint4 q = *reinterpret_cast<const uint4*>(src + 2 * i);
        out[i] = q.x; out[i + 1] = q.y; out[i + 2] = q.z; out[i + 3] = q.w;
      }
    } else if constexpr (n % 4 == 0) {
#pragma unroll
      for (int i = 0; i < n / 2; i += 2) {
        const uint2 q = *reinterpret_cast<const uint2*>(src + 2 * i);
        out[i] = q.x; out[i + 1] = q.y;
      }
    } else if constexpr (n % 2 == 0) {
#pragma unroll
      for (int i = 0; i < n / 2; ++i) out[i] = *reinterpret_cast<const uint32_t*>(src + 2 * i);
    } else {
#pragma unroll
      for (int i = 0; i < n; ++i) out[i / 2] = i & 1 ? out[i / 2] | ((uint32_t)src[i] << 16) : (uint32_t)src[i];
    }
  };
  // The loads of a span carry no condition, so that the compiler counts them and a span waits for its own and not for those of
  // the next one (with conditions it drains them all: a round trip to memory per span).  What lies past K is fetched from the
  // span's first positions instead and cleared on its way into LDS.
  auto fetch = [&](Loads& d, int span, int begin) {
    const int k_left = a.K - span * 128;  // reduction positions from the span on
    const bool in = chunk * 16 < k_left, half_in = chunk * 16 + 8 < k_left;
    const bf16_t* src = v_at + (int64_t)span * (8 * C::VPC) - (in ? 0 : chunk * C::VPC);
    if constexpr (WHOLE) {
      load_run(src, std::integral_constant<int, C::VPC>{}, d.v);
    } else {  // K % 16 == 8: rows begin on half a chunk, and the last chunk may be half of one
      constexpr int HALF = C::VPC / 2;
      const bf16_t* second = src + (half_in ? HALF : 0);
      if constexpr (HALF % 2 == 0) {
        load_run(src, std::integral_constant<int, HALF>{}, d.v);
        load_run(second, std::integral_constant<int, HALF>{}, d.v + HALF / 2);
      } else {
#pragma unroll
        for (int i = 0; i < C::VW; ++i) d.v[i] = 0;
#pragma unroll
        for (int j = 0; j < C::VPC; ++j) d.v[j / 2] |= (uint32_t)(j < HALF ? src[j] : second[j - HALF]) << (16 * (j & 1));
      }
    }
    const int64_t word = C::field_word(span, begin, chunk, in);
    d.f[0] = f_at[word];
    if constexpr (C::WORDS == 2) d.f[1] = f_at[word + 1 < nw ? word + 1 : word];
    const unsigned char* x = x_base + (int64_t)span * 256;
    const uint32_t back = (tid & 15) * 8 < k_left ? 0u : (uint32_t)(tid & 15) * 16;
#pragma unroll
    for (int i = 0; i < C::PIECES; ++i) d.x[i] = *reinterpret_cast<const u32x4_t*>(x + (x_off[i] - back));
  };
  auto clear_past = [&](Loads& d, int span) {  // the last span, where K ends inside it
    const int k_left = a.K - span * 128;
#pragma unroll
    for (int j = 0; j < C::VPC; ++j)
      if (chunk * 16 + (j < C::VPC / 2 ? 0 : 8) >= k_left) d.v[j / 2] &= j & 1 ? 0xFFFFu : 0xFFFF0000u;
    if ((tid & 15) * 8 >= k_left)
#pragma unroll
      for (int i = 0; i < C::PIECES; ++i) d.x[i] = u32x4_t{0, 0, 0, 0};
  };
  // a span into its LDS buffer, the weight decoded; 16-byte pieces of a row are XOR-swizzled with the row
  auto put = [&](Loads& d, int span, unsigned char* buf, int begin, auto whole_span) {
    if constexpr (!decltype(whole_span)::value)
      if (a.K - span * 128 < 128) clear_past(d, span);
    const int step = chunk >> 2, c = chunk & 3;
    const int shift = (begin + chunk * C::BITS) & 31;
    uint32_t fields = d.f[0] >> shift;
    if constexpr (C::WORDS == 2) fields = __builtin_amdgcn_alignbit(d.f[1], d.f[0], shift);
    unsigned char* at = buf + C::X_SPAN + step * C::A_STEP + row * C::A_ROWB;
    if constexpr (C::SPARSE) {
      const uint32_t sel = put_sparse_piece<N, M>(at + (c ^ ((row >> 1) & 3)) * 16, d.v, fields);
      *reinterpret_cast<uint16_t*>(buf + C::X_SPAN + C::STEPS * C::A_STEP + step * C::S_STEP + (row >> 5) * 256 + (row & 15) * 16 +
                                   c * 4 + ((row >> 4) & 1) * 2) = (uint16_t)sel;
    } else {
      const int key = row & 7;
      *reinterpret_cast<u32x4_t*>(at + ((2 * c) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
      *reinterpret_cast<u32x4_t*>(at + ((2 * c + 1) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
      // (the index fields of groups past K may be anything: their values, zero, stay inside their groups)
#pragma unroll
      for (int j = 0; j < C::VPC; ++j) {
        const uint32_t pos = (uint32_t)(j / N * M) + ((fields >> (C::B * j)) & (uint32_t)(M - 1));
        *reinterpret_cast<uint16_t*>(at + (((2 * c + (pos >> 3)) ^ key) * 16) + (pos & 7) * 2) = (uint16_t)(d.v[j / 2] >> (16 * (j & 1)));
      }
    }
#pragma unroll
    for (int i = 0; i < C::PIECES; ++i) {
      const int t = (tid >> 4) + C::NT / 16 * i, p = tid & 15;
      *reinterpret_cast<u32x4_t*>(buf + (p >> 3) * C::X_STEP + t * 128 + (((p & 7) ^ (t & 7)) * 16)) = d.x[i];
    }
  };

  f32x4_t acc[C::OT][C::TT];
  const int o_wave = o0 + wo * C::OT * 16;
#pragma unroll
  for (int i = 0; i < C::OT; ++i) {
    f32x4_t b = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (a.bias != nullptr)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (o_wave + 16 * i + kb * 4 + e < a.O) b[e] = a.bias[o_wave + 16 * i + kb * 4 + e];
#pragma unroll
    for (int j = 0; j < C::TT; ++j) acc[i][j] = b;
  }

  auto multiply = [&](const unsigned char* buf, int steps) {
#pragma unroll
    for (int st = 0; st < C::STEPS; ++st) {
      if (st >= steps) break;
      const unsigned char* x = buf + st * C::X_STEP + (wt * C::TT * 16 + r16) * 128;
      const unsigned char* w = buf + C::X_SPAN + st * C::A_STEP + (wo * C::OT * 16 + r16) * C::A_ROWB;
      const int xk = r16 & 7;
      if constexpr (C::SPARSE) {
        u32x4_t af[C::OT];
        int sel[C::OT / 2];
        u32x8_t b[C::TT];
#pragma unroll
        for (int i = 0; i < C::OT; ++i) af[i] = *reinterpret_cast<const u32x4_t*>(w + i * 16 * C::A_ROWB + (kb ^ ((r16 >> 1) & 3)) * 16);
#pragma unroll
        for (int i = 0; i < C::OT / 2; ++i)
          sel[i] = (int)*reinterpret_cast<const uint32_t*>(buf + C::X_SPAN + C::STEPS * C::A_STEP + st * C::S_STEP +
                                                           (wo * C::OT / 2 + i) * 256 + r16 * 16 + kb * 4);
#pragma unroll
        for (int j = 0; j < C::TT; ++j) {
          const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(x + j * 2048 + ((kb ^ xk) * 16));
          const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(x + j * 2048 + (((4 + kb) ^ xk) * 16));
          b[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
#pragma unroll
        for (int j = 0; j < C::TT; ++j) {
#pragma unroll
          for (int i = 0; i < C::OT; i += 2) {
            acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, af[i]), __builtin_bit_cast(bf16x16_t, b[j]), acc[i][j], sel[i / 2], 0, 0);
            acc[i + 1][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, af[i + 1]), __builtin_bit_cast(bf16x16_t, b[j]), acc[i + 1][j], sel[i / 2], 0, 1);
          }
        }
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int at = ((4 * h + kb) ^ xk) * 16;
          u32x4_t af[C::OT], b[C::TT];
#pragma unroll
          for (int i = 0; i < C::OT; ++i) af[i] = *reinterpret_cast<const u32x4_t*>(w + i * 16 * C::A_ROWB + at);
#pragma unroll
          for (int j = 0; j < C::TT; ++j) b[j] = *reinterpret_cast<const u32x4_t*>(x + j * 2048 + at);
#pragma unroll
          for (int j = 0; j < C::TT; ++j)
#pragma unroll
            for (int i = 0; i < C::OT; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, af[i]), __builtin_bit_cast(bf16x8_t, b[j]), acc[i][j], 0, 0, 0);
        }
      }
    }
  };

  // Two register sets and two LDS buffers, as in the kernel above.
  constexpr int p0 = 0, p1 = C::ODD_BITS;
  Loads even, odd;
  fetch(even, 0, p0);
  if (spans == 1) {
    put(even, 0, smem, p0, std::false_type{});
    __syncthreads();
    multiply(smem, nk);
  } else {
    fetch(odd, 1, p1);
    int span = 0;
    for (; span + 3 < spans; span += 2) {  // two whole spans: no conditions, so that a span's decoding and the products interleave
      put(even, span, smem, p0, std::true_type{});
      fetch(even, span + 2, p0);
      __syncthreads();
      multiply(smem, C::STEPS);
      put(odd, span + 1, smem + C::SPAN, p1, std::true_type{});
      fetch(odd, span + 3, p1);
      __syncthreads();
      multiply(smem + C::SPAN, C::STEPS);
    }
    if (span + 2 < spans) {  // three are left, two of them whole
      put(even, span, smem, p0, std::true_type{});
      fetch(even, span + 2, p0);
      __syncthreads();
      multiply(smem, C::STEPS);
      put(odd, span + 1, smem + C::SPAN, p1, std::true_type{});
      __syncthreads();
      multiply(smem + C::SPAN, C::STEPS);
      span += 2;
    }
    put(even, span, smem, p0, std::false_type{});
    __syncthreads();
    multiply(smem, nk - span * C::STEPS);
    if (span + 1 < spans) {
      put(odd, span + 1, smem + C::SPAN, p1, std::false_type{});
      __syncthreads();
      multiply(smem + C::SPAN, nk - (span + 1) * C::STEPS);
    }
  }

  const int64_t row0 = t0 + wt * C::TT * 16, col0 = o_wave;
  if (a.again) {
    uint32_t which = 0;  // bit 4 (i TT + j) + e
    static_assert(C::OT * C::TT <= 8, "one bit per sum");
#pragma unroll
    for (int i = 0; i < C::OT; ++i)
#pragma unroll
      for (int j = 0; j < C::TT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) which |= (__builtin_isnan(acc[i][j][e]) ? 1u : 0u) << (4 * (i * C::TT + j) + e);
    for (; which != 0; which &= which - 1) {
      const int bit = __ffs(which) - 1;
      const int64_t t = row0 + (bit >> 2) % C::TT * 16 + r16, o = col0 + (bit >> 2) / C::TT * 16 + kb * 4 + (bit & 3);
      if (t >= a.T || o >= a.O) continue;
      const float y = gather_output(a.values, a.indices, a.K, N, M, a.X + t * a.ldx, a.bias, o);
#pragma unroll
      for (int i = 0; i < C::OT; ++i)
#pragma unroll
        for (int j = 0; j < C::TT; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (bit == 4 * (i * C::TT + j) + e) acc[i][j][e] = y;
    }
  }
  __syncthreads();  // every wave is done with the buffers
  auto get = [&](int i, int j) { return __builtin_bit_cast(u32x4_t, acc[i][j]); };
  unsigned char* slice = smem + wave * wave_tile_slice_bytes<C::OT, 4>();
  if (a.rows16) {
    if (a.out_bf16) write_wave_tile_pieces<C::OT, C::TT, 2>(slice, lane, get, a.Y, a.ldy, row0, col0, a.T, a.O);
    else write_wave_tile_pieces<C::OT, C::TT, 4>(slice, lane, get, a.Y, a.ldy, row0, col0, a.T, a.O);
  } else {
    if (a.out_bf16) write_wave_tile_rows<C::OT, C::TT, 2>(slice, lane, get, a.Y, a.ldy, row0, col0, a.T, a.O);
    else write_wave_tile_rows<C::OT, C::TT, 4>(slice, lane, get, a.Y, a.ldy, row0, col0, a.T, a.O);
  }
}

template <int N, int M, int TOKS, bool PACKED, int ROWS = 32>
hipError_t launch_tokens(const DirectArgs& g, hipStream_t s) {
  using C = DirectCfg<N, M, TOKS, ROWS>;
  auto kern = nm_direct_kernel<N, M, TOKS, ROWS, PACKED>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((g.O + ROWS - 1) / ROWS), (unsigned)((g.T + TOKS - 1) / TOKS)), dim3(256),
                     C::LDS_BYTES, s, g);
  return hipGetLastError();
}

// Blocks of 16 tokens: of 16 out-features, which halves what a lane decodes before the first product, while each has a unit to itself,
// and where several passes of four spans follow one another; of 32 for a wide shallow weight, whose blocks of 16 are many and mostly
// start and end.  32 and 16 (in a graph): 8 tokens x 768 -> 1000 at 4:8 4.25 and 3.74 us, 16 x 1024 -> 768 at 1:16 4.14 and 3.63, 1 x 4096
// -> 16384 at 4:8 35.1 and 29.2, 16 x 2048 -> 8192 at 4:8 9.5 and 8.2; 16 x 1024 -> 8192 at 4:8 5.06 and 5.22, -> 16384 at 1:8 5.2 and 6.6.
template <int N, int M, bool PACKED>
hipError_t launch_sixteen(const DirectArgs& g, hipStream_t s) {
  if (g.O <= 16 * 256 || g.K > 1024) return launch_tokens<N, M, 16, PACKED, 16>(g, s);
  return launch_tokens<N, M, 16, PACKED>(g, s);
}

// Up to 16 tokens a block of 64 would bring, store and skip rows of zeros, and its two spans in flight make two round trips of
// K = 768; up to 32 tokens the same holds for blocks of 32 while round trips bound the launch (in blocks of 64 and of 32, in a graph:
// 20 tokens x 768 -> 1000 at 2:8 5.3 and 4.8 us, at 4:8 5.5 and 4.6, 32 x 3072 -> 3072 at 1:8 11.7 and 10.4, x 2048 -> 4096 at 4:8 10.6 and
// 9.0, x 1024 -> 32768 at 1:8 19.2 and 16.7).  A large weight is bound by what its blocks pull in and decode, and there the longer run of
// a block of 64 is the faster one.  The limits are in kept values, near where the two cross: 2:4 form 32 x 2048 -> 8192 at 2:8
// (4 M) 9.3 and 8.8, x 3072 -> 16384 (12 M) 23.8 and 25.0, x 4096 -> 32768 (32 M) 56.9 and 63.0; dense form 32 x 3072 -> 8192 at 4:8
// (12 M) 14.6 and 14.2, 3072 -> 16384 (24 M) 27.8 and 28.1, 20 x 4096 -> 16384 (32 M) 35.4 and 37.8.
template <int N, int M, bool PACKED>
hipError_t launch_level(const DirectArgs& g, hipStream_t s) {
  if (g.T <= 16) return launch_sixteen<N, M, PACKED>(g, s);
  const int64_t kept = (int64_t)g.O * (g.K / M * N);
  if (g.T <= 32 && kept < (N <= 2 ? 1 << 23 : 1 << 24)) return launch_tokens<N, M, 32, PACKED>(g, s);
  return launch_tokens<N, M, 64, PACKED>(g, s);
}

template <int N, int M, bool WHOLE>
hipError_t launch_wide(const DirectArgs& g, hipStream_t s) {
  using C = WideCfg<N, M>;
  auto kern = nm_direct_wide_kernel<N, M, WHOLE>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((g.O + C::ROWS - 1) / C::ROWS), (unsigned)((g.T + C::TOKS - 1) / C::TOKS)), dim3(C::NT),
                     C::LDS_BYTES, s, g);
  return hipGetLastError();
}

template <int N, int M>
hipError_t launch_wide_level(const DirectArgs& g, hipStream_t s) {
  if constexpr (M < 16)
    if (g.K % 16) return launch_wide<N, M, false>(g, s);
  return launch_wide<N, M, true>(g, s);
}

}  // namespace

// The levels whose packed form the matrix instructions cannot read as it lies and whose 16 weights have at most 32 bits
// of fields.
bool direct_level(int N, int M) {
  switch (N * 32 + M) {
    case 1 * 32 + 4: case 3 * 32 + 4: case 1 * 32 + 8: case 2 * 32 + 8: case 3 * 32 + 8: case 4 * 32 + 8:
    case 1 * 32 + 16: case 2 * 32 + 16: case 4 * 32 + 16: return true;
    default: return false;
  }
}

// Words of a row's index stream that the kernels of the level load at a reduction of K, up to the last one of them.
template <int N, int M>
static int64_t index_words_reached(bool wide, int64_t K) {
  const int64_t nw = (K / M * N * log2_of(M) + 31) / 32;
  const int nk = (int)((K + 63) / 64);
  int64_t end = 0;
  auto load = [&](int64_t word, bool two) {
    end = std::max(end, word + 1);
    if (two) end = std::max(end, (word + 1 < nw ? word + 1 : word) + 1);
  };
  if (wide) {
    using C = WideCfg<N, M>;
    const int spans = (nk + C::STEPS - 1) / C::STEPS;
    auto fetch = [&](int span, int begin) {
      for (int chunk = 0; chunk < 8; ++chunk)
        load(C::field_word(span, begin, chunk, chunk * 16 < (int)K - span * 128), C::WORDS == 2);
    };
    for (int span = 0; span < spans; ++span) fetch(span, span % 2 ? C::ODD_BITS : 0);
  } else {
    using C = DirectCfg<N, M, 64, 32>;
    for (int span = 0; span < (nk + kSteps - 1) / kSteps; ++span)
      for (int chunk = 0; chunk < 16; ++chunk)
        load(C::field_word(span, chunk, chunk * 16 < (int)K - span * 256), C::WORDS == 2);
  }
  return end;
}

// Not in the public header, for tests: the above; -1 where the level is not one of these kernels'.
extern "C" int64_t nm_internal_direct_index_words(int32_t wide, int32_t N, int32_t M, int64_t K) {
  switch (N * 32 + M) {
#define X(n, m) case n * 32 + m: return index_words_reached<n, m>(wide != 0, K);
    X(1, 4) X(3, 4) X(1, 8) X(2, 8) X(3, 8) X(4, 8) X(1, 16) X(2, 16) X(4, 16)
#undef X
    default: return -1;
  }
}

// The caller has checked the operands (K % 64 == 0, or K % 16 == 0 in the tiled kernel's order; 16-byte aligned X rows and
// values, sizes as the tiled kernel's).  wide: blocks of 64 out-features x 128 tokens, the tiled kernel's order only, and K % 8 == 0 is
// enough (at M = 16 K is a multiple of 16 anyway).  again: a prepared call multiplies the layer on the ragged form of the tiled
// kernel also where K % 64 == 0, so what that form does with sums that end as NaN is done here.
hipError_t launch_direct(const SpmmArgs& a, bool packed_order, bool wide, bool again, hipStream_t s) {
  DirectArgs g;
  g.values = a.values; g.indices = a.indices; g.X = a.X; g.bias = a.bias; g.Y = a.Y;
  g.ldx = a.ldx; g.ldy = a.ldy;
  g.O = (int32_t)a.O; g.K = (int32_t)a.K; g.T = (int32_t)a.T;
  g.out_bf16 = a.out_bf16;
  g.pieces = (a.O % 4 == 0) && (a.ldy % 4 == 0) && ((uintptr_t)a.Y & (a.out_bf16 ? 7u : 15u)) == 0;
  const int per_piece = a.out_bf16 ? 8 : 4;
  g.again = again || a.K % 64 != 0;
  g.rows16 = (a.O % per_piece == 0) && (a.ldy % per_piece == 0) && ((uintptr_t)a.Y & 15u) == 0;
  if (wide) {
    switch (a.N * 32 + a.M) {
#define X(n, m) case n * 32 + m: return launch_wide_level<n, m>(g, s);
      X(1, 4) X(3, 4) X(1, 8) X(2, 8) X(3, 8) X(4, 8) X(1, 16) X(2, 16) X(4, 16)
#undef X
      default: return hipErrorInvalidValue;
    }
  }
  switch (a.N * 32 + a.M) {
#define X(n, m)                                                                              \
  case n * 32 + m:                                                                           \
    return packed_order ? launch_level<n, m, true>(g, s) : launch_level<n, m, false>(g, s);
    X(1, 4) X(1, 8) X(2, 8) X(4, 8) X(1, 16) X(2, 16) X(4, 16)
#undef X
    case 3 * 32 + 4: return launch_level<3, 4, false>(g, s);
    case 3 * 32 + 8: return launch_level<3, 8, false>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nm
