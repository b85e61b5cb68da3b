// One launch from the packed weight to the product of a few tokens.  A call that brings a packed weight and no prepared
// copy of it otherwise runs the stream-order pre-pass over the weight and then the tiled kernel; at up to a few dozen
// tokens the pre-pass is the longer of the two and its output is read once.  Here a block decodes the weight of its 32
// out-features into LDS as the operand of the matrix instructions and multiplies it with up to 64 tokens.
//
// What bounds it: latency.  768 -> 1000 at 4:8 and 8 tokens is 1.3 MB, under 1 us of HBM time; what takes time is one
// round trip to memory, decoding 16 weights per lane and pass (a 2-byte LDS write per kept value), and a serial chain of
// K / 64 steps.  So a block is small (768 out-features are 24 of them per 64 tokens), all four waves decode, the loads
// of two spans of 256 reduction positions are in flight in registers while a third is multiplied, and a span has one
// barrier; in blocks of 16 or 32 tokens four spans share one (launch_level).  Which products it takes is decided in nm_spmm.hip
// (direct_takes).  In a graph, pre-pass and product before: 768 -> 1000 at 4:8 and 8 tokens 9.4 -> 4.6 us, 3072 -> 768 at
// 1:4 16.4 -> 9.4, 1024 -> 4096 at 4:8 16.3 -> 6.0.
//
// Two summation orders, so that a product is the same bytes whichever kernel of its route computes it:
//   PACKED = false  the tiled kernel's (nm_spmm.hip): the sum starts from the bias; the dense instruction takes the
//                   positions of a 64-wide step as 0 .. 31 and 32 .. 63
//   PACKED = true   the few-token kernel's (nm_fewtok.hip): the bias is added last; the dense instruction takes the even
//                   and the odd runs of 8 positions
#include "nm_launch.h"
#include "nm_mma.h"

namespace nm {
namespace {

constexpr int kRows = 32, kSteps = 4;  // of a block: out-features, 64-wide steps per span; TOKS: its tokens, 64, 32 or 16

struct DirectArgs {
  const bf16_t* values;
  const uint32_t* indices;
  const bf16_t* X;
  const float* bias;  // nullable
  void* Y;
  int64_t ldx, ldy;
  int32_t O, K, T;
  int32_t out_bf16, pieces;  // pieces: rows of Y are made of aligned runs of four outputs
};

template <int N, int M, int TOKS>
struct DirectCfg {
  static constexpr int X_STEP = TOKS * 128, X_SPAN = kSteps * X_STEP;  // bytes of the activations of a step, of a span
  static constexpr int SETS = TOKS == 64 ? 2 : 4;      // spans in flight
  static constexpr bool SPARSE = N <= 2 && N < M;
  static constexpr int B = log2_of(M);
  static constexpr int VPC = 16 / M * N;               // kept values of 16 weights
  static constexpr int BITS = VPC * B;                 // their index fields
  static constexpr int WORDS = 32 % BITS == 0 ? 1 : 2;  // 32-bit words those may lie in
  static constexpr int A_ROWB = SPARSE ? 64 : 128;     // bytes of a weight row per step
  static constexpr int A_STEP = kRows * A_ROWB;
  static constexpr int S_STEP = SPARSE ? 256 : 0;      // a selector word per pair of rows and lane group
  static constexpr int SPAN = X_SPAN + kSteps * (A_STEP + S_STEP);
  static constexpr int LDS_BYTES = SETS * SPAN;
  static constexpr int VW = (VPC + 1) / 2;             // registers of a chunk's values
  static_assert(BITS <= 32 && LDS_BYTES <= 160 * 1024, "chunk fields and LDS budget");
};

// What a lane brings of a span: the packed form of two 16-weight chunks and TOKS / 8 16-byte pieces of X.
template <int N, int M, int TOKS>
struct DirectLoads {
  using C = DirectCfg<N, M, TOKS>;
  uint32_t v[2][C::VW], f[2][C::WORDS];
  u32x4_t x[TOKS / 8];
};

template <int N, int M, int TOKS, bool PACKED>
__global__ void __launch_bounds__(256) nm_direct_kernel(const DirectArgs a) {
  using C = DirectCfg<N, M, TOKS>;
  using Loads = DirectLoads<N, M, TOKS>;
  constexpr int kXStep = C::X_STEP, kXSpan = C::X_SPAN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kb = lane >> 4;
  const int o0 = (int)blockIdx.x * kRows, t0 = (int)blockIdx.y * TOKS;
  const int nk = (a.K + 63) >> 6, spans = (nk + kSteps - 1) / kSteps;  // a last step may be short (K % 16 == 0)
  const int64_t nf = (int64_t)a.K / M * N;
  const int64_t nw = (nf * C::B + 31) / 32;

  // a lane's chunks are tid and tid + 256 of the span's 32 rows x 16, its pieces of X tid + 256 i of TOKS rows x 32
  auto fetch = [&](Loads& d, int span) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int o = o0 + (tid >> 4) + 16 * u, c = span * 16 + (tid & 15);
#pragma unroll
      for (int i = 0; i < C::VW; ++i) d.v[u][i] = 0;
#pragma unroll
      for (int i = 0; i < C::WORDS; ++i) d.f[u][i] = 0;
      if (o < a.O && c * 16 < a.K) {  // rows past O and chunks past K are zero
        const bf16_t* src = a.values + o * nf + (int64_t)c * C::VPC;
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
        const int64_t w = ((int64_t)c * C::BITS) >> 5;
        d.f[u][0] = a.indices[o * nw + w];
        if constexpr (C::WORDS == 2) {
          if (w + 1 < nw) d.f[u][1] = a.indices[o * nw + w + 1];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < TOKS / 8; ++i) {
      const int t = t0 + (tid >> 5) + 8 * i, k = span * 256 + (tid & 31) * 8;
      d.x[i] = u32x4_t{0, 0, 0, 0};
      if (t < a.T && k < a.K) d.x[i] = *reinterpret_cast<const u32x4_t*>(a.X + t * a.ldx + k);
    }
  };
  // the same into the span's LDS buffer, the weight decoded.  16-byte pieces of a row are XOR-swizzled with the row.
  auto put = [&](const Loads& d, int span, unsigned char* buf) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = (tid >> 4) + 16 * u, step = (tid & 15) >> 2, c = tid & 3;
      uint64_t fields = d.f[u][0];
      if constexpr (C::WORDS == 2)
        fields = (fields | (uint64_t)d.f[u][1] << 32) >> (((uint32_t)(span * 16 + (tid & 15)) * C::BITS) & 31);
      else
        fields >>= ((uint32_t)(tid & 15) * C::BITS) & 31;  // a span starts on a word
      unsigned char* at = buf + kXSpan + step * C::A_STEP + row * C::A_ROWB;
      if constexpr (C::SPARSE) {
        // the 2:4 form: the first kept value of a run of four in slot 2 run, a second one in slot 2 run + 1
        at += (c ^ ((row >> 1) & 3)) * 16;
        *reinterpret_cast<u32x4_t*>(at) = u32x4_t{0, 0, 0, 0};
        uint32_t sel = 0, prev = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < C::VPC; ++j) {
          const uint32_t pos = (uint32_t)(j / N * M) + ((uint32_t)(fields >> (C::B * j)) & (uint32_t)(M - 1));
          const uint32_t run = pos >> 2, second = run == prev ? 1u : 0u;
          prev = run;
          *reinterpret_cast<uint16_t*>(at + 4 * run + 2 * second) = (uint16_t)(d.v[u][j / 2] >> (16 * (j & 1)));
          sel |= (pos & 3u) << (4 * run + 2 * second);
        }
        *reinterpret_cast<uint16_t*>(buf + kXSpan + kSteps * C::A_STEP + step * C::S_STEP + (row & 15) * 16 + c * 4 +
                                     (row >> 4) * 2) = (uint16_t)sel;
      } else {
        const int key = row & 7;
        *reinterpret_cast<u32x4_t*>(at + ((2 * c) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
        *reinterpret_cast<u32x4_t*>(at + ((2 * c + 1) ^ key) * 16) = u32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < C::VPC; ++j) {
          const uint32_t pos = (uint32_t)(j / N * M) + ((uint32_t)(fields >> (C::B * j)) & (uint32_t)(M - 1));
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
  // block of 16 out-features (acc[0]), the lower one in the even waves
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
  for (int i = 0; i < 2; ++i) acc[i] = PACKED ? f32x4_t{0.f, 0.f, 0.f, 0.f} : bias_of(TOKS == 64 ? i : wave & 1);

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
    const unsigned char* x = buf + ((wave >> 1) * 16 + r16) * 128;
    const unsigned char* w = buf + kXSpan + ((wave & 1) * 16 + r16) * C::A_ROWB;
    const int xk = r16 & 7;
    auto one = [&](int st) {
      if constexpr (C::SPARSE) {
        const u32x4_t a0 = *reinterpret_cast<const u32x4_t*>(w + st * C::A_STEP + (kb ^ ((r16 >> 1) & 3)) * 16);
        const uint32_t sel = *reinterpret_cast<const uint32_t*>(buf + kXSpan + kSteps * C::A_STEP + st * C::S_STEP + r16 * 16 + kb * 4);
        const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(x + st * kXStep + ((kb ^ xk) * 16));
        const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(x + st * kXStep + (((4 + kb) ^ xk) * 16));
        const u32x8_t b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc[0] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, a0), __builtin_bit_cast(bf16x16_t, b), acc[0],
                                                           (int)(sel >> (16 * (wave & 1))), 0, 0);
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
    // that every wave reaches only after it has multiplied the first.
    Loads even, odd;
    fetch(even, 0);
    if (spans > 1) fetch(odd, 1);
    for (int span = 0; span < spans; span += 2) {
      put(even, span, smem);
      if (span + 2 < spans) fetch(even, span + 2);
      __syncthreads();
      multiply(smem, span);
      if (span + 1 < spans) {
        put(odd, span + 1, smem + C::SPAN);
        if (span + 3 < spans) fetch(odd, span + 3);
        __syncthreads();
        multiply(smem + C::SPAN, span + 1);
      }
    }
  } else {
    // Four spans at a time, all their loads in flight together and one barrier for them.
    Loads d[4];
    const bool stored = (wave >> 1) * 16 < TOKS && t0 + (wave >> 1) * 16 < a.T;  // some token of this wave's 16 is
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

  const int t = t0 + (TOKS == 64 ? wave : wave >> 1) * 16 + r16;
  if (t >= a.T) return;
#pragma unroll
  for (int i = 0; i < (TOKS == 64 ? 2 : 1); ++i) {
    const int o = o_lane + 16 * (TOKS == 64 ? i : wave & 1);
    if (o >= a.O) continue;
    f32x4_t y = PACKED ? acc[i] + bias_of(TOKS == 64 ? i : wave & 1) : acc[i];
    if (a.K & 63) {  // a sum that ended as NaN again by the definition, as the ragged form of the tiled kernel has it
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

template <int N, int M, int TOKS, bool PACKED>
hipError_t launch_tokens(const DirectArgs& g, hipStream_t s) {
  using C = DirectCfg<N, M, TOKS>;
  auto kern = nm_direct_kernel<N, M, TOKS, PACKED>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((g.O + kRows - 1) / kRows), (unsigned)((g.T + TOKS - 1) / TOKS)), dim3(256),
                     C::LDS_BYTES, s, g);
  return hipGetLastError();
}

// Up to 16 tokens a block of 64 would bring, store and skip rows of zeros, and its two spans in flight make two round trips of
// K = 768: 768 -> 1000 at 4:8 and 8 tokens 5.8 -> 4.6 us, 3072 -> 768 at 1:4 12.6 -> 9.4, 16 tokens x
// 1024 -> 4096 at 4:8 7.0 -> 6.0, one token x 256 -> 128 at 2:8 3.1 -> 2.8 (in a graph).  Up to 32 the same holds for the dense
// form (24 tokens x 768 -> 1000 at 4:8 5.8 -> 5.2, 20 x 2048 -> 2048 at 4:16 10.3 -> 8.8); the 2:4 form, with half the matrix
// instructions and LDS reads per step, gains nothing on average (32 x 768 -> 768 at 1:4 5.0 and 4.9, x 768 -> 3072 at 1:16 4.7
// and 4.8).  In the dense form this holds while round trips bound the launch.  A large weight is bound by what its blocks pull in and
// decode, and there the longer run of a block of 64 is the faster one, the earlier the more tokens there are.  The limits are in
// kept values, where the two cross at 4:8, 4:16, 3:8 and 3:4: 32 tokens x 2048 -> 4096 at 4:8 (4 M) 12.1 us in blocks of 64 and 11.2,
// x 3072 -> 16384 (25 M) 31.6 and 35.2; 28 tokens x 3072 -> 6144 (9 M) 16.7 and 16.0, x 3072 -> 16384 31.4 and 32.4; up to 24 tokens a
// weight beyond the memory-side cache (24 tokens x 8192 -> 32768, 134 M, 150 and 177).  At 3:4 the two waves that multiply in a block
// of 16 hold up a large weight (16 tokens x 3072 -> 8192, 19 M: 19.0 in blocks of 64, 20.8 in blocks of 16, 18.5 in blocks of 32).
template <int N, int M, bool PACKED>
hipError_t launch_level(const DirectArgs& g, hipStream_t s) {
  if constexpr (N <= 2) {
    if (g.T <= 16) return launch_tokens<N, M, 16, PACKED>(g, s);
  } else {
    const int64_t kept = (int64_t)g.O * (g.K / M * N), full = 1 << 24;
    if (kept < (g.T <= 24 ? 6 * full : g.T <= 28 ? full : g.T <= 32 ? full / 2 : 0)) {
      if (g.T <= 16 && (M > 4 || kept < full)) return launch_tokens<N, M, 16, PACKED>(g, s);
      return launch_tokens<N, M, 32, PACKED>(g, s);
    }
  }
  return launch_tokens<N, M, 64, PACKED>(g, s);
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

// The caller has checked the operands (K % 64 == 0, or K % 16 == 0 in the tiled kernel's order; 16-byte aligned X rows and
// values, sizes as the tiled kernel's).
hipError_t launch_direct(const SpmmArgs& a, bool packed_order, hipStream_t s) {
  DirectArgs g;
  g.values = a.values; g.indices = a.indices; g.X = a.X; g.bias = a.bias; g.Y = a.Y;
  g.ldx = a.ldx; g.ldy = a.ldy;
  g.O = (int32_t)a.O; g.K = (int32_t)a.K; g.T = (int32_t)a.T;
  g.out_bf16 = a.out_bf16;
  g.pieces = (a.O % 4 == 0) && (a.ldy % 4 == 0) && ((uintptr_t)a.Y & (a.out_bf16 ? 7u : 15u)) == 0;
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
