// Sparse-weight x dense-activation product from the packed N:M layout (Section 2, Fig. 2 lower
// part): Y[t, o] = sum_g sum_{j<N} X[t, g*M + idx[o,g,j]] * val[o,g,j], fp32 accumulation.
//
// Two matrix-core formulations on gfx950, W as the first (row) operand so that a lane's four
// accumulators are four consecutive out-features of one token (contiguous in Y):
//
//  * levels with N <= 2: every aligned run of 4 weights holds at most 2 kept values, which is the
//    pattern v_smfmac_f32_16x16x64_bf16 consumes (8 compressed values + eight 2-bit selectors per
//    lane per instruction).  The packed 2:4 layout already IS that operand order; the other levels
//    are re-coded into it (explicit zeros fill the free slots) by a small pre-pass.  The instruction
//    then performs half of the dense multiply-accumulates.
//  * levels with N > 2 (4:8, 4:16, 3:8, ... and N = M): the packed weight is expanded to a dense
//    zero-filled operand by the pre-pass and multiplied with v_mfma_f32_16x16x32_bf16.
//
// Tiling: a block owns BO x BT outputs; per 64-wide K step the W tile (compressed rows + selector
// words, or dense rows) and the X tile are copied global -> LDS asynchronously, two to four stages
// deep with one barrier per step; each wave reads its operand fragments with 16-byte LDS reads
// (XOR-swizzled rows, conflict free) and keeps an (OT*16) x (TT*16) accumulator tile.
// A reduction that is no whole number of steps, or X and Y at any alignment, run the ragged form of the same tiles from a
// workspace; what is left (K < 64, no workspace, an unaligned X at 2:4 and N = M, whose weight is read as packed) runs a
// plain gather kernel.
#include "nm_device.h"
#include "nm_launch.h"
#include "nm_mma.h"

#include <type_traits>
#include <utility>

namespace nm {

// ---------------------------------------------------------------------------------------------
// Pre-pass: the weight in "stream order", the form every matrix-core kernel here reads it in (the persistent
// kernel always; the tiled kernel except at 2:4 and N = M, whose packed layouts it reads as they lie): exactly the LDS image
// of every (16-row group, K step) as one contiguous 1 KB block, so that the product kernel's
// loads are whole contiguous kilobytes (a 16-row x 64-byte slice of a row-major weight touches 16
// cache lines for one kilobyte, and the selector words one line per 8 bytes).
//   values/dense block (rg, ks) at ((rg * nk) + ks) * 1024: piece i (16 bytes) = row 16*rg + i/4,
//     16-byte chunk (i & 3) ^ ((i >> 4) & 3) of that row's 64 bytes of step ks  (the XOR is the
//     LDS swizzle; a step is 32 compressed values = 64 dense k, or 32 dense weights)
//   selector block (o_tile, ks) at ((o_tile * nk) + ks) * 2048: row r of the tile at r*8, 2 words
// Rows from O up to the next multiple of 256 are written as zeros.
// Levels with N <= 2 are re-coded as a 2:4 weight.  Slot rule: run q (4 weights) owns slots 2q and 2q+1; the first
// kept value of the run goes to slot 2q with selector = its offset in the run, a second one to slot 2q+1; free slots
// hold +0 with selector 0 (the matrix instruction is a plain multiplexer per slot, so any selector of a zero slot
// is harmless).
//
// One lane per 16 consecutive weights of a row (one 16-byte piece of the 2:4 form, two of the dense form).  K need
// not be a whole number of steps: K_pad is K rounded up to one, and what lies past K is zero.  The kept values go to
// their places through 32 bytes of LDS per lane: a 2-byte LDS write per value instead of a comparison with every
// place it could have.
template <int N, int M>
__global__ void __launch_bounds__(256)
operand_stream_kernel(const bf16_t* __restrict__ values, const uint32_t* __restrict__ indices, int64_t O, int64_t O_pad,
                      int64_t K, int64_t K_pad, int wide, unsigned char* __restrict__ vals_s,
                      unsigned char* __restrict__ sel_s) {
  constexpr int B = log2_of(M);
  constexpr int VPC = 16 / M * N;  // kept values of a chunk
  constexpr bool SPARSE = N <= 2 && N < M;
  constexpr int BYTES = SPARSE ? 16 : 32, STRIDE = BYTES + 16;
  __shared__ __attribute__((aligned(16))) unsigned char places[256 * STRIDE];
  const int64_t per_row = K_pad / 16;
  const int64_t id = flat_lane_256();
  if (id >= O_pad * per_row) return;
  int64_t o, kc;
  if (O_pad * per_row < (int64_t)1 << 31) {  // the 32-bit division is a fifth of the 64-bit one
    o = (uint32_t)id / (uint32_t)per_row;
    kc = (uint32_t)id % (uint32_t)per_row;
  } else {
    o = id / per_row;
    kc = id % per_row;
  }
  unsigned char* mine = places + threadIdx.x * STRIDE;
#pragma unroll
  for (int i = 0; i < BYTES / 16; ++i) reinterpret_cast<uint4*>(mine)[i] = make_uint4(0, 0, 0, 0);
  uint32_t sel = 0;
  const int64_t nf = K / M * N, f0 = kc * VPC;
  if (o < O && f0 < nf) {
    const int64_t nw = (nf * B + 31) / 32;
    const uint32_t* row = indices + o * nw;
    const int64_t w0 = (f0 * B) >> 5;
    const int sh = (int)((f0 * B) & 31);
    uint64_t fields = row[w0];
    if (sh + VPC * B > 32 && w0 + 1 < nw) fields |= (uint64_t)row[w0 + 1] << 32;
    fields >>= sh;
    if (VPC * B > 32 && sh && w0 + 2 < nw) fields |= (uint64_t)row[w0 + 2] << (64 - sh);
    uint32_t v[VPC];
    const bf16_t* src = values + o * nf + f0;
    if (wide) {  // whole chunks at aligned addresses
      if constexpr (VPC % 8 == 0) {
#pragma unroll
        for (int j = 0; j < VPC; j += 8) {
          const uint4 q = *reinterpret_cast<const uint4*>(src + j);
          v[j] = q.x & 0xFFFFu; v[j + 1] = q.x >> 16; v[j + 2] = q.y & 0xFFFFu; v[j + 3] = q.y >> 16;
          v[j + 4] = q.z & 0xFFFFu; v[j + 5] = q.z >> 16; v[j + 6] = q.w & 0xFFFFu; v[j + 7] = q.w >> 16;
        }
      } else if constexpr (VPC % 2 == 0) {
#pragma unroll
        for (int j = 0; j < VPC; j += 2) {
          const uint32_t q = *reinterpret_cast<const uint32_t*>(src + j);
          v[j] = q & 0xFFFFu; v[j + 1] = q >> 16;
        }
      } else {
#pragma unroll
        for (int j = 0; j < VPC; ++j) v[j] = src[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < VPC; ++j) v[j] = f0 + j < nf ? src[j] : 0u;
    }
    uint32_t prev_run = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < VPC; ++j) {
      if (!wide && f0 + j >= nf) break;
      const uint32_t pos = (uint32_t)(j / N * M) + ((uint32_t)(fields >> (B * j)) & (uint32_t)(M - 1));
      if constexpr (SPARSE) {
        const uint32_t run = pos >> 2;
        const uint32_t second = run == prev_run ? 1u : 0u;
        prev_run = run;
        *reinterpret_cast<uint16_t*>(mine + 4 * run + 2 * second) = (uint16_t)v[j];
        sel |= (pos & 3u) << (4 * run + 2 * second);
      } else {
        *reinterpret_cast<uint16_t*>(mine + 2 * pos) = (uint16_t)v[j];
      }
    }
  }
  if constexpr (SPARSE) {
    const int64_t nk = K_pad / 64;
    *reinterpret_cast<uint4*>(vals_s + stream_piece_offset(o, kc >> 2, (int)(kc & 3), nk)) = *reinterpret_cast<const uint4*>(mine);
    // rows r and r+16 of a 32-row pair share the selector word of a lane (r mod 16, chunk): low half = the first
    // row's 16 bits, high half = the second row's, which is what the matrix instruction's ABID modifier selects
    *reinterpret_cast<uint16_t*>(sel_s + stream_selector_offset(o, kc >> 2, (int)(kc & 3), nk)) = (uint16_t)sel;
  } else {
    const int64_t nk = K_pad / 32, ks = kc >> 1;
    const int c0 = (int)(kc & 1) * 2;
    *reinterpret_cast<uint4*>(vals_s + stream_piece_offset(o, ks, c0, nk)) = reinterpret_cast<const uint4*>(mine)[0];
    *reinterpret_cast<uint4*>(vals_s + stream_piece_offset(o, ks, c0 + 1, nk)) = reinterpret_cast<const uint4*>(mine)[1];
  }
}

// dense form of a TRANSPOSED weight: the operand rows are the columns of Ws [R, I] (row-major, ld ldw), the
// reduction runs over its rows.  A block turns 64 columns x 64 reduction rows through LDS: it reads 128 bytes of a row at
// a time and writes the whole contiguous kilobytes of four 16-row groups and two steps (a lane that gathers its piece from
// eight rows writes 16 bytes every 64: the four weights of a block at C = 768 28.2 us, this 21.7).  Columns past I
// (up to the tile edge) are zero.  WIDE: rows of Ws in whole 16-byte pieces.
template <bool WIDE>
__global__ void __launch_bounds__(256)
transpose_stream_kernel(const bf16_t* __restrict__ Ws, int64_t R, int64_t I, int64_t ldw, int n_i,
                        unsigned char* __restrict__ dense_s) {
  constexpr int PITCH = 64 + 2;  // elements of an LDS row: the 16-bit reads down a column spread over the banks
  __shared__ __attribute__((aligned(16))) bf16_t tile[64 * PITCH];
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)(blockIdx.x % (unsigned)n_i) * 64, r0 = (int64_t)(blockIdx.x / (unsigned)n_i) * 64;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int row = (tid >> 3) + 32 * u, c = (tid & 7) * 8;
    const bf16_t* src = Ws + (r0 + row) * ldw + i0 + c;  // R is a multiple of 64
    uint32_t w[4] = {0, 0, 0, 0};
    if (WIDE && i0 + c + 8 <= I) {
      const uint4 q = *reinterpret_cast<const uint4*>(src);
      w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (i0 + c + e < I) w[e / 2] |= (uint32_t)src[e] << (16 * (e & 1));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) *reinterpret_cast<uint32_t*>(tile + row * PITCH + c + 2 * e) = w[e];
  }
  __syncthreads();
  const int64_t nk = R / 32;
#pragma unroll
  for (int u = 0; u < 2; ++u) {  // piece: column i0 + col, 8 reduction rows; a wave writes one (16-row group, step) kilobyte
    const int unit = (tid >> 6) + 4 * u, lane = tid & 63;
    const int col = (unit & 3) * 16 + (lane >> 2), step = unit >> 2;
    const int chunk = lane & 3;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bf16_t* at = tile + (step * 32 + chunk * 8 + 2 * e) * PITCH + col;
      w[e] = (uint32_t)at[0] | ((uint32_t)at[PITCH] << 16);
    }
    *reinterpret_cast<uint4*>(dense_s + stream_piece_offset(i0 + col, r0 / 32 + step, chunk, nk)) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// ---------------------------------------------------------------------------------------------
// Tiled matrix-core product.
//
// Operand tiles travel global -> LDS directly (global_load_lds_dwordx4: each lane names its own
// 16 global bytes, the wave's 64 pieces land in 1 KB of consecutive LDS), STAGES buffers deep, so
// that two K steps of loads are in flight while a third is multiplied and no register is spent on
// staging.  The compiler does not track these loads; the kernel counts them itself: every wave
// issues exactly LPW loads per stage and waits with s_waitcnt vmcnt(LPW) (one younger stage may
// still be in flight) or vmcnt(0) before the one barrier of the step.
// LDS rows are not padded (the DMA writes 1 KB runs); instead the 16-byte pieces of a row are
// XOR-swizzled with the row number on the way in, and the fragment reads apply the same XOR, which
// keeps 8 consecutive rows on distinct banks.
// ---------------------------------------------------------------------------------------------
struct GemmArgs {
  const bf16_t* A;      // SPARSE: compressed values [O, K/2]; dense: W_s [O, K]
  const uint32_t* sel;  // SPARSE: selector words [O, K/32]
  const bf16_t* X;
  const float* bias;
  void* Y;
  float* partial = nullptr;  // splits > 1: fp32 partial sums [splits][T][O] (rows of O floats), added up by the reduce kernel
  int64_t O, K, T, ldx, ldy;
  int n_o_tiles, n_t_tiles;
  uint8_t out_bf16;
  uint8_t vec_store;    // Y rows split into whole aligned 16-byte pieces (ldy, O multiples of 8 (bf16) / 4 (fp32))
  uint8_t stream_form;  // A (and sel) lie in stream order (the pre-pass's output), else row-major as packed
  uint8_t splits = 1;   // ranges the reduction is cut into (tiled kernel only; 1 = the whole K in one block)
  uint8_t rot = 0;      // tiled kernel: XCD x takes the layer's share number (x + rot) mod 8
  uint8_t x_aligned = 0;  // every X row starts on 16 bytes
  // ragged form only: the packed weight itself, for the sums that are computed a second time
  uint8_t N = 0, M = 0;
  const bf16_t* values = nullptr;
  const uint32_t* indices = nullptr;
};
// (a launch that sets only what it knows leaves no share number to chance)
static_assert([] { GemmArgs g; return g.rot == 0 && g.splits == 1 && g.partial == nullptr && g.values == nullptr; }());

template <bool SPARSE, int WO, int WT, int OT, int TT, int STAGES_>
struct GemmCfg {
  static constexpr int STAGES = STAGES_;
  static constexpr int NW = WO * WT;
  static constexpr int NT = NW * 64;
  static constexpr int BO = WO * OT * 16;
  static constexpr int BT = WT * TT * 16;
  static constexpr int KC = 64;                         // dense k per stage
  static constexpr int H = SPARSE ? 1 : 2;              // sub-steps (32 matrix instructions each) per stage
  static constexpr int A_ROWB = SPARSE ? 64 : 128;      // bytes of one W row per stage
  static constexpr int X_BYTES = BT * 128;
  static constexpr int A_BYTES = BO * A_ROWB;
  static constexpr int S_BYTES = SPARSE ? BO * 8 : 0;   // two selector words per row per stage
  static constexpr int STAGE = X_BYTES + A_BYTES + S_BYTES;
  static constexpr int LDS_BYTES = STAGES * STAGE;
  static constexpr int X_LOADS = X_BYTES / 1024;        // wave-wide 16-byte loads per stage
  static constexpr int A_LOADS = A_BYTES / 1024;
  static constexpr int S_LOADS = S_BYTES / 256;         // wave-wide 4-byte loads per stage
  static constexpr int X_PW = (X_LOADS + NW - 1) / NW;  // per wave (surplus waves repeat a load)
  static constexpr int A_PW = (A_LOADS + NW - 1) / NW;
  static constexpr int S_PW = SPARSE ? (S_LOADS + NW - 1) / NW : 0;
  static constexpr int LPW = X_PW + A_PW + S_PW;
  static_assert(STAGES >= 2 && STAGES <= 4, "LDS stages");
  static_assert(STAGES * LPW < 64, "vmcnt is a 6-bit counter");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// Accumulator start value of the 16 x 16 block whose four out-features start at o: the bias (so
// that no load sits between the stores of the epilogue), or zero.
__device__ __forceinline__ f32x4_t bias_init(const float* bias, int64_t o, int64_t O, bool vec) {
  f32x4_t v = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (bias) {
    if (vec) {
      if (o < O) {
        const float4 b = *reinterpret_cast<const float4*>(bias + o);
        v = f32x4_t{b.x, b.y, b.z, b.w};
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (o + e < O) v[e] = bias[o + e];
    }
  }
  return v;
}

// One tile of one layer; `block` is the block's number among the layer's blocks (a multiple of 8 of them, so
// that block mod 8 is the XCD the block runs on).
// STREAM: the weight lies in stream order (the pre-pass's output: every 16-row x K-step slice one contiguous,
// already swizzled kilobyte; selector words interleaved per 32-row pair), else row-major (the packed 2:4 layout
// or a dense level's values, read as they lie).
// X_REGS: not 0: the operands travel through registers instead of by asynchronous copies, so that rows of X may start anywhere and K
// may end anywhere, loaded that many stages ahead (2 or 4; see the loop); two stages of LDS.
// TAIL: K, a multiple of 8, may end inside the last step (rows of X still start on 16 bytes).  The pieces of that step past K are fetched
// from its first piece instead (what lies behind a row's end may be no memory at all) and cleared in LDS by the lanes
// that brought them, so they never enter a sum.
template <bool SPARSE, int WO, int WT, int OT, int TT, int STAGES, bool STREAM, int X_REGS = 0, bool TAIL = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, unsigned block, unsigned char* smem) {
  using C = GemmCfg<SPARSE, WO, WT, OT, TT, STAGES>;
  static_assert(!STREAM || (OT % 2 == 0 && C::BO % 32 == 0 && 256 % C::BO == 0), "stream order: whole 32-row pairs inside one 256-row tile");
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  // XCD-aware tile order: consecutive block ids land on different XCDs (8 of them, each with its
  // own L2); give every XCD a contiguous range of tiles so that the blocks sharing an L2 share X rows.
  // A layer with few tiles and a long reduction is cut along K as well: unit = (tile, K range); every range of a
  // tile writes fp32 partial sums of its own, which splitk_reduce_kernel adds in range order.
  const int n_splits = a.splits > 1 ? a.splits : 1;
  const int n_units = a.n_o_tiles * a.n_t_tiles * n_splits;
  const int per_xcd = (n_units + 7) >> 3;
  // (the shares at the end of the list may be short or empty; `rot` says which XCDs get those, so that the layers
  // of a launch can leave them to different ones)
  const int unit = (int)((block + a.rot) & 7) * per_xcd + (int)(block >> 3);
  if (unit >= n_units) return;
  const int tile = unit / n_splits, split = unit - tile * n_splits;
  const int o_tile = tile % a.n_o_tiles;
  const int t_tile = tile / a.n_o_tiles;
  const int64_t o0 = (int64_t)o_tile * C::BO;
  const int64_t t0 = (int64_t)t_tile * C::BT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave % WO;
  const int wt = wave / WO;
  const int r16 = lane & 15;
  const int kb = lane >> 4;

  // ---- per-lane source offsets and per-wave LDS destinations of this wave's loads (fixed over K)
  const int64_t a_ld = SPARSE ? (a.K >> 1) : a.K;  // elements per row of A
  uint32_t x_voff[C::X_PW], a_voff[C::A_PW], s_voff[C::S_PW > 0 ? C::S_PW : 1];
  uint32_t x_dst[C::X_PW], a_dst[C::A_PW], s_dst[C::S_PW > 0 ? C::S_PW : 1];
  const int64_t t_last = a.T - 1 - t0, o_last = a.O - 1 - o0;  // rows past the edge re-read the last valid row
#pragma unroll
  for (int i = 0; i < C::X_PW; ++i) {
    const int j = (wave + i * C::NW) % C::X_LOADS;
    int64_t row = 8 * j + (lane >> 3);
    const int c = (lane & 7) ^ (int)(row & 7);
    if (row > t_last) row = t_last;
    x_voff[i] = (uint32_t)((row * a.ldx + c * 8) * 2);
    x_dst[i] = (uint32_t)(j * 1024);
  }
  const int nk_all = (int)((a.K + C::KC - 1) / C::KC);  // K steps of the layer
  const int per_split = (nk_all + n_splits - 1) / n_splits;
  const int ks0 = split * per_split;                    // this block's steps: ks0 .. ks0 + nk - 1
  const int nk = nk_all - ks0 < per_split ? nk_all - ks0 : per_split;
#pragma unroll
  for (int i = 0; i < C::A_PW; ++i) {
    const int j = (wave + i * C::NW) % C::A_LOADS;
    if constexpr (STREAM) {
      // load j brings one kilobyte: 16-row group rg of the tile at the stage's K step (2:4 form), or at its
      // first (h = 0) or second (h = 1) 32-wide step (dense form, two stream steps per stage)
      constexpr int GROUPS = C::BO / 16;
      const int rg = j % GROUPS, h = j / GROUPS;
      a_voff[i] = ((uint32_t)(rg * (SPARSE ? nk_all : 2 * nk_all) + h) << 10) + (uint32_t)(lane * 16);
      a_dst[i] = (uint32_t)(C::X_BYTES + h * (C::BO * 64) + rg * 1024);
    } else {
      int64_t row;
      int c;
      if (SPARSE) { row = 16 * j + (lane >> 2); c = (lane & 3) ^ (int)((row >> 1) & 3); }
      else { row = 8 * j + (lane >> 3); c = (lane & 7) ^ (int)(row & 7); }
      if (row > o_last) row = o_last;
      a_voff[i] = (uint32_t)((row * a_ld + c * 8) * 2);
      a_dst[i] = (uint32_t)(C::X_BYTES + j * 1024);
    }
  }
  if (SPARSE) {
#pragma unroll
    for (int i = 0; i < C::S_PW; ++i) {
      const int j = (wave + i * C::NW) % C::S_LOADS;
      if constexpr (STREAM) {
        // the tile's share of the (256-row tile, step) selector block: 256 bytes per 32-row pair
        s_voff[i] = (uint32_t)((((o0 & 255) >> 5) + j) * 256 + lane * 4);
      } else {
        int64_t row = 32 * j + (lane >> 1);
        if (row > o_last) row = o_last;
        s_voff[i] = (uint32_t)((row * (a.K >> 5) + (lane & 1)) * 4);
      }
      s_dst[i] = (uint32_t)(C::X_BYTES + C::A_BYTES + j * 256);
    }
  }
  // elements the weight and selector pointers advance per stage
  constexpr int A_STEP = STREAM ? (SPARSE ? 512 : 1024) : (SPARSE ? 32 : 64);
  constexpr int S_STEP = STREAM ? 512 : 2;
  const bf16_t* x_base = a.X + t0 * a.ldx + (int64_t)ks0 * 64;
  const bf16_t* a_base = a.A + (STREAM ? (o0 >> 4) * (int64_t)nk_all * A_STEP : o0 * a_ld) + (int64_t)ks0 * A_STEP;
  const uint32_t* s_base =
      SPARSE ? a.sel + (STREAM ? (o0 >> 8) * (int64_t)nk_all * S_STEP : o0 * (a.K >> 5)) + (int64_t)ks0 * S_STEP : nullptr;
  // where the block's sums go: the output, or its range's partial sums (plain fp32 rows of O, no bias yet)
  void* out_ptr = a.Y;
  int64_t out_ld = a.ldy;
  bool out_bf16 = a.out_bf16 != 0, out_vec = a.vec_store != 0;
  const float* bias = a.bias;
  if (a.splits > 1) {
    out_ptr = a.partial + (int64_t)split * a.T * a.O;
    out_ld = a.O;
    out_bf16 = false;
    out_vec = (a.O & 3) == 0;
    bias = nullptr;
  }

  // The stage to be loaded next, as three running uniform pointers (X rows at the stage's k, weight, selectors),
  // advanced by constants: the step loop then holds no address products.
  uniform_ptr_t x_next = make_uniform(x_base), a_next = make_uniform(a_base), s_next = make_uniform(s_base);
  // the d-th of this wave's LPW loads of that stage into LDS buffer buf (d is a compile-time index)
  auto issue_one = [&](auto d_tag, int buf) {
    constexpr int d = decltype(d_tag)::value;
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)buf * C::STAGE);
    if constexpr (d < C::X_PW) {
      dma16(x_next, x_voff[d], lds + x_dst[d]);
    } else if constexpr (d < C::X_PW + C::A_PW) {
      dma16(a_next, a_voff[d - C::X_PW], lds + a_dst[d - C::X_PW]);
    } else {
      dma4(s_next, s_voff[d - C::X_PW - C::A_PW], lds + s_dst[d - C::X_PW - C::A_PW]);
    }
    if constexpr (d == C::LPW - 1) {  // the stage is out: on to the next one
      x_next += 64 * sizeof(bf16_t);
      a_next += A_STEP * sizeof(bf16_t);
      s_next += S_STEP * sizeof(uint32_t);
    }
  };
  auto issue_stage = [&](int buf) {
    [&]<int... D>(std::integer_sequence<int, D...>) {
      (issue_one(std::integral_constant<int, D>{}, buf), ...);
    }(std::make_integer_sequence<int, C::LPW>{});
  };

  f32x4_t acc[OT][TT];
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    const f32x4_t b = bias_init(bias, o0 + (wo * OT + i) * 16 + kb * 4, a.O, a.vec_store);
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = b;
  }

  // fragment read offsets inside a stage (the XOR undoes the swizzle applied by the loads)
  const int x_sw = r16 & 7;
  const int x_row = (wt * TT * 16 + r16) * 128;
  // stream order keeps 64-byte weight rows in both forms (the dense stage is two such sub-tiles)
  constexpr int A_ROWB = STREAM ? 64 : C::A_ROWB;
  const int a_row = C::X_BYTES + (wo * OT * 16 + r16) * A_ROWB;
  const int a_sw = (SPARSE || STREAM) ? ((r16 >> 1) & 3) : (r16 & 7);
  const int s_row = STREAM ? C::X_BYTES + C::A_BYTES + (wo * OT / 2) * 256 + r16 * 16 + kb * 4
                           : C::X_BYTES + C::A_BYTES + (wo * OT * 16 + r16) * 8 + (kb >> 1) * 4;

  // One sub-step = 32 matrix instructions per wave.  SPARSE: a stage is one sub-step (K = 64 through
  // v_smfmac 16x16x64).  Dense: a stage is two sub-steps of K = 32 (v_mfma 16x16x32), h selects the half.
  // SPARSE lane (r16, kb) of the W operand covers dense k = 16*kb .. 16*kb+15 of the step (compressed
  // values 8*kb .. 8*kb+7 and 16 selector bits); the X operand holds k = 8*kb+e (e < 8) and
  // 32 + 8*kb + e - 8 (e >= 8).
  constexpr int H = C::H;
  u32x4_t af[OT];
  int sel[OT];
  u32x8_t bs[SPARSE ? TT : 1];
  u32x4_t bd[SPARSE ? 1 : TT];
  auto read_frags = [&](int buf, int h) {
    const unsigned char* base = smem + buf * C::STAGE;
    if (SPARSE) {
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        af[i] = *reinterpret_cast<const u32x4_t*>(base + a_row + i * 16 * A_ROWB + ((kb ^ a_sw) * 16));
        if constexpr (STREAM) {
          // one word serves the two 16-row blocks of a pair: low half / high half, picked by the instruction
          sel[i] = (int)*reinterpret_cast<const uint32_t*>(base + s_row + (i / 2) * 256);
        } else {
          const uint32_t w = *reinterpret_cast<const uint32_t*>(base + s_row + i * 16 * 8);
          sel[i] = (int)(w >> ((kb & 1) * 16));
        }
      }
#pragma unroll
      for (int j = 0; j < TT; ++j) {
        const unsigned char* row = base + x_row + j * 16 * 128;
        const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(row + ((kb ^ x_sw) * 16));
        const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(row + (((4 + kb) ^ x_sw) * 16));
        bs[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    } else {
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if constexpr (STREAM)
          af[i] = *reinterpret_cast<const u32x4_t*>(base + a_row + h * (C::BO * 64) + i * 16 * A_ROWB + ((kb ^ a_sw) * 16));
        else
          af[i] = *reinterpret_cast<const u32x4_t*>(base + a_row + i * 16 * A_ROWB + (((h * 4 + kb) ^ a_sw) * 16));
      }
#pragma unroll
      for (int j = 0; j < TT; ++j)
        bd[j] = *reinterpret_cast<const u32x4_t*>(base + x_row + j * 16 * 128 + (((h * 4 + kb) ^ x_sw) * 16));
    }
  };
  // 32 matrix instructions; when `load` is set, this wave's LPW loads of stage (lks -> lbuf) are issued
  // between them, one every few instructions, so that the memory pipe is fed evenly instead of in bursts
  constexpr int MMA = OT * TT;
  constexpr int EVERY = MMA / C::LPW > 0 ? MMA / C::LPW : 1;
  auto multiply = [&](bool load, int lbuf) {
    [&]<int... Q>(std::integer_sequence<int, Q...>) {
      ([&] {
        constexpr int j = Q / OT, i = Q % OT;
        if (SPARSE)
          acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, af[i]),
                                                                __builtin_bit_cast(bf16x16_t, bs[j]), acc[i][j],
                                                                sel[i], 0, STREAM ? (i & 1) : 0);
        else
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, af[i]),
                                                              __builtin_bit_cast(bf16x8_t, bd[j]), acc[i][j], 0, 0, 0);
        if constexpr (Q % EVERY == EVERY - 1 && Q / EVERY < C::LPW) {
          if (load) issue_one(std::integral_constant<int, Q / EVERY>{}, lbuf);
          __builtin_amdgcn_sched_barrier(0);
        }
      }(), ...);
    }(std::make_integer_sequence<int, MMA>{});
  };
  // stage s has landed in this wave's view once at most the loads of the younger stages issued so far
  // are outstanding: `younger` of them (0, 1 or 2)
  auto wait_stage = [&](int younger) {
    if (younger >= 2) wait_loads_outstanding<2 * C::LPW>();
    else if (younger == 1) wait_loads_outstanding<C::LPW>();
    else wait_loads_outstanding<0>();
  };

  if constexpr (X_REGS != 0) {
    // Rows of X that start anywhere, and a K that ends anywhere.  Every operand travels through registers: plain loads, which
    // need no alignment, X_REGS stages ahead, and written to LDS where the asynchronous copies of the other form put them.  The loads carry no
    // condition, so that the wait before a stage's write leaves the younger ones in flight: past K a piece is the row's last
    // eight elements, shifted and cleared on its way to LDS (so is the weight there: what lies behind a row's end never enters a sum);
    // past the last stage it is that one again.  Bound by the latency of a stage's loads where a unit has one block: with one stage in
    // flight and its wait in the same step, a step took 0.6 - 0.9 us, now 0.25.  Where units have several, the registers of further stages
    // cost blocks: two stages, and four only for long reductions of the dense form on few tiles (518 x 2164 -> 528 at 4:4 12.5 us, 13.0 with
    // two; 10403 x 100 -> 279 at 4:4 in the small tiles 9.3 with four, 7.3 with two).  Products, us, one stage in flight and now: 926 x 2740
    // -> 96 at 1:4 27.5 and 12.3, 518 x 2164 -> 528 24.3 and 12.5, 4345 x 3468 -> 128 at 1:4 61.0 and 15.6, 8000 x 516 -> 2052 at 4:4
    // 69.5 and 40.3, 3000 x 1028 -> 1400 at 3:4 31.0 and 21.6, 969 x 244 -> 3040 at 4:4 7.6 and 6.8, 35674 x 84 -> 2697 at 2:4 82.6 and 88.0.
    static_assert(STAGES == 2 && STREAM && X_REGS % 2 == 0, "register-staged form");
    constexpr int DEPTH = X_REGS;
    u32x4_t xr[DEPTH][C::X_PW], ar[DEPTH][C::A_PW];
    uint32_t sr[DEPTH][C::S_PW > 0 ? C::S_PW : 1];
    struct __attribute__((packed, aligned(2))) Piece { u32x4_t v; };
    const bf16_t* x_row_ptr[C::X_PW];
    int x_k[C::X_PW];  // the piece's first k inside a step
#pragma unroll
    for (int i = 0; i < C::X_PW; ++i) {
      const int j = (wave + i * C::NW) % C::X_LOADS;
      int64_t row = 8 * j + (lane >> 3);
      x_k[i] = ((lane & 7) ^ (int)(row & 7)) * 8;
      if (row > t_last) row = t_last;
      x_row_ptr[i] = a.X + (t0 + row) * a.ldx;
    }
    auto fetch = [&](auto set_tag, int ks) {
      constexpr int S = decltype(set_tag)::value;
      if (ks >= nk) ks = nk - 1;
#pragma unroll
      for (int i = 0; i < C::X_PW; ++i) {
        const int k = ks * 64 + x_k[i];
        xr[S][i] = reinterpret_cast<const Piece*>(x_row_ptr[i] + (k <= (int)a.K - 8 ? k : (int)a.K - 8))->v;
      }
      const unsigned char* src = reinterpret_cast<const unsigned char*>(a_base + (int64_t)ks * A_STEP);
#pragma unroll
      for (int i = 0; i < C::A_PW; ++i) ar[S][i] = *reinterpret_cast<const u32x4_t*>(src + a_voff[i]);
      if constexpr (SPARSE) {
        const unsigned char* sel_src = reinterpret_cast<const unsigned char*>(s_base + (int64_t)ks * S_STEP);
#pragma unroll
        for (int i = 0; i < C::S_PW; ++i) sr[S][i] = *reinterpret_cast<const uint32_t*>(sel_src + s_voff[i]);
      }
    };
    auto put = [&](auto set_tag, int ks, int buf) {
      constexpr int S = decltype(set_tag)::value;
      unsigned char* base = smem + buf * C::STAGE;
      if (ks == nk - 1) {
#pragma unroll
        for (int i = 0; i < C::X_PW; ++i) {
          const int n = (int)a.K - (ks * 64 + x_k[i]);  // elements left of the piece; a multiple of 4: K is one
          const u32x4_t v = xr[S][i];
          xr[S][i] = n >= 8 ? v : n >= 4 ? u32x4_t{v[2], v[3], 0, 0} : u32x4_t{0, 0, 0, 0};
        }
      }
#pragma unroll
      for (int i = 0; i < C::X_PW; ++i) *reinterpret_cast<u32x4_t*>(base + x_dst[i] + lane * 16) = xr[S][i];
#pragma unroll
      for (int i = 0; i < C::A_PW; ++i) *reinterpret_cast<u32x4_t*>(base + a_dst[i] + lane * 16) = ar[S][i];
      if constexpr (SPARSE) {
#pragma unroll
        for (int i = 0; i < C::S_PW; ++i) *reinterpret_cast<uint32_t*>(base + s_dst[i] + lane * 4) = sr[S][i];
      }
    };
    auto everyone = [&]() {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
    };
    [&]<int... D>(std::integer_sequence<int, D...>) {
      (fetch(std::integral_constant<int, D>{}, D), ...);
    }(std::make_integer_sequence<int, DEPTH>{});
    put(std::integral_constant<int, 0>{}, 0, 0);
    // Steps first .. first + DEPTH - 1: stage ks lies in LDS, stages ks + 1 .. ks + DEPTH are on their way.  STEADY: all of them load one.
    auto round = [&](auto steady, int first) {
      [&]<int... B>(std::integer_sequence<int, B...>) {
        ([&] {
          constexpr bool STEADY = decltype(steady)::value;
          constexpr int buf = B & 1;
          using Next = std::integral_constant<int, (B + 1) % DEPTH>;
          const int ks = first + B;
          if (!STEADY && ks >= nk) return;
#pragma unroll
          for (int h = 0; h < H; ++h) {
            read_frags(buf, h);
            multiply(false, 0);
          }
          if (!STEADY && ks + 1 == nk) return;
          put(Next{}, ks + 1, buf ^ 1);
          if (STEADY || ks + 1 + DEPTH < nk) fetch(Next{}, ks + 1 + DEPTH);
          everyone();
        }(), ...);
      }(std::make_integer_sequence<int, DEPTH>{});
    };
    int first = 0;
    if (nk > 2 * DEPTH) {
      fetch(std::integral_constant<int, 0>{}, DEPTH);
      everyone();
      for (; first + 2 * DEPTH < nk; first += DEPTH) round(std::true_type{}, first);
    } else {
      if (DEPTH < nk) fetch(std::integral_constant<int, 0>{}, DEPTH);
      everyone();
    }
    for (; first < nk; first += DEPTH) round(std::false_type{}, first);
  } else {
    static_assert(!TAIL || C::X_LOADS % C::NW == 0, "every piece is brought by one lane");
    const int k_tail = (int)(a.K - (int64_t)(nk_all - 1) * 64);  // elements of the last step, 8 .. 64
    int x_piece[C::X_PW];
    if constexpr (TAIL) {
#pragma unroll
      for (int i = 0; i < C::X_PW; ++i) {
        const int row = 8 * (wave + i * C::NW) + (lane >> 3);
        x_piece[i] = (lane & 7) ^ (row & 7);
      }
    }
    auto last_sources = [&]() {  // the next stage to be issued is the last one
#pragma unroll
      for (int i = 0; i < C::X_PW; ++i)
        if (x_piece[i] * 8 >= k_tail) x_voff[i] -= (uint32_t)x_piece[i] * 16;
    };
    auto clear_tail = [&](int buf) {
#pragma unroll
      for (int i = 0; i < C::X_PW; ++i) {
        if (x_piece[i] * 8 >= k_tail)
          *reinterpret_cast<u32x4_t*>(smem + buf * C::STAGE + x_dst[i] + lane * 16) = u32x4_t{0, 0, 0, 0};
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
      if (s < STAGES - 1 && s < nk) {
        if (TAIL && s == nk - 1) last_sources();
        issue_stage(s);
      }

    // One barrier per stage; the buffer multiplied in the previous step is refilled right after the barrier,
    // STAGES-1 stages ahead.  A wave issues one instruction at a time, so whatever the step spends on addresses and
    // conditions its matrix instructions do not get: the steady state (every step has a stage to load) runs STAGES
    // steps at a time, which makes every LDS buffer a constant and leaves the step without branches; the last steps
    // run the general form.
    int ks = 0;
    for (; ks + 2 * STAGES - 2 < nk - (TAIL ? 1 : 0); ks += STAGES) {
      [&]<int... B>(std::integer_sequence<int, B...>) {
        ([&] {
          constexpr int buf = B, nbuf = (B + STAGES - 1) % STAGES;
          wait_stage(STAGES - 2);
          __builtin_amdgcn_s_barrier();
#pragma unroll
          for (int h = 0; h < H; ++h) {
            read_frags(buf, h);
            multiply(h == 0, nbuf);
          }
        }(), ...);
      }(std::make_integer_sequence<int, STAGES>{});
    }
    {
      int buf = 0;  // ks is a multiple of STAGES here
      for (; ks < nk; ++ks) {
        wait_stage(nk - 1 - ks < STAGES - 2 ? nk - 1 - ks : STAGES - 2);
        if (TAIL && ks + 1 == nk && k_tail < 64) clear_tail(buf);
        __builtin_amdgcn_s_barrier();
        if (TAIL && ks + STAGES == nk) last_sources();
        int nbuf = buf + STAGES - 1;
        if (nbuf >= STAGES) nbuf -= STAGES;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          read_frags(buf, h);
          multiply(h == 0 && ks + STAGES - 1 < nk, nbuf);
        }
        if (++buf == STAGES) buf = 0;
      }
    }
  }

  // ---- epilogue.  A lane holds out-features o .. o+3 (accumulator element e -> row 4*kb + e of the
  // 16-row tile) of token r16, i.e. 8 or 16 contiguous bytes of a Y row.  For aligned outputs every
  // wave transposes 16 tokens at a time through its own LDS slice so that the global stores are
  // 16 bytes per lane and whole row segments of the wave tile (OW elements) are written contiguously.
  __builtin_amdgcn_s_barrier();  // every wave is done with the operand stages
  auto get = [&](int i, int j) { return __builtin_bit_cast(u32x4_t, acc[i][j]); };
  const int64_t row0 = t0 + wt * TT * 16, col0 = o0 + wo * OT * 16;
  static_assert(C::NW * wave_tile_slice_bytes<OT, 4>() <= C::LDS_BYTES, "write-out slices");
  if (out_vec) {
    if (out_bf16)
      write_wave_tile_pieces<OT, TT, 2>(smem + wave * wave_tile_slice_bytes<OT, 2>(), lane, get, out_ptr, out_ld, row0, col0, a.T, a.O);
    else
      write_wave_tile_pieces<OT, TT, 4>(smem + wave * wave_tile_slice_bytes<OT, 4>(), lane, get, out_ptr, out_ld, row0, col0, a.T, a.O);
  } else if (out_bf16) {
    write_wave_tile_rows<OT, TT, 2>(smem + wave * wave_tile_slice_bytes<OT, 4>(), lane, get, out_ptr, out_ld, row0, col0, a.T, a.O);
  } else {
    write_wave_tile_rows<OT, TT, 4>(smem + wave * wave_tile_slice_bytes<OT, 4>(), lane, get, out_ptr, out_ld, row0, col0, a.T, a.O);
  }

  if constexpr (X_REGS != 0 || TAIL) {
    // The shapes of the ragged form are the gather kernel's when there is no workspace, and an infinity or NaN among the
    // activations must not change a product by the way it was computed: a zero of the padded weight makes NaN of it
    // where the gather skips it.  Sums that ended as NaN are computed again by the definition.  The test is one
    // comparison per two sums (1579 x 1000 -> 1001 at 2:8: no measurable time).
    bool any = false;
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
      for (int j = 0; j < TT; ++j)
        any |= __builtin_isunordered(acc[i][j][0], acc[i][j][1]) || __builtin_isunordered(acc[i][j][2], acc[i][j][3]);
    if (any) {
      uint64_t which = 0;  // bit 4 (i TT + j) + e
#pragma unroll
      for (int i = 0; i < OT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            which |= (uint64_t)(__builtin_isnan(acc[i][j][e]) ? 1 : 0) << (4 * (i * TT + j) + e);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // another lane of this wave has stored the element: it is out
      for (; which != 0; which &= which - 1) {
        const int bit = __ffsll((unsigned long long)which) - 1;
        const int64_t o = col0 + (bit >> 2) / TT * 16 + kb * 4 + (bit & 3), t = row0 + (bit >> 2) % TT * 16 + r16;
        if (o >= a.O || t >= a.T) continue;
        const float y = gather_output(a.values, a.indices, a.K, a.N, a.M, a.X + t * a.ldx, a.bias, o);
        if (out_bf16) reinterpret_cast<bf16_t*>(out_ptr)[t * out_ld + o] = (bf16_t)f32_to_bf16_rne(y);
        else reinterpret_cast<float*>(out_ptr)[t * out_ld + o] = y;
      }
    }
  }
}

// Both weight orders live in one kernel (a block-uniform branch): the layers of a launch may differ in it (2:4 and
// N = M are read as packed, the other levels in stream order), and every launch more is a partly filled chip more.
template <bool SPARSE, int WO, int WT, int OT, int TT, int STAGES>
__global__ void __launch_bounds__(WO * WT * 64)
nm_gemm_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  if (a.stream_form) gemm_tile<SPARSE, WO, WT, OT, TT, STAGES, true>(a, blockIdx.x, smem);
  else gemm_tile<SPARSE, WO, WT, OT, TT, STAGES, false>(a, blockIdx.x, smem);
}

// Any K, any alignment of X and Y: the weight in stream order (K padded with zeros to whole steps), X by asynchronous
// copies where its rows are whole 16-byte pieces, else through registers.
template <bool SPARSE, int WO, int WT, int OT, int TT, int STAGES, int X_REGS>
__global__ void __launch_bounds__(WO * WT * 64)
nm_gemm_ragged_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  gemm_tile<SPARSE, WO, WT, OT, TT, STAGES, true, X_REGS, X_REGS == 0>(a, blockIdx.x, smem);
}

// The tiles of many small layers in one launch, whatever their operand form and weight order: products of a few
// tokens are a handful of tiles each, far fewer than the chip has compute units, and independent ones fill it
// together (two launches, one per form, would each end in a partly filled chip and run one after the other).
// A block finds its layer in the running block counts (whole multiples of 8 per layer) by bisection and takes the
// branch of that layer's form; the table entry is the layer's arguments packed to 80 bytes, so that the 48 linears
// of a 12-block model fit one kernel argument segment.
constexpr int kTileLayersMax = 50;
struct TileLayer {
  const bf16_t* A;
  const uint32_t* sel;
  const bf16_t* X;
  const float* bias;
  void* Y;
  float* partial;
  int64_t ldy;
  uint32_t O, T;           // O <= 2^24, T < 2^31
  uint32_t K : 23, rot : 3;  // K <= 2^22
  uint32_t ldx : 23, out_bf16 : 1, vec_store : 1, stream_form : 1, sparse_form : 1, splits : 4, narrow : 1;
  uint32_t block_end;      // exclusive prefix end, in blocks
};
struct TileGroup {
  int32_t count;
  TileLayer layer[kTileLayersMax];
};
static_assert(sizeof(TileLayer) == 80 && sizeof(TileGroup) <= 4096, "the table must fit the kernel argument segment");

// SS, SD: LDS stages of the 2:4-form and of the dense-form tiles (the launch's LDS is the larger of the two).  NARROW: a
// layer may take tiles of half the out-features, three stages in either form (tile_group_narrow).
template <int WO, int WT, int OT, int TT, int SS, int SD, bool NARROW>
__global__ void __launch_bounds__(WO * WT * 64)
nm_gemm_group_kernel(const TileGroup g) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int lo = 0, hi = g.count - 1;  // the first layer whose end lies beyond this block
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (blockIdx.x >= g.layer[mid].block_end) lo = mid + 1;
    else hi = mid;
  }
  const TileLayer& L = g.layer[lo];
  const unsigned block = blockIdx.x - (lo ? g.layer[lo - 1].block_end : 0u);
  GemmArgs a;
  a.A = L.A; a.sel = L.sel; a.X = L.X; a.bias = L.bias; a.Y = L.Y; a.partial = L.partial;
  a.O = L.O; a.K = L.K; a.T = L.T; a.ldx = L.ldx; a.ldy = L.ldy;
  const uint32_t rows = WO * OT * 16 >> (NARROW ? L.narrow : 0);
  a.n_o_tiles = (int)((L.O + rows - 1) / rows);
  a.n_t_tiles = (int)((L.T + WT * TT * 16 - 1) / (WT * TT * 16));
  a.out_bf16 = L.out_bf16; a.vec_store = L.vec_store; a.stream_form = L.stream_form; a.splits = L.splits;
  a.rot = L.rot;
  if constexpr (NARROW) {
    if (L.narrow) {
      if (L.sparse_form) {
        if (L.stream_form) gemm_tile<true, WO, WT, OT / 2, TT, 3, true>(a, block, smem);
        else gemm_tile<true, WO, WT, OT / 2, TT, 3, false>(a, block, smem);
      } else {
        if (L.stream_form) gemm_tile<false, WO, WT, OT / 2, TT, 3, true>(a, block, smem);
        else gemm_tile<false, WO, WT, OT / 2, TT, 3, false>(a, block, smem);
      }
      return;
    }
  }
  if (L.sparse_form) {
    if (L.stream_form) gemm_tile<true, WO, WT, OT, TT, SS, true>(a, block, smem);
    else gemm_tile<true, WO, WT, OT, TT, SS, false>(a, block, smem);
  } else {
    if (L.stream_form) gemm_tile<false, WO, WT, OT, TT, SD, true>(a, block, smem);
    else gemm_tile<false, WO, WT, OT, TT, SD, false>(a, block, smem);
  }
}

// The partial sums of layers whose reduction was cut into ranges, added up in range order (so the result does not
// depend on which block finished first), plus the bias, rounded to the output type.  One launch serves every such
// layer of a call; a thread owns four consecutive out-features of one token.
constexpr int kSplitLayersMax = 60;
struct SplitLayer {
  const float* partial;  // [splits][T][O]
  const float* bias;     // nullable
  void* Y;
  int64_t ldy;
  int32_t T, O, splits, out_bf16;
  uint32_t block_end;    // exclusive prefix end, in blocks of 256 threads
  int32_t vec;           // Y rows in whole aligned pieces of four outputs
};
struct SplitGroup {
  int32_t count;
  SplitLayer layer[kSplitLayersMax];
};
static_assert(sizeof(SplitGroup) <= 4096, "the table must fit the kernel argument segment");

__global__ void __launch_bounds__(256) splitk_reduce_kernel(const SplitGroup g) {
  int l = 0;
#pragma unroll 4
  for (int i = 0; i + 1 < g.count; ++i) l += blockIdx.x >= g.layer[i].block_end ? 1 : 0;
  const SplitLayer& L = g.layer[l];
  const unsigned first = l ? g.layer[l - 1].block_end : 0u;
  const int quads = (L.O + 3) >> 2;
  const int64_t q = (int64_t)(blockIdx.x - first) * 256 + threadIdx.x;
  if (q >= (int64_t)L.T * quads) return;
  const int64_t t = q / quads;
  const int o = (int)(q - t * quads) * 4;
  const int64_t plane = (int64_t)L.T * L.O;
  const float* src = L.partial + t * L.O + o;
  float y[4] = {0.f, 0.f, 0.f, 0.f};
  const int n = L.O - o < 4 ? L.O - o : 4;
  if ((L.O & 3) == 0) {
    for (int sp = 0; sp < L.splits; ++sp) {
      const float4 v = *reinterpret_cast<const float4*>(src + sp * plane);
      y[0] += v.x; y[1] += v.y; y[2] += v.z; y[3] += v.w;
    }
  } else {
    for (int sp = 0; sp < L.splits; ++sp)
      for (int e = 0; e < n; ++e) y[e] += src[sp * plane + e];
  }
  if (L.bias != nullptr)
    for (int e = 0; e < n; ++e) y[e] += L.bias[o + e];
  if (L.out_bf16) {
    bf16_t* dst = reinterpret_cast<bf16_t*>(L.Y) + t * L.ldy + o;
    if (L.vec) {
      uint2 pk;
      pk.x = pack_bf16x2(y[0], y[1]);
      pk.y = pack_bf16x2(y[2], y[3]);
      *reinterpret_cast<uint2*>(dst) = pk;
    } else {
      for (int e = 0; e < n; ++e) dst[e] = (bf16_t)f32_to_bf16_rne(y[e]);
    }
  } else {
    float* dst = reinterpret_cast<float*>(L.Y) + t * L.ldy + o;
    if (L.vec) *reinterpret_cast<float4*>(dst) = make_float4(y[0], y[1], y[2], y[3]);
    else
      for (int e = 0; e < n; ++e) dst[e] = y[e];
  }
}

// ---------------------------------------------------------------------------------------------
// Persistent streamed product for large layers.
//
// One block of 8 waves (4 along O x 2 along T, 64 x 16 TT outputs each) per CU walks over its share of
// the output tiles, 256 out-features x 32 TT tokens; the LDS stage ring and the load pipeline run across tile boundaries,
// so the first stages of the next tile are already in flight (and its first fragments in registers)
// while the current tile is being written out, and the stores of one tile drain while the next one
// is multiplied.  A K step is 4 TT matrix instructions per wave for both operand forms: K = 64 of
// the 2:4 form through v_smfmac_f32_16x16x64_bf16, K = 32 of the dense form through
// v_mfma_f32_16x16x32_bf16.
// Per step a wave keeps its 4 W fragments in registers and reads the TT X fragments three groups or more ahead
// of the four instructions that consume each; the fragments of the next step are
// fetched during the last groups of the current one.  Before anything of stage g+1 is read (group BAR of stage g) every wave
// has issued all its reads of stage g: it drains them, makes sure its
// share of stage g+1 has landed, meets the others at the step's only barrier and then refills the
// buffer of stage g with stage g+STAGES, two full steps or more ahead of its use.
// The tiles that share X rows (same tokens, other out-features) run on one XCD at the same time; each
// walks K from its own starting step and wraps around, so that they do not miss on the same lines together.
// The weight arrives in stream order (see the pre-pass above): every W load is one contiguous
// kilobyte.  A ragged last token tile is shifted back inside X (it recomputes a few rows of its
// neighbour but stores only its own) and the weight is zero-padded to whole tiles, so every tile is
// full and lane offsets never change.
// ---------------------------------------------------------------------------------------------
template <bool SPARSE, int TT_, bool I8 = false>
struct StreamCfg {
  // Tiles are 256 out-features x 32 TT tokens on 8 waves (one block per CU, two waves per SIMD); a wave holds 64
  // out-features x 16 TT tokens (WO 4, WT 2), 4 TT accumulator blocks of 16 x 16.  The height
  // is chosen per launch (stream_height): 256 tokens move the fewest operand bytes per product, but 12608 tokens x 768
  // out-features are 150 such tiles on 256 compute units, and 198 of 192 tokens are done sooner.
  // Measured and no faster on transformer-sized layers: WO 2, WT 4 (128 x 64 per wave: a fifth fewer fragment
  // bytes, the same time in the 2:4 form and 4 % more in the dense form), 4 waves of 128 x 128 (one per SIMD
  // with the 512-register budget: a lone wave does not hide its own LDS and issue latency), and 256 x 128 tiles
  // with two stages (two blocks of 4 waves per CU).
  static constexpr int WO = 4, WT = 2, BO = 256, OT = BO / (WO * 16), TT = TT_;
  static constexpr int TW = TT * 16, BT = TW * WT;       // tokens per wave, per tile
  static constexpr int NW = WO * WT, NT = NW * 64;
  static constexpr int OW = OT * 16;                     // out-features per wave
  // The int8 forms (v_smfmac_i32_16x16x128_i8, v_mfma_i32_16x16x64_i8) have the same geometry in bytes with
  // twice the K per step; only the selectors differ: a lane's 16 compressed values need a whole 32-bit word,
  // so a row takes 16 bytes of selectors per step instead of 8 and no two rows share a word.
  static constexpr int ES = I8 ? 1 : 2;                  // bytes per operand element
  static constexpr int X_ROWB = SPARSE ? 128 : 64;       // bytes of one X row per stage
  static constexpr int KSTEP = X_ROWB / ES;              // dense k per stage
  static constexpr int A_ROWB = 64;                      // compressed values of the 2:4 form, or dense weights
  static constexpr int X_BYTES = BT * X_ROWB;
  static constexpr int A_BYTES = BO * A_ROWB;
  static constexpr int S_ROWB = I8 ? 16 : 8;
  static constexpr int S_BYTES = SPARSE ? BO * S_ROWB : 0;
  static constexpr int STAGE = X_BYTES + A_BYTES + S_BYTES;
  // as many stages as fit: three of the 2:4 form's, four of the smaller ones
  static constexpr int STAGES = 4 * STAGE + 4 * BO * 4 <= 160 * 1024 ? 4 : 3;
  // Per-out-feature constants of a tile travel through LDS: the bias (one slice of BO floats per stage buffer,
  // read when the tile starts), or for int8 the weight scales and the bias (read when the tile ends, so the
  // slices alternate with the tile's parity instead: two pairs)
  static constexpr int BIAS0 = STAGES * STAGE;
  static constexpr int LDS_BYTES = BIAS0 + (I8 ? 4 : STAGES) * BO * 4;
  static constexpr int X_LOADS = X_BYTES / 1024;         // wave-wide loads of a stage
  static constexpr int X_PW = (X_LOADS + NW - 1) / NW;   // of a wave; waves from X_FULL on have one less
  static constexpr int X_FULL = X_LOADS % NW == 0 ? NW : X_LOADS % NW;
  static constexpr int A_PW = A_BYTES / 1024 / NW;
  static constexpr int S_PW = SPARSE ? S_BYTES / 256 / NW : 0;
  static constexpr int LPW = X_PW + A_PW + S_PW;
  // Schedule of a step of TT groups (4 matrix instructions each): the barrier stands before group BAR.  After it the
  // weight fragments of the next stage are read in two groups from W_GROUP on and its first PRE X fragments one per
  // group; the other X fragments are read in their own step, before the barrier.  Where the registers allow it
  // (everywhere but in the highest 2:4-form tile) the last of those reads is two groups before the barrier, which
  // drains them, and the weight comes first after it: 3 - 8 % on the dense form of 160 to 224 tokens, nothing on the
  // 2:4 form.
  static constexpr bool ROOMY = !(SPARSE && TT == 8);
  static constexpr int BAR = TT == 4 ? 1 : (ROOMY ? TT - 4 : TT - 3), PRE = TT - BAR;
  static constexpr int W_GROUP = ROOMY ? BAR : TT - 2;
  static constexpr int read_group(int f) {               // group that reads X fragment f (PRE <= f < TT) of its own step
    return !ROOMY ? f - PRE : TT == 8 ? (f == 4 ? 0 : f == 7 ? 2 : 1) : (TT == 7 && f == 6 ? 1 : 0);
  }
  static_assert(BO * 4 == 1024, "the bias slice of a tile is one wave-load");
  static_assert(LDS_BYTES <= 160 * 1024 && STAGES * (LPW + 2) < 64, "LDS budget and vmcnt range");
};

// One launch serves a list of layers of the same operand form: their tiles form one list (layer after layer),
// which the blocks share as they share the tiles of a single layer.  A stack of independent products then ends
// in ONE partial round of tiles instead of one per layer (591 tiles on 256 compute units are 2.3 rounds and
// cost 3).  The table travels in the kernel arguments.
struct StreamLayer {
  const bf16_t* A;      // stream-order values (2:4 form) or dense weight
  const uint32_t* sel;  // stream-order selectors (2:4 form)
  const bf16_t* X;
  const float* bias;    // nullable
  const float* scale;   // int8: per-out-feature weight scales, nullable (= 1)
  void* Y;
  int32_t O, T, nk, ldx, ldy;  // nk: K steps of the form; ldx, ldy in elements
  int32_t n_o_tiles;
  int32_t n_tiles;      // tiles of this layer
  float x_scale;        // int8: activation scale
  int32_t out_kind;     // NM_OUT_F32 / NM_OUT_BF16 / NM_OUT_I32 (int8 only)
  int32_t reserved;
};
constexpr int kStreamLayersMax = 44;
struct StreamGroup {
  int32_t count, n_tiles;
  StreamLayer layer[kStreamLayersMax];
};
static_assert(sizeof(StreamGroup) <= 4096, "the table must fit the kernel argument segment");

// TURN_IN_LDS (2:4 form): which write-out, and when the W loads leave; see there.
template <bool SPARSE, int TT_, bool I8, bool TURN_IN_LDS>
__global__ void __launch_bounds__(512, 2)
nm_stream_kernel(const StreamGroup g) {
  using C = StreamCfg<SPARSE, TT_, I8>;
  constexpr int OT = C::OT, TT = C::TT, STAGES = C::STAGES;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  // ---- this block's tiles: every XCD (block id mod 8) owns a contiguous eighth of the tiles of EVERY layer,
  // out-feature tiles fastest; its list is those ranges layer after layer, and its blocks take the entries
  // round-robin.  So the blocks sharing an L2 work on neighbouring tiles (same X rows) at the same time, and
  // every XCD gets the same share of each layer's work, whatever the layers' K.
  const int xcd = (int)(blockIdx.x & 7);
  const int slots = (int)(gridDim.x >> 3);
  auto xcd_share = [&](int layer) {  // how many tiles of the layer this XCD owns
    const int n = g.layer[layer].n_tiles;
    const int per = (n + 7) >> 3;
    const int left = n - xcd * per;
    return left < 0 ? 0 : (left < per ? left : per);
  };
  int entries = 0;
  for (int l = 0; l < g.count; ++l) entries += xcd_share(l);
  const int first = (int)(blockIdx.x >> 3);
  if (first >= entries) return;
  const int my_tiles = (entries - first + slots - 1) / slots;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave % C::WO;
  const int wt = wave / C::WO;
  const int r16 = lane & 15;
  const int kb = lane >> 4;

  // ---- per-lane source offsets (they depend on the layer: its row pitch and K steps) and per-wave LDS
  // destinations of this wave's loads.  The W piece a load brings is the one of 16-row group (wave + 8 i) of
  // the tile: group and lane are folded into the lane offset, so every load of a stage uses one of three
  // running base pointers.
  uint32_t x_voff[C::X_PW], w_voff[C::A_PW];
  uint32_t x_dst[C::X_PW], a_dst[C::A_PW];
#pragma unroll
  for (int i = 0; i < C::X_PW; ++i) x_dst[i] = (uint32_t)((wave + i * C::NW) * 1024);
#pragma unroll
  for (int i = 0; i < C::A_PW; ++i) a_dst[i] = (uint32_t)(C::X_BYTES + (wave + i * C::NW) * 1024);
  auto layer_offsets = [&](int ldx, int nk) {
#pragma unroll
    for (int i = 0; i < C::X_PW; ++i) {
      const int j = wave + i * C::NW;
      int row, c;
      if (SPARSE) { row = 8 * j + (lane >> 3); c = (lane & 7) ^ (row & 7); }
      else { row = 16 * j + (lane >> 2); c = (lane & 3) ^ ((row >> 1) & 3); }
      x_voff[i] = (uint32_t)((int64_t)row * ldx * C::ES + c * 16);
    }
#pragma unroll
    for (int i = 0; i < C::A_PW; ++i)
      w_voff[i] = ((uint32_t)((wave + i * C::NW) * nk) << 10) + (uint32_t)(lane * 16);  // < 16 * 2^16 * 2^10
  };
  uint32_t s_voff[C::S_PW > 0 ? C::S_PW : 1], s_dst[C::S_PW > 0 ? C::S_PW : 1];
#pragma unroll
  for (int i = 0; i < C::S_PW; ++i) {
    s_voff[i] = (uint32_t)((wave + i * C::NW) * 256 + lane * 4);
    s_dst[i] = (uint32_t)(C::X_BYTES + C::A_BYTES + (wave + i * C::NW) * 256);
  }

  // ---- the block's n-th tile: its layer (tiles come in ascending order, so the search resumes where it
  // stopped), out-feature tile and token rows.  A ragged last token tile is shifted back inside X.
  struct ListPos { int layer, begin; };  // a layer and the XCD-list entry its range starts at
  auto tile_place = [&](int n, ListPos& at, int& o_tile, int64_t& t_lo, int64_t& t0) {
    const int entry = first + n * slots;
    int share = xcd_share(at.layer);
    while (entry >= at.begin + share) {
      at.begin += share;
      share = xcd_share(++at.layer);
    }
    // The table is read at this point of the program and not earlier: a scalar load the compiler starts before
    // the K steps for use after them stays in flight through the steps, and with it in flight every wait for a
    // fragment read has to drain the wave's whole LDS queue (scalar loads return out of order).
    int layer = at.layer;
    asm volatile("" : "+s"(layer));
    const int local = xcd * ((g.layer[layer].n_tiles + 7) >> 3) + (entry - at.begin);
    const int n_o = g.layer[layer].n_o_tiles;
    o_tile = local % n_o;
    t_lo = (int64_t)(local / n_o) * C::BT;
    const int64_t T = g.layer[layer].T;
    t0 = t_lo + C::BT <= T ? t_lo : T - C::BT;
  };

  // ---- load cursor = the stage to be issued next (tile number in this block, k step) as running pointers: X
  // rows of the tile at the step's k, W and selector blocks of the step
  int ld_n = 0, ld_ks = 0, ld_nk = 1, ld_wrap = 1, ld_offsets_of = -1;
  ListPos ld_at{0, 0};
  uint32_t ld_bias_voff = 0;
  int ld_consts = 0;  // nonzero while the cursor's tile still has per-out-feature constants for this wave to fetch
  const float* ld_bias = nullptr;
  const float* ld_scale = nullptr;
  const unsigned char* ld_x = nullptr;
  const unsigned char* ld_w = nullptr;
  const unsigned char* ld_s = nullptr;
  auto cursor_tile = [&](int n) {
    int o_tile;
    int64_t t_lo, t0;
    tile_place(n, ld_at, o_tile, t_lo, t0);
    const int ld_layer = ld_at.layer;
    const StreamLayer& L = g.layer[ld_layer];
    ld_nk = L.nk;
    if (ld_offsets_of != ld_layer) {
      layer_offsets(L.ldx, ld_nk);
      ld_offsets_of = ld_layer;
    }
    ld_x = reinterpret_cast<const unsigned char*>(L.X) + t0 * L.ldx * C::ES;
    ld_w = reinterpret_cast<const unsigned char*>(L.A) + (((int64_t)o_tile * 16 * ld_nk) << 10);
    ld_s = SPARSE ? reinterpret_cast<const unsigned char*>(L.sel) + (int64_t)o_tile * ld_nk * C::S_BYTES : nullptr;
    // bias[o0 + 4 lane ..]: past the last out-feature re-read the last four (never stored)
    const int64_t ob = (int64_t)o_tile * C::BO + lane * 4;
    ld_bias = L.bias;
    ld_scale = L.scale;
    ld_bias_voff = (uint32_t)((ob + 4 <= L.O ? ob : L.O - 4) * 4);
    ld_consts = (wave == 0 && (ld_bias != nullptr || (I8 && ld_scale != nullptr))) ? 1 : 0;
    // The tiles that share the tile's X rows (same tokens, other out-features) run on the same XCD at the
    // same time; each starts at its own K step and wraps around, so they ask for different slices of those rows
    // at any moment and find the others' slices in L2 instead of missing on them together.  The start depends on
    // the out-features alone, so that a sum is added up in the same order whatever the tile height.
    ld_wrap = ld_nk - (int)((unsigned)o_tile % (unsigned)ld_nk);  // steps until the walk wraps to K step 0
    const int64_t k0 = ld_nk - ld_wrap;
    ld_x += k0 * C::X_ROWB;
    ld_w += k0 * 1024;
    if (SPARSE) ld_s += k0 * C::S_BYTES;
    ld_n = n;
    ld_ks = 0;
  };
  auto cursor_advance = [&]() {
    ld_x += C::X_ROWB;
    ld_w += 1024;
    if (SPARSE) ld_s += C::S_BYTES;
    // past the block's last stage the cursor walks the last tile again: the step below then needs no
    // conditions (the surplus stages land in buffers nobody reads any more)
    if (++ld_ks == ld_wrap) {
      ld_x -= (int64_t)ld_nk * C::X_ROWB;
      ld_w -= (int64_t)ld_nk * 1024;
      if (SPARSE) ld_s -= (int64_t)ld_nk * C::S_BYTES;
    }
    if (ld_ks == ld_nk) cursor_tile(ld_n + 1 < my_tiles ? ld_n + 1 : ld_n);
  };
  // the d-th of this wave's LPW loads of the cursor's stage into the stage buffer at LDS offset stage_off
  auto issue_one = [&](auto d_tag, uint32_t stage_off) {
    constexpr int d = decltype(d_tag)::value;
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds0 + stage_off);
    if constexpr (d == 0) {
      // a tile's first stage brings the tile's bias slice along (older than the stage's own loads, so
      // every wait that covers the stage covers it); slice s belongs to stage buffer s
      if (ld_consts) {  // wave 0 also fetches the tile's per-out-feature constants, once (one test per step)
        ld_consts = 0;
        if constexpr (I8) {
          const uint32_t pair = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)C::BIAS0 + (uint32_t)(ld_n & 1) * (2 * C::BO * 4));
          if (ld_scale != nullptr) dma16(make_uniform(ld_scale), ld_bias_voff, pair);
          if (ld_bias != nullptr) dma16(make_uniform(ld_bias), ld_bias_voff, pair + C::BO * 4);
        } else if (ld_bias != nullptr) {
          dma16(make_uniform(ld_bias), ld_bias_voff,
                __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)C::BIAS0 + stage_off / (uint32_t)C::STAGE * (C::BO * 4)));
        }
      }
    }
    if constexpr (d < C::X_PW) {
      if (d + 1 < C::X_PW || C::X_FULL == C::NW || wave < C::X_FULL)
        dma16_at(make_uniform(ld_x), x_voff[d], lds, __builtin_amdgcn_readfirstlane(x_dst[d]));
    } else if constexpr (d < C::X_PW + C::A_PW) {
      constexpr int q = d - C::X_PW;
      dma16_at(make_uniform(ld_w), w_voff[q], lds, __builtin_amdgcn_readfirstlane(a_dst[q]));
    } else {
      constexpr int q = d - C::X_PW - C::A_PW;
      dma4_at(make_uniform(ld_s), s_voff[q], lds, __builtin_amdgcn_readfirstlane(s_dst[q]));
    }
  };
  // at most this wave's loads of STAGES - 2 whole stages, and HEADS of the one after, outstanding
  auto wait_younger = [&](auto heads_tag) {
    constexpr int HEADS = decltype(heads_tag)::value;
    constexpr int LESS = HEADS >= C::X_PW ? 1 : 0;  // the load the later waves do not have is the last X load of a stage
    if (C::X_FULL == C::NW || wave < C::X_FULL) wait_loads_outstanding<(STAGES - 2) * C::LPW + HEADS>();
    else wait_loads_outstanding<(STAGES - 2) * (C::LPW - 1) + HEADS - LESS>();
  };

  // ---- fragment readers (the XOR undoes the swizzle applied by the loads).  A lane's four fragment
  // addresses inside a stage buffer (W values, its 16 selector bits, the two halves of an X row) are kept
  // for the current and for the next buffer; the two sets swap roles from step to step, so a step spends
  // four vector additions on addresses and none on moving fragments: vector ALU instructions take issue
  // slots from the matrix instructions of both waves of the SIMD.
  using bfrag_t = std::conditional_t<SPARSE, u32x8_t, u32x4_t>;
  struct FragAddr { uint32_t a, s, xlo, xhi; };  // byte offsets into the dynamic LDS
  FragAddr at0;
  at0.a = (uint32_t)(C::X_BYTES + (wo * C::OW + r16) * C::A_ROWB + ((kb ^ ((r16 >> 1) & 3)) * 16));
  at0.s = (uint32_t)(C::X_BYTES + C::A_BYTES + (I8 ? wo * OT : wo * C::OW / 32) * 256 + r16 * 16 + kb * 4);
  at0.xlo = (uint32_t)((wt * C::TW + r16) * C::X_ROWB + (SPARSE ? ((kb ^ (r16 & 7)) * 16) : ((kb ^ ((r16 >> 1) & 3)) * 16)));
  at0.xhi = (uint32_t)((wt * C::TW + r16) * C::X_ROWB + ((4 + kb) ^ (r16 & 7)) * 16);
  auto frag_addr = [&](uint32_t stage_off) {
    return FragAddr{at0.a + stage_off, at0.s + stage_off, at0.xlo + stage_off, at0.xhi + stage_off};
  };
  // W fragments come in pairs of 16-row blocks: for bfloat16 one selector word serves both (low / high half),
  // for int8 each block has its own word (sv holds the pair)
  constexpr int SV = I8 ? 2 : 1;  // selector registers per pair of blocks
  auto read_a2 = [&](const FragAddr& at, int ip, u32x4_t& av0, u32x4_t& av1, int* sv) {
    av0 = *reinterpret_cast<const u32x4_t*>(smem + at.a + (2 * ip) * 16 * C::A_ROWB);
    av1 = *reinterpret_cast<const u32x4_t*>(smem + at.a + (2 * ip + 1) * 16 * C::A_ROWB);
#pragma unroll
    for (int q = 0; q < SV; ++q)
      sv[q] = SPARSE ? (int)*reinterpret_cast<const uint32_t*>(smem + at.s + (ip * SV + q) * 256) : 0;
  };
  auto read_b = [&](const FragAddr& at, int j, bfrag_t& bv) {
    if constexpr (SPARSE) {
      const u32x4_t lo = *reinterpret_cast<const u32x4_t*>(smem + at.xlo + j * 16 * C::X_ROWB);
      const u32x4_t hi = *reinterpret_cast<const u32x4_t*>(smem + at.xhi + j * 16 * C::X_ROWB);
      bv = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      bv = *reinterpret_cast<const u32x4_t*>(smem + at.xlo + j * 16 * C::X_ROWB);
    }
  };

  // ---- prologue: three stages in flight, the first one landed, its first fragments in registers
  // A stage's loads leave LPG at a time (one, when there are as many groups as loads), SPREAD groups apart, from
  // the barrier that frees the buffer (before group BAR) round to the groups before the next step's barrier:
  // loads d LPG .. d LPG + LPG - 1 after group (BAR + d SPREAD) mod TT.
  // HEAD of them fall into the step that freed the buffer, the others into the next one.  The requests of the
  // eight waves then reach the CU's one load path spread over the step instead of in one burst, behind which
  // every wave's matrix instructions would queue (a wave issues in order).
  // TURN_IN_LDS: the W loads of a stage leave in the next step, after the write-out of a tile that ended with the buffer's
  // step: the write-out uses the part of the buffer that they refill.  Where the even spacing brings them earlier, the X
  // loads and selectors go into the groups of the step that freed the buffer and the W loads into the first ones of the next.
  constexpr int LPG = (C::LPW + C::TT - 1) / C::TT;                     // loads that leave together
  constexpr int SLOTS = (C::LPW + LPG - 1) / LPG;
  constexpr int SPREAD = 2 * SLOTS <= C::TT ? 2 : 1;
  constexpr bool EVEN = !TURN_IN_LDS || C::X_PW / LPG * SPREAD >= C::PRE;
  constexpr int EARLY = C::X_PW + C::S_PW;                              // loads that are not of W
  constexpr int EARLY_PER = (EARLY + C::PRE - 1) / C::PRE;
  constexpr int LAST = EVEN ? C::LPW - 1 : C::X_PW + C::A_PW - 1;       // the load that completes a stage
  auto since_of = [](int d) constexpr {                                 // groups between the barrier and the d-th load
    if (EVEN) return d / LPG * SPREAD;
    const int q = d - C::X_PW;
    if (q >= 0 && q < C::A_PW) return C::PRE + (q < C::BAR ? q : C::BAR - 1);
    return (q < 0 ? d : d - C::A_PW) / EARLY_PER;
  };
  constexpr int HEAD_EVEN = (C::PRE + SPREAD - 1) / SPREAD * LPG;
  constexpr int HEAD = !EVEN ? EARLY : HEAD_EVEN < C::LPW ? HEAD_EVEN : C::LPW;  // loads that leave in the step that freed the buffer
  static_assert(since_of(C::LPW - 1) < C::TT && since_of(LAST) < C::TT && HEAD <= C::LPW, "the last load must be out before the next step's wait");
  static_assert(!TURN_IN_LDS || since_of(C::X_PW) >= C::PRE && since_of(C::X_PW + C::A_PW - 1) >= C::PRE, "W loads follow the write-out");
  cursor_tile(0);
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    [&]<int... D>(std::integer_sequence<int, D...>) {  // the last one's tail leaves in the first step
      ([&] {
        constexpr int d = D;
        if (s + 1 < STAGES || since_of(d) < C::PRE) issue_one(std::integral_constant<int, d>{}, (uint32_t)(s * C::STAGE));
      }(), ...);
    }(std::make_integer_sequence<int, C::LPW>{});
    if (s + 1 < STAGES || HEAD == C::LPW) cursor_advance();
  }
  wait_younger(std::integral_constant<int, HEAD>{});
  __builtin_amdgcn_s_barrier();

  u32x4_t afr[2][OT];  // W fragments of the current step and of the next one; the roles alternate
  int sfr[2][OT / 2 * SV];
  FragAddr at[2];      // likewise the fragment addresses in the current and in the next buffer
  bfrag_t bq[TT];
  at[0] = at0;
#pragma unroll
  for (int ip = 0; ip < OT / 2; ++ip) read_a2(at[0], ip, afr[0][2 * ip], afr[0][2 * ip + 1], &sfr[0][ip * SV]);
#pragma unroll
  for (int j = 0; j < C::PRE; ++j) read_b(at[0], j, bq[j]);

  uint32_t cur_off = 0;  // LDS offset of the buffer that holds the current stage
  using acc_t = std::conditional_t<I8, i32x4_t, f32x4_t>;
  acc_t acc[OT][TT];

  // One K step, free of conditions: a wave issues one instruction at a time, in order, so every other
  // instruction of the step is time its matrix instructions do not get.  PP names the fragment and address
  // set the step multiplies with.  Every other group takes the W fragments backwards, so that an operand stays between two
  // instructions: a loop of dense instructions fed from LDS 0.590 -> 0.580 us a step, int8 0.615 -> 0.583, the sparse ones the same;
  // of the products nothing that their spread shows (0.1 to 0.2 % on average over 360 bfloat16 and 240 int8 shapes).  Every step refills the buffer it has consumed and prefetches fragments
  // of the next stage, also past the block's last stage.
  auto step = [&](auto pp_tag) {
    constexpr int PP = decltype(pp_tag)::value;
    uint32_t nxt_off = cur_off + C::STAGE;
    if (nxt_off == (uint32_t)(STAGES * C::STAGE)) nxt_off = 0;
    at[PP ^ 1] = frag_addr(nxt_off);
    const uint32_t prev_off = cur_off == 0 ? (uint32_t)((STAGES - 1) * C::STAGE) : cur_off - (uint32_t)C::STAGE;
    [&]<int... J>(std::integer_sequence<int, J...>) {
      ([&] {
        constexpr int j = J;
        if constexpr (j == C::BAR) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // all this wave's reads of the stage are back
          wait_younger(std::integral_constant<int, 0>{});     // this wave's share of the next stage has landed
          __builtin_amdgcn_s_barrier();
        }
        if constexpr (j < C::BAR) {
          [&]<int... F>(std::integer_sequence<int, F...>) {
            ([&] {
              if constexpr (C::PRE + F < TT && C::read_group(C::PRE + F) == j) read_b(at[PP], C::PRE + F, bq[C::PRE + F]);
            }(), ...);
          }(std::make_integer_sequence<int, TT>{});
        } else {
          if constexpr (j >= C::W_GROUP && j < C::W_GROUP + 2) {
            constexpr int part = j - C::W_GROUP;
#pragma unroll
            for (int ip = part * (OT / 2) / 2; ip < (part + 1) * (OT / 2) / 2; ++ip)
              read_a2(at[PP ^ 1], ip, afr[PP ^ 1][2 * ip], afr[PP ^ 1][2 * ip + 1], &sfr[PP ^ 1][ip * SV]);
          }
          read_b(at[PP ^ 1], j - C::BAR, bq[j - C::BAR]);
        }
        [&]<int... I>(std::integer_sequence<int, I...>) {
          ([&] {
            constexpr int i = j & 1 ? OT - 1 - I : I;  // back and forth
            if constexpr (SPARSE && I8)
              acc[i][j] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(__builtin_bit_cast(i32x4_t, afr[PP][i]),
                                                                   __builtin_bit_cast(i32x8_t, bq[j]), acc[i][j],
                                                                   sfr[PP][i], 0, 0);
            else if constexpr (I8)
              acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4_t, afr[PP][i]),
                                                                __builtin_bit_cast(i32x4_t, bq[j]), acc[i][j], 0, 0, 0);
            else if constexpr (SPARSE)
              acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8_t, afr[PP][i]),
                                                                    __builtin_bit_cast(bf16x16_t, bq[j]),
                                                                    acc[i][j], sfr[PP][i / 2], 0, i & 1);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, afr[PP][i]),
                                                                  __builtin_bit_cast(bf16x8_t, bq[j]), acc[i][j],
                                                                  0, 0, 0);
          }(), ...);
        }(std::make_integer_sequence<int, OT>{});
        {
          // the load that leaves after this group, if any: into the buffer this step has consumed (free since the
          // barrier), or the rest of the stage begun in the previous step into the buffer consumed there
          constexpr int since = (j - C::BAR + TT) % TT;  // groups since the barrier
          [&]<int... D>(std::integer_sequence<int, D...>) {
            ([&] {
              constexpr int d = D;
              if constexpr (since_of(d) == since) {
                issue_one(std::integral_constant<int, d>{}, j >= C::BAR ? cur_off : prev_off);
                if constexpr (d == LAST) cursor_advance();
              }
            }(), ...);
          }(std::make_integer_sequence<int, C::LPW>{});
        }
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, TT>{});
    cur_off = nxt_off;
  };

  ListPos cp_at{0, 0};
  for (int n = 0; n < my_tiles; ++n) {
    int o_tile;
    int64_t t_lo, t0;
    tile_place(n, cp_at, o_tile, t_lo, t0);
    const StreamLayer& L = g.layer[cp_at.layer];
    const int nk = L.nk;
    const int64_t o0 = (int64_t)o_tile * C::BO;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if constexpr (I8) {
#pragma unroll
        for (int j = 0; j < TT; ++j) acc[i][j] = i32x4_t{0, 0, 0, 0};
      } else {
        // the accumulators start from the bias, which came with the tile's first stage
        f32x4_t b = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (L.bias != nullptr)
          b = *reinterpret_cast<const f32x4_t*>(smem + C::BIAS0 + cur_off / (uint32_t)C::STAGE * (C::BO * 4) +
                                                (wo * C::OW + i * 16 + kb * 4) * 4);
#pragma unroll
        for (int j = 0; j < TT; ++j) acc[i][j] = b;
      }
    }

    // The layer's output geometry goes into registers now: read through the table entry after the steps, every
    // store would wait for a scalar load of its own (and for everything else the wave has in flight with it).
    int32_t ldy_s = L.ldy, o_s = L.O, kind_s = L.out_kind;
    uint64_t y_s = reinterpret_cast<uint64_t>(L.Y);
    asm volatile("" : "+s"(ldy_s), "+s"(o_s), "+s"(kind_s), "+s"(y_s));
    // Nothing of this wave's LDS or scalar reads is in flight when the steps begin (it costs nothing here: all of
    // them have just been used); the compiler then counts the fragment reads inside the steps exactly instead of
    // draining the queue at the first waits of every pair of steps.
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only

    // steps in pairs, so that every tile starts with fragment set 0; an odd count ends with a copy
    for (int ks = 0; ks + 1 < nk; ks += 2) {
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
    }
    if (nk & 1) {
      step(std::integral_constant<int, 0>{});
      at[0] = at[1];
#pragma unroll
      for (int i = 0; i < OT; ++i) afr[0][i] = afr[1][i];
#pragma unroll
      for (int i = 0; i < OT / 2 * SV; ++i) sfr[0][i] = sfr[1][i];
    }
    if (n + 1 == my_tiles) wait_loads_outstanding<0>();  // the surplus stages: nothing in flight when the block ends

    // ---- write the tile out.  A lane holds out-features o .. o+3 of token r16 per 16 x 16 block; for bfloat16 the eight
    // pieces of a token row's 128 bytes (the wave's 64 out-features) are brought into eight consecutive lanes: a store
    // instruction is merged only across consecutive lanes, and whole lines leave as single requests.  The stores
    // carry the non-temporal hint: the output is never read back by this kernel, and lines that linger in L2 until
    // write-back push out the X rows the neighbouring tiles still need (with the hint the launch fetches a quarter
    // less; on half lines the same hint costs 40 % more written bytes).
    // int8: the sums are rescaled first, y = fma(float(acc), x_scale * w_scale[o], bias[o]); the tile's scales
    // and bias came with its first stage (pair n mod 2, so the next tile's do not overwrite them)
    f32x4_t sc[I8 ? OT : 1], bi[I8 ? OT : 1];
    if constexpr (I8) {
      const unsigned char* pair = smem + C::BIAS0 + (n & 1) * (2 * C::BO * 4);
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        const int off = (wo * C::OW + i * 16 + kb * 4) * 4;
        sc[i] = f32x4_t{L.x_scale, L.x_scale, L.x_scale, L.x_scale};
        bi[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (L.scale != nullptr) sc[i] *= *reinterpret_cast<const f32x4_t*>(pair + off);
        if (L.bias != nullptr) bi[i] = *reinterpret_cast<const f32x4_t*>(pair + C::BO * 4 + off);
      }
    }
    auto value = [&](int i, int j) -> f32x4_t {
      if constexpr (I8) {
        f32x4_t y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fmaf((float)acc[i][j][e], sc[i][e], bi[i][e]);
        return y;
      } else {
        return acc[i][j];
      }
    };
    // global address space, so that the stores are not counted with the LDS operations
    using gbyte_t = __attribute__((address_space(1))) unsigned char;
    using gpiece_t = __attribute__((address_space(1))) u32x4_t;
    const int first_row = (int)(t_lo - t0);  // rows of a shifted last tile below this one belong to its neighbour
    if (kind_s == 1) {
      // Whole 128-byte lines per store: a wave's 64 out-features are one line of a token row.  lines_of(j) gives a lane
      // its pieces of token rows lane / 8 and lane / 8 + 8 of 16-row block j.
      static_assert(OT == 4 && C::A_PW == 2, "a line is four blocks; two kilobytes per wave");
      struct Lines { u32x4_t first, second; };
      // 2:4 form: the wave turns 16 token rows at a time through two kilobytes of LDS, the places of its own W loads in the
      // buffer that the last step has freed (they leave in the next step): 8 bytes per lane and block in, 16-byte pieces
      // of whole rows out, the pieces of a row XOR-swizzled with the row (rows 8..15 on the other parity than rows 0..7, which
      // lie on the same banks: without it every write takes two passes).  The LDS operations of a wave run in order, so
      // nothing waits between a write and a read.  Against the exchange below: 12608 tokens x 768 -> 768 15.1 -> 14.5 us,
      // 3072 -> 768 36.3 -> 35.0, 50432 x 768 -> 3072 145 -> 140; int8 by tile height, see stream_i8_turns.
      // The dense form, whose loads would have to move for it, loses up to 6 % (3072 -> 768 54.0 -> 57.4).
      const uint32_t freed = cur_off == 0 ? (uint32_t)((STAGES - 1) * C::STAGE) : cur_off - (uint32_t)C::STAGE;
      unsigned char* slice = smem + freed + C::X_BYTES + wave * 1024;     // rows 0..7; rows 8..15 lie C::NW kilobytes further
      unsigned char* put = slice + (r16 >> 3) * (C::NW * 1024) + (r16 & 7) * 128 + (kb & 1) * 8;
      uint32_t put_at[OT];
#pragma unroll
      for (int i = 0; i < OT; ++i) put_at[i] = (uint32_t)(((2 * i + (kb >> 1)) ^ (r16 & 7) ^ (r16 >> 3)) * 16);
      const unsigned char* get = slice + (lane >> 3) * 128 + ((lane & 7) ^ (lane >> 3)) * 16;
      const unsigned char* get_second = slice + C::NW * 1024 + (lane >> 3) * 128 + ((lane & 7) ^ (lane >> 3) ^ 1) * 16;
      // Dense form: the two 16-byte pieces a lane holds for a token block (out-feature pairs 0 and 1, after the exchange
      // between lane rows) are pushed to the lanes that store them: lane 8m + p stores piece p (0..7) of token row m
      // (first store) and of token row m + 8 (second store).
      const int qk = ((kb & 1) << 1) | (kb >> 1);            // place of this lane's piece inside its pair's 64 bytes
      const int hi_rows = r16 >> 3;                          // this lane's token row belongs to the second store
      const int dest_a = (8 * (r16 & 7) + 4 * hi_rows + qk) * 4;
      const int dest_b = (8 * (r16 & 7) + 4 * (1 - hi_rows) + qk) * 4;
      const bool upper = (lane >> 2) & 1;                    // as a storing lane: pieces 4..7 (out-feature pair 1)
      auto swapped = [&](int j, int ip) {  // ip: out-feature pair (blocks 2 ip and 2 ip + 1)
        const f32x4_t v0 = value(2 * ip, j), v1 = value(2 * ip + 1, j);
        const uint32_t a0 = pack_bf16x2(v0[0], v0[1]), a1 = pack_bf16x2(v0[2], v0[3]);
        const uint32_t b0 = pack_bf16x2(v1[0], v1[1]), b1 = pack_bf16x2(v1[2], v1[3]);
        const auto s0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
        return u32x4_t{(uint32_t)s0[0], (uint32_t)s1[0], (uint32_t)s0[1], (uint32_t)s1[1]};
      };
      auto lines_of = [&](int j) {
        if constexpr (TURN_IN_LDS) {
          asm volatile("" ::: "memory");  // (nor does the compiler move them past one another)
#pragma unroll
          for (int i = 0; i < OT; ++i) {
            const f32x4_t v = value(i, j);
            *reinterpret_cast<uint2*>(put + put_at[i]) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
          }
          asm volatile("" ::: "memory");
          return Lines{*reinterpret_cast<const u32x4_t*>(get), *reinterpret_cast<const u32x4_t*>(get_second)};
        } else {
          const u32x4_t p0 = swapped(j, 0), p1 = swapped(j, 1);
          u32x4_t ra, rb;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // rows 0..7 send pair 0 the first way and pair 1 the second way, rows 8..15 the other way round
            const int send_a = hi_rows ? (int)p1[e] : (int)p0[e];
            const int send_b = hi_rows ? (int)p0[e] : (int)p1[e];
            ra[e] = (uint32_t)__builtin_amdgcn_ds_permute(dest_a, send_a);
            rb[e] = (uint32_t)__builtin_amdgcn_ds_permute(dest_b, send_b);
          }
          Lines l;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            l.first[e] = upper ? rb[e] : ra[e];
            l.second[e] = upper ? ra[e] : rb[e];
          }
          return l;
        }
      };
      const int row = wt * C::TW + (lane >> 3);                            // this lane's row of the tile in block j = 0, first store
      const int64_t col = o0 + wo * C::OW + (lane & 7) * 8;              // its out-features in line 0
      gbyte_t* dst = (gbyte_t*)y_s + ((t0 + row) * (int64_t)ldy_s + col) * 2;
      const int64_t half_bytes = (int64_t)ldy_s * 16;                    // 8 token rows further
      const bool col_ok = col < o_s;
      Lines cur = lines_of(0);
#pragma unroll
      for (int j = 0; j < TT; ++j) {
        Lines nxt = cur;
        if (j + 1 < TT) nxt = lines_of(j + 1);
        if (row + j * 16 >= first_row && col_ok) __builtin_nontemporal_store(cur.first, (gpiece_t*)dst);
        if (row + j * 16 + 8 >= first_row && col_ok) __builtin_nontemporal_store(cur.second, (gpiece_t*)(dst + half_bytes));
        dst += 2 * half_bytes;
        cur = nxt;
      }
    } else {
      const int row = wt * C::TW + r16;
      const int64_t col = o0 + wo * C::OW + kb * 4;
      gbyte_t* dst = (gbyte_t*)y_s + ((t0 + row) * (int64_t)ldy_s + col) * 4;
      const int64_t block_bytes = (int64_t)ldy_s * 64;
      bool col_ok[OT];
#pragma unroll
      for (int i = 0; i < OT; ++i) col_ok[i] = col + i * 16 < o_s;
#pragma unroll
      for (int j = 0; j < TT; ++j) {
#pragma unroll
        for (int i = 0; i < OT; ++i) {
          u32x4_t piece;
          if (I8 && kind_s == 2) piece = __builtin_bit_cast(u32x4_t, acc[i][j]);  // the integer sums themselves
          else piece = __builtin_bit_cast(u32x4_t, value(i, j));
          if (row + j * 16 >= first_row && col_ok[i]) *(gpiece_t*)(dst + i * 64) = piece;
        }
        dst += block_bytes;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Plain gather kernel for shapes the tiles cannot take: one thread per output.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
spmm_general_kernel(const bf16_t* __restrict__ values, const uint32_t* __restrict__ indices, int64_t O, int64_t K, int N,
                    int M, const bf16_t* __restrict__ X, int64_t T, int64_t ldx, const float* __restrict__ bias,
                    void* __restrict__ Y, int64_t ldy, int out_bf16, int64_t n_o_tiles) {
  const int64_t o = (blockIdx.x % n_o_tiles) * 16 + (threadIdx.x & 15);
  const int64_t t = (blockIdx.x / n_o_tiles) * 16 + (threadIdx.x >> 4);
  if (o >= O || t >= T) return;
  const float acc = gather_output(values, indices, K, N, M, X + t * ldx, bias, o);
  if (out_bf16) reinterpret_cast<bf16_t*>(Y)[t * ldy + o] = (bf16_t)f32_to_bf16_rne(acc);
  else reinterpret_cast<float*>(Y)[t * ldy + o] = acc;
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
static inline bool aligned_to(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

static bool tiles_ok(int64_t K, const void* X, int64_t ldx, const void* values, const void* indices, int64_t O,
                     int64_t T) {
  if (K % 64) return false;
  if (!aligned_to(X, 16) || (ldx % 8)) return false;
  if (!aligned_to(values, 16) || !aligned_to(indices, 8)) return false;
  if (O > (1 << 24) || T >= (1ll << 31)) return false;
  if (ldx > (1 << 22) || K > (1 << 22)) return false;  // per-lane byte offsets inside a tile stay below 2^32
  return true;
}

// Estimated durations (microseconds) of the product kernels: models fitted to measured launches on DeiT- and Swin-shaped
// and generic layers.
//   persistent: one block per compute unit walks ceil(tiles / 256) tiles of 256 x 32 TT; a tile takes `nk` steps of
//               step0 + step1 TT and epi0 + epi1 TT to write out, and everything takes up to 1 + busy times as long
//               when the whole chip works on it (memory and power are shared: at 3072 -> 768 a step of the highest
//               2:4 tile takes 0.63 us on 30 compute units and 0.95 on 255).  Fitted on 35 shapes from 1576 to 200704
//               tokens in every height; the height it picks is within 5 % of the best one on all of them (0.3 % on
//               average) and 12 % (2:4 form), 18 % (dense), 7 % and 12 % (int8) faster than always 256 tokens.
//   tiled:      a compute unit works through ceil(tiles / 256) tiles of 128 x 128 (one after the other or two at
//               a time, the rate per unit is the same), `tiled_step_us` per K step of 64 (0.34 us in the 2:4
//               form, 0.5 us in the dense form, whose step holds twice the matrix instructions).
struct StreamModel {
  double step0, step1, epi0, epi1, start, busy;
  double tile(int64_t nk, int tt) const { return (double)nk * (step0 + step1 * tt) + epi0 + epi1 * tt; }
};
constexpr StreamModel kStreamModel[2][2] = {  // [int8][2:4 form]
    {{0.082, 0.050, 0.02, 0.447, 3.4, 0.48}, {0.168, 0.046, 0.06, 0.388, 4.0, 0.60}},
    {{0.092, 0.044, 0.17, 0.476, 3.9, 0.51}, {0.116, 0.035, 0.02, 0.296, 4.9, 1.32}}};
constexpr int kStreamHeights[] = {8, 7, 6, 5, 4};
constexpr double kModelUnits = 256.0;  // compute units of the chip the models were fitted on

// Duration of one layer's launch with tiles of 32 tt tokens.
static double stream_estimate(const StreamModel& m, int64_t O, int64_t T, int64_t nk, int tt) {
  const double tiles = (double)((O + 255) / 256) * (double)((T + 32 * tt - 1) / (32 * tt));
  const double full = (double)(int64_t)(tiles / kModelUnits), rest = tiles - full * kModelUnits;
  return m.start + m.tile(nk, tt) * (full * (1.0 + m.busy) + (rest > 0 ? 1.0 + m.busy * rest / kModelUnits : 0.0));
}
static double stream_estimate(const StreamModel& m, int64_t O, int64_t T, int64_t nk) {
  double best = 0;
  for (int tt : kStreamHeights)
    if (const double e = stream_estimate(m, O, T, nk, tt); tt == kStreamHeights[0] || e < best) best = e;
  return best;
}

// `steps` K steps of 64 or 128, step_us each
static double tiled_estimate(int64_t O, int64_t T, int64_t steps, double step_us) {
  const int64_t tiles = ((O + 127) / 128) * ((T + 127) / 128);
  return (double)((tiles + 255) / 256) * ((double)steps * step_us + 1.5) + 3.0;
}

// Which product kernel a layer of O out-features runs at T tokens: 0 = the persistent kernel, 2 = the tiled kernel with
// 128 x 128 tiles, 3 = with 64 x 64 tiles: the smaller estimate.  A layer with fewer than 64 tiles of 128 x 128 takes
// 64 x 64 tiles: the few tiles there are finish sooner.
static int pick_tile(int64_t O, int64_t T, int64_t stream_steps, const StreamModel& m, int64_t tiled_steps, double tiled_step_us,
                     double margin = 1.0) {
  const int64_t tiles_mid = ((O + 127) / 128) * ((T + 127) / 128);
  if (tiles_mid < 64) return 3;
  if (T < 256) return 2;
  return stream_estimate(m, O, T, stream_steps) <= margin * tiled_estimate(O, T, tiled_steps, tiled_step_us) ? 0 : 2;
}
static int pick_tile(int64_t O, int64_t K, int64_t T, bool sparse_form) {
  // A layer takes the persistent kernel where it is 10 % (2:4 form) or 12 % (dense) faster by the estimates: within that
  // the tiled one, whose tile is chosen afterwards (tile_kind), wins (45581 x 512 -> 384 at 2:16 in fp32
  // 31.9 and 27.7 us).  A tile of one 64-wide step has no step to load the next one under: a quarter more (6666 x 64 ->
  // 1176 at 2:8 14.7 and 11.4).  An output beyond 200 MB leaves the memory-side
  // cache, and the persistent kernel's stores, which do not linger there, make up for it (dense form, 35857 x 64 -> 4096
  // 54 and 91 us).  Measured on 43000 shapes in every kernel and tile, buffers in the cache and not: of 10300 dense-form
  // ones 890 lost over 5 % to a fixed tile by shape alone without the two last rules, a margin and tile_kind's, 510 with them.
  double margin = sparse_form ? 0.9 : 0.88;
  if (K == 64) margin *= 0.75;
  if (T * O > 100000000) margin = sparse_form ? 0.9 : 1.0;
  return pick_tile(O, T, sparse_form ? K / 64 : K / 32, kStreamModel[0][sparse_form], K / 64, sparse_form ? 0.34 : 0.5, margin);
}

// A reduction that is no whole number of 64-wide steps: the ragged form of the tiled kernel multiplies it from stream
// order padded with zeros.  The workspace it needs is optional (without it the gather kernel reads the packed layout);
// a reduction shorter than one step is left to the gather kernel and asks for none.
static bool ragged_shape(int64_t O, int64_t K, int64_t T) {
  return (K % 64) != 0 && K > 64 && O <= (1 << 24) && T < (1ll << 31) && K <= (1 << 22);
}
static int64_t padded_k(int64_t K) { return (K + 63) / 64 * 64; }

// The form in which the product kernels read a layer's weight at T tokens.
//   FORM_PACKED  as packed: the gather kernel, or the tiled kernel at 2:4 and at N = M, whose packed layouts already
//                are the row-major 2:4 / dense operands
//   FORM_STREAM  stream order in the workspace (2:4 form for N <= 2, dense form otherwise): every other level, every
//                level on the persistent kernel, and every level where K is no whole number of steps
enum { FORM_PACKED = 0, FORM_STREAM = 1 };
static int operand_form(int64_t O, int64_t K, int64_t T, int N, int M, bool* sparse_form) {
  *sparse_form = N <= 2 && N < M;
  if (K % 64) return ragged_shape(O, K, T) ? FORM_STREAM : FORM_PACKED;
  const bool as_packed = (N == 2 && M == 4) || N == M;
  return (pick_tile(O, K, T, *sparse_form) != 0 && as_packed) ? FORM_PACKED : FORM_STREAM;
}

// whether the layer's weight lies in stream order without padding along K (what a packing kernel can write as it goes)
bool spmm_stream_order(int64_t O, int64_t K, int64_t T, int N, int M, bool* sparse_form) {
  return K % 64 == 0 && operand_form(O, K, T, N, M, sparse_form) == FORM_STREAM;
}

// Ranges the reduction of a layer on the tiled kernel is cut into: a layer with far fewer tiles than the chip has
// compute units and a long K (one image through a wide MLP: 197 tokens, K = 4096) leaves most units idle for many
// steps; cut into ranges of at least 12 steps, it fills them, at the price of fp32 partial sums through memory and
// a reduce launch (about 5 us: below 64 steps the cut gains nothing; measured on ViT-S .. ViT-H shaped layers).
// A function of the shape alone.
static int split_count(int64_t O, int64_t K, int64_t T, bool sparse_form) {
  const int64_t steps = K / 64;
  if (K % 64 || steps < 64) return 1;
  const int pick = pick_tile(O, K, T, sparse_form);
  if (pick == 0) return 1;
  const int64_t side = pick == 2 ? 128 : 64;
  const int64_t tiles = ((O + side - 1) / side) * ((T + side - 1) / side);
  if (tiles >= 128) return 1;
  int64_t n = 256 / tiles;
  if (n > steps / 12) n = steps / 12;
  if (n > 8) n = 8;
  while (n > 1 && (n - 1) * ((steps + n - 1) / n) >= steps) --n;  // no empty range
  return n < 2 ? 1 : (int)n;
}
static size_t operand_bytes(int64_t O, int64_t K, int N, int M, int64_t T, bool* sparse_form) {
  if (operand_form(O, K, T, N, M, sparse_form) != FORM_STREAM) return 0;
  const size_t o_pad = (size_t)((O + 255) / 256) * 256;  // whole 256-row tiles
  const size_t k_pad = (size_t)padded_k(K);
  return *sparse_form ? o_pad * k_pad + o_pad * k_pad / 8 : o_pad * k_pad * 2;
}

// The part of the workspace a product cannot do without: the operand-order copy.  With no more than that the
// reduction stays in one piece.  (A ragged reduction can do without: the gather kernel takes it then.)
size_t spmm_operand_workspace_bytes(int64_t O, int64_t K, int N, int M, int64_t T) {
  if (K % 64) return 0;
  bool sparse_form = false;
  return operand_bytes(O, K, N, M, T, &sparse_form);
}

// Partial sums of a cut reduction.  They belong to one call: a prepared layer's workspace serves calls on several streams at
// once, and two layers of a batched call may share it, so a call that does not own its workspace brings them beside it.
size_t spmm_partial_bytes(int64_t O, int64_t K, int N, int M, int64_t T) {
  const int splits = split_count(O, K, T, N <= 2 && N < M);
  return splits < 2 ? 0 : (size_t)splits * (size_t)T * (size_t)O * 4;
}

// Workspace of a product: the operand-order copy (if the level needs one), then the partial sums of a cut reduction.
size_t spmm_workspace_bytes(int64_t O, int64_t K, int N, int M, int64_t T) {
  bool sparse_form = false;
  const size_t operand = operand_bytes(O, K, N, M, T, &sparse_form);
  const size_t partial = spmm_partial_bytes(O, K, N, M, T);
  return partial ? ((operand + 255) / 256) * 256 + partial : operand;
}

void spmm_scratch_behind_operand(SpmmArgs* a) {
  bool sparse_form = false;
  const size_t at = (operand_bytes(a->O, a->K, a->N, a->M, a->T, &sparse_form) + 255) / 256 * 256;
  if (a->workspace == nullptr || a->workspace_bytes <= at) return;
  a->scratch = static_cast<unsigned char*>(a->workspace) + at;
  a->scratch_bytes = a->workspace_bytes - at;
}

// The reduce launch of layers whose reduction was cut: split_group_append lists a layer (false: table full),
// launch_split_reduce adds their partial sums up.
static bool split_group_append(SplitGroup& sg, const GemmArgs& g) {
  if (sg.count >= kSplitLayersMax) return false;
  const int64_t quads = g.T * ((g.O + 3) / 4);
  const int64_t first = sg.count ? sg.layer[sg.count - 1].block_end : 0;
  if (first + (quads + 255) / 256 > 0x7FFFFFF0) return false;
  SplitLayer& L = sg.layer[sg.count++];
  L.partial = g.partial; L.bias = g.bias; L.Y = g.Y; L.ldy = g.ldy;
  L.T = (int32_t)g.T; L.O = (int32_t)g.O; L.splits = g.splits; L.out_bf16 = g.out_bf16;
  L.block_end = (uint32_t)(first + (quads + 255) / 256);
  L.vec = (g.O % 4 == 0) && (g.ldy % 4 == 0) && aligned_to(g.Y, g.out_bf16 ? 8 : 16);
  return true;
}
static hipError_t launch_split_reduce(SplitGroup& sg, hipStream_t s) {
  if (sg.count == 0) return hipSuccess;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3(sg.layer[sg.count - 1].block_end), dim3(256), 0, s, sg);
  sg.count = 0;
  return hipGetLastError();
}

template <bool SPARSE, int WO, int WT, int OT, int TT, int STAGES>
static hipError_t launch_gemm(GemmArgs g, hipStream_t s) {
  using C = GemmCfg<SPARSE, WO, WT, OT, TT, STAGES>;
  auto kern = nm_gemm_kernel<SPARSE, WO, WT, OT, TT, STAGES>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  g.n_o_tiles = (int)((g.O + C::BO - 1) / C::BO);
  g.n_t_tiles = (int)((g.T + C::BT - 1) / C::BT);
  const int64_t n_units = (int64_t)g.n_o_tiles * g.n_t_tiles * (g.splits > 1 ? g.splits : 1);
  const int64_t grid = ((n_units + 7) / 8) * 8;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(C::NT), C::LDS_BYTES, s, g);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (g.splits > 1) {
    SplitGroup sg;
    sg.count = 0;
    split_group_append(sg, g);
    return launch_split_reduce(sg, s);
  }
  return hipSuccess;
}

// Tiled kernel, many layers in one launch.  tile_group_append fills the table (false: full, launch it and retry;
// a layer with more blocks than a grid holds never fits and is launched alone).
template <int BO, int BT>
static int64_t tile_layer_units(const TileLayer& L) {
  const int bo = BO >> L.narrow;
  const int64_t tiles = (int64_t)((L.O + bo - 1) / bo) * ((L.T + BT - 1) / BT);
  return tiles * (L.splits > 1 ? L.splits : 1);
}
template <int BO, int BT>
static int64_t tile_layer_blocks(const TileLayer& L) { return (tile_layer_units<BO, BT>(L) + 7) / 8 * 8; }
constexpr double kTileBlockUs = 2.0;   // a block's start and write-out
constexpr double kNarrowShare = 1.5, kNarrowShareDeep = 1.25;
// estimated duration of one of the layer's blocks (the model of pick_tile): the order of the launch
static double tile_layer_cost(const TileLayer& L) {
  const int n = L.splits > 1 ? L.splits : 1;
  return (double)((L.K / 64 + n - 1) / n) * (L.sparse_form ? 0.34 : 0.5) * (L.narrow ? 0.6 : 1.0);
}

// A launch ends with its longest blocks, and a deep layer's may run far longer than the launch's even share of work.
// Where a block of 128 out-features would run 1.25 times that share, the layer takes tiles of 64 out-features: twice the
// blocks, each a little over half as long.  One image (in a graph): 4 linears at C = 768 36 -> 23 us, 12 of them 36.5 ->
// 26.9, 24 43.0 -> 32.7, 32 at C = 512 32.6 -> 25.9.  The line, with weights from memory: 48 linears at C = 768 whose deep
// dense layers run 1.28 or 1.29 shares 60.2 -> 57.9 and 60.0 -> 57.4 us, 44 (1.41) 58.5 -> 52.5, 32 (the 2:4 form at 1.33
// too) 48.6 -> 45.0; below it the activations read by twice the blocks cost more: 48 with more such layers (1.23) 61.6 and
// 62.1 narrow, 61.7 and 62.7, 40 with the 2:4 form at 1.08 narrow as well 50.9 and 53.9.
// Shallow layers, where most of a block is its start and write-out, take narrow tiles from 1.5 shares on.  792 calls of 1 to 12
// blocks at C = 128 to 768, 1 to 4 images: between 1.25 and 1.5 narrow tiles gain 2 to 8 % on average in the deep layers (K >= 1024;
// single level draws from 5 % slower to 13 % faster), 1 to 2 % in the 2:4 form from K = 256 on, nothing in the dense form of K = 256
// to 640 (0.95 to 1.05), and lose at K = 128 (40 linears of 394 tokens 9.8 us, 11.0 narrow; 44 9.9 and 11.1).
// The 2:4 form of more than 512 tokens, whose X is then read by many more blocks, keeps its tiles (8 linears at 788 tokens
// 31.0, 33.4 narrow).
template <int BO, int BT>
static void tile_group_narrow(TileGroup& grp) {
  double total = 0;
  for (int i = 0; i < grp.count; ++i)
    total += (double)tile_layer_units<BO, BT>(grp.layer[i]) * (tile_layer_cost(grp.layer[i]) + kTileBlockUs);
  const double even = total / (2.0 * kModelUnits);  // two blocks share a unit
  for (int i = 0; i < grp.count; ++i) {
    TileLayer& L = grp.layer[i];
    const double share = L.K >= (L.sparse_form ? 256u : 1024u) ? kNarrowShareDeep : kNarrowShare;
    L.narrow = L.splits <= 1 && !(L.sparse_form && L.T > 512) && tile_layer_cost(L) + kTileBlockUs > share * even;
  }
}

template <int WO, int WT, int OT, int TT>
static bool tile_group_append(TileGroup& grp, const GemmArgs& g, bool sparse_form) {
  if (grp.count >= kTileLayersMax) return false;
  TileLayer& L = grp.layer[grp.count];
  L.A = g.A; L.sel = g.sel; L.X = g.X; L.bias = g.bias; L.Y = g.Y; L.partial = g.partial;
  L.ldy = g.ldy;
  L.O = (uint32_t)g.O; L.K = (uint32_t)g.K; L.T = (uint32_t)g.T;   // tiles_ok has bounded them
  L.ldx = (uint32_t)g.ldx; L.out_bf16 = g.out_bf16; L.vec_store = g.vec_store; L.stream_form = g.stream_form;
  L.sparse_form = sparse_form; L.splits = g.splits > 1 ? g.splits : 1;
  L.block_end = 0; L.rot = 0; L.narrow = 0;
  int64_t total = tile_layer_blocks<WO * OT * 16, WT * TT * 16>(L);
  for (int i = 0; i < grp.count; ++i) total += tile_layer_blocks<WO * OT * 16, WT * TT * 16>(grp.layer[i]);
  if (total > 0x7FFFFFF0) return false;
  ++grp.count;
  return true;
}

// Not in the public header, for tests: which layers of one launch of 128 x 128 tiles take tiles of 64 out-features.
extern "C" int32_t nm_internal_narrow_layers(int32_t count, const int64_t* O, const int64_t* K, const int64_t* T,
                                             const int32_t* sparse_form, int32_t* narrow) {
  TileGroup grp;
  grp.count = 0;
  for (int i = 0; i < count; ++i) {
    GemmArgs g = {};
    g.O = O[i]; g.K = K[i]; g.T = T[i]; g.splits = 1;
    if (!tile_group_append<2, 2, 4, 4>(grp, g, sparse_form[i])) return -1;
  }
  tile_group_narrow<128, 128>(grp);
  for (int i = 0; i < count; ++i) narrow[i] = (int32_t)grp.layer[i].narrow;
  return 0;
}

template <int WO, int WT, int OT, int TT, int SS, int SD, bool NARROW>
static hipError_t launch_gemm_group(TileGroup& grp, hipStream_t s) {
  using CS = GemmCfg<true, WO, WT, OT, TT, SS>;
  using CD = GemmCfg<false, WO, WT, OT, TT, SD>;
  constexpr int LDS = CS::LDS_BYTES > CD::LDS_BYTES ? CS::LDS_BYTES : CD::LDS_BYTES;
  static_assert(!NARROW || GemmCfg<false, WO, WT, OT / 2, TT, 3>::LDS_BYTES <= LDS, "LDS of the narrow tiles");
  if (grp.count == 0) return hipSuccess;
  auto kern = nm_gemm_group_kernel<WO, WT, OT, TT, SS, SD, NARROW>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, LDS, lds_limit); e != hipSuccess) return e;
  if constexpr (NARROW) tile_group_narrow<CS::BO, CS::BT>(grp);
  // longest blocks first (insertion sort, stable), so that the launch ends with the shortest ones
  for (int i = 1; i < grp.count; ++i) {
    const TileLayer L = grp.layer[i];
    const double cost = tile_layer_cost(L);
    int j = i;
    for (; j > 0 && tile_layer_cost(grp.layer[j - 1]) < cost; --j) grp.layer[j] = grp.layer[j - 1];
    grp.layer[j] = L;
  }
  // A layer's blocks are a whole multiple of 8, one share per XCD; the last shares are short or empty.  Each layer
  // turns its shares against the XCDs so that the estimated work per XCD stays as even as the list allows.
  uint32_t end = 0;
  double load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = 0; i < grp.count; ++i) {
    TileLayer& L = grp.layer[i];
    const int64_t blocks = tile_layer_blocks<CS::BO, CS::BT>(L);
    const int64_t per_xcd = blocks / 8;
    const int64_t units = tile_layer_units<CS::BO, CS::BT>(L);
    const double cost = tile_layer_cost(L) + kTileBlockUs;
    double share[8];
    for (int sl = 0; sl < 8; ++sl) {
      int64_t u = units - sl * per_xcd;
      u = u < 0 ? 0 : (u > per_xcd ? per_xcd : u);
      share[sl] = cost * (double)u;
    }
    int best = 0;
    double best_sq = 0;  // the turn that leaves the sum of squared loads smallest
    for (int rot = 0; rot < 8; ++rot) {
      double sq = 0;
      for (int x = 0; x < 8; ++x) {
        const double v = load[x] + share[(x + rot) & 7];
        sq += v * v;
      }
      if (rot == 0 || sq < best_sq) { best = rot; best_sq = sq; }
    }
    for (int x = 0; x < 8; ++x) load[x] += share[(x + best) & 7];
    L.rot = (uint32_t)best;
    end += (uint32_t)blocks;
    L.block_end = end;
  }
  hipLaunchKernelGGL(kern, dim3(end), dim3(CS::NT), LDS, s, grp);
  grp.count = 0;
  return hipGetLastError();
}

template <bool SPARSE, bool I8>
static constexpr int stream_stages(int tt) {
  return tt == 4   ? StreamCfg<SPARSE, 4, I8>::STAGES
         : tt == 5 ? StreamCfg<SPARSE, 5, I8>::STAGES
         : tt == 6 ? StreamCfg<SPARSE, 6, I8>::STAGES
         : tt == 7 ? StreamCfg<SPARSE, 7, I8>::STAGES
                   : StreamCfg<SPARSE, 8, I8>::STAGES;
}
// int8: the per-tile constants alternate between two LDS slices, so a tile has to have as many steps as stages.
template <bool SPARSE>
static constexpr int stream_i8_min_steps() {
  int least = stream_stages<SPARSE, true>(kStreamHeights[0]);
  for (int tt : kStreamHeights)
    if (stream_stages<SPARSE, true>(tt) < least) least = stream_stages<SPARSE, true>(tt);
  return least;
}

// The tile height of a launch: the smallest estimate; 0 when no height can take it.  The tiles of several layers form
// one list, which ends in one partial round.
template <bool SPARSE, bool I8>
static int stream_height(const StreamGroup& grp) {
  const StreamModel& m = kStreamModel[I8][SPARSE];
  int best_tt = 0;
  double best = 0;
  for (int tt : kStreamHeights) {
    if (I8 && grp.layer[0].nk < stream_stages<SPARSE, I8>(tt)) continue;
    double e = 0;
    if (grp.count == 1) {
      e = stream_estimate(m, grp.layer[0].O, grp.layer[0].T, grp.layer[0].nk, tt);
    } else {
      double longest = 0;
      for (int i = 0; i < grp.count; ++i) {
        const StreamLayer& L = grp.layer[i];
        const double tile = m.tile(L.nk, tt);
        e += (double)L.n_o_tiles * (double)(((int64_t)L.T + 32 * tt - 1) / (32 * tt)) * tile / kModelUnits;
        longest = tile > longest ? tile : longest;
      }
      e = (e < longest ? longest : e) + longest / 2;
    }
    if (best_tt == 0 || e < best) { best = e; best_tt = tt; }
  }
  return best_tt;
}

template <bool SPARSE, int TT, bool I8, bool TURN = SPARSE>
static hipError_t launch_stream_kernel(StreamGroup& grp, hipStream_t s) {
  using C = StreamCfg<SPARSE, TT, I8>;
  auto kern = nm_stream_kernel<SPARSE, TT, I8, TURN>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  int cus = 0;
  if (hipError_t e = compute_units(&cus); e != hipSuccess) return e;
  const int n_cu = cus > 8 ? (cus / 8) * 8 : 8;
  int64_t tiles = 0;
  for (int i = 0; i < grp.count; ++i) {
    StreamLayer& L = grp.layer[i];
    const int64_t n = (int64_t)L.n_o_tiles * (((int64_t)L.T + C::BT - 1) / C::BT);
    L.n_tiles = (int32_t)n;
    tiles += n;
  }
  if (tiles > 0x7FFFFFF0) return hipErrorInvalidValue;
  grp.n_tiles = (int32_t)tiles;
  const int64_t want = ((tiles + 7) / 8) * 8;
  const unsigned grid = (unsigned)(want < n_cu ? want : n_cu);  // persistent blocks: one per compute unit
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::NT), C::LDS_BYTES, s, grp);
  return hipGetLastError();
}

// Whether the 2:4 form of int8 turns its rows in LDS, for which the W loads leave late (but for 256 tokens, where they leave at the
// same time).  bfloat16 gains 4 to 6 % in tiles of 128 and 3 to 5 % in those of 160, 192 and 256 tokens.  Tiles of 224 gain 2 to 3 %
// at the levels sparser than 2:4; at 2:4 (full), whose operand holds twice the weights that are not zero, long launches of them take
// up to a quarter more on two of six cards (18912 x 768 -> 3072 46.2 us, 58.9; 23640 53.4 and 59.9; 2 to 3 % less on the others).
// 32-bit rows need no turn: at 160 to 224 tokens the late loads alone cost up to 14 % on four of five cards (18912 x 1024 -> 3072 73.1
// us, 84.6; 7880 35.8 and 38.8), at 128 they gain 2 to 3 %.
static bool stream_i8_turns(int tt, int out_kind, bool full) { return out_kind == 1 ? !(tt == 7 && full) : tt == 4 || tt == 8; }

template <bool SPARSE, bool I8 = false>
static hipError_t launch_stream_group(StreamGroup& grp, hipStream_t s, bool full = false) {
  const int tt = stream_height<SPARSE, I8>(grp);
  if constexpr (SPARSE && I8)
    if (!stream_i8_turns(tt, grp.layer[0].out_kind, full)) switch (tt) {
      case 5: return launch_stream_kernel<true, 5, true, false>(grp, s);
      case 6: return launch_stream_kernel<true, 6, true, false>(grp, s);
      case 7: return launch_stream_kernel<true, 7, true, false>(grp, s);
      default: return hipErrorInvalidValue;
    }
  switch (tt) {
    case 4: return launch_stream_kernel<SPARSE, 4, I8>(grp, s);
    case 5: return launch_stream_kernel<SPARSE, 5, I8>(grp, s);
    case 6: return launch_stream_kernel<SPARSE, 6, I8>(grp, s);
    case 7: return launch_stream_kernel<SPARSE, 7, I8>(grp, s);
    case 8: return launch_stream_kernel<SPARSE, 8, I8>(grp, s);
    default: return hipErrorInvalidValue;
  }
}

// Appends a layer to the table of a launch; false when its tiles would overflow the list.
template <bool SPARSE>
static bool group_append(StreamGroup& grp, const GemmArgs& g) {
  using C = StreamCfg<SPARSE, 8>;
  const int64_t n_o = (g.O + C::BO - 1) / C::BO, n_t = (g.T + 127) / 128;  // of the lowest tiles
  const int64_t end = (int64_t)grp.n_tiles + n_o * n_t;
  if (grp.count >= kStreamLayersMax || end > 0x7FFFFFF0) return false;
  StreamLayer& L = grp.layer[grp.count++];
  L.A = g.A; L.sel = g.sel; L.X = g.X; L.bias = g.bias; L.scale = nullptr; L.Y = g.Y;
  L.O = (int32_t)g.O; L.T = (int32_t)g.T; L.nk = (int32_t)(g.K / C::KSTEP);
  L.ldx = (int32_t)g.ldx; L.ldy = (int32_t)g.ldy;
  L.n_o_tiles = (int32_t)n_o;
  L.n_tiles = (int32_t)(n_o * n_t);
  L.x_scale = 1.f; L.out_kind = g.out_bf16 ? 1 : 0; L.reserved = 0;
  grp.n_tiles = (int32_t)end;
  return true;
}

template <bool SPARSE>
static hipError_t launch_stream(const GemmArgs& g, hipStream_t s) {
  StreamGroup grp;
  grp.count = 0; grp.n_tiles = 0;
  if (!group_append<SPARSE>(grp, g)) return hipErrorInvalidValue;
  return launch_stream_group<SPARSE>(grp, s);
}

// The int8 layer on the persistent kernel.  The operands are in stream order (see nm_int8.hip's pre-pass).
bool stream_i8_takes(int64_t O, int64_t K, int64_t T, int N, int M) {
  const bool sparse_form = N <= 2 && N < M;
  const int64_t kstep = sparse_form ? 128 : 64;
  const int64_t min_steps = sparse_form ? stream_i8_min_steps<true>() : stream_i8_min_steps<false>();
  return pick_tile(O, T, K / kstep, kStreamModel[1][sparse_form], K / 128, sparse_form ? 0.5 : 1.0) == 0 && K % kstep == 0 && K / kstep >= min_steps && O <= (1 << 24) && T < (1ll << 31) && K <= (1 << 22);
}

// Not in the public header, for tests: tokens per tile and LDS stages of a launch of the persistent kernel for one layer
// of nk steps (0: no height takes it).
extern "C" int32_t nm_internal_stream_tile(int32_t int8, int32_t sparse_form, int64_t O, int64_t T, int64_t nk, int32_t* stages) {
  StreamGroup grp;
  grp.count = 1; grp.n_tiles = 0;
  StreamLayer& L = grp.layer[0];
  L.O = (int32_t)O; L.T = (int32_t)T; L.nk = (int32_t)nk; L.n_o_tiles = (int32_t)((O + 255) / 256);
  int tt = 0;
  auto ask = [&](auto sparse, auto i8) {
    tt = stream_height<decltype(sparse)::value, decltype(i8)::value>(grp);
    *stages = tt ? stream_stages<decltype(sparse)::value, decltype(i8)::value>(tt) : 0;
  };
  if (sparse_form) int8 ? ask(std::true_type{}, std::true_type{}) : ask(std::true_type{}, std::false_type{});
  else int8 ? ask(std::false_type{}, std::true_type{}) : ask(std::false_type{}, std::false_type{});
  return 32 * tt;
}

// Not in the public header, for tests: whether the 2:4 form of an int8 layer of nk steps turns its rows in LDS.
extern "C" int32_t nm_internal_stream_i8_turns(int64_t O, int64_t T, int64_t nk, int32_t out_kind, int32_t full) {
  int32_t stages;
  return stream_i8_turns(nm_internal_stream_tile(1, 1, O, T, nk, &stages) / 32, out_kind, full);
}

hipError_t launch_stream_i8(const StreamI8Args& a, hipStream_t s) {
  StreamGroup grp;
  grp.count = 1;
  StreamLayer& L = grp.layer[0];
  const int64_t kstep = a.sparse_form ? 128 : 64;
  const int64_t n_o = (a.O + 255) / 256, n_t = (a.T + 255) / 256;
  if (n_o * n_t > 0x7FFFFFF0) return hipErrorInvalidValue;
  L.A = reinterpret_cast<const bf16_t*>(a.values); L.sel = a.sel; L.X = reinterpret_cast<const bf16_t*>(a.X);
  L.bias = a.bias; L.scale = a.w_scale; L.Y = a.Y;
  L.O = (int32_t)a.O; L.T = (int32_t)a.T; L.nk = (int32_t)(a.K / kstep);
  L.ldx = (int32_t)a.ldx; L.ldy = (int32_t)a.ldy;
  L.n_o_tiles = (int32_t)n_o; L.n_tiles = (int32_t)(n_o * n_t);
  L.x_scale = a.x_scale; L.out_kind = a.out_kind; L.reserved = 0;
  grp.n_tiles = L.n_tiles;
  return a.sparse_form ? launch_stream_group<true, true>(grp, s, a.full) : launch_stream_group<false, true>(grp, s);
}

// Tiles of the tiled kernel for one layer alone.  Its blocks are bound by the bytes their compute unit pulls into LDS
// (about 100 GB/s per unit: a step of a 64 x 64 tile brings 12.5 KB for 4096 outputs, of a 128 x 128 tile 25 KB for
// 16384), so larger tiles are cheaper per output and smaller ones spread a small layer over more units: 1576 tokens x
// 768 out-features are 78 tiles of 128 x 128 and 150 of 128 x 64.  Durations (microseconds) by the same kind of model
// as the persistent kernel's, fitted on 28 shapes of 8 to 200704 tokens per form (rms 4 - 11 %); the tile it picks is
// within 4 % of the best one on average.  K = 3072 -> 768 at 1576 tokens 17.8 -> 11.9 us (128 x 128 before), K = 768 ->
// 2304 at 788 7.1 -> 5.9, in the dense form 22.1 -> 16.5 and 9.5 -> 7.0.
enum TileKind { TILE_64, TILE_128_64, TILE_128_TWO, TILE_128, TILE_KINDS };  // _TWO: two LDS stages instead of three
struct TileModel {
  int bo, bt;
  double start, step, epi, busy;
};
constexpr TileModel kTileModel[2][TILE_KINDS] = {  // [2:4 form]
    {{64, 64, 2.52, 0.154, 0.38, 0.12}, {128, 64, 2.59, 0.215, 0.65, 0.31}, {128, 128, 2.09, 0.413, 1.14, 0.13},
     {128, 128, 1.88, 0.338, 2.19, 0.26}},
    {{64, 64, 2.75, 0.099, 0.31, 0.30}, {128, 64, 2.81, 0.127, 0.40, 0.65}, {128, 128, 2.46, 0.359, 0.85, 0.06},
     {128, 128, 2.68, 0.215, 0.97, 0.45}}};
static double tile_estimate(const TileModel& m, int64_t O, int64_t K, int64_t T) {
  const double tiles = (double)((O + m.bo - 1) / m.bo) * (double)((T + m.bt - 1) / m.bt);
  const double full = (double)(int64_t)(tiles / kModelUnits), rest = tiles - full * kModelUnits;
  return m.start + ((double)(K / 64) * m.step + m.epi) *
                       (full * (1.0 + m.busy) + (rest > 0 ? 1.0 + m.busy * rest / kModelUnits : 0.0));
}
// The 128 x 128 or 64 x 64 tile of pick_tile's choice keeps the layer unless another is 2 % faster.
static TileKind tile_kind(int64_t O, int64_t K, int64_t T, bool sparse_form, int pick) {
  const int64_t tiles = ((O + 127) / 128) * ((T + 127) / 128);  // of 128 x 128
  // Tiles of 64 tokens read the weight up to twice as often as those of 128.  Of a weight past the L2s (16 MB) that is memory
  // traffic, which the model does not see: with the chip at least half full of 128 x 128 tiles, 65 tokens x 4096 -> 16384 in
  // the dense form take 28.5 us on those and 42.8 on 128 x 64, 65 x 1024 -> 16384 at 2:8 8.4 and 10.2.
  const double weight = (double)((O + 255) / 256 * 256) * (double)K * (sparse_form ? 1.125 : 2.0);
  const bool reread = pick != 3 && weight > 16e6 && tiles >= 128 && T > 64;
  int best = pick == 3 ? TILE_64 : TILE_128;
  double least = 0.98 * tile_estimate(kTileModel[sparse_form][best], O, K, T);
  for (int k = 0; k < TILE_KINDS; ++k) {
    if (reread && (k == TILE_64 || k == TILE_128_64)) continue;
    if (k == TILE_128_TWO && !sparse_form && tiles <= 256) continue;  // a block per unit: two stages leave it waiting
    if (const double e = tile_estimate(kTileModel[sparse_form][k], O, K, T); e < least) { best = k; least = e; }
  }
  return (TileKind)best;
}

// Tile and LDS stages.  pick: pick_tile's choice.  A cut reduction keeps the tile its range count was computed for.
// A fourth stage pays where a unit has one block and that block 32 steps or more: 64 x 64 8.6 -> 8.3 us (dense form
// 13.8 -> 11.6) at 394 x 3072 -> 768, 128 x 64 14.5 -> 11.9 at 1576 x 3072 -> 768, 128 x 128 23.7 -> 21.0 at 3136 x
// 4096 -> 1024; at K = 768 it costs 2 - 5 %, with two blocks on a unit it gains nothing, and neither does a fifth.
struct TileChoice {
  TileKind kind;
  int stages;
};
static TileChoice tile_choice(int64_t O, int64_t K, int64_t T, bool sparse_form, int pick, int splits) {
  const TileKind kind = splits > 1 ? (pick == 2 ? TILE_128 : TILE_64) : tile_kind(O, K, T, sparse_form, pick);
  if (kind == TILE_128_TWO) return {kind, 2};
  const TileModel& m = kTileModel[sparse_form][kind];
  const bool deep = splits <= 1 && K >= 2048 && ((O + m.bo - 1) / m.bo) * ((T + m.bt - 1) / m.bt) <= 256;
  return {kind, deep ? 4 : 3};
}

template <bool SPARSE>
static hipError_t dispatch_gemm(const GemmArgs& g, int pick, hipStream_t s) {
  if (pick == 0) return launch_stream<SPARSE>(g, s);
  const TileChoice c = tile_choice(g.O, g.K, g.T, SPARSE, pick, g.splits);
  const bool deep = c.stages == 4;
  switch (c.kind) {
    case TILE_64: return deep ? launch_gemm<SPARSE, 2, 2, 2, 2, 4>(g, s) : launch_gemm<SPARSE, 2, 2, 2, 2, 3>(g, s);
    case TILE_128_64: return deep ? launch_gemm<SPARSE, 2, 2, 4, 2, 4>(g, s) : launch_gemm<SPARSE, 2, 2, 4, 2, 3>(g, s);
    case TILE_128_TWO: return launch_gemm<SPARSE, 2, 2, 4, 4, 2>(g, s);
    default: return deep ? launch_gemm<SPARSE, 2, 2, 4, 4, 4>(g, s) : launch_gemm<SPARSE, 2, 2, 4, 4, 3>(g, s);
  }
}

// Tiles of the ragged form where X travels through registers: 64 x 64, or, from 150 of them on, 128 x 128 where those are estimated
// faster.  The blocks of a unit's list run `at_once` of them together; `share` is what the units' number of blocks adds beyond whole
// lists.  `pieces`: rows of Y in whole aligned 16-byte pieces; without, a large tile's write-out is most of a short reduction.  Fitted on
// 24800 shapes (60 to 40000 tokens, 72 .. 4096 deep and wide; rms 5 and 6 %); the choice takes 1.0015 of the better tile's time on
// average, 1.1 % of the shapes lose more than 5 %.  (Two thresholds on the tiles, 208 and 336, took 1.042.)  64 and 128, us: 7410 x 84 ->
// 1317 at 2:4 in bfloat16 13.5 and 17.8, 18048 x 476 -> 159 at 3:4 in float32 12.1 and 17.2; 33413 x 140 -> 1896 at 2:4 in bfloat16 51.5
// and 41.5, 9906 x 1932 -> 648 at 1:4 41.6 and 31.8, 35674 x 84 -> 2697 at 2:4 in float32 122 and 94.
struct RaggedModel {
  double start, step, busy, share;
  double byte[2];    // a MB of output: [pieces]
  double epi[2][2];  // [bfloat16][pieces]
  int at_once;
};
constexpr RaggedModel kRaggedModel[2][2] = {  // [2:4 form][128 x 128]
    {{4.20, 0.284, 0.643, 0, {0.047, 0.082}, {{0.449, 0.160}, {0.576, 0.115}}, 4},
     {4.78, 0.620, 0.549, 0.101, {0.075, 0.135}, {{1.792, 0.264}, {3.139, 0.109}}, 2}},
    {{4.23, 0.244, 0.536, 0, {0.051, 0.046}, {{0.535, 0.422}, {0.715, 0.297}}, 4},
     {4.37, 0.470, 0.499, 0.077, {0.054, 0.094}, {{2.177, 0.912}, {3.492, 0.528}}, 2}}};
static double ragged_estimate(bool sparse_form, bool large, int64_t O, int64_t K, int64_t T, bool out_bf16, bool pieces) {
  const RaggedModel& m = kRaggedModel[sparse_form][large];
  const int64_t side = large ? 128 : 64, tiles = ((O + side - 1) / side) * ((T + side - 1) / side);
  const int64_t list = ((tiles + 7) / 8 + 31) / 32, rest = list % m.at_once;  // blocks of a unit; of those, past the last full set
  const double steps = (double)((K + 63) / 64);
  return m.start + (steps * m.step + m.epi[out_bf16][pieces]) * ((double)(list / m.at_once) * (1.0 + m.busy * (m.at_once - 1)) +
                                                                 (rest ? 1.0 + m.busy * (double)(rest - 1) : 0.0)) +
         m.byte[pieces] * 1e-6 * (double)O * (double)T * (out_bf16 ? 2.0 : 4.0) + m.share * steps * (double)tiles / kModelUnits;
}
static int ragged_tile(bool sparse_form, int64_t O, int64_t K, int64_t T, bool out_bf16, bool pieces) {
  if (((O + 127) / 128) * ((T + 127) / 128) < 150) return 64;
  auto estimate = [&](bool large) { return ragged_estimate(sparse_form, large, O, K, T, out_bf16, pieces); };
  return estimate(true) < estimate(false) ? 128 : 64;
}
// Not in the public header, for tests.
extern "C" int32_t nm_internal_ragged_tile(int32_t sparse_form, int64_t O, int64_t K, int64_t T, int32_t out_bf16, int32_t pieces) {
  return ragged_tile(sparse_form != 0, O, K, T, out_bf16 != 0, pieces != 0);
}

// The ragged form of the tiled kernel.  K and the rows of X in whole 16-byte pieces: the
// tile of the aligned form.  A product of 1579 x 1000 -> 1001 at 2:8 takes 8.0 us that way and 11.0 through registers.
// Other rows: ragged_tile's choice.  (The gather kernel, which still takes such shapes when there is no workspace: 1096 us.)
template <bool SPARSE>
static hipError_t launch_ragged(GemmArgs g, hipStream_t s) {
  auto go = [&](auto kern, auto cfg, PerDeviceOnce& once) {
    using C = decltype(cfg);
    if (hipError_t e = raise_dynamic_lds_limit(kern, C::LDS_BYTES, once); e != hipSuccess) return e;
    g.n_o_tiles = (int)((g.O + C::BO - 1) / C::BO);
    g.n_t_tiles = (int)((g.T + C::BT - 1) / C::BT);
    const int64_t grid = (((int64_t)g.n_o_tiles * g.n_t_tiles + 7) / 8) * 8;
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(C::NT), C::LDS_BYTES, s, g);
    return hipGetLastError();
  };
  const int64_t tiles_mid = ((g.O + 127) / 128) * ((g.T + 127) / 128);
  static PerDeviceOnce once[7];
  if (g.x_aligned && g.K % 8 == 0 && g.ldx <= (1 << 22)) {  // (per-lane byte offsets inside a tile stay below 2^32)
    switch (tile_kind(g.O, padded_k(g.K), g.T, SPARSE, tiles_mid < 64 ? 3 : 2)) {
      case TILE_64: return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 2, 2, 3, 0>, GemmCfg<SPARSE, 2, 2, 2, 2, 3>{}, once[0]);
      case TILE_128_64: return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 4, 2, 3, 0>, GemmCfg<SPARSE, 2, 2, 4, 2, 3>{}, once[1]);
      case TILE_128_TWO: return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 4, 4, 2, 0>, GemmCfg<SPARSE, 2, 2, 4, 4, 2>{}, once[2]);
      default: return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 4, 4, 3, 0>, GemmCfg<SPARSE, 2, 2, 4, 4, 3>{}, once[3]);
    }
  }
  if (ragged_tile(SPARSE, g.O, g.K, g.T, g.out_bf16 != 0, g.vec_store != 0) == 128)
    return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 4, 4, 2, 2>, GemmCfg<SPARSE, 2, 2, 4, 4, 2>{}, once[4]);
  if constexpr (!SPARSE)
    if (tiles_mid < 64 && g.K >= 1280) return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 2, 2, 2, 4>, GemmCfg<SPARSE, 2, 2, 2, 2, 2>{}, once[6]);
  return go(nm_gemm_ragged_kernel<SPARSE, 2, 2, 2, 2, 2, 2>, GemmCfg<SPARSE, 2, 2, 2, 2, 2>{}, once[5]);
}

static hipError_t launch_general(const SpmmArgs& a, hipStream_t s) {
  const int64_t n_o_tiles = (a.O + 15) / 16, n_t_tiles = (a.T + 15) / 16;
  if (n_o_tiles * n_t_tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(spmm_general_kernel, dim3((unsigned)(n_o_tiles * n_t_tiles)), dim3(256), 0, s, a.values, a.indices,
                     a.O, a.K, a.N, a.M, a.X, a.T, a.ldx, a.bias, a.Y, a.ldy, a.out_bf16, n_o_tiles);
  return hipGetLastError();
}

// Out[t, i] = sum_r Q[t, r] * Ws[r, i] on the persistent dense kernel: the weight is written transposed into
// stream order first (a pass over the weight only), then it is an ordinary product with I out-features and a
// reduction of R.  Shapes: enough tiles, R % 64 == 0, Out rows in whole aligned 16-byte pieces.
// The alternative, nm_grad.hip's kernel, reads the weight as it lies, so the pass over the weight counts: 2.5 us and a
// quarter of one per MB, about half of that beside a short reduction, whose tiles the estimates make 30 % too cheap at
// R = 64.  Over 8200 shapes (256 to 200704 tokens, buffers from memory) the choice is 1.8 % from the better of the two on
// average, 4.2 % without the pass in it: 5388 tokens x 64 -> 904 7.1 and 11.8 us, 12608 x 64 -> 768 9.2 and 12.2.
static bool dense_transposed_takes(int64_t R, int64_t I, int64_t T) {
  if (R % 64 || ((I + 127) / 128) * ((T + 127) / 128) < 64 || T < 256) return false;
  const double weight_mb = (double)((I + 255) / 256 * 256) * (double)R * 2e-6;
  const double pass = R > 192 ? 2.5 + 0.25 * weight_mb : 1.3;
  return stream_estimate(kStreamModel[0][0], I, T, R / 32) + pass <= tiled_estimate(I, T, R / 64, 0.5) * (R == 64 ? 0.7 : 1.0);
}

// What the persistent kernel does not take, few tokens above all, the tiled kernel multiplies from the same copy where the two are
// estimated faster (by a fifth where the result is four times as wide as the reduction is long) than nm_grad.hip's kernel, whose
// tiles of 128 x 256 are a handful of blocks then, each with the whole reduction in a row, 0.32 us per 32 positions.  Tokens x
// reduction -> width, float32: 197 x 3072 -> 768 37.1 -> 17.2 us, x 768 -> 768 13.5 -> 8.6, 1576 x 4096 -> 1024 52.4 -> 27.3; 394 x 768 ->
// 3072, 14.1 us, would take 15.2.  The sums are the same bits.  The copy is optional: without the workspace for it the
// call runs as it did.  The constants are fitted on 865 shapes of 1 to 20000 tokens, 64 .. 4096 wide and deep, float32 (rms 5 % for the one
// kernel, 10 % for the two); of 10400 other shapes that this chose the two launches take 0.55 of the one kernel's time on average (0.57
// in bfloat16).
static bool dense_transposed_tiles(int64_t R, int64_t I, int64_t T) {
  if (R % 64 || R > (1 << 22) || I > (1 << 24) || T >= (1ll << 31) || dense_transposed_takes(R, I, T)) return false;
  const double weight_mb = (double)((I + 255) / 256 * 256) * (double)R * 2e-6;
  double tiles = 1e30;
  for (const TileModel& m : kTileModel[0])
    if (const double e = tile_estimate(m, I, R, T); e < tiles) tiles = e;
  constexpr TileModel kGrad = {256, 128, 2.92, 0.638, 1.56, 0.81};  // (a step of 64; its 256-wide side runs along the tokens)
  return tiles + 2.74 + 0.615 * weight_mb < (I >= 4 * R ? 0.8 : 0.95) * tile_estimate(kGrad, T, R, I);
}

// Of these, with the output type known: what the one kernel writes in bfloat16 takes it up to a sixth less, and many tokens cost the two
// launches their way through memory as well, which the estimates above do not see.  Fitted on 10400 shapes that they chose (rms 3 and
// 2 % for the one kernel, 8 % for the two).  On the estimates above alone 62 (float32) and 98 (bfloat16) of them lost more than 3 % against
// the one kernel, up to 25; now 8 and 25.  One kernel and two launches, us: 1576 x 768 -> 2048 in bfloat16 13.9 and 15.7, 7205 x 576
// -> 1600 20.6 and 25.1, 13056 x 1792 -> 640 in float32 33.4 and 41.8; 1576 x 4096 -> 1024 in bfloat16 51.4 and 26.7.
bool dense_transposed_pays(int64_t R, int64_t I, int64_t T, int out_bf16) {
  const double weight_mb = (double)((I + 255) / 256 * 256) * (double)R * 2e-6;
  double tiles = 1e30;
  for (const TileModel& m : kTileModel[0])
    if (const double e = tile_estimate(m, I, R, T); e < tiles) tiles = e;
  const double two = 3.62 + 0.487 * weight_mb + 0.89 * tiles + 0.047e-6 * (double)T * (double)R +
                     (out_bf16 ? 0.855e-6 : 1.585e-6) * (double)T * (double)I;
  constexpr TileModel kGrad[2] = {{256, 128, 5.34, 0.656, 0, 0.276}, {256, 128, 4.65, 0.654, 0, 0.316}};  // [bfloat16]
  return two < tile_estimate(kGrad[out_bf16], T, R, I) + (out_bf16 ? 0.388e-6 : 1.13e-6) * (double)T * (double)I;
}
// *required: the layer is the persistent kernel's, and a call without the workspace is refused.
size_t dense_transposed_workspace_bytes(int64_t R, int64_t I, int64_t T, bool* required) {
  *required = dense_transposed_takes(R, I, T);
  if (!*required && !dense_transposed_tiles(R, I, T)) return 0;
  return (size_t)(((I + 255) / 256) * 256) * (size_t)R * 2;
}

hipError_t launch_dense_transposed(const bf16_t* Ws, int64_t R, int64_t I, int64_t ldw, const bf16_t* Q, int64_t T,
                                   int64_t ldq, void* Out, int64_t ldo, int out_bf16, void* workspace,
                                   size_t workspace_bytes, hipStream_t s, bool* taken) {
  *taken = false;
  bool persistent = false;
  const size_t need = dense_transposed_workspace_bytes(R, I, T, &persistent);
  const int per_piece = out_bf16 ? 8 : 4;
  if (!need || workspace == nullptr || workspace_bytes < need || !aligned_to(workspace, 256)) return hipSuccess;
  if (!aligned_to(Q, 16) || (ldq % 8) || !aligned_to(Ws, 2) || (ldo % per_piece) || !aligned_to(Out, 16) || (I % per_piece))
    return hipSuccess;
  if (I > (1 << 24) || T >= (1ll << 31) || ldq > (1 << 22) || R > (1 << 22) || ldo > 0x7FFFFFFF) return hipSuccess;
  const int64_t i_pad = ((I + 255) / 256) * 256;
  const int64_t n_i = i_pad / 64, blocks = n_i * (R / 64);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  auto turn = aligned_to(Ws, 16) && ldw % 8 == 0 ? transpose_stream_kernel<true> : transpose_stream_kernel<false>;
  hipLaunchKernelGGL(turn, dim3((unsigned)blocks), dim3(256), 0, s, Ws, R, I, ldw, (int)n_i, reinterpret_cast<unsigned char*>(workspace));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  GemmArgs g;
  g.A = reinterpret_cast<const bf16_t*>(workspace); g.sel = nullptr;
  g.X = Q; g.bias = nullptr; g.Y = Out;
  g.O = I; g.K = R; g.T = T; g.ldx = ldq; g.ldy = ldo;
  g.n_o_tiles = g.n_t_tiles = 0;
  g.out_bf16 = (uint8_t)out_bf16; g.vec_store = 1; g.stream_form = 1; g.splits = 1; g.partial = nullptr;
  *taken = true;
  return dispatch_gemm<false>(g, persistent ? 0 : ((I + 127) / 128) * ((T + 127) / 128) < 64 ? 3 : 2, s);
}

#define NM_FOR_EACH_LEVEL(X)                                                                         \
  X(1, 4) X(2, 4) X(3, 4) X(4, 4)                                                                    \
  X(1, 8) X(2, 8) X(3, 8) X(4, 8) X(5, 8) X(6, 8) X(7, 8) X(8, 8)                                    \
  X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(6, 16) X(7, 16) X(8, 16) X(9, 16) X(10, 16)         \
  X(11, 16) X(12, 16) X(13, 16) X(14, 16) X(15, 16) X(16, 16)

// The stream-order pre-pass of a layer into its workspace.
static hipError_t launch_stream_prepass(const SpmmArgs& a, bool sparse_form, hipStream_t s) {
  unsigned char* ws = reinterpret_cast<unsigned char*>(a.workspace);
  const int64_t o_pad = ((a.O + 255) / 256) * 256, k_pad = padded_k(a.K);
  unsigned char* sel_s = sparse_form ? ws + (size_t)o_pad * (size_t)k_pad : nullptr;
  const dim3 grid = flat_grid_256(o_pad * (k_pad / 16));
  const int wide = (a.K % 16 == 0) && aligned_to(a.values, 16);  // every 16-weight chunk is whole and its values aligned
  switch (a.N * 32 + a.M) {
#define X(n_, m_)                                                                                                  \
  case n_ * 32 + m_:                                                                                               \
    hipLaunchKernelGGL((operand_stream_kernel<n_, m_>), grid, dim3(256), 0, s, a.values, a.indices, a.O, o_pad, a.K, \
                       k_pad, wide, ws, sel_s);                                                                    \
    break;
    NM_FOR_EACH_LEVEL(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Operands of the matrix-core kernels for a layer whose form is known.
static void fill_gemm_args(const SpmmArgs& a, int form, bool sparse_form, GemmArgs* g) {
  g->X = a.X; g->bias = a.bias; g->Y = a.Y;
  g->O = a.O; g->K = a.K; g->T = a.T; g->ldx = a.ldx; g->ldy = a.ldy;
  g->N = (uint8_t)a.N; g->M = (uint8_t)a.M; g->values = a.values; g->indices = a.indices;
  g->out_bf16 = a.out_bf16;
  g->n_o_tiles = g->n_t_tiles = 0;
  g->rot = 0;
  g->x_aligned = aligned_to(a.X, 16) && a.ldx % 8 == 0;
  // 16-byte pieces of Y rows: every row start and the row end fall on a piece boundary
  const int per_piece = a.out_bf16 ? 8 : 4;
  g->vec_store = (a.ldy % per_piece == 0) && aligned_to(a.Y, 16) && (a.O % per_piece == 0) &&
                 (a.bias == nullptr || aligned_to(a.bias, 16));
  g->stream_form = form == FORM_STREAM;
  {
    int splits = split_count(a.O, a.K, a.T, sparse_form);
    if (splits > 1 && (a.scratch == nullptr || !aligned_to(a.scratch, 256) ||
                       a.scratch_bytes < (size_t)splits * (size_t)a.T * (size_t)a.O * 4))
      splits = 1;
    g->splits = (uint8_t)splits;
    g->partial = splits > 1 ? static_cast<float*>(a.scratch) : nullptr;
  }
  if (form == FORM_STREAM) {
    const int64_t o_pad = ((a.O + 255) / 256) * 256;
    unsigned char* ws = reinterpret_cast<unsigned char*>(a.workspace);
    g->A = reinterpret_cast<const bf16_t*>(ws);
    g->sel = sparse_form ? reinterpret_cast<const uint32_t*>(ws + (size_t)o_pad * (size_t)padded_k(a.K)) : nullptr;
  } else {
    g->A = a.values;  // 2:4: values + index words are the row-major 2:4 operand; N = M: the dense weight
    g->sel = sparse_form ? a.indices : nullptr;
  }
}

// The persistent kernel writes Y in 16-byte pieces only; other outputs of layers of its size take the ragged form of the
// tiled kernel, whichever of the two the estimates name (the ragged form does not multiply an activation at a pruned
// position that is not finite, and that must not hang on an estimate).
static bool unaligned_output(const SpmmArgs& a, const GemmArgs& g, int pick) {
  if (pick == 0) return !g.vec_store || a.ldy > 0x7FFFFFFF;
  return g.stream_form && !g.vec_store && a.O > 128 && ((a.O + 127) / 128) * ((a.T + 127) / 128) > 256;
}

// A layer whose operand-order workspace is missing (or too small) and which the few-token kernel can multiply
// from the packed format instead.
static bool packed_path(const SpmmArgs& a) {
  if (!tiles_ok(a.K, a.X, a.ldx, a.values, a.indices, a.O, a.T)) return false;
  const size_t need = spmm_operand_workspace_bytes(a.O, a.K, a.N, a.M, a.T);
  if (!need || (a.workspace != nullptr && a.workspace_bytes >= need && aligned_to(a.workspace, 256))) return false;
  return fewtok_takes(a);
}

// A call that prepares and multiplies in one takes the kernel that decodes the weight itself (nm_direct.hip) where its
// estimate is below the pre-pass and the tiled kernel together.  It decodes the weight once per 64 tokens, so it wins as
// long as its blocks of 32 out-features x 64 tokens are few rounds on the chip, later for a shallow weight.  Both estimates were fitted on
// 3000 shapes per form (64 .. 16384 deep, 64 .. 49152 wide, 1 .. 1000 tokens, in a graph) when the loads of blocks of 64 tokens still
// carried conditions, and they know neither the smaller blocks of up to 32 tokens (launch_level there) nor the faster loads.  They still
// choose well between the two: over 47300 shapes (1 .. 50000 tokens, 64 .. 8192 deep, 64 .. 24576 wide, both output types) the choice takes
// 1.003 of the better one's time on average, 1.9 % of the shapes lose more than 5 %.  Pre-pass and product against it: 768 -> 1000 at
// 4:8 and 8 tokens 8.1 and 3.7 us, 768 -> 768 at 394 tokens 9.0 and 5.8, 1024 -> 4096 at 197 tokens 17.4 and 9.6.
// Its sums are those of the tiled kernel; a layer that the persistent kernel or a cut reduction would sum in another
// order stays there.
constexpr TileModel kDirectModel[2] = {{32, 64, 3.81, 0.130, 0.57, 1.09}, {32, 64, 3.22, 0.117, 0.85, 0.68}};  // [2:4 form]
// Its second form, blocks of 64 out-features x 128 tokens, takes what is beyond the first one's few rounds and still not worth the two
// launches: spans of 128 reduction positions, and of a block's span and its write-out the parts that grow with the kept
// values of 16 weights and with the bytes of an output.  Fitted on 3200 shapes (40 .. 8000 tokens, 64 .. 4096 deep and wide, whole and
// ragged, in a graph) with an rms of 8 %, but for the smallest, which take 4.5 us where the model has 3.7.  It has to be a fifth
// faster than the first form, whose estimate is the rougher one.  Where it is chosen it takes 0.73 of the better other route's time on
// average (8400 of 60500 shapes as above), 0.5 % of them lose more than 5 %: 551 x 256 -> 129 at 4:8 stays with the first form
// (3.6 us, 5.7), 788 x 768 -> 2304 at 1:8 6.9 and 10.8 in two launches, 1576 x 3072 -> 768 at 2:8 17.4 in two and 22.8.
// It is not asked up to 64 tokens, where half its block would be empty, nor for reductions of 3072 and more, which it was not fitted on;
// both leave something: 42 x 2232 -> 16032 at 4:8 takes 41 us in two launches and would take 22, 204 x 3968 -> 7488 at 4:16 52 and 29.
// Of all 60500 shapes 10 % are more than 5 % from their best route, 1.02 of its time on average.
struct WideModel {
  double start, span, kept, epi, byte, busy;
};
constexpr WideModel kWideModel[2] = {{1.30, 0.650, 0.029, 1.24, 0.12, 0.29}, {1.55, 0.572, 0.016, 1.18, 0.092, 0.37}};  // [2:4 form]
static double wide_estimate(int64_t O, int64_t K, int N, int M, int64_t T, bool out_bf16) {
  const WideModel& m = kWideModel[N <= 2];
  const double tiles = (double)((O + 63) / 64) * (double)((T + 127) / 128);
  const double full = (double)(int64_t)(tiles / kModelUnits), rest = tiles - full * kModelUnits;
  const double block = (double)((K + 127) / 128) * (m.span + m.kept * (double)(16 / M * N)) + m.epi + m.byte * (out_bf16 ? 2.0 : 4.0);
  const double e = m.start + block * (full * (1.0 + m.busy) + (rest > 0 ? 1.0 + m.busy * rest / kModelUnits : 0.0));
  return e < 4.5 ? 4.5 : e;
}

// Many tokens on most of the units, where every unit waits for memory and not for its own chain, are outside of what the estimate
// was fitted on: of 755 shapes of 1500 to 50000 tokens the two launches won at 4490 x 1216 -> 440 at 1:8 (252 blocks; 13.3 us, 16.2 in one),
// 8969 x 1096 -> 156 (213; 12.9 and 14.4), 8830 x 416 -> 392 (483; 12.4 and 16.1), 9911 x 80 -> 436 (546; 12.4 and 14.9), the one launch at
// 1579 x 1000 -> 1001 (208; 13.5 and 11.6), 5222 x 448 -> 312 (205; 8.9 and 7.1), 4003 x 104 -> 832 (416; 9.0 and 7.8).
static bool wide_in_range(int64_t O, int64_t K, int64_t T) {
  const int64_t tiles = ((O + 63) / 64) * ((T + 127) / 128), spans = (K + 127) / 128;
  return tiles <= 192 || T <= 2560 || (tiles <= 256 && spans <= 5) || (tiles <= 512 && spans == 1 && T <= 8192);
}

enum DirectForm { DIRECT_NONE, DIRECT_FIRST, DIRECT_WIDE };
static DirectForm direct_form(int64_t O, int64_t K, int N, int M, int64_t T, bool out_bf16, int pick) {
  const bool sparse_form = N <= 2;
  const int64_t steps_k = padded_k(K);
  if (pick == 0 || !direct_level(N, M) || split_count(O, steps_k, T, sparse_form) != 1) return DIRECT_NONE;
  const int64_t blocks = ((O + 31) / 32) * ((T + 63) / 64);
  if ((T + 63) / 64 > 65535 || blocks > (1 << 20)) return DIRECT_NONE;  // (a grid's second dimension)
  double two = 1e30;
  for (const TileModel& m : kTileModel[sparse_form])
    if (const double e = tile_estimate(m, O, steps_k, T); e < two) two = e;
  two += 3.85 + (sparse_form ? 0.49 : 0.85) * 1e-6 * (double)((O + 255) / 256 * 256) * (double)steps_k;
  const double first = K % 16 == 0 ? tile_estimate(kDirectModel[sparse_form], O, steps_k, T) : 1e30;
  // (a reduction of one span of the first form, on one round of its blocks, is 0.80 - 0.92 of the two spans' time in the second:
  // 507 x 208 -> 893 at 4:16 4.4 us and 6.2)
  const bool one_span = K <= 256 && K % 16 == 0 && blocks <= (int64_t)kModelUnits;
  if (T > 64 && K < 3072 && !one_span && wide_in_range(O, K, T))
    if (const double e = wide_estimate(O, K, N, M, T, out_bf16); e < 0.8 * first && e < two) return DIRECT_WIDE;
  return first < two ? DIRECT_FIRST : DIRECT_NONE;
}

// A ragged reduction is decoded likewise, of whole 16-weight chunks (210 x 144 -> 332 at 1:16 8.5 us in two launches, 4.4 here) or of
// eight more, which the second form takes.
static DirectForm direct_form_ragged(int64_t O, int64_t K, int N, int M, int64_t T, bool out_bf16) {
  return K % 8 == 0 ? direct_form(O, K, N, M, T, out_bf16, 2) : DIRECT_NONE;
}

// A call without a workspace takes it up to four rounds of blocks, and at one block of tokens in any case; beyond, it would
// decode a wide weight two to four times, and the kernel of nm_fewtok.hip, with the same sums, is the faster one (12288 ->
// 49152 at 1:8 and 208 tokens 370 us, 1080 that way; 2048 -> 16384 at 130 tokens 38.7 and 53.3; 768 -> 1000 at 4:8 and 16
// tokens 23.0 and 5.4).
static bool direct_takes_packed(int64_t O, int64_t T) { return T <= 64 || ((O + 31) / 32) * ((T + 63) / 64) <= 1024; }

hipError_t launch_spmm(const SpmmArgs& a, hipStream_t s, bool* workspace_short, int phases) {
  *workspace_short = false;
  const bool prepare = phases & SPMM_PREPARE, product = phases & SPMM_PRODUCT;
  bool sparse_form = false;
  const int form = operand_form(a.O, a.K, a.T, a.N, a.M, &sparse_form);
  // The ragged form of the tiled kernel: stream order in the workspace, any X and Y.  For K % 64 == 0 (an X that the
  // other kernels cannot take) the weight has to be one that the prepare call, which does not see X, has written.
  auto ragged_product = [&]() {
    GemmArgs g;
    fill_gemm_args(a, form, sparse_form, &g);
    g.splits = 1; g.partial = nullptr;
    return sparse_form ? launch_ragged<true>(g, s) : launch_ragged<false>(g, s);
  };
  const bool copy_fits = form == FORM_STREAM && a.workspace != nullptr && aligned_to(a.workspace, 256) &&
                         a.workspace_bytes >= operand_bytes(a.O, a.K, a.N, a.M, a.T, &sparse_form);
  if (!tiles_ok(a.K, a.X, a.ldx, a.values, a.indices, a.O, a.T)) {
    // without the workspace the gather kernel reads the packed layout itself
    const bool ragged = copy_fits && (a.K % 64 != 0 || tiles_ok(a.K, nullptr, a.K, a.values, a.indices, a.O, a.T));
    if (ragged && prepare && product && a.K % 64 != 0 && aligned_to(a.X, 16) && a.ldx % 8 == 0 && aligned_to(a.values, 16))
      if (const DirectForm f = direct_form_ragged(a.O, a.K, a.N, a.M, a.T, a.out_bf16);
          f == DIRECT_FIRST || (f == DIRECT_WIDE && a.ldx <= (1 << 22)))
        return launch_direct(a, false, f == DIRECT_WIDE, true, s);
    if (ragged && prepare) {
      hipError_t e = launch_stream_prepass(a, sparse_form, s);
      if (e != hipSuccess) return e;
    }
    if (!product) return hipSuccess;
    return ragged ? ragged_product() : launch_general(a, s);
  }
  const size_t need = spmm_operand_workspace_bytes(a.O, a.K, a.N, a.M, a.T);
  if (need && (a.workspace == nullptr || a.workspace_bytes < need || !aligned_to(a.workspace, 256))) {
    // no workspace: few tokens can still be multiplied straight from the packed format
    if (!packed_path(a)) {
      *workspace_short = true;
    } else if (product) {
      if (direct_takes_packed(a.O, a.T)) return launch_direct(a, true, false, false, s);
      const SpmmArgs* one = &a;
      return launch_fewtok(&one, 1, s);
    }
    return hipSuccess;
  }
  const int pick = pick_tile(a.O, a.K, a.T, sparse_form);
  GemmArgs g;
  fill_gemm_args(a, form, sparse_form, &g);
  const bool unaligned = unaligned_output(a, g, pick);
  if (prepare && product)
    if (const DirectForm f = direct_form(a.O, a.K, a.N, a.M, a.T, a.out_bf16, pick); f != DIRECT_NONE)
      return launch_direct(a, false, f == DIRECT_WIDE, unaligned, s);
  if (prepare && form == FORM_STREAM) {
    hipError_t e = launch_stream_prepass(a, sparse_form, s);
    if (e != hipSuccess) return e;
  }
  if (!product) return hipSuccess;
  if (unaligned) return ragged_product();
  return sparse_form ? dispatch_gemm<true>(g, pick, s) : dispatch_gemm<false>(g, pick, s);
}

// Not in the public header, for tests: the kernel that a product of aligned operands takes at one layer's shape and, for
// the tiled and the persistent one and the second form of the one that decodes itself (bfloat16 output), its tile
// (out-features, tokens, LDS stages).
// call: 0 the weight is prepared in the same call, 1 it has been, 2 there is no workspace.
extern "C" int32_t nm_internal_product_route(int32_t call, int64_t O, int64_t K, int32_t N, int32_t M, int64_t T, int32_t* tile) {
  enum { ROUTE_GENERAL, ROUTE_TILED, ROUTE_PERSISTENT, ROUTE_RAGGED, ROUTE_DIRECT, ROUTE_FEWTOK };
  const bool sparse_form = N <= 2 && N < M;
  auto direct = [&](DirectForm f) {
    if (f == DIRECT_WIDE) { tile[0] = 64; tile[1] = 128; tile[2] = 2; }
    return f != DIRECT_NONE;
  };
  if (K % 64) {
    if (call == 2 || !ragged_shape(O, K, T)) return ROUTE_GENERAL;
    return call == 0 && direct(direct_form_ragged(O, K, N, M, T, true)) ? ROUTE_DIRECT : ROUTE_RAGGED;
  }
  const int pick = pick_tile(O, K, T, sparse_form);
  if (call == 2 && spmm_operand_workspace_bytes(O, K, N, M, T) != 0)
    return !fewtok_shape(O, K, N, M, T) ? -1 : direct_takes_packed(O, T) ? ROUTE_DIRECT : ROUTE_FEWTOK;
  if (call == 0 && direct(direct_form(O, K, N, M, T, true, pick))) return ROUTE_DIRECT;
  if (pick == 0) {
    tile[0] = 256;
    tile[1] = nm_internal_stream_tile(0, sparse_form, O, T, sparse_form ? K / 64 : K / 32, &tile[2]);
    return ROUTE_PERSISTENT;
  }
  const TileChoice c = tile_choice(O, K, T, sparse_form, pick, split_count(O, K, T, sparse_form));
  tile[0] = kTileModel[sparse_form][c.kind].bo;
  tile[1] = kTileModel[sparse_form][c.kind].bt;
  tile[2] = c.stages;
  return ROUTE_TILED;
}

// nm_linear_forward on a scratch of a given size.  The operand copy of a ragged reduction may be larger than that: the
// layer is then prepared and multiplied a run of out-features at a time, as many 256-row tiles as fit.  An output's
// sum does not depend on the tiles around it, so the bytes are those of the whole layer in one workspace.
hipError_t launch_spmm_on_scratch(const SpmmArgs& a, hipStream_t s, bool* workspace_short) {
  bool sparse_form = false;
  const size_t tile_bytes = ragged_shape(a.O, a.K, a.T) ? operand_bytes(256, a.K, a.N, a.M, a.T, &sparse_form) : 0;
  const int64_t rows = tile_bytes ? (int64_t)(a.workspace_bytes / tile_bytes) * 256 : 0;
  if (rows == 0) return launch_spmm(a, s, workspace_short, SPMM_PREPARE | SPMM_PRODUCT);
  const int64_t nf = values_per_row(a.K, a.N, a.M), nw = index_words_per_row(a.K, a.N, a.M);
  for (int64_t o = 0; o < a.O; o += rows) {
    SpmmArgs part = a;
    part.values += o * nf;
    part.indices += o * nw;
    if (part.bias) part.bias += o;
    part.Y = static_cast<unsigned char*>(a.Y) + o * (a.out_bf16 ? 2 : 4);
    part.O = a.O - o < rows ? a.O - o : rows;
    if (hipError_t e = launch_spmm(part, s, workspace_short, SPMM_PREPARE | SPMM_PRODUCT); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The product of a prepared layer on the tiled kernel, as a table entry (the operands launch_spmm would hand the
// kernel): false when the layer takes another path.
static bool tiled_entry(const SpmmArgs& a, GemmArgs* g, bool* sparse_form, int* pick) {
  if (packed_path(a)) return false;
  if (!tiles_ok(a.K, a.X, a.ldx, a.values, a.indices, a.O, a.T)) return false;
  const int form = operand_form(a.O, a.K, a.T, a.N, a.M, sparse_form);
  *pick = pick_tile(a.O, a.K, a.T, *sparse_form);
  if (*pick == 0) return false;
  fill_gemm_args(a, form, *sparse_form, g);
  return !unaligned_output(a, *g, *pick);
}

// The product of a prepared layer on the persistent kernel, as a table entry: false when this layer takes
// another path (too few tiles, a shape or alignment the kernel does not handle).
static bool stream_entry(const SpmmArgs& a, GemmArgs* g, bool* sparse_form) {
  if (packed_path(a)) return false;
  if (!tiles_ok(a.K, a.X, a.ldx, a.values, a.indices, a.O, a.T)) return false;
  const int form = operand_form(a.O, a.K, a.T, a.N, a.M, sparse_form);
  if (pick_tile(a.O, a.K, a.T, *sparse_form) != 0) return false;
  fill_gemm_args(a, form, *sparse_form, g);
  if (!g->vec_store || a.ldy > 0x7FFFFFFF) return false;
  return true;
}

bool spmm_workspace_short(const SpmmArgs& a) {
  if (packed_path(a)) return false;
  if (!tiles_ok(a.K, a.X, a.ldx, a.values, a.indices, a.O, a.T)) return false;  // the gather kernel needs none
  const size_t need = spmm_operand_workspace_bytes(a.O, a.K, a.N, a.M, a.T);
  return need && (a.workspace == nullptr || a.workspace_bytes < need || !aligned_to(a.workspace, 256));
}

// A layer alone takes 64 x 64 tiles when 128 x 128 ones would leave most compute units idle; the layers of a
// call fill the chip together, so they take the larger tiles (half the operand traffic into the compute
// units per output) as soon as the call holds enough of them.  A sum is accumulated in the same order under
// either tile size, so the outputs are the same bytes.
static bool batch_promotes(const SpmmArgs* layers, int count) {
  int64_t mid_tiles = 0;
  for (int i = 0; i < count; ++i) {
    GemmArgs g;
    bool sparse_form = false;
    int pick = 0;
    if (tiled_entry(layers[i], &g, &sparse_form, &pick))
      mid_tiles += ((layers[i].O + 127) / 128) * ((layers[i].T + 127) / 128);
  }
  return mid_tiles >= 256;
}

size_t spmm_batched_scratch(SpmmArgs* layers, int count, void* scratch, size_t scratch_bytes) {
  size_t end = 0;
  for (int i = 0; i < count; ++i) {
    SpmmArgs& a = layers[i];
    const size_t bytes = spmm_partial_bytes(a.O, a.K, a.N, a.M, a.T);
    if (bytes == 0) continue;
    if (scratch != nullptr && scratch_bytes >= end + bytes) {
      a.scratch = static_cast<unsigned char*>(scratch) + end;
      a.scratch_bytes = bytes;
    }
    end += (bytes + 255) / 256 * 256;
  }
  return end != 0 && batch_promotes(layers, count) ? 0 : end;  // (such a call cuts nothing)
}

// LDS stages of the dense-form 128 x 128 tiles in a shared launch: two (64 KB) instead of three (96 KB) keep the
// launch's LDS at the 2:4 form's 75 KB, so that two blocks share a compute unit (48 layers at 197 tokens: 62 us
// against 70 us with three).
constexpr int kGroupDenseStages = 2;

// Products of many prepared layers: those the persistent kernel takes share launches (one table per operand form,
// flushed when full), the small ones share one launch of the tiled kernel per tile size (both forms together),
// few-token layers without a workspace one launch of the packed-format kernel; what is left is launched alone.
hipError_t launch_spmm_batched(const SpmmArgs* layers, int count, hipStream_t s) {
  StreamGroup sparse_grp, dense_grp;
  sparse_grp.count = dense_grp.count = 0;
  sparse_grp.n_tiles = dense_grp.n_tiles = 0;
  hipError_t e = hipSuccess;
  auto flush = [&](StreamGroup& grp, bool sparse) {
    if (grp.count == 0) return hipSuccess;
    // Deepest layers first (insertion sort, stable): the blocks take the list in order, so the launch then ends
    // with the cheapest tiles and its last, partly filled round is as short as the list allows.
    for (int i = 1; i < grp.count; ++i) {
      const StreamLayer L = grp.layer[i];
      int j = i;
      for (; j > 0 && grp.layer[j - 1].nk < L.nk; --j) grp.layer[j] = grp.layer[j - 1];
      grp.layer[j] = L;
    }
    const hipError_t r = sparse ? launch_stream_group<true>(grp, s) : launch_stream_group<false>(grp, s);
    grp.count = 0; grp.n_tiles = 0;
    return r;
  };
  SplitGroup split_grp;
  split_grp.count = 0;
  TileGroup tile_grp[2];  // 128 x 128 and 64 x 64 tiles, both operand forms in each
  for (TileGroup& t : tile_grp) t.count = 0;
  auto tile_append = [&](int which, const GemmArgs& g, bool sparse_form) {
    return which == 0 ? tile_group_append<2, 2, 4, 4>(tile_grp[0], g, sparse_form)
                      : tile_group_append<2, 2, 2, 2>(tile_grp[1], g, sparse_form);
  };
  auto tile_flush = [&](int which) {
    return which == 0 ? launch_gemm_group<2, 2, 4, 4, 3, kGroupDenseStages, true>(tile_grp[0], s)
                      : launch_gemm_group<2, 2, 2, 2, 3, 3, false>(tile_grp[1], s);
  };
  const bool promote = batch_promotes(layers, count);
  // few tokens and no workspace: all such layers of the call in one launch of the kernel that reads the packed format
  {
    constexpr int kChunk = 64;
    const SpmmArgs* few[kChunk];
    int n_few = 0;
    for (int i = 0; i < count; ++i) {
      if (!packed_path(layers[i])) continue;
      few[n_few++] = &layers[i];
      if (n_few == kChunk) {
        if ((e = launch_fewtok(few, n_few, s)) != hipSuccess) return e;
        n_few = 0;
      }
    }
    if (n_few && (e = launch_fewtok(few, n_few, s)) != hipSuccess) return e;
  }
  for (int i = 0; i < count; ++i) {
    GemmArgs g;
    bool sparse_form = false;
    if (packed_path(layers[i])) continue;
    if (stream_entry(layers[i], &g, &sparse_form)) {
      StreamGroup& grp = sparse_form ? sparse_grp : dense_grp;
      bool ok = sparse_form ? group_append<true>(grp, g) : group_append<false>(grp, g);
      if (!ok) {
        if ((e = flush(grp, sparse_form)) != hipSuccess) return e;
        ok = sparse_form ? group_append<true>(grp, g) : group_append<false>(grp, g);
        if (!ok) return hipErrorInvalidValue;
      }
    } else if (int pick = 0; tiled_entry(layers[i], &g, &sparse_form, &pick)) {
      // small layers: the tiled kernel, all layers of one operand form and tile size in one launch
      const int which = (pick == 2 || promote) ? 0 : 1;
      // a call that fills the chip with whole tiles has no use for cut reductions (their partial sums would only
      // add traffic and a launch): such a call's sums differ from the single calls' in rounding order only
      if (promote) { g.splits = 1; g.partial = nullptr; }
      bool listed = tile_append(which, g, sparse_form);
      if (!listed) {
        if ((e = tile_flush(which)) != hipSuccess) return e;
        listed = tile_append(which, g, sparse_form);
        if (!listed) {  // more blocks than a grid holds: alone
          bool short_ws = false;
          if ((e = launch_spmm(layers[i], s, &short_ws, SPMM_PRODUCT)) != hipSuccess) return e;
        }
      }
      // a layer whose reduction is cut into ranges: its partial sums are added up after the tile launches
      if (listed && g.splits > 1 && !split_group_append(split_grp, g)) {
        for (int w = 0; w < 2; ++w)
          if ((e = tile_flush(w)) != hipSuccess) return e;
        if ((e = launch_split_reduce(split_grp, s)) != hipSuccess) return e;
        split_group_append(split_grp, g);  // its tiles have just run; the table is empty again
      }
    } else {
      bool short_ws = false;
      if ((e = launch_spmm(layers[i], s, &short_ws, SPMM_PRODUCT)) != hipSuccess) return e;
    }
  }
  if ((e = flush(sparse_grp, true)) != hipSuccess) return e;
  if ((e = flush(dense_grp, false)) != hipSuccess) return e;
  for (int which = 0; which < 2; ++which)
    if ((e = tile_flush(which)) != hipSuccess) return e;
  return launch_split_reduce(split_grp, s);
}

}  // namespace nm
