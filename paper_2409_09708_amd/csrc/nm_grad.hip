// Training products of one sparse linear layer (Section 3.2: the gradient of the loss is taken with
// respect to the sparse weights of the chosen configuration; Section 3.1, weight-update figure: the
// sparse matrix of the applied level is what is trained inside the shared weight).  With the mask of
// the step held fixed and Y = X (W (.) m)^T:
//
//   dX[t, k] = sum_o dY[t, o] * (W (.) m)[o, k]            reduction over the out-features
//   dW[o, k] = sum_t dY[t, o] * X[t, k]   ((.) m[o, k])     reduction over the tokens
//
// Both are dense products (the weight is N:M along k, which is an OUTPUT index of dX, so no term of
// the reduction can be skipped), and in both the reduction index is the ROW index of an operand as
// it lies in memory: W (.) m is [O, K], dY is [T, O], X is [T, K].  The matrix instruction wants, per
// lane, 8 consecutive reduction indices of one row.  Instead of transposing operands in HBM, a tile
// travels global -> LDS as it lies (rows = reduction index) and the fragments are read with the
// transposing LDS read of gfx950 (ds_read_b64_tr_b16): in each group of 16 lanes, lanes 4e .. 4e+3
// name the 16 elements of "row" e (4 each), and lane i receives element i of rows 0 .. 3, i.e. four
// consecutive reduction indices of column i.
//
// One kernel serves both products:  C[i, j] = sum_r P[r, i] * Q(j, r), stored as Out[j, i]:
//   dX: P = W (.) m [r = o, i = k], Q = dY as [j = t, r = o] (reduction contiguous), Out = dX [t, k]
//   dW: P = X       [r = t, i = k], Q = dY as [r = t, j = o] (reduction = row),       Out = dW [o, k]
// The token reduction of dW is long and its output small (a few dozen 128 x 256 tiles), so it is cut
// into `splits` ranges; every block leaves an fp32 partial tile, of its range or of a pair of neighbouring ones, and a second
// kernel adds the partial tiles in order (the result does not depend on scheduling), applies the mask and rounds.
#include "nm_device.h"
#include "nm_launch.h"
#include "nm_mma.h"

#include <type_traits>
#include <utility>

namespace nm {

namespace {

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t* lds_i16x4_ptr;

struct TGemmArgs {
  const bf16_t* P;  // [R, I], ld ldp
  const bf16_t* Q;  // Q_STRIDED: [R, J], else [J, R]; ld ldq
  int64_t I, J, R, ldp, ldq;
  void* out;        // Out[J, I], ld ldo (when partial is NULL)
  int64_t ldo;
  int out_bf16;
  int vec_store;    // Out rows split into whole aligned 16-byte pieces
  int n_i_tiles, n_j_tiles;
  int splits;       // ranges the reduction is cut into (>= 1)
  float* partial;   // not NULL: fp32 partial tiles [range, or pair of ranges][tile][accumulator][thread] (16 bytes per
                    // thread) instead of Out
};

struct TCfg {
  // 4 waves (2 x 2), each 64 (i) x 128 (j) outputs: a wave reads 12 fragments per 32 matrix instructions (the
  // LDS read rate is what bounds these kernels; 64 x 64 per wave needs 8 per 16).  Two blocks share a compute
  // unit (72 KiB of LDS each), so one block's barrier and write-out overlap the other's arithmetic.
  static constexpr int WI = 2, WJ = 2, IT = 4, JT = 8;
  static constexpr int NW = WI * WJ, NT = NW * 64;
  static constexpr int BI = WI * IT * 16, BJ = WJ * JT * 16;  // 128 x 256 outputs per block
  static constexpr int RS = 32;                                // reduction indices per stage: one instruction deep
  static constexpr int STAGES = 3;
  static constexpr int P_ROWB = BI * 2, Q_ROWB = BJ * 2;       // bytes of a row of a reduction-major tile
  static constexpr int P_BYTES = RS * BI * 2, Q_BYTES = RS * BJ * 2;
  static constexpr int STAGE = P_BYTES + Q_BYTES;
  static constexpr int LDS_BYTES = STAGES * STAGE;
  static constexpr int P_PW = P_BYTES / 1024 / NW, Q_PW = Q_BYTES / 1024 / NW;  // wave-wide loads per wave
  static constexpr int LPW = P_PW + Q_PW;
  static constexpr int MMA = IT * JT;
  static_assert(P_PW * NW * 1024 == P_BYTES && Q_PW * NW * 1024 == Q_BYTES && STAGES * LPW < 64, "load split");
  static_assert(2 * LDS_BYTES <= 160 * 1024, "two blocks per compute unit");
};

// Transposing fragment read from a tile stored as [RS rows (reduction)][ROWB / 2 columns], the 16-byte pieces
// of row r at slot (piece ^ 2 (r & 3) ^ 8 ((r >> 3) & 1)): the 16 lanes of a group touch four rows, and the
// first term puts their 32-byte runs on different banks; two groups are served together and their rows lie 8
// apart, the second term sends them to different halves of the 64 banks.  Lane (c16 = lane % 16, kb = lane / 16) receives the reduction indices
// 8 kb .. 8 kb + 7 of column 16 * block + c16.
template <int ROWB>
__device__ __forceinline__ u32x4_t read_transposed(const unsigned char* tile, int block, int c16, int kb) {
  const int sub = c16 >> 2;  // row inside the group of four; also (row & 3)
  const int off = (8 * kb + sub) * ROWB + (((2 * (block ^ sub) + ((c16 & 3) >> 1)) ^ (8 * (kb & 1))) << 4) + (c16 & 1) * 8;
  const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(tile + off));
  const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(tile + off + 4 * ROWB));
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const u32x2_t l = __builtin_bit_cast(u32x2_t, lo), h = __builtin_bit_cast(u32x2_t, hi);
  return u32x4_t{l[0], l[1], h[0], h[1]};
}

// Where lane `lane` of the n-th wave-wide load (1 KiB of consecutive LDS) of a reduction-major tile reads:
// row of the stage and 16-byte piece of that row (before the edge clamp).
template <int ROWB>
__device__ __forceinline__ void strided_load_place(int n, int lane, int* row, int* piece) {
  constexpr int PER_ROW = ROWB / 16, ROWS = 1024 / ROWB;
  *row = n * ROWS + lane / PER_ROW;
  *piece = (lane % PER_ROW) ^ (2 * (*row & 3)) ^ (8 * ((*row >> 3) & 1));
}

// PAIR (split reductions only): a block of eight waves, two halves of four, each half a tile of its own range as above with its
// own LDS stages.  The halves of a block take two neighbouring ranges of one tile and add their sums through LDS before they
// leave, so half as many partial tiles are written and read back: those bytes (64 MB written and 64 MB read by the sum, whatever
// the layer) and the wait for them at the end, when every block writes at once, were what the kernels of a layer at 12608 tokens
// spent most of their time on beside the instructions.  The ranges stay as they were, so no sum gets longer.  The second half runs one
// barrier behind the first: on every SIMD one wave reads its fragments while the other multiplies.  12608 tokens, both
// kernels: 768 -> 2304 59.4 -> 51.7 us, 768 -> 768 33.5 -> 29.0, 768 -> 3072 67.6 -> 61.8; 25216 x 768 -> 3072 115 -> 104.
// Blocks of the paired form: one per tile and pair of ranges, and one per two tiles for the last of an odd number of ranges.
__host__ __device__ constexpr int64_t pair_blocks(int64_t n_tiles, int splits) {
  return n_tiles * (splits / 2) + (splits % 2 ? (n_tiles + 1) / 2 : 0);
}

template <bool Q_STRIDED, bool PAIR>
__global__ void __launch_bounds__(PAIR ? 2 * TCfg::NT : TCfg::NT, 2)
nm_tgemm_kernel(const TGemmArgs a) {
  using C = TCfg;
  constexpr int IT = C::IT, JT = C::JT, STAGES = C::STAGES;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_all[];
  const int half = PAIR ? (int)__builtin_amdgcn_readfirstlane(threadIdx.x / C::NT) : 0;
  unsigned char* const smem = smem_all + half * C::LDS_BYTES;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  // Block -> (tile, split).  Consecutive block ids land on different XCDs (8, each with its own L2); every
  // XCD takes a contiguous run of (split, tile) pairs, tiles fastest and i fastest among the tiles, so the
  // blocks that share an L2 share rows of Q, and each range of rows of a split reduction is fetched into one
  // L2 (two where a split straddles a boundary).
  const int n_tiles = a.n_i_tiles * a.n_j_tiles;
  const int64_t n_paired = PAIR ? (int64_t)n_tiles * (a.splits / 2) : 0;
  const int64_t n_blocks = PAIR ? pair_blocks(n_tiles, a.splits) : (int64_t)n_tiles * a.splits;
  const int64_t per_xcd = (n_blocks + 7) >> 3;
  const int64_t virt = (int64_t)(blockIdx.x & 7) * per_xcd + (int64_t)(blockIdx.x >> 3);
  if (virt >= n_blocks) return;
  // PAIR: the halves take ranges 2p and 2p + 1 of one tile, or the last range of two neighbouring tiles
  const bool paired = PAIR && virt < n_paired;
  const int plane = (int)(PAIR && !paired ? a.splits / 2 : virt / n_tiles);  // partial tile it is stored as
  const int split = !PAIR ? plane : paired ? 2 * plane + half : a.splits - 1;
  const int tile = (int)(PAIR && !paired ? 2 * (virt - n_paired) + half : virt % n_tiles);
  const int64_t i0 = (int64_t)(tile % a.n_i_tiles) * C::BI;
  const int64_t j0 = (int64_t)(tile / a.n_i_tiles) * C::BJ;

  // this block's reduction steps
  const int64_t steps_all = (a.R + C::RS - 1) / C::RS;
  int64_t step_first = 0, nk = steps_all;
  if (a.splits > 1) {
    const int64_t share = steps_all / a.splits, extra = steps_all % a.splits;
    step_first = split * share + (split < extra ? split : extra);
    nk = share + (split < extra ? 1 : 0);
  }
  // PAIR: both halves pass the same barriers: the second range of a pair is never the longer one, and a half without a tile
  // only keeps step
  const int64_t nk_block = PAIR && half && paired ? nk + (split - 1 < steps_all % a.splits && split >= steps_all % a.splits ? 1 : 0) : nk;
  if (PAIR && tile >= n_tiles) nk = 0;
  const int64_t r_first = step_first * C::RS;

  const int tid = PAIR ? threadIdx.x % C::NT : threadIdx.x;  // in the half
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave % C::WI;
  const int wj = wave / C::WI;
  const int c16 = lane & 15;
  const int kb = lane >> 4;

  // ---- this wave's loads of a stage.  Columns of a reduction-major tile past the edge re-read the last whole
  // piece of the row (those outputs are never stored).  Rows past R are clamped to stay inside the operand
  // and zeroed in LDS before use.
  int p_row[C::P_PW], q_row[C::Q_PW];       // row inside the stage (reduction-major) or inside the tile
  uint32_t p_col[C::P_PW], q_col[C::Q_PW];  // byte offset inside the row
  uint32_t p_dst[C::P_PW], q_dst[C::Q_PW];
  const int64_t p_last_piece = (a.I - i0) / 8 - 1;
#pragma unroll
  for (int d = 0; d < C::P_PW; ++d) {
    const int n = wave + d * C::NW;
    int piece;
    strided_load_place<C::P_ROWB>(n, lane, &p_row[d], &piece);
    if (piece > p_last_piece) piece = (int)p_last_piece;
    p_col[d] = (uint32_t)(piece * 16);
    p_dst[d] = (uint32_t)(n * 1024);
  }
  const int64_t q_last_piece = (a.J - j0) / 8 - 1, q_last_row = a.J - 1 - j0;
#pragma unroll
  for (int d = 0; d < C::Q_PW; ++d) {
    const int n = wave + d * C::NW;
    if (Q_STRIDED) {
      int piece;
      strided_load_place<C::Q_ROWB>(n, lane, &q_row[d], &piece);
      if (piece > q_last_piece) piece = (int)q_last_piece;
      q_col[d] = (uint32_t)(piece * 16);
    } else {
      // [BJ rows j][32 reduction indices]: 64 bytes per row, load n covers rows 16n .. 16n+15, lane ->
      // (row 16n + lane / 4, slot lane % 4), the slot holds piece slot ^ ((row >> 1) & 3)
      int64_t row = 16 * n + (lane >> 2);
      const int piece = (lane & 3) ^ (int)((row >> 1) & 3);
      if (row > q_last_row) row = q_last_row;
      q_row[d] = (int)row;
      q_col[d] = (uint32_t)(piece * 16);
    }
    q_dst[d] = (uint32_t)(C::P_BYTES + n * 1024);
  }
  const bf16_t* p_base = a.P + i0;
  // lane byte offsets of the loads of a stage with all its rows (the common case; a ragged last stage clamps)
  uint32_t p_voff[C::P_PW], q_voff[C::Q_PW];
#pragma unroll
  for (int d = 0; d < C::P_PW; ++d) p_voff[d] = (uint32_t)p_row[d] * (uint32_t)(a.ldp * 2) + p_col[d];
#pragma unroll
  for (int d = 0; d < C::Q_PW; ++d) q_voff[d] = (uint32_t)q_row[d] * (uint32_t)(a.ldq * 2) + q_col[d];
  const bf16_t* q_base = Q_STRIDED ? a.Q + j0 : a.Q + j0 * a.ldq;
  const uint32_t ldp2 = (uint32_t)(a.ldp * 2), ldq2 = (uint32_t)(a.ldq * 2);

  // A stage's sources: the (wave-uniform) operand addresses at its first reduction index and the rows it has
  struct StageSrc { uniform_ptr_t p, q; int rows; };
  auto stage_src = [&](int64_t r) {
    StageSrc src;
    src.p = make_uniform(p_base + r * a.ldp);
    src.q = make_uniform(Q_STRIDED ? q_base + r * a.ldq : q_base + r);
    src.rows = (int)((a.R - r) < C::RS ? (a.R - r) : C::RS);  // >= 1
    return src;
  };
  // the d-th load of a stage into LDS buffer buf
  auto issue_one = [&](auto d_tag, const StageSrc& src, int buf) {
    constexpr int d = decltype(d_tag)::value;
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)buf * C::STAGE);
    const bool ragged = src.rows < C::RS;  // wave-uniform; only the last stage of the reduction
    if constexpr (d < C::P_PW) {
      uint32_t voff = p_voff[d];
      if (ragged && p_row[d] >= src.rows) voff = (uint32_t)(src.rows - 1) * ldp2 + p_col[d];
      dma16(src.p, voff, lds + p_dst[d]);
    } else if constexpr (Q_STRIDED) {
      uint32_t voff = q_voff[d - C::P_PW];
      if (ragged && q_row[d - C::P_PW] >= src.rows) voff = (uint32_t)(src.rows - 1) * ldq2 + q_col[d - C::P_PW];
      dma16(src.q, voff, lds + q_dst[d - C::P_PW]);
    } else {
      dma16(src.q, q_voff[d - C::P_PW], lds + q_dst[d - C::P_PW]);
    }
  };
  auto issue_stage = [&](int64_t r, int buf) {
    const StageSrc src = stage_src(r);
    [&]<int... D>(std::integer_sequence<int, D...>) {
      (issue_one(std::integral_constant<int, D>{}, src, buf), ...);
    }(std::make_integer_sequence<int, C::LPW>{});
  };

  f32x4_t acc[IT][JT];
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int j = 0; j < JT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  u32x4_t pf[IT], qf[JT];
  auto read_frags = [&](int buf) {
    const unsigned char* base = smem + buf * C::STAGE;
#pragma unroll
    for (int i = 0; i < IT; ++i) pf[i] = read_transposed<C::P_ROWB>(base, wi * IT + i, c16, kb);
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      if (Q_STRIDED) {
        qf[j] = read_transposed<C::Q_ROWB>(base + C::P_BYTES, wj * JT + j, c16, kb);
      } else {
        const int row = (wj * JT + j) * 16 + c16;
        qf[j] = *reinterpret_cast<const u32x4_t*>(base + C::P_BYTES + row * 64 + ((kb ^ ((c16 >> 1) & 3)) << 4));
      }
    }
  };
  // 32 matrix instructions; the wave's loads of a later stage are issued between them
  auto multiply = [&](bool load, int64_t lr, int lbuf) {
    const StageSrc src = stage_src(load ? lr : r_first);
    [&]<int... Q>(std::integer_sequence<int, Q...>) {
      ([&] {
        constexpr int j = Q / IT, i = j & 1 ? IT - 1 - Q % IT : Q % IT;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pf[i]),
                                                            __builtin_bit_cast(bf16x8_t, qf[j]), acc[i][j], 0, 0, 0);
        if constexpr (Q % 4 == 3 && Q / 4 < C::LPW) {
          if (load) issue_one(std::integral_constant<int, Q / 4>{}, src, lbuf);
          __builtin_amdgcn_sched_barrier(0);
        }
      }(), ...);
    }(std::make_integer_sequence<int, C::MMA>{});
  };
  auto wait_stage = [&](int younger) {
    [&]<int... Y>(std::integer_sequence<int, Y...>) {
      ((younger == Y ? wait_loads_outstanding<Y * C::LPW>() : void()), ...);
    }(std::make_integer_sequence<int, STAGES - 1>{});
  };

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue_stage(r_first + (int64_t)s * C::RS, s);

  // PAIR: the second half runs one barrier behind the first
  auto turn = [&] {
    if constexpr (PAIR) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (half) turn();
  // One barrier per stage; the buffer multiplied in the previous step is refilled right after the barrier,
  // STAGES - 1 stages ahead.
  {
    int buf = 0;
    int64_t ks = 0;
    // Steady state, free of conditions: while the stage to be fetched exists and has all its rows (then so has
    // the one being multiplied), the waits are fixed, no row is clamped or cleared, and the operand addresses
    // advance by additions.  A wave issues in order, so every scalar and vector instruction saved here is issue
    // time its matrix instructions get.  The last STAGES - 1 steps (and a ragged last stage of the reduction)
    // take the general form below.
    int64_t n_fast = nk - (STAGES - 1);
    if (n_fast > 0 && a.R - (r_first + (nk - 1) * C::RS) < C::RS) --n_fast;
    if (n_fast > 0) {
      const int64_t r_load = r_first + (int64_t)(STAGES - 1) * C::RS;
      const unsigned char* fp = reinterpret_cast<const unsigned char*>(p_base + r_load * a.ldp);
      const unsigned char* fq = reinterpret_cast<const unsigned char*>(Q_STRIDED ? q_base + r_load * a.ldq : q_base + r_load);
      const int64_t p_step = (int64_t)C::RS * a.ldp * 2, q_step = Q_STRIDED ? (int64_t)C::RS * a.ldq * 2 : (int64_t)C::RS * 2;
      uint32_t lds_load = lds0 + (uint32_t)((STAGES - 1) * C::STAGE);  // LDS address of the buffer to be refilled
      for (; ks < n_fast; ++ks) {
        wait_loads_outstanding<(STAGES - 2) * C::LPW>();
        __builtin_amdgcn_s_barrier();
        read_frags(buf);
        turn();
        const uniform_ptr_t up = make_uniform(fp), uq = make_uniform(fq);
        const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_load);
        [&]<int... Q>(std::integer_sequence<int, Q...>) {
          ([&] {
            constexpr int j = Q / IT, i = j & 1 ? IT - 1 - Q % IT : Q % IT;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pf[i]),
                                                                __builtin_bit_cast(bf16x8_t, qf[j]), acc[i][j], 0, 0, 0);
            if constexpr (Q % 4 == 3 && Q / 4 < C::LPW) {
              constexpr int d = Q / 4;
              if constexpr (d < C::P_PW) dma16(up, p_voff[d], lds + p_dst[d]);
              else dma16(uq, q_voff[d - C::P_PW], lds + q_dst[d - C::P_PW]);
              __builtin_amdgcn_sched_barrier(0);
            }
          }(), ...);
        }(std::make_integer_sequence<int, C::MMA>{});
        fp += p_step;
        fq += q_step;
        lds_load += (uint32_t)C::STAGE;
        if (lds_load == lds0 + (uint32_t)(STAGES * C::STAGE)) lds_load = lds0;
        if (++buf == STAGES) buf = 0;
      }
    }
    for (; ks < nk; ++ks) {
      const int64_t ahead = nk - 1 - ks;  // stages after this one; the loads of at most STAGES - 2 of them are out
      wait_stage(ahead < STAGES - 2 ? (int)ahead : STAGES - 2);
      const int64_t r = r_first + ks * C::RS;
      if (a.R - r < C::RS) {
        // ragged last stage of the reduction: this wave's own loads have landed; it clears the rows past R
        // it fetched (reduction-major tiles only; the other form requires R % 32 == 0)
        const int rows_left = (int)(a.R - r);
        unsigned char* base = smem + buf * C::STAGE;
#pragma unroll
        for (int d = 0; d < C::P_PW; ++d)
          if (p_row[d] >= rows_left) *reinterpret_cast<u32x4_t*>(base + p_dst[d] + lane * 16) = u32x4_t{0, 0, 0, 0};
        if (Q_STRIDED) {
#pragma unroll
          for (int d = 0; d < C::Q_PW; ++d)
            if (q_row[d] >= rows_left) *reinterpret_cast<u32x4_t*>(base + q_dst[d] + lane * 16) = u32x4_t{0, 0, 0, 0};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      __builtin_amdgcn_s_barrier();
      int nbuf = buf + STAGES - 1;
      if (nbuf >= STAGES) nbuf -= STAGES;
      read_frags(buf);
      turn();
      multiply(ks + STAGES - 1 < nk, r + (int64_t)(STAGES - 1) * C::RS, nbuf);
      if (++buf == STAGES) buf = 0;
    }
    if constexpr (PAIR)
      for (; ks < nk_block; ++ks) {
        turn();
        turn();
      }
  }
  if (PAIR && !half) turn();

  // ---- split reduction: the partial tile, 16 bytes per lane and accumulator, fully coalesced
  if (a.partial) {
    f32x4_t* mine = reinterpret_cast<f32x4_t*>(a.partial) + ((size_t)plane * n_tiles + tile) * (C::MMA * C::NT) + tid;
    if (PAIR && paired) {
      // the two ranges are added here: each half hands the other 16 of its 32 accumulators through its own stages
      static_assert(C::MMA / 2 * C::NT * 16 <= C::LDS_BYTES && JT % 2 == 0, "half the accumulators fit the half's stages");
      turn();  // nobody reads operands any more
      auto swap_and_store = [&](auto keep_tag) {
        constexpr int KEEP = decltype(keep_tag)::value * (JT / 2), GIVE = JT / 2 - KEEP;
        f32x4_t* out = reinterpret_cast<f32x4_t*>(smem) + tid;
        const f32x4_t* in = reinterpret_cast<const f32x4_t*>(smem_all + (1 - half) * C::LDS_BYTES) + tid;
#pragma unroll
        for (int j = 0; j < JT / 2; ++j)
#pragma unroll
          for (int i = 0; i < IT; ++i) out[(j * IT + i) * C::NT] = acc[i][GIVE + j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        turn();
#pragma unroll
        for (int j = 0; j < JT / 2; ++j)
#pragma unroll
          for (int i = 0; i < IT; ++i) mine[(i * JT + KEEP + j) * C::NT] = acc[i][KEEP + j] + in[(j * IT + i) * C::NT];
      };
      if (half) swap_and_store(std::integral_constant<int, 1>{});
      else swap_and_store(std::integral_constant<int, 0>{});
      return;
    }
    if (PAIR && tile >= n_tiles) return;
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int j = 0; j < JT; ++j) mine[(i * JT + j) * C::NT] = acc[i][j];
    return;
  }

  // ---- write-out.  A lane holds columns i .. i+3 (accumulator element e -> row 4 kb + e of the 16-row block)
  // of output row j = c16, i.e. 8 or 16 contiguous bytes of an Out row.  For aligned outputs every wave
  // transposes 16 output rows at a time through its own LDS slice, so that the global stores are 16 bytes
  // per lane and whole row segments of the wave tile are written contiguously.
  __builtin_amdgcn_s_barrier();  // every wave is done with the operand stages
  auto get = [&](int i, int j) { return __builtin_bit_cast(u32x4_t, acc[i][j]); };
  const int64_t row0 = j0 + wj * JT * 16, col0 = i0 + wi * IT * 16;
  static_assert(C::NW * wave_tile_slice_bytes<IT, 4>() <= C::LDS_BYTES, "write-out slices");
  if (a.vec_store) {
    if (a.out_bf16)
      write_wave_tile_pieces<IT, JT, 2>(smem + wave * wave_tile_slice_bytes<IT, 2>(), lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
    else
      write_wave_tile_pieces<IT, JT, 4>(smem + wave * wave_tile_slice_bytes<IT, 4>(), lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  } else if (a.out_bf16) {
    write_wave_tile_rows<IT, JT, 2>(smem + wave * wave_tile_slice_bytes<IT, 4>(), lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  } else {
    write_wave_tile_rows<IT, JT, 4>(smem + wave * wave_tile_slice_bytes<IT, 4>(), lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  }
}

// dW of a short reduction in one launch.  A block walks the whole reduction of a tile of 128 x 128 and adds the sums of its
// ranges itself, range by range (pair by pair) in the order in which grad_reduce_kernel adds the partial tiles: the same bits,
// without the partial tiles (up to 64 MB written and read back, whatever the layer) and without the second launch, which bound the
// short reductions.  The smaller tile makes twice the blocks of them, as nothing else spreads the work.  A step of 32 tokens takes
// 0.29 us, some 610 cycles, and keeps nothing busy: at 1576 x 768 -> 2304 the fragments hold LDS for 0.22 of a unit's cycles (48 KB a
// step, and 16 KB of copies beside them), the matrix pipes run for 0.26, and the waves, one block of them to a unit, are stalled at a
// wait for 0.35 of their time and wait to issue for 0.28: what bounds it is the chain of a step, barrier, reads, products.  Eight waves of 64 x 32
// and fragments read one step ahead: with one wave of 64 x 64 on each SIMD nothing covers a range's additions and the waits, and a step
// takes 0.38; with eight stages instead of four it is no faster.  us, f32 gradients, in two launches and here: 20 tokens x 768 -> 2304
// 10.8 and 4.9, 197 x 768 -> 2304 13.9 and 7.2, 394 x 1024 -> 4096 28.5 and 11.3, 788 x 768 -> 3072 28.2 and 13.7, 1576 x 768 -> 2304
// 27.6 and 21.3.
struct SCfg {
  static constexpr int WI = 2, WJ = 4, IT = 4, JT = 2;
  static constexpr int NW = WI * WJ, NT = NW * 64;
  static constexpr int BI = WI * IT * 16, BJ = WJ * JT * 16;
  static constexpr int RS = 32, STAGES = 4;
  static constexpr int ROWB = BI * 2, P_BYTES = RS * BI * 2, Q_BYTES = RS * BJ * 2;  // (rows of both operands are 256 bytes)
  static constexpr int STAGE = P_BYTES + Q_BYTES, LDS_BYTES = STAGES * STAGE;
  static constexpr int P_PW = P_BYTES / 1024 / NW, Q_PW = Q_BYTES / 1024 / NW, LPW = P_PW + Q_PW;
  static constexpr int MMA = IT * JT;
  static_assert(BI == BJ && RS == TCfg::RS && LDS_BYTES <= 160 * 1024 && STAGES * LPW < 64, "one block of 160 KiB at most");
};

template <bool PAIRED>
__global__ void __launch_bounds__(SCfg::NT, 2)
nm_wgrad_kernel(const TGemmArgs a, const uint32_t* __restrict__ mask) {
  using C = SCfg;
  constexpr int IT = C::IT, JT = C::JT, STAGES = C::STAGES;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const int n_tiles = a.n_i_tiles * a.n_j_tiles;
  const int per_xcd = (n_tiles + 7) >> 3;
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);  // an XCD's tiles share rows of Q
  if (tile >= n_tiles) return;
  const int64_t i0 = (int64_t)(tile % a.n_i_tiles) * C::BI, j0 = (int64_t)(tile / a.n_i_tiles) * C::BJ;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave % C::WI, wj = wave / C::WI, c16 = lane & 15, kb = lane >> 4;

  // loads of a stage, as in the kernel above: columns past the edge re-read the last piece, rows past R the last row (and are cleared)
  int row[C::P_PW];
  uint32_t p_col[C::P_PW], q_col[C::P_PW], p_voff[C::P_PW], q_voff[C::P_PW];
  static_assert(C::P_PW == C::Q_PW, "one set of rows");
  const int64_t p_last = (a.I - i0) / 8 - 1, q_last = (a.J - j0) / 8 - 1;
  const uint32_t ldp2 = (uint32_t)(a.ldp * 2), ldq2 = (uint32_t)(a.ldq * 2);
#pragma unroll
  for (int d = 0; d < C::P_PW; ++d) {
    int piece;
    strided_load_place<C::ROWB>(wave + d * C::NW, lane, &row[d], &piece);
    p_col[d] = (uint32_t)((piece > p_last ? (int)p_last : piece) * 16);
    q_col[d] = (uint32_t)((piece > q_last ? (int)q_last : piece) * 16);
    p_voff[d] = (uint32_t)row[d] * ldp2 + p_col[d];
    q_voff[d] = (uint32_t)row[d] * ldq2 + q_col[d];
  }
  const int steps = (int)((a.R + C::RS - 1) / C::RS);
  const int last_rows = (int)(a.R - (int64_t)(steps - 1) * C::RS);  // of the last step
  const unsigned char* fp = reinterpret_cast<const unsigned char*>(a.P + i0);
  const unsigned char* fq = reinterpret_cast<const unsigned char*>(a.Q + j0);
  const int64_t p_step = (int64_t)C::RS * a.ldp * 2, q_step = (int64_t)C::RS * a.ldq * 2;
  auto issue_one = [&](auto d_tag, uniform_ptr_t up, uniform_ptr_t uq, uint32_t lds) {
    constexpr int d = decltype(d_tag)::value;
    if constexpr (d < C::P_PW) dma16(up, p_voff[d], lds + (uint32_t)((wave + d * C::NW) * 1024));
    else dma16(uq, q_voff[d - C::P_PW], lds + (uint32_t)(C::P_BYTES + (wave + (d - C::P_PW) * C::NW) * 1024));
  };
  // the last step's missing rows are fetched from its last one
  auto clamp_rows = [&]() {
#pragma unroll
    for (int d = 0; d < C::P_PW; ++d)
      if (row[d] >= last_rows) {
        p_voff[d] = (uint32_t)(last_rows - 1) * ldp2 + p_col[d];
        q_voff[d] = (uint32_t)(last_rows - 1) * ldq2 + q_col[d];
      }
  };
  auto issue_stage = [&](int s, int buf) {
    if (s == steps - 1) clamp_rows();
    const uniform_ptr_t up = make_uniform(fp + s * p_step), uq = make_uniform(fq + s * q_step);
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)buf * C::STAGE);
    [&]<int... D>(std::integer_sequence<int, D...>) {
      (issue_one(std::integral_constant<int, D>{}, up, uq, lds), ...);
    }(std::make_integer_sequence<int, C::LPW>{});
  };

  // the mask words of this lane's outputs: rows j, 64 columns; in flight under the reduction
  const int64_t row0 = j0 + wj * JT * 16, col0 = i0 + wi * IT * 16;
  uint32_t word[JT][IT / 2];
  const int64_t nw = (a.I + 31) / 32;
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int h = 0; h < IT / 2; ++h) {
      const int64_t jj = row0 + j * 16 + c16, w = (col0 >> 5) + h;
      word[j][h] = !mask ? ~0u : mask[(jj < a.J ? jj : a.J - 1) * nw + (w < nw ? w : nw - 1)];
    }

  // A step's fragments are read under the matrix instructions of the step before.
  f32x4_t acc[IT][JT], sum[IT][JT], first[PAIRED ? IT : 1][PAIRED ? JT : 1];
  u32x4_t pf[2][IT], qf[2][JT];
  const int share = steps / a.splits, extra = steps % a.splits;
  int range = 0, left = share + (0 < extra ? 1 : 0);
  bool fresh = true;  // the next step begins a range
  auto end_range = [&]() {  // the sums of `range` are complete
    auto each = [&](auto f) {
#pragma unroll
      for (int q = 0; q < C::MMA; ++q) f(q / JT, q % JT);
    };
    if constexpr (PAIRED) {
      if (range & 1) each([&](int i, int j) { acc[i][j] = first[i][j] + acc[i][j]; });
      else if (range + 1 < a.splits) each([&](int i, int j) { first[i][j] = acc[i][j]; });
    }
    if (!PAIRED || (range & 1) || range + 1 == a.splits) {
      if (range < (PAIRED ? 2 : 1)) each([&](int i, int j) { sum[i][j] = acc[i][j]; });
      else each([&](int i, int j) { sum[i][j] += acc[i][j]; });
    }
    ++range;
    left = share + (range < extra ? 1 : 0);
    fresh = true;
  };
  auto read_frags = [&](auto set_tag, int buf) {
    constexpr int S = decltype(set_tag)::value;
    const unsigned char* base = smem + buf * C::STAGE;
#pragma unroll
    for (int i = 0; i < IT; ++i) pf[S][i] = read_transposed<C::ROWB>(base, wi * IT + i, c16, kb);
#pragma unroll
    for (int j = 0; j < JT; ++j) qf[S][j] = read_transposed<C::ROWB>(base + C::P_BYTES, wj * JT + j, c16, kb);
  };
  auto clear_rows = [&](int buf) {  // this wave's own loads have landed: it clears the rows past R that it fetched
    unsigned char* base = smem + buf * C::STAGE;
#pragma unroll
    for (int d = 0; d < C::P_PW; ++d)
      if (row[d] >= last_rows) {
        *reinterpret_cast<u32x4_t*>(base + (wave + d * C::NW) * 1024 + lane * 16) = u32x4_t{0, 0, 0, 0};
        *reinterpret_cast<u32x4_t*>(base + C::P_BYTES + (wave + d * C::NW) * 1024 + lane * 16) = u32x4_t{0, 0, 0, 0};
      }
  };
  auto wait_landed = [&](int ahead) {  // ... a stage after which `ahead` stages have been asked for
    if (ahead >= 2) wait_loads_outstanding<2 * C::LPW>();
    else if (ahead == 1) wait_loads_outstanding<C::LPW>();
    else wait_loads_outstanding<0>();
  };
  static_assert(STAGES == 4, "the cases above");

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < steps) issue_stage(s, s);
  wait_landed(steps - 1 < STAGES - 2 ? steps - 1 : STAGES - 2);
  if (steps == 1 && last_rows < C::RS) clear_rows(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  read_frags(std::integral_constant<int, 0>{}, 0);

  int buf = 0;
  // Step ks with fragment set S: stage ks + 1 has landed, everybody has read stage ks - 1 and has stage ks in registers.
  auto step = [&](auto set_tag, int ks, auto fast_tag) {
    constexpr int S = decltype(set_tag)::value;
    constexpr bool FAST = decltype(fast_tag)::value;
    int next = buf + 1 == STAGES ? 0 : buf + 1;
    if (FAST) {
      wait_loads_outstanding<(STAGES - 3) * C::LPW>();
    } else if (ks + 1 < steps) {
      wait_landed(steps - 2 - ks < STAGES - 3 ? steps - 2 - ks : STAGES - 3);
      if (ks + 2 == steps && last_rows < C::RS) clear_rows(next);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (FAST || ks + 1 < steps) read_frags(std::integral_constant<int, S ^ 1>{}, next);
    // the buffer of stage ks - 1, which nobody reads any more
    const int free_buf = buf == 0 ? STAGES - 1 : buf - 1;
    uniform_ptr_t up = 0, uq = 0;
    uint32_t lds = 0;
    const bool load = FAST || ks + STAGES - 1 < steps;
    if (load) {
      if (!FAST && ks + STAGES - 1 == steps - 1) clamp_rows();
      up = make_uniform(fp + (ks + STAGES - 1) * p_step);
      uq = make_uniform(fq + (ks + STAGES - 1) * q_step);
      lds = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)free_buf * C::STAGE);
    }
    auto products = [&](auto fresh_tag) {
      [&]<int... Q>(std::integer_sequence<int, Q...>) {
        ([&] {
          constexpr int j = Q / IT, i = j & 1 ? IT - 1 - Q % IT : Q % IT;
          const f32x4_t c = decltype(fresh_tag)::value ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[i][j];
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pf[S][i]),
                                                              __builtin_bit_cast(bf16x8_t, qf[S][j]), c, 0, 0, 0);
          if constexpr (Q % 4 == 3 && Q / 4 < C::LPW) {
            if (load) issue_one(std::integral_constant<int, Q / 4>{}, up, uq, lds);
            __builtin_amdgcn_sched_barrier(0);
          }
        }(), ...);
      }(std::make_integer_sequence<int, C::MMA>{});
    };
    if (fresh) products(std::true_type{});
    else products(std::false_type{});
    fresh = false;
    buf = next;
    if (--left == 0) end_range();
  };
  // Steady state: a whole stage to load
  const int n_fast = steps - (STAGES - 1) - (last_rows < C::RS ? 1 : 0);
  int ks = 0;
  for (; ks + 1 < n_fast; ks += 2) {
    step(std::integral_constant<int, 0>{}, ks, std::true_type{});
    step(std::integral_constant<int, 1>{}, ks + 1, std::true_type{});
  }
  for (; ks < steps; ks += 2) {
    step(std::integral_constant<int, 0>{}, ks, std::false_type{});
    if (ks + 1 < steps) step(std::integral_constant<int, 1>{}, ks + 1, std::false_type{});
  }

  // ---- the mask of the step, then as the kernel above
  if (mask) {
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!((word[j][i / 2] >> (16 * (i & 1) + kb * 4 + e)) & 1u)) sum[i][j][e] = 0.f;
  }
  __builtin_amdgcn_s_barrier();  // every wave is done with the operand stages
  auto get = [&](int i, int j) { return __builtin_bit_cast(u32x4_t, sum[i][j]); };
  static_assert(C::NW * wave_tile_slice_bytes<IT, 4>() <= C::LDS_BYTES, "write-out slices");
  unsigned char* slice = smem + wave * wave_tile_slice_bytes<IT, 4>();
  if (a.vec_store) {
    if (a.out_bf16) write_wave_tile_pieces<IT, JT, 2>(slice, lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
    else write_wave_tile_pieces<IT, JT, 4>(slice, lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  } else if (a.out_bf16) {
    write_wave_tile_rows<IT, JT, 2>(slice, lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  } else {
    write_wave_tile_rows<IT, JT, 4>(slice, lane, get, a.out, a.ldo, row0, col0, a.J, a.I);
  }
}

// Sum of the partial tiles (of a range, or of a pair of ranges: `planes` of them for each tile) in order, the mask of the step
// (bit k % 32 of word k / 32 of row o; NULL = every weight receives its gradient) and the rounding.  One lane per accumulator of
// the tile kernel.  Bound by reading the partial tiles, and by its launch (72 tiles in 4 planes, 47 MB in all, 8.3 us; 12.2 with
// the 7 single ranges; 32 in 8 7.4, 10.8 with 15).  Up to 10 tiles the few wavefronts do not hide a load and a lane reads six at
// a time, else two (both kernels, six and two: 1 tile in 64 planes 16.4 us and 20.6, 2 in 64 21.3 and 25.7, 8 in 25 25.2 and
// 26.2, 10 in 15 19.1 and 19.4; from 12 tiles on they differ by 1 % either way: 12 in 20 24.8 and 25.0, 16 in 15 27.3 and 27.0,
// 32 in 8 37.2 and 36.1, 65 in 8 69.8 and 69.6, 75 in 7 74.7 and 74.7).
__global__ void __launch_bounds__(256)
grad_reduce_kernel(const float* __restrict__ partial, int planes, int n_tiles, int n_i_tiles, int64_t I, int64_t J,
                   const uint32_t* __restrict__ mask, void* __restrict__ out, int64_t ldo, int out_bf16) {
  using C = TCfg;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)n_tiles * C::MMA * C::NT) return;
  const int tid = (int)(id % C::NT);
  const int q = (int)((id / C::NT) % C::MMA);
  const int tile = (int)(id / (C::NT * C::MMA));
  const f32x4_t* src = reinterpret_cast<const f32x4_t*>(partial) + id;
  const size_t stride = (size_t)n_tiles * (C::MMA * C::NT);
  f32x4_t sum = src[0];
  int s = 1;
  if (n_tiles <= 10) {
    for (; s + 6 <= planes; s += 6) {
      f32x4_t p[6];
#pragma unroll
      for (int u = 0; u < 6; ++u) p[u] = src[(size_t)(s + u) * stride];
#pragma unroll
      for (int u = 0; u < 6; ++u) sum += p[u];
    }
  }
  for (; s + 2 <= planes; s += 2) {
    const f32x4_t p0 = src[(size_t)s * stride], p1 = src[(size_t)(s + 1) * stride];
    sum += p0;
    sum += p1;
  }
  if (s < planes) sum += src[(size_t)s * stride];
  const int lane = tid & 63, wave = tid >> 6;
  const int wi = wave % C::WI, wj = wave / C::WI;
  const int i = q / C::JT, j = q % C::JT;
  const int64_t ii = (int64_t)(tile % n_i_tiles) * C::BI + (wi * C::IT + i) * 16 + (lane >> 4) * 4;
  const int64_t jj = (int64_t)(tile / n_i_tiles) * C::BJ + (wj * C::JT + j) * 16 + (lane & 15);
  if (jj >= J || ii >= I) return;
  if (mask) {
    const uint32_t w = mask[jj * ((I + 31) / 32) + (ii >> 5)] >> (ii & 31);  // I % 4 == 0: the four bits share a word
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!((w >> e) & 1u)) sum[e] = 0.f;
  }
  if (out_bf16) {
    bf16_t* dst = reinterpret_cast<bf16_t*>(out) + jj * ldo + ii;
    if (ii + 3 < I && ((uintptr_t)dst & 7) == 0) {
      *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3]));
    } else {
      for (int e = 0; e < 4 && ii + e < I; ++e) dst[e] = (bf16_t)f32_to_bf16_rne(sum[e]);
    }
  } else {
    float* dst = reinterpret_cast<float*>(out) + jj * ldo + ii;
    if (ii + 3 < I && ((uintptr_t)dst & 15) == 0) {
      *reinterpret_cast<f32x4_t*>(dst) = sum;
    } else {
      for (int e = 0; e < 4 && ii + e < I; ++e) dst[e] = sum[e];
    }
  }
}

// Any shape and alignment: one lane per output, a plain loop over the reduction.
__global__ void __launch_bounds__(256)
backward_input_general_kernel(const bf16_t* __restrict__ Ws, int64_t O, int64_t K, int64_t ldw,
                              const bf16_t* __restrict__ dY, int64_t T, int64_t ldy, void* __restrict__ dX, int64_t ldx,
                              int out_bf16) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= T * K) return;
  const int64_t t = id / K, k = id % K;
  float acc = 0.f;
  for (int64_t o = 0; o < O; ++o) acc = fmaf(bf16_to_f32(dY[t * ldy + o]), bf16_to_f32(Ws[o * ldw + k]), acc);
  if (out_bf16) reinterpret_cast<bf16_t*>(dX)[t * ldx + k] = (bf16_t)f32_to_bf16_rne(acc);
  else reinterpret_cast<float*>(dX)[t * ldx + k] = acc;
}

__global__ void __launch_bounds__(256)
backward_weight_general_kernel(const bf16_t* __restrict__ dY, int64_t T, int64_t O, int64_t ldy,
                               const bf16_t* __restrict__ X, int64_t K, int64_t ldx, const uint32_t* __restrict__ mask,
                               void* __restrict__ dW, int64_t lddw, int out_bf16) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= O * K) return;
  const int64_t o = id / K, k = id % K;
  float acc = 0.f;
  if (!mask || ((mask[o * ((K + 31) / 32) + (k >> 5)] >> (k & 31)) & 1u))
    for (int64_t t = 0; t < T; ++t) acc = fmaf(bf16_to_f32(dY[t * ldy + o]), bf16_to_f32(X[t * ldx + k]), acc);
  if (out_bf16) reinterpret_cast<bf16_t*>(dW)[o * lddw + k] = (bf16_t)f32_to_bf16_rne(acc);
  else reinterpret_cast<float*>(dW)[o * lddw + k] = acc;
}

inline bool aligned_to(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

template <bool Q_STRIDED, bool PAIR = false>
hipError_t launch_tgemm(TGemmArgs g, hipStream_t s) {
  using C = TCfg;
  constexpr int HALVES = PAIR ? 2 : 1;
  auto kern = nm_tgemm_kernel<Q_STRIDED, PAIR>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, HALVES * C::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  const int64_t n_tiles = (int64_t)g.n_i_tiles * g.n_j_tiles;
  const int64_t grid = ((PAIR ? pair_blocks(n_tiles, g.splits) : n_tiles * g.splits) + 7) / 8 * 8;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(HALVES * C::NT), HALVES * C::LDS_BYTES, s, g);
  return hipGetLastError();
}

template <bool PAIRED>
hipError_t launch_wgrad(const TGemmArgs& g, const uint32_t* mask, hipStream_t s) {
  auto kern = nm_wgrad_kernel<PAIRED>;
  static PerDeviceOnce lds_limit;
  if (hipError_t e = raise_dynamic_lds_limit(kern, SCfg::LDS_BYTES, lds_limit); e != hipSuccess) return e;
  const unsigned grid = (unsigned)((g.n_i_tiles * g.n_j_tiles + 7) / 8 * 8);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(SCfg::NT), SCfg::LDS_BYTES, s, g, mask);
  return hipGetLastError();
}

// Ranges of the token reduction of dW.  Two blocks fit a compute unit, 512 at once on a 256-unit chip; the
// smallest count that fills at least 90 % of a whole number of such rounds is taken (else the fullest), with
// at least four steps per range where the reduction is long enough.
struct WeightGradPlan {
  bool tiles;  // the matrix-core kernel takes this shape
  int n_i_tiles, n_j_tiles, splits;
};
WeightGradPlan weight_grad_plan(int64_t O, int64_t K, int64_t T) {
  WeightGradPlan p{false, 0, 0, 0};
  if ((O % 8) || (K % 8) || O > (1 << 24) || K > (1 << 22) || T > (1ll << 31)) return p;
  const int64_t ni = (K + TCfg::BI - 1) / TCfg::BI, nj = (O + TCfg::BJ - 1) / TCfg::BJ;
  if (ni * nj > (1 << 20)) return p;
  p.tiles = true;
  p.n_i_tiles = (int)ni;
  p.n_j_tiles = (int)nj;
  const int64_t steps = (T + TCfg::RS - 1) / TCfg::RS, tiles = ni * nj;
  int best = 1;
  double best_fill = 0.0;
  for (int s = 1; s <= 64; ++s) {
    if (s > 1 && steps / s < 4) break;
    const int64_t blocks = tiles * s, rounds = (blocks + 511) / 512;
    const double fill = (double)blocks / (double)(rounds * 512);
    if (fill > best_fill + 1e-9) { best = s; best_fill = fill; }
    if (fill >= 0.9) break;
  }
  p.splits = best;
  return p;
}

// Whether the ranges are taken in pairs (see nm_tgemm_kernel).  Up to 256 ranges of tiles have a compute unit each to themselves
// as single blocks.  Below 16 steps the ranges are so short that an odd last one, which stays alone, is a third of the work
// (400 tokens x 1024 -> 4096 in 3 ranges 28.7 us, 30.5 in pairs; 600 in 4 32.4 and 30.2).  Past 200 steps a range the bytes of
// the partial tiles no longer count and eight waves in step lose to two free blocks (50432 x 768 -> 3072, 225 steps, 215 us,
// 220 in pairs; 25216 x 1024 -> 4096, 197 steps, 182 and 175).
// Many ranges of fewer than 5.5 steps on 368 (beyond 32 ranges: 328) to 431 blocks stay single: pairs leave a fifth of the units
// empty there.  7880 x 384 -> 384 in 61 ranges 24.0 us, 25.6 in pairs; 10638 x 320 -> 320 in 64 24.8 and 27.0 (but x 256 -> 768 23.5
// and 21.3: of 700 shapes of short ranges pairs take 1.03 of the time on average there).  Fewer blocks gain (1182 x 512 -> 2048, 288,
// 26.1 and 23.4; 1200 x 1024 -> 1280, 360, 27.4 and 25.9), as do more (2364 x 512 -> 2048, 480, 28.1 and 26.6), at most 8 ranges
// (788 x 768 -> 3072 in 6, 31.1 and 28.3) and longer ones (at 5.5 to 6 steps 0.93 to 1.13 either way).
bool weight_grad_paired(const WeightGradPlan& p, int64_t T) {
  const int64_t steps = (T + TCfg::RS - 1) / TCfg::RS, blocks = (int64_t)p.n_i_tiles * p.n_j_tiles * p.splits;
  if (p.splits < 2 || blocks <= 256 || steps < 16 || steps > 200 * p.splits) return false;
  return !(p.splits > 8 && 2 * steps < 11 * p.splits && blocks >= (p.splits > 32 ? 328 : 368) && blocks < 432);
}

// Partial tiles of a tile: one per pair, and the last of an odd number of ranges by itself.
int weight_grad_planes(const WeightGradPlan& p, int64_t T) { return weight_grad_paired(p, T) ? (p.splits + 1) / 2 : p.splits; }

// Whether one launch takes the whole reduction (nm_wgrad_kernel) rather than ranges of it to many blocks and the sum over them.
// Times in us, least squares over 1230 shapes of 1 to 16000 tokens and 64 to 9000 features (rms 6 and 10 %).  One launch: the steps
// of a tile one after another, in rounds of one tile to a compute unit, and the output.  Two: the steps of a range, in rounds of 512
// blocks, and the partial tiles.  Single ranges, many, on 257 to 431 blocks write them partly under the others' arithmetic (0.85).
// 1.0 us and 5 % are left for the two launches.  With them the one launch takes 0.97 of the time or less wherever it is chosen, and of
// the 28.7 % that always choosing right would save 28.4 are had.  us, two launches and one, near the border: 394 x 256 -> 256 9.1
// and 9.9 (two), 394 x 768 -> 768 13.2 and 9.5; 788 x 256 -> 256 9.9 and 13.3 (two), 788 x 768 -> 768 17.1 and 13.8; 1576 x 768 -> 2304
// 28.3 and 21.0, 3152 x 768 -> 2304 30.3 and 36.9 (two).
bool weight_grad_one_launch(const WeightGradPlan& p, int64_t O, int64_t K, int64_t T) {
  const int64_t steps = (T + TCfg::RS - 1) / TCfg::RS, tiles = (int64_t)p.n_i_tiles * p.n_j_tiles, blocks = tiles * p.splits;
  const int64_t small = ((K + SCfg::BI - 1) / SCfg::BI) * ((O + SCfg::BJ - 1) / SCfg::BJ);
  const bool pair = weight_grad_paired(p, T);
  const double one = 2.8 + (1.66 + 0.325 * (double)steps) * (double)((small + 255) / 256) + 0.009 * (double)small;
  const double rounds = (double)(pair ? ((blocks + 1) / 2 + 255) / 256 : (blocks + 511) / 512);
  double two = 6.4 + 0.59 * (double)((steps + p.splits - 1) / p.splits) * rounds + 0.063 * (double)tiles * weight_grad_planes(p, T);
  if (!pair && p.splits > 8 && blocks > 256) two *= 0.85;
  return one + 1.0 < 0.95 * two;
}

}  // namespace

// Not in the public header, for tests: whether the weight gradient of the shape is one launch.
extern "C" int32_t nm_internal_weight_grad_one_launch(int64_t O, int64_t K, int64_t T) {
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  return p.tiles && weight_grad_one_launch(p, O, K, T);
}

// Not in the public header, for tests: tiles of the weight gradient, ranges of its reduction, and partial tiles of a tile that
// the sum over them reads (fewer than ranges where they are taken in pairs).  0: another kernel takes the shape.
extern "C" int32_t nm_internal_weight_grad_plan(int64_t O, int64_t K, int64_t T, int32_t* ranges, int32_t* planes) {
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  *ranges = p.splits;
  *planes = weight_grad_planes(p, T);
  return p.n_i_tiles * p.n_j_tiles;
}

size_t backward_input_workspace_bytes(int64_t O, int64_t K, int64_t T) {
  bool required = false;
  const size_t need = dense_transposed_workspace_bytes(O, K, T, &required);
  return required ? need : 0;
}
size_t backward_input_scratch_bytes(int64_t O, int64_t K, int64_t T) {
  bool required = false;
  return dense_transposed_workspace_bytes(O, K, T, &required);
}

// A call that is launched by itself takes the host 7.4 to 8.0 us with the two launches and the scratch (5.9 without the scratch on the
// fastest host seen).  A reduction of up to 256 on one round of blocks takes the one kernel less: us a call, one and two, 4 x 256 -> 256
// in float32 7.0 and 7.9, in bfloat16 6.5 and 7.9, 1576 x 256 -> 256 in bfloat16 7.3 and 7.5 (in float32 8.6 and 7.5, which copies);
// at 320 4 tokens in float32 take 7.8 and 7.6.  In a graph only the device counts: 4 x 256 -> 256 7.0 and 5.3.
bool backward_input_scratch_pays(int64_t O, int64_t K, int64_t T, int out_bf16, hipStream_t s) {
  bool required = false;
  if (dense_transposed_workspace_bytes(O, K, T, &required) == 0) return false;
  if (required) return true;
  if (!dense_transposed_pays(O, K, T, out_bf16)) return false;
  const int64_t tiles = ((K + TCfg::BI - 1) / TCfg::BI) * ((T + TCfg::BJ - 1) / TCfg::BJ);
  if (O > 256 || tiles > 256 || !(out_bf16 || T <= 64)) return true;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (s != nullptr && hipStreamIsCapturing(s, &status) != hipSuccess) {
    (void)hipGetLastError();  // (a later launch does not report it)
    status = hipStreamCaptureStatusNone;
  }
  return status == hipStreamCaptureStatusActive;
}

// Not in the public header, for tests: whether dX of aligned operands multiplies a transposed copy where its scratch is brought.
extern "C" int32_t nm_internal_backward_input_copies(int64_t O, int64_t K, int64_t T, int32_t out_bf16) {
  bool required = false;
  return dense_transposed_workspace_bytes(O, K, T, &required) != 0 && (required || dense_transposed_pays(O, K, T, out_bf16 != 0));
}

hipError_t launch_backward_input(const bf16_t* Ws, int64_t O, int64_t K, int64_t ldw, const bf16_t* dY, int64_t T,
                                 int64_t ldy, void* dX, int64_t ldx, int out_bf16, void* workspace,
                                 size_t workspace_bytes, hipStream_t s, bool optional, bool* workspace_short) {
  *workspace_short = false;
  // Large layers: dX = dY * Ws is the forward product of a layer whose weight is Ws^T, so once the weight has
  // been written transposed into stream order (a pass over the weight only) the persistent dense kernel of the
  // forward path computes it.  Small ones whose copy is worth its while take the tiled kernel of that path, where the
  // caller has brought the scratch for it (optional).
  bool required = false;
  const size_t need = dense_transposed_workspace_bytes(O, K, T, &required);
  const bool there = workspace != nullptr && workspace_bytes >= need && aligned_to(workspace, 256);
  if (required && !there) {
    *workspace_short = true;
    return hipSuccess;
  }
  const bool tiles = (O % 32 == 0) && (K % 8 == 0) && (ldw % 8 == 0) && (ldy % 8 == 0) && aligned_to(Ws, 16) &&
                     aligned_to(dY, 16) && K <= (1 << 24) && T <= (1ll << 31) && ldw <= (1 << 22) && ldy <= (1 << 22);
  if (need && there && (required || (optional && (!tiles || dense_transposed_pays(O, K, T, out_bf16))))) {
    bool taken = false;
    hipError_t e = launch_dense_transposed(Ws, O, K, ldw, dY, T, ldy, dX, ldx, out_bf16, workspace, workspace_bytes, s,
                                           &taken);
    if (e != hipSuccess || taken) return e;
  }
  if (!tiles) {
    if (T * K > 0x7FFFFFFFll * 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(backward_input_general_kernel, dim3((unsigned)((T * K + 255) / 256)), dim3(256), 0, s, Ws, O, K, ldw,
                       dY, T, ldy, dX, ldx, out_bf16);
    return hipGetLastError();
  }
  TGemmArgs g;
  g.P = Ws; g.Q = dY; g.I = K; g.J = T; g.R = O; g.ldp = ldw; g.ldq = ldy;
  g.out = dX; g.ldo = ldx; g.out_bf16 = out_bf16;
  const int per_piece = out_bf16 ? 8 : 4;
  g.vec_store = (ldx % per_piece == 0) && aligned_to(dX, 16);  // K % 8 == 0 holds here
  g.n_i_tiles = (int)((K + TCfg::BI - 1) / TCfg::BI);
  g.n_j_tiles = (int)((T + TCfg::BJ - 1) / TCfg::BJ);
  g.splits = 1; g.partial = nullptr;
  return launch_tgemm<false>(g, s);
}

// (of every range, also where pairs leave half of it unused)
size_t backward_weight_workspace_bytes(int64_t O, int64_t K, int64_t T) {
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  if (!p.tiles) return 0;
  return (size_t)p.splits * (size_t)p.n_i_tiles * (size_t)p.n_j_tiles * (size_t)(TCfg::BI * TCfg::BJ) * sizeof(float);
}

// (none where one launch adds the ranges itself)
size_t backward_weight_scratch_bytes(int64_t O, int64_t K, int64_t T) {
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  return p.tiles && weight_grad_one_launch(p, O, K, T) ? 0 : backward_weight_workspace_bytes(O, K, T);
}

// need: bytes of the workspace without which the call is refused (0 only with one_launch)
static hipError_t launch_weight_grad(const WeightGradPlan& p, bool one_launch, size_t need, const bf16_t* dY, int64_t T, int64_t O,
                                     int64_t ldy, const bf16_t* X, int64_t K, int64_t ldx, const uint32_t* mask, void* dW,
                                     int64_t lddw, int out_bf16, void* workspace, size_t workspace_bytes, hipStream_t s,
                                     bool* workspace_short) {
  *workspace_short = false;
  const bool tiles = p.tiles && (ldy % 8 == 0) && (ldx % 8 == 0) && aligned_to(dY, 16) && aligned_to(X, 16) &&
                     ldx <= (1 << 22) && ldy <= (1 << 22);
  if (!tiles) {
    if (O * K > 0x7FFFFFFFll * 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(backward_weight_general_kernel, dim3((unsigned)((O * K + 255) / 256)), dim3(256), 0, s, dY, T, O, ldy,
                       X, K, ldx, mask, dW, lddw, out_bf16);
    return hipGetLastError();
  }
  if (need && (workspace == nullptr || workspace_bytes < need || !aligned_to(workspace, 256))) {
    *workspace_short = true;
    return hipSuccess;
  }
  TGemmArgs g;
  g.P = X; g.Q = dY; g.I = K; g.J = O; g.R = T; g.ldp = ldx; g.ldq = ldy;
  g.out = nullptr; g.ldo = 0; g.out_bf16 = 0; g.vec_store = 0;
  g.n_i_tiles = p.n_i_tiles; g.n_j_tiles = p.n_j_tiles;
  g.splits = p.splits; g.partial = reinterpret_cast<float*>(workspace);
  const bool pair = weight_grad_paired(p, T);
  if (one_launch) {
    g.partial = nullptr;
    g.out = dW; g.ldo = lddw; g.out_bf16 = out_bf16;
    g.vec_store = (lddw % (out_bf16 ? 8 : 4) == 0) && aligned_to(dW, 16);  // K % 8 == 0 holds here
    g.n_i_tiles = (int)((K + SCfg::BI - 1) / SCfg::BI);
    g.n_j_tiles = (int)((O + SCfg::BJ - 1) / SCfg::BJ);
    return pair ? launch_wgrad<true>(g, mask, s) : launch_wgrad<false>(g, mask, s);
  }
  const int planes = weight_grad_planes(p, T);
  hipError_t e = pair ? launch_tgemm<true, true>(g, s) : launch_tgemm<true>(g, s);
  if (e != hipSuccess) return e;
  const int64_t n = (int64_t)p.n_i_tiles * p.n_j_tiles * TCfg::MMA * TCfg::NT;
  hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g.partial, planes,
                     p.n_i_tiles * p.n_j_tiles, p.n_i_tiles, K, O, mask, dW, lddw, out_bf16);
  return hipGetLastError();
}

hipError_t launch_backward_weight(const bf16_t* dY, int64_t T, int64_t O, int64_t ldy, const bf16_t* X, int64_t K,
                                  int64_t ldx, const uint32_t* mask, void* dW, int64_t lddw, int out_bf16, void* workspace,
                                  size_t workspace_bytes, hipStream_t s, bool used_only, bool* workspace_short) {
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  const size_t need = used_only ? backward_weight_scratch_bytes(O, K, T) : backward_weight_workspace_bytes(O, K, T);
  return launch_weight_grad(p, p.tiles && weight_grad_one_launch(p, O, K, T), need, dY, T, O, ldy, X, K, ldx, mask, dW, lddw, out_bf16,
                            workspace, workspace_bytes, s, workspace_short);
}

// Not in the public header, for tests: dW in two launches also where one is chosen.  Arguments as nm_linear_backward_weight has checked
// them; 0, or -1 where the workspace is too small or a launch fails.
extern "C" int32_t nm_internal_weight_grad_two_launches(const bf16_t* dY, int64_t T, int64_t O, int64_t ldy, const bf16_t* X, int64_t K,
                                                        int64_t ldx, const uint32_t* mask, float* dW, int64_t lddw, void* workspace,
                                                        size_t workspace_bytes, hipStream_t s) {
  bool workspace_short = false;
  const WeightGradPlan p = weight_grad_plan(O, K, T);
  const hipError_t e = launch_weight_grad(p, false, backward_weight_workspace_bytes(O, K, T), dY, T, O, ldy, X, K, ldx, mask, dW, lddw, 0,
                                          workspace, workspace_bytes, s, &workspace_short);
  return e == hipSuccess && !workspace_short ? 0 : -1;
}

}  // namespace nm
