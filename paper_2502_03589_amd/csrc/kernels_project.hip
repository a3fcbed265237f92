// QKV generation (Sec. 4, Eq. 1) fused with quantize-on-write (Sec. 5.2 quantizer,
// Sec. 5.3 partitioning), the front half of the paper's prefill kernel (Sec. 6).
//
// The projection is one GEMM: out[token][n] = sum_i E[token][i] W[n][i], where the
// output channels n are the H_q query heads' 128 channels, then the H_kv key heads',
// then the H_kv value heads'.  One workgroup of four or eight 64-lane waves computes a tile
// of one or two heads of 32 to 256 tokens of one sequence (choose_project_tile):
//   main loop  K steps of 32 or 64 input channels through three or four LDS stages (the E
//              rows and the W rows of the step, 16-byte chunks XOR-swizzled so that fragment
//              reads hit distinct banks).  The stages are filled by direct global-to-LDS loads
//              (global_load_lds_dwordx4, 1 KB per wave instruction, no registers) issued two
//              or three steps ahead, so those steps' matrix work covers each load's latency;
//              one barrier per step publishes a stage and frees the one computed before it.
//              The products are v_mfma_f32_32x32x16_f16 (fp32 accumulators); at 256 x 256 a
//              wave computes 128 x 64, so each 16-byte LDS read feeds 21 multiply-adds per
//              lane.  A step of a small tile is a chain of barrier, LDS reads and a few
//              products, so its steps are twice as deep (250 tokens, hidden 4096: 32.9 us
//              with 32 channels a step, 28.3 with 64; one 256 x 256 tile per head pair 106).
//   epilogue   the tile is rounded to fp16 into the stage buffers; then, for each of its
//              heads: a query head is written out in fp16 (the prefill attention
//              quantizes Q itself); a key head is quantized per (token, partition) and a
//              value head per (V block, channel) straight into the cache, with the same
//              quantizer and element indices as hack_quantize, including the fp16 open
//              V block.  The fp16 K and V never reach device memory.
// Tiles are numbered so that the workgroups one XCD runs at a time share their E and
// W tiles (groups of 1024 tokens per channel tile, contiguous ranges per XCD), so
// each slab is fetched into that XCD's L2 once for several workgroups.
#include "hack_internal.hpp"
#include "launch_rules.hpp"

namespace hack {

namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kXcds = 8;          // workgroups are dealt to the XCDs round-robin
constexpr int kGroupTokens = 1024;  // tokens whose tiles share each channel tile in the numbering
typedef __attribute__((address_space(3))) void lvoid;

// One tile shape: BM tokens x BN output channels (one or two heads) by WM x WN waves, in steps
// of BK input channels through NST LDS stages.
template <int BM_, int BN_, int WM_, int WN_, int BK_, int NST_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, BK = BK_, NST = NST_;
  static constexpr int kThreads = 64 * WM * WN;
  static constexpr int kTM = BM / WM / 32, kTN = BN / WN / 32;  // 32x32 products of a wave
  static constexpr int kStageH = (BM + BN) * BK;  // halves per stage: BM E rows, then BN W rows
  static constexpr int kChunks = BK / 8;           // 16-byte chunks of a row
  static constexpr int kRows = 64 / kChunks;       // rows of a 1-KB direct-to-LDS load
  static constexpr int kPieces = (BM + BN) / kRows;  // loads per step
  static constexpr int kDma = kPieces / (WM * WN); // of one wave
  static constexpr int kGroupM = kGroupTokens / BM;
  static_assert(kPieces % (WM * WN) == 0 && NST * kStageH >= BM * BN && (NST - 2) * kDma < 64, "tile shape");
};

// Position of 16-byte chunk c of staged row r: the chunks are XOR-swizzled so that the eight
// rows an LDS cycle reads (32-row fragment reads, eight lanes per cycle) cover all eight
// 16-byte slots of 128 bytes (two rows of 64 bytes, or one of 128).
template <int CHUNKS>
__device__ __forceinline__ int stage_chunk(int r, int c) {
  return CHUNKS == 4 ? c ^ ((r >> 1) & 3) : c ^ (r & 7);
}

// 16 bytes per lane from global memory straight into LDS: lane l reads base + off and
// writes LDS bytes lds + 16 l (base and lds wave-uniform, lds via M0).  Issued as inline
// assembly so that the compiler does not add waits for it before LDS reads of other
// stages; the kernel waits for each stage's loads explicitly (vmcnt) before the barrier
// that publishes it.  The per-lane offset is a register that stays live for the whole
// main loop, so no later instruction (in particular no matrix-core result) overwrites
// an address operand while a load is still in flight.
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}

// Workgroup barrier that orders LDS accesses without waiting for outstanding
// direct-to-LDS loads (a fence would wait for all of them); each wave waits for its
// own loads of a stage explicitly before it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Waits until at most min(MAX, left) steps' loads (N per step) of this wave are in flight.
template <int MAX, int N>
__device__ __forceinline__ void wait_steps(int left) {
  if constexpr (MAX == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (left >= MAX) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX * N) : "memory");
    else wait_steps<MAX - 1, N>(left);
  }
}

__device__ __forceinline__ v16f mfma_f16(v8h a, v8h b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

}  // namespace

template <int BITS, int PI, class Shape>
__global__ __launch_bounds__(Shape::kThreads, 1) void project_kernel(ProjectArgs p) {
  constexpr int kBM = Shape::BM, kBN = Shape::BN, kThreads = Shape::kThreads, kDma = Shape::kDma, kGroupM = Shape::kGroupM;
  constexpr int kBK = Shape::BK, kChunks = Shape::kChunks, kRows = Shape::kRows;
  constexpr int NST = Shape::NST, TM = Shape::kTM, TN = Shape::kTN, kStageH = Shape::kStageH;
  __shared__ __attribute__((aligned(1024))) __half st[NST * kStageH];
  const CacheView& c = p.c;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / Shape::WN, wn = wave % Shape::WN;

  // ---- tile of this workgroup: contiguous ranges per XCD, then groups of kGroupM
  // token tiles sharing each head tile ----
  const int64_t wg = blockIdx.x;
  const int64_t xcd = wg % kXcds, idx = wg / kXcds;
  const int64_t per = p.total / kXcds, rem = p.total % kXcds;
  const int64_t tl = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
  const int64_t mt_all = p.total / p.ntiles;
  const int64_t group = tl / ((int64_t)kGroupM * p.ntiles);
  const int64_t first_m = group * kGroupM;
  const int64_t gsize = min((int64_t)kGroupM, mt_all - first_m);
  const int64_t local = tl - group * kGroupM * p.ntiles;
  const int64_t mtile = first_m + local % gsize;
  const int ntile = (int)(local / gsize);
  const int s = (int)(mtile / p.mtiles);
  const int t0 = (int)(mtile % p.mtiles) * kBM;
  const __half* e_rows = p.e + ((int64_t)s * p.len + t0) * p.hidden;
  const int nrows = p.nheads * 128;  // output channels
  const __half* w_rows = p.w + (int64_t)ntile * kBN * p.hidden;

  // ---- main loop ----
  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  const int nk = p.hidden / kBK;
  const int rows_valid = min(kBM, p.len - t0);
  const int wrows_valid = min(kBN, nrows - ntile * kBN);
  // Direct-to-LDS loads: wave w fills 1-KB pieces q = kDma w + i of a stage (kRows staged
  // rows each, the E rows first), lane l row kRows q + l / kChunks at chunk slot l % kChunks.  Rows past the
  // sequence (or the last head) read the last valid row.
  const uint8_t* gbase[kDma];
  uint32_t goff[kDma];
#pragma unroll
  for (int i = 0; i < kDma; ++i) {
    const int q = kDma * wave + i, r = kRows * q + lane / kChunks;
    const bool is_e = q < kBM / kRows;
    gbase[i] = is_e ? reinterpret_cast<const uint8_t*>(e_rows) : reinterpret_cast<const uint8_t*>(w_rows);
    const int row = is_e ? min(r, rows_valid - 1) : min(r - kBM, wrows_valid - 1);
    goff[i] = (uint32_t)((row * p.hidden + 8 * stage_chunk<kChunks>(r, lane % kChunks)) * 2);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lvoid*)st + 1024u * (uint32_t)(kDma * wave);
  auto load_stage = [&](int stage, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kDma; ++i)
      dma16(gbase[i] + (int64_t)k * kBK * 2, goff[i], lds0 + (uint32_t)(stage * kStageH * 2 + 1024 * i));
  };
  // fragment reads: lane l reads staged row (base + l % 32), chunk 2 kk + l / 32
  const int frow = lane & 31;
  auto compute = [&](int stage) __attribute__((always_inline)) {
    const __half* s0 = st + stage * kStageH;
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      const int ck = 2 * kk + (lane >> 5);
      v8h af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = 32 * TM * wm + 32 * i + frow;
        af[i] = *reinterpret_cast<const v8h*>(s0 + r * kBK + 8 * stage_chunk<kChunks>(r, ck));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int r = kBM + 32 * TN * wn + 32 * j + frow;
        bf[j] = *reinterpret_cast<const v8h*>(s0 + r * kBK + 8 * stage_chunk<kChunks>(r, ck));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_f16(af[i], bf[j], acc[i][j]);
    }
  };
  // step k: wait for this wave's loads of stage k (the loads of the NST - 2 steps after it may
  // stay in flight), barrier (every wave's loads of stage k are in LDS, and every wave is done
  // with step k - 1, whose stage takes step k + NST - 1), then load and compute
#pragma unroll
  for (int i = 0; i < NST - 1; ++i)
    if (i < nk) load_stage(i, i);
  auto step = [&](int k, int stage) __attribute__((always_inline)) {
    wait_steps<NST - 2, kDma>(nk - 1 - k);
    stage_barrier();
    if (k + NST - 1 < nk) load_stage((stage + NST - 1) % NST, k + NST - 1);
    compute(stage);
  };
  for (int ks = 0; ks < nk; ks += NST) {
#pragma unroll
    for (int i = 0; i < NST; ++i)
      if (ks + i < nk) step(ks + i, i);
  }
  stage_barrier();  // every wave is done reading the stages

  // ---- the tile in fp16 (round to nearest even), 128 channels per row, one head after the
  // other ----
  // accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = 32 * TN * wn + 32 * j + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * TM * wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        st[((col >> 7) * kBM + row) * 128 + (col & 127)] = __float2half_rn(acc[i][j][r]);
      }
    }
  __syncthreads();
  const int valid = rows_valid;
  const int Hq = p.q_heads, H = p.kv_heads;
  constexpr int D = 128, P = D / PI;
#pragma unroll 1
  for (int hh = 0; hh < kBN / 128; ++hh) {
    const int head = kBN / 128 * ntile + hh;  // output head: query heads, then key heads, then value heads
    if (head >= p.nheads) break;
    auto tile_row = [&](int row) __attribute__((always_inline)) -> const __half* {
      return st + (hh * kBM + row) * 128;
    };
    if (head < Hq) {
      // query head: 128-channel fp16 rows, 16 bytes per thread and step
      __half* dst = p.q + (((int64_t)s * Hq + head) * p.len + t0) * D;
      for (int i = tid; i < valid * (D / 8); i += kThreads) {
        const int row = i / (D / 8), part = i % (D / 8);
        *reinterpret_cast<uint4*>(dst + (int64_t)row * D + 8 * part) =
            *reinterpret_cast<const uint4*>(tile_row(row) + 8 * part);
      }
    } else if (head < Hq + H) {
      // key head: one thread per (token, partition along the head dimension)
      const int h = head - Hq;
      for (int task = tid; task < valid * P; task += kThreads) {
        const int row = task / P, pp = task % P, t = t0 + row;
        float x[PI];
#pragma unroll
        for (int e = 0; e < PI; e += 8) {
          const uint4 raw = *reinterpret_cast<const uint4*>(tile_row(row) + pp * PI + e);
          const __half2* h2 = reinterpret_cast<const __half2*>(&raw);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float2 f = __half22float2(h2[q]);
            x[e + 2 * q] = f.x;
            x[e + 2 * q + 1] = f.y;
          }
        }
        uint32_t w[(PI * BITS + 31) / 32];
        uint16_t mb, sb;
        const uint32_t sum = quantize_values<BITS, PI>(x, PI, p.stochastic != 0, p.key_k,
                                                       element_index(s, H, h, t, D, pp * PI), 1ull, w, mb, sb);
        const int64_t kr = k_row(c, s, h, t);
        store_codes<BITS, PI>(c.k_codes + kr * (D * BITS / 8) + pp * (PI * BITS / 8), w);
        reinterpret_cast<uint32_t*>(c.k_meta)[kr * P + pp] = (uint32_t)mb | ((uint32_t)sb << 16);
        store_sum(c.k_sums, kr * P + pp, c.sum_bytes, sum);
      }
    } else {
      // value head: one thread per (V block of PI tokens, channel); the open block is
      // quantized with n = T and its fp16 values kept in the open-block buffer
      const int h = head - Hq - H;
      const int F = p.len / PI, T = p.len - F * PI;
      constexpr int NBT = kBM / PI;  // V blocks per tile
      for (int task = tid; task < NBT * D; task += kThreads) {
        const int bl = task / D, ch = task % D;
        const int blk = t0 / PI + bl;
        if (blk > F || (blk == F && T == 0)) continue;
        const int n = blk < F ? PI : T;
        float x[PI];
#pragma unroll
        for (int e = 0; e < PI; ++e) x[e] = e < n ? __half2float(tile_row(bl * PI + e)[ch]) : 0.0f;
        uint32_t w[(PI * BITS + 31) / 32];
        uint16_t mb, sb;
        const uint32_t sum = quantize_values<BITS, PI>(x, n, p.stochastic != 0, p.key_v,
                                                       element_index(s, H, h, blk * PI, D, ch), (uint64_t)D, w, mb, sb);
        const int64_t vb = v_block<PI>(c, s, h, blk * PI);
        store_codes<BITS, PI>(c.v_codes + (vb * D + ch) * (PI * BITS / 8), w);
        reinterpret_cast<uint32_t*>(c.v_meta)[vb * D + ch] = (uint32_t)mb | ((uint32_t)sb << 16);
        store_sum(c.v_sums, vb * D + ch, c.sum_bytes, sum);
        if (blk == F) {
          __half* tail = c.v_tail + (((int64_t)s * H + h) * PI) * D + ch;
          for (int e = 0; e < T; ++e) tail[(int64_t)e * D] = tile_row(bl * PI + e)[ch];
        }
      }
    }
  }
}

template <int BITS, int PI, int INDEX, class Shape>
static hipError_t project_tile(ProjectArgs& a, hipStream_t stream) {
  constexpr ProjectTile t = kProjectTiles[INDEX];
  static_assert(t.bm == Shape::BM && t.bn == Shape::BN && t.threads == Shape::kThreads, "the rule's tile");
  a.mtiles = (a.len + Shape::BM - 1) / Shape::BM;
  a.ntiles = (a.nheads * 128 + Shape::BN - 1) / Shape::BN;
  a.total = project_workgroups(t, a.batch, a.len, a.nheads);
  if (a.total * Shape::kThreads > kMaxLaunchThreads) return hipErrorInvalidValue;
  hipLaunchKernelGGL((project_kernel<BITS, PI, Shape>), dim3((unsigned)a.total), dim3(Shape::kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int BITS, int PI>
static hipError_t project_impl(ProjectArgs& a, hipStream_t stream) {
  switch (choose_project_tile(a.batch, a.len, a.nheads, a.hidden, PI)) {
    case 0:
      if constexpr (PI <= 32) return project_tile<BITS, PI, 0, Tile<32, 128, 1, 4, 64, 4>>(a, stream);
      return hipErrorInvalidValue;
    case 1:
      if constexpr (PI <= 64) return project_tile<BITS, PI, 1, Tile<64, 128, 2, 2, 64, 3>>(a, stream);
      return hipErrorInvalidValue;
    case 2: return project_tile<BITS, PI, 2, Tile<128, 128, 2, 4, 64, 4>>(a, stream);
    case 3: return project_tile<BITS, PI, 3, Tile<256, 128, 4, 2, 64, 3>>(a, stream);
    default: return project_tile<BITS, PI, 4, Tile<256, 256, 2, 4, 32, 4>>(a, stream);
  }
}

hipError_t launch_project(const hack_kv_layout& lay, const ProjectArgs& args, hipStream_t stream) {
  ProjectArgs a = args;
  a.nheads = a.q_heads + 2 * a.kv_heads;
  a.stochastic = lay.rounding == HACK_ROUND_STOCHASTIC;
  a.key_k = lay.seed ^ (1ull << 56);
  a.key_v = lay.seed ^ (2ull << 56);
  switch (lay.kv_bits * 1000 + lay.partition) {
    case 2016: return project_impl<2, 16>(a, stream);
    case 2032: return project_impl<2, 32>(a, stream);
    case 2064: return project_impl<2, 64>(a, stream);
    case 2128: return project_impl<2, 128>(a, stream);
    case 4016: return project_impl<4, 16>(a, stream);
    case 4032: return project_impl<4, 32>(a, stream);
    case 4064: return project_impl<4, 64>(a, stream);
    case 4128: return project_impl<4, 128>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hack
