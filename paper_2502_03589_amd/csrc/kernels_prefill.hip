// Prefill attention on quantized Q/K/V/P (Sec. 5.3 with L_Q = L_KV; Eq. 2-4).
//
// One workgroup of four 64-lane wavefronts per (32 RT query rows, HW query heads of one kv
// group, sequence), HW RT = 4: wave w owns 32 rows of one head.  The workgroup walks the V
// blocks (PI tokens each) up to the causal diagonal:
//   staging  the 256 threads load block kb+1 (packed K and V codes, per-token K and
//            per-channel V metadata) into registers while the waves compute block kb, then
//            write it to the other LDS buffer: codes spread to bytes (packed at partition
//            128), metadata as matrix-core operands (below).
//   S^T = K'Q'^T  v_mfma_i32_32x32x32_i8, per 32-token tile and K partition: A = K codes
//            (lane = token), B = Q codes minus 2^(b-1) quantized in registers in the same
//            channel order (lane = query row).  Token order inside a tile is chosen so that
//            lane (row n, half h) receives PI/32 runs of 16 consecutive tokens, all in half h
//            of the block, and the order inside 16 codes is the one shifts and masks give.
//   Eq. 4    the factors of an integer product form an outer product of a token-side and a
//            row-side vector, so the matrix cores form them in the tile's layout: s_q s_k of
//            a partition by one v_mfma_f32_32x32x16_bf16, the rank-1 terms m~_q s_k sum k~' +
//            R m~_k by another (all sides as bf16 pieces, whose products are exact: as accurate
//            as an fp32 product at any magnitude).  K and V codes are centred (k~' = k' -
//            2^(b-1), m~_k = m_k + 2^(b-1) s_k).  The VALU converts the integer products and
//            takes one fused multiply-add each.
//   softmax  online per row with a lazily raised reference max; causal mask.
//   P        8-bit per (row, V block) with round-to-nearest-even codes; the masked
//            zeros inside the diagonal block are quantized with it.  The lane's codes
//            are already the B operand of the P.V product (no transpose).
//   O^T = V'^T P'^T  the same products with A = V codes (lane = channel), the row side
//            s_p, and (s_p sum p~' + n m~_p, m~_p) against (m_v, s_v sum v').
//   open block  (len mod PI tokens): fp16 products of V with unquantized p in three pieces.
//
// What bounds it: instruction issue.  A wave issues about 680 VALU and 32 matrix instructions
// per 32 x 64 scores (partition 64) at no more than one in four cycles, two waves share a SIMD
// (246 VGPRs), and VALU and matrix cycles of the two overlap only in part (0.79 and 0.30 busy).  Measured against
// the layout before (16 x 16 products, eight waves of 16 rows, row blocks in the fastest grid
// dimension), 32/8 heads: 8192 tokens, 4 bits, partition 64: 1177 -> 773 us; 2 bits, partition
// 128: 1071 -> 577; two prompts of 1999 tokens, 2 bits, partition 32: 452 -> 187 (its 8-byte LDS
// reads conflicted, and half of each 16x16x32 product was idle).  The rank-1 terms as fp32
// products (64 matrix cycles each, half as many in bf16) took 817, 617 and 204 us; with codes
// counted from the partition's minimum they were several times the score and bf16 pieces lost
// precision, with centred codes the error is lower than either (a row's median error against
// 64 bits at 1500 tokens 1.7e-6 -> 5.3e-7 of its norm).
#include <type_traits>

#include "hack_internal.hpp"
#include "launch_rules.hpp"

namespace hack {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

namespace {

constexpr int kWaveRows = 32;    // query rows per wave
constexpr int kGroupThreads = 256;  // four waves: they share the K and V of a staged block
constexpr float kScale = 0.12751743074941640f;  // log2(e) / sqrt(128)
constexpr float kSlack = 8.0f;   // reference max raised only beyond this (log2 units)

template <int BITS, int PI>
struct PrefillCfg {
  static constexpr int D = 128;
  static constexpr int P = D / PI;        // K partitions per token
  static constexpr int NT = PI / 32;      // 32-token tiles per block
  static constexpr int SW = BITS / 2;     // dwords of 16 packed codes
  static constexpr int KWD = PI * BITS / 64;  // dwords of half a partition (K) or half a block (V)
  // Codes enter the products centred, as (code - kCentre) kUnit: the top BITS of a signed byte
  // (the code's high bit flipped).  Around a partition's middle instead of its minimum the
  // rank-1 terms are about a tenth of the score, so their rounding no longer sets its error.
  static constexpr int kCentre = 1 << (BITS - 1), kUnit = 1 << (8 - BITS);
  static constexpr uint32_t kFlip = BITS == 2 ? 0xAAAAAAAAu : 0x88888888u;
  // LDS row strides of the packed codes (bytes).  A lane reads one 16-byte vector (or less)
  // per row half; the pads give the 8 lanes of an LDS cycle distinct 16-byte slots.
  // Codes are spread to bytes on their way into LDS at partitions 32 and 64 (each wave would
  // otherwise spend a tenth of its instructions on shifts and masks); at 128 two workgroups'
  // stages of bytes do not fit a compute unit, and every wave unpacks what it reads.
  static constexpr bool BYTES = PI < 128;
  static constexpr int VB = PI * BITS / 8;
  static constexpr int KHALF = BYTES ? 64 : 8 * BITS;      // bytes of one half of a K row
  static constexpr int VHALF = BYTES ? PI / 2 : VB / 2;    // and of a V row
  static constexpr int KROW = 2 * KHALF + 16;
  static constexpr int VROW = BYTES ? PI + 16 : (VB == 64 ? 80 : VB + VB / 2);
};

// LDS of one staged V block.  K rows are in tile order: row 32 st + i holds the token that
// row i of the tile's product stands for (tile_pos); each row holds the two halves of every
// partition's channels apart: [half][partition].
template <int BITS, int PI>
struct Stage {
  using C = PrefillCfg<BITS, PI>;
  uint8_t k[PI * C::KROW];
  uint8_t v[128 * C::VROW];
  u32x4 ks[C::P][PI];      // scale operand: s_k
  u32x4 vs[128];           // scale operand: s_v
  u32x4 kr[C::P][2][PI];   // rank-1 operand of (partition, half, row): m~_k | s_k sum k~'
  u32x4 vr[2][128];        // rank-1 operand of (half, channel): m~_v | s_v sum v~'
};

__device__ __forceinline__ v16i mfma_i8(v4i a, v4i b, v16i c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v16f mfma_bf16(u32x4 a, u32x4 b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}
__device__ __forceinline__ v16f mfma_f16(u32x4 a, u32x4 b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}
__device__ __forceinline__ v16f zero16() {
  v16f z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

// Row of a 32x32 product held by register r of lane half h.
__device__ __forceinline__ constexpr int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }
// LDS row of token t of a block: tile 32 st + i, where the tokens of half h of the block are
// the rows of lane half h in register order (token h PI/2 + 16 st + r).
template <int PI>
__device__ __forceinline__ int tile_pos(int t) {
  const int h = t / (PI / 2), u = t % (PI / 2);
  return 32 * (u >> 4) + acc_row(u & 15, h);
}

// Two floats rounded to bf16, one dword.
typedef __bf16 v2b __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{lo, hi}), v2b));
}
// x as three bf16 values x1 + x2 + x3 (exact; the last two remainders are exact in fp32).
// Rounded, not cut (cut_bf16): x2 and x3 are half as large and of either sign, which the scale
// products' error below rests on.  The rank-1 products take all products of their pieces but the
// smallest, so truncation, one instruction a piece instead of three, serves them as well.
struct Pieces {
  float x1, x2, x3;
};
__device__ __forceinline__ Pieces split_bf16(float x) {
  Pieces p;
  p.x1 = __uint_as_float(pack_bf16(x, x) & 0xFFFF0000u);
  const float r = x - p.x1;
  p.x2 = __uint_as_float(pack_bf16(r, r) & 0xFFFF0000u);
  p.x3 = r - p.x2;
  return p;
}

// Operands of the scale products, eight k slots in each lane half: every product of the
// pieces of x (three) and of y, an fp16 value (two).  The matrix core adds the eight products
// of a half at the precision of the largest, so the large ones are in half 0 and the small
// ones in half 1 (rms error against 64 bits 0.42 units of 2^-24; all in one half 0.82).
// (x1 y1, x1 y2) | (x2 y1, x2 y2, x3 y1, x3 y2).
__device__ __forceinline__ u32x4 row_scale(float x, int half) {
  const Pieces p = split_bf16(x);
  const float a = half ? p.x2 : p.x1, b = half ? p.x3 : 0.0f;
  return u32x4{pack_bf16(a, a), pack_bf16(b, b), 0u, 0u};
}
__device__ __forceinline__ u32x4 token_scale(float y) {
  const float y1 = __uint_as_float(pack_bf16(y, y) & 0xFFFF0000u);
  const uint32_t d = pack_bf16(y1, y - y1);
  return u32x4{d, d, d, d};
}
// Operands of the rank-1 products, one term in each lane half: both factors cut into three
// bf16 values (x1 + x2 + x3 exactly, eight bits each), all their products but x3 y3 (2^-28).
// (x1 y1, x1 y2, x2 y1, x2 y2, x1 y3, x3 y1, x2 y3, x3 y2).
struct Cut {
  uint32_t x, r, t;  // x1, x2, x3 in the upper halves
};
__device__ __forceinline__ Cut cut_bf16(float x) {
  const float r = x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
  const float t = r - __uint_as_float(__float_as_uint(r) & 0xFFFF0000u);
  return Cut{__float_as_uint(x), __float_as_uint(r), __float_as_uint(t)};
}
__device__ __forceinline__ uint32_t upper_halves(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}
__device__ __forceinline__ u32x4 row_rank(float x) {
  const Cut c = cut_bf16(x);
  return u32x4{upper_halves(c.x, c.x), upper_halves(c.r, c.r), upper_halves(c.x, c.t), upper_halves(c.r, c.t)};
}
__device__ __forceinline__ u32x4 token_rank(float y) {
  const Cut c = cut_bf16(y);
  const uint32_t y12 = upper_halves(c.x, c.r);
  return u32x4{y12, y12, upper_halves(c.t, c.x), upper_halves(c.t, c.r)};
}
// 16 packed codes with their high bits flipped -> 16 int8 lanes of an operand; operand byte b
// of dword q is element code_element<BITS>(q, b).
template <int BITS>
__device__ __forceinline__ v4i unpack16(const uint32_t* w) {
  if constexpr (BITS == 2) {
    const uint32_t x = w[0];
    return v4i{(int)((x << 6) & 0xC0C0C0C0u), (int)((x << 4) & 0xC0C0C0C0u), (int)((x << 2) & 0xC0C0C0C0u),
               (int)(x & 0xC0C0C0C0u)};
  } else {
    const uint32_t x = w[0], y = w[1];
    return v4i{(int)((x << 4) & 0xF0F0F0F0u), (int)(x & 0xF0F0F0F0u), (int)((y << 4) & 0xF0F0F0F0u),
               (int)(y & 0xF0F0F0F0u)};
  }
}
template <int BITS>
__device__ __forceinline__ constexpr int code_element(int q, int b) {
  return BITS == 2 ? 4 * b + q : 8 * (q >> 1) + 2 * b + (q & 1);
}

// N dwords (1, 2, 4 or 8) from or to an address aligned to min(4 N, 16) bytes.
template <int N>
__device__ __forceinline__ void get_words(const uint8_t* p, uint32_t* w) {
  if constexpr (N == 1) {
    w[0] = *reinterpret_cast<const uint32_t*>(p);
  } else if constexpr (N == 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    w[0] = v.x; w[1] = v.y;
  } else {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const uint4 v = reinterpret_cast<const uint4*>(p)[i];
      w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
    }
  }
}
template <int N>
__device__ __forceinline__ void put_words(uint8_t* p, const uint32_t* w) {
  if constexpr (N == 1) {
    *reinterpret_cast<uint32_t*>(p) = w[0];
  } else if constexpr (N == 2) {
    *reinterpret_cast<uint2*>(p) = uint2{w[0], w[1]};
  } else {
#pragma unroll
    for (int i = 0; i < N / 4; ++i)
      reinterpret_cast<uint4*>(p)[i] = uint4{w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]};
  }
}

// N operands of 16 codes each from a staged row.
template <int BITS, bool BYTES, int N>
__device__ __forceinline__ void load_codes(const uint8_t* p, v4i* x) {
  if constexpr (BYTES) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int4 w = reinterpret_cast<const int4*>(p)[i];
      x[i] = v4i{w.x, w.y, w.z, w.w};
    }
  } else {
    uint32_t w[N * BITS / 2];
    get_words<N * BITS / 2>(p, w);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = unpack16<BITS>(w + i * (BITS / 2));
  }
}

// Max / min / sum over the two lane halves (lanes l, l^32).
__device__ __forceinline__ float xh_max(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float xh_min(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float xh_sum(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ __forceinline__ int xh_sum_i(int x) {
  const auto a = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  return (int)a[0] + (int)a[1];
}

struct PrefillArgs {
  CacheView c;
  const __half* q;   // [B][H_q][L][128]
  float* out;        // [B][H_q][L][128]
  int num_q_heads;
  int group;
  int head_groups;   // workgroups per (kv head, row block): ceil(group / HW)
  int hw_log2;       // log2 of HW, the heads of a workgroup (4, 2 or 1); it takes 4 / HW row tiles
  int len;
  int causal;
  int nqb;           // row blocks of 32 * 4 / HW rows
  int batch;
  int grid_x, workgroups;  // workgroup index = x + y grid_x, below workgroups
  float qmax;        // 2^b_QP - 1 of the transient Q and P codes (15 or 255)
  float inv_qmax;    // 1 / qmax
  int qoff;          // Q codes enter the signed int8 MFMA as code - qoff, qoff = 2^(b_QP - 1)
  float qoff_f;
  // P codes enter as code - poff: 128 at 8 bits (bit 7 flipped, pflip), 0 at 4 bits.  A shift
  // before the rounding (to 120 + code, one flip for both widths) rounded at an ulp of 1.5e-5
  // and so took codes that close to a tie the other way.
  int poff;
  float poff_f;
  uint32_t pflip;
  uint64_t key_q, key_p;  // stochastic rounding of the Q and P codes (streams 3 and 4)
};

// Bytes of one cached code sum: 1 when b + log2(PI) <= 8, else 2 (Sec. 5.3).
template <int BITS, int PI>
constexpr int sum_bytes() {
  int need = BITS;
  for (int v = 1; v < PI; v <<= 1) ++need;
  return need <= 8 ? 1 : 2;
}

// One block on its way to LDS: a thread holds half a partition of K codes of one token, half
// a block of V codes of one channel, and the metadata of one (token, partition) (threads
// 0-127) or channel (threads 128-255).
template <int BITS, int PI>
struct StageRegs {
  using C = PrefillCfg<BITS, PI>;
  uint32_t k[C::KWD], v[C::KWD];
  uint32_t meta, sum;

  // Section bases of the block are wave-uniform; each thread adds a 32-bit offset.
  __device__ __forceinline__ void load(const CacheView& c, int64_t page, int hkv, int slot0, bool with_v) {
    constexpr int P = C::P, SB = sum_bytes<BITS, PI>();
    const int tid = threadIdx.x % kGroupThreads;
    const int64_t krow0 = (page * c.kv_heads + hkv) * c.page_tokens + slot0;
    const int64_t vb = (page * c.kv_heads + hkv) * (c.page_tokens / PI) + slot0 / PI;
    uint32_t off = (uint32_t)(tid * C::KWD * 4);
    get_words<C::KWD>(c.k_codes + krow0 * (C::D * BITS / 8) + off, k);
    if (with_v) {
      get_words<C::KWD>(c.v_codes + vb * (C::D * C::VB) + off, v);
    } else {
#pragma unroll
      for (int i = 0; i < C::KWD; ++i) v[i] = 0u;
    }
    meta = 0u;
    sum = 0u;
    const uint32_t e = (uint32_t)tid & 127u;
    if (tid < 128) {
      meta = reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(c.k_meta) + krow0 * (P * 4))[e];
      const uint8_t* z = c.k_sums + krow0 * (P * SB);
      sum = SB == 1 ? (uint32_t)z[e] : (uint32_t)reinterpret_cast<const uint16_t*>(z)[e];
    } else if (with_v) {
      meta = reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(c.v_meta) + vb * (C::D * 4))[e];
      const uint8_t* z = c.v_sums + vb * (C::D * SB);
      sum = SB == 1 ? (uint32_t)z[e] : (uint32_t)reinterpret_cast<const uint16_t*>(z)[e];
    }
  }

  static __device__ __forceinline__ void put_codes(uint8_t* dst, const uint32_t* packed) {
    uint32_t w[C::KWD];
#pragma unroll
    for (int i = 0; i < C::KWD; ++i) w[i] = packed[i] ^ C::kFlip;
    if constexpr (C::BYTES) {
#pragma unroll
      for (int i = 0; i < C::KWD / C::SW; ++i) {
        const v4i x = unpack16<BITS>(w + i * C::SW);
        reinterpret_cast<int4*>(dst)[i] = int4{x[0], x[1], x[2], x[3]};
      }
    } else {
      put_words<C::KWD>(dst, w);
    }
  }
  __device__ __forceinline__ void store(Stage<BITS, PI>& st) const {
    constexpr int P = C::P;
    const int tid = threadIdx.x % kGroupThreads;
    // K: thread -> (token, partition, half of its channels)
    const int tt = tid / (2 * P), piece = tid % (2 * P);
    put_codes(st.k + tile_pos<PI>(tt) * C::KROW + (piece & 1) * C::KHALF + (piece >> 1) * (C::KHALF / P), k);
    // V: thread -> (channel, half of the block's tokens)
    put_codes(st.v + (tid >> 1) * C::VROW + (tid & 1) * C::VHALF, v);
    const float m = __half2float(__ushort_as_half((uint16_t)(meta & 0xFFFFu)));
    const float s = __half2float(__ushort_as_half((uint16_t)(meta >> 16)));
    const int e = tid & 127;
    const bool is_k = tid < 128;
    const int kp = e % P, kt = tile_pos<PI>(e / P);
    u32x4* r0 = is_k ? &st.kr[kp][0][kt] : &st.vr[0][e];
    u32x4* r1 = is_k ? &st.kr[kp][1][kt] : &st.vr[1][e];
    u32x4* sc = is_k ? &st.ks[kp][kt] : &st.vs[e];
    *r0 = token_rank(fmaf((float)C::kCentre, s, m));
    *r1 = token_rank(s * (float)((int)sum - C::kCentre * PI));  // exact: 11 significant bits times an integer below 2^11
    *sc = token_scale(s * (1.0f / C::kUnit));
  }
};

}  // namespace

// Two waves per SIMD (256 VGPRs): the 32 rows of a wave hold 64 registers of O and PI/2 of
// scores, and their products are long enough (32 matrix cycles each) that two waves cover
// each other's dependences.
// SR: the Q and P codes are rounded stochastically (the layout's rounding mode).
// KG: key groups of four waves; group g of a workgroup takes the V blocks kb = g mod KG of the
// same rows, with stages of its own, and group 0 merges the groups' (max, sum, O) at the end.
// Two groups halve the longest chain of blocks (launch_prefill).
template <int BITS, int PI, bool SR, int KG>
__global__ __launch_bounds__(kGroupThreads* KG, 2) void prefill_kernel(PrefillArgs a) {
  using C = PrefillCfg<BITS, PI>;
  constexpr int D = 128, P = C::P, NT = C::NT;
  constexpr int NJ = PI / 32;  // 32-channel products per K partition

  __shared__ __attribute__((aligned(16))) Stage<BITS, PI> all_stages[KG][2];
  static_assert(KG == 1 || sizeof(all_stages) >= 4 * 66 * 64 * 4, "the merge takes 66 floats a lane of one group");

  const CacheView& c = a.c;
  const int tid = threadIdx.x;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wave = wave_all % 4, kg = KG == 1 ? 0 : wave_all / 4;
  Stage<BITS, PI>(&stages)[2] = all_stages[kg];
  const int col = lane & 31, half = lane >> 5;
  // Workgroups are numbered with the heads fastest, then the sequences, then the row blocks
  // (causal: the longest first).  All long rows start before any short ones, so none is left
  // to run alone at the end (row blocks fastest: 952 us for 8192 tokens, 1.4 waves per SIMD
  // resident), and with a multiple of eight heads an XCD's L2 sees one kv head's blocks.
  const int nh = c.kv_heads * a.head_groups;
  const int wg = (int)blockIdx.y * a.grid_x + (int)blockIdx.x;
  if (wg >= a.workgroups) return;
  const int hk = wg % nh, sq_qb = wg / nh;
  const int hkv = hk % c.kv_heads, hg = hk / c.kv_heads;
  const int s = sq_qb % a.batch;
  const int hw = 1 << a.hw_log2;
  const int qb = a.causal ? a.nqb - 1 - sq_qb / a.batch : sq_qb / a.batch;
  const int wg_rows = kWaveRows * (4 >> a.hw_log2);
  const int L = a.len;
  const int gh = hg * hw + (wave & (hw - 1));
  const int r0 = qb * wg_rows + kWaveRows * (wave >> a.hw_log2);  // this wave's first row
  const bool live = gh < a.group && r0 < L;
  const int hq = hkv * a.group + (gh < a.group ? gh : 0);
  const int row = r0 + col;  // this lane's query row
  const int F = L / PI, T = L - F * PI;
  const int nblk_q = F + (T > 0 ? 1 : 0);
  const int last_row = min(qb * wg_rows + wg_rows, L) - 1;
  const int nblk = a.causal ? min(nblk_q, last_row / PI + 1) : nblk_q;

  // page of block kb: a scalar load, requested one block before the block's loads need it
  auto page_entry = [&](int kb) __attribute__((always_inline)) -> int {
    if (c.block_table == nullptr) return s;
    const auto* bt = (const __attribute__((address_space(4))) int32_t*)(uintptr_t)c.block_table;
    return bt[(int64_t)s * c.mbps + kb * PI / c.page_tokens];
  };
  auto stage_load = [&](StageRegs<BITS, PI>& sr, int kb, int entry) __attribute__((always_inline)) {
    const int64_t page = entry < 0 ? 0 : (entry >= c.num_pages ? c.num_pages - 1 : (int64_t)entry);
    const int slot0 = c.block_table == nullptr ? kb * PI : kb * PI % c.page_tokens;
    sr.load(c, page, hkv, slot0, kb < F);
  };
  StageRegs<BITS, PI> sr;
  if (kg < nblk) stage_load(sr, kg, page_entry(kg));
  int next_page = kg + KG < nblk ? page_entry(kg + KG) : 0;

  // ---- Q row: codes per partition (float32 metadata), in MFMA operand layout: this lane
  // holds channels [p PI + half PI/2, + PI/2) of each partition p ----
  v4i qop[P][NJ];
  // Partition 128 has no register left at 4 bits or with stochastic codes; its rank-1 operand is
  // rebuilt for every tile from one (two prompts of 1999 tokens, 32/8 heads: 4 bits 103.2 us with
  // the operand kept, 98.8 rebuilt; 2 bits stochastic 223.3 and 219.2; but 2 bits to nearest,
  // 246 to 252 registers, 91.1 and 93.2).  Left in scratch: four to six registers at 4 bits to
  // nearest, all but one reload of them outside the block loop.
  constexpr bool kRebuild = PI == 128 && (BITS == 4 || SR);
  float rank_f[P];
  u32x4 rank_b[P], scale_b[P];
  {
    const bool rv = live && row < L;
    const __half* qrow = a.q + (((int64_t)s * a.num_q_heads + hq) * L + (rv ? row : 0)) * D;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      constexpr int N = PI / 2;
      const int c0 = p * PI + half * N;
      float x[N];
#pragma unroll
      for (int e = 0; e < N; e += 8) {
        uint4 raw = uint4{0u, 0u, 0u, 0u};
        if (rv) raw = *reinterpret_cast<const uint4*>(qrow + c0 + e);
        const __half2* h2 = reinterpret_cast<const __half2*>(&raw);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 f = __half22float2(h2[i]);
          x[e + 2 * i] = f.x;
          x[e + 2 * i + 1] = f.y;
        }
      }
      float mn = x[0], mx = x[0];
#pragma unroll
      for (int e = 1; e < N; ++e) {
        mn = fminf(mn, x[e]);
        mx = fmaxf(mx, x[e]);
      }
      mn = xh_min(mn);
      mx = xh_max(mx);
      int csum = 0;
      float s32;
      {
#pragma clang fp contract(off)
        s32 = __fdiv_rn(__fsub_rn(mx, mn), a.qmax);
        const float r = s32 != 0.0f ? __fdiv_rn(1.0f, s32) : 0.0f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const int e = 16 * j + code_element<BITS>(q, b);
              const float t = __fmul_rn(__fsub_rn(x[e], mn), r);
              int code = 0;
              // Stochastic: on every lane (t = 0 and so the code is 0 where s32 = 0).  A branch a
              // value that leaves few rows in it lowers the clock (36 tokens: 25.2 us; all: 15.1).
              if constexpr (SR) {
                const float u = sr_threshold(a.key_q, qp_index(s, a.num_q_heads, hq, row, c0 + e));
                code = (int)round_stochastic(t, u, a.qmax);
              } else if (s32 != 0.0f) {
                code = (int)fminf(rintf(t), a.qmax);
              }
              csum += code;
              v |= (uint32_t)((code - a.qoff) & 0xFF) << (8 * b);
            }
            qop[p][j][q] = (int)v;
          }
      }
      csum = xh_sum_i(csum);
      // Eq. 4 coefficients in log2 units: s_q, m~_q = m_q + qoff s_q, R = s_q sum q' + n m_q
      const float sq = kScale * s32;
      const float mq = kScale * (mn + a.qoff_f * s32);
      const float rq = kScale * (s32 * (float)csum + (float)PI * mn);
      rank_f[p] = half ? mq : rq;
      rank_b[p] = row_rank(rank_f[p]);
      scale_b[p] = row_scale(sq, half);
    }
  }

  float m_ref = -INFINITY, l_run = 0.0f;
  v16f o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = zero16();

  if (kg < nblk) sr.store(stages[0]);
  __syncthreads();

  // One V block: quantized blocks run in the main loop; the fp16 open block (at most
  // one, the last) runs after it, so the loop body holds no branch on the block kind.
  auto block = [&](const int kb, const Stage<BITS, PI>& st, auto tail_tag) __attribute__((always_inline)) {
    constexpr bool is_tail = decltype(tail_tag)::value;  // the fp16 open block
    const int tb0 = kb * PI;

    if (live && !(a.causal && tb0 > r0 + kWaveRows - 1)) {
      // ---------------- S^T tiles and Eq. 4 (lane: row `row`, tokens half PI/2 + 16 t + r) ----------------
      v16f sv[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int kr = 32 * t + col;
        v4i kx[4];
        load_codes<BITS, C::BYTES, 4>(st.k + kr * C::KROW + half * C::KHALF, kx);
        v16f acc = zero16();
#pragma unroll
        for (int p = 0; p < P; ++p) {
          if constexpr (kRebuild) {
            float x = rank_f[p];
            asm volatile("" : "+v"(x));
            acc = mfma_bf16(st.kr[p][half][kr], row_rank(x), acc);
          } else {
            acc = mfma_bf16(st.kr[p][half][kr], rank_b[p], acc);
          }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const v16f sc = mfma_bf16(st.ks[p][kr], scale_b[p], zero16());
          v16i ci;
#pragma unroll
          for (int r = 0; r < 16; ++r) ci[r] = 0;
#pragma unroll
          for (int j = 0; j < NJ; ++j) ci = mfma_i8(kx[p * NJ + j], qop[p][j], ci);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[r] = fmaf(sc[r], (float)ci[r], acc[r]);
        }
        sv[t] = acc;
      }
      // The scores are complete before the branch below (the compiler would otherwise copy
      // their last multiply-adds into both of its sides, and spill).
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(sv[t][r]));
      // masking is needed only in the block holding the length or this wave's diagonal
      if (is_tail || tb0 + PI > L || (a.causal && tb0 + PI - 1 > r0)) {
        const int last = (a.causal ? min(row, L - 1) : L - 1) - tb0 - half * (PI / 2);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) sv[t][r] = 16 * t + r > last ? -INFINITY : sv[t][r];
      }

      // ---------------- softmax and P codes ----------------
      float bmax = sv[0][0], bmin = sv[0][0];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          bmax = fmaxf(bmax, sv[t][r]);
          bmin = fminf(bmin, sv[t][r]);
        }
      bmax = xh_max(bmax);
      if (bmax > m_ref + kSlack || (m_ref == -INFINITY && bmax > -INFINITY)) {  // raise the reference max
        const float alpha = __builtin_amdgcn_exp2f(m_ref - bmax);
        l_run *= alpha;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] *= alpha;
        m_ref = bmax;
      }
      float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // four chains: a dependent add issues at a quarter of the rate
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sv[t][r] = __builtin_amdgcn_exp2f(sv[t][r] - m_ref);  // masked: exp2(-inf) = 0
          ls[r & 3] += sv[t][r];
        }
      l_run += (ls[0] + ls[1]) + (ls[2] + ls[3]);

      if constexpr (!is_tail) {
        bmin = xh_min(bmin);
        const float pmax = bmax > -INFINITY ? __builtin_amdgcn_exp2f(bmax - m_ref) : 0.0f;
        const float pmin = bmin > -INFINITY ? __builtin_amdgcn_exp2f(bmin - m_ref) : 0.0f;
        const float dp = pmax - pmin;
        const float r = dp > 0.0f ? a.qmax * __builtin_amdgcn_rcpf(dp) : 0.0f;
        const float bias = -pmin * r;
        v4i pop[NT];
        uint32_t zsum = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const int e = code_element<BITS>(q, b);
              if constexpr (SR) {
                const int tok = tb0 + half * (PI / 2) + 16 * t + e;
                const float u = sr_threshold(a.key_p, qp_index(s, a.num_q_heads, hq, row, tok));
                v = __builtin_amdgcn_cvt_pk_u8_f32(round_stochastic(fmaf(sv[t][e], r, bias), u, a.qmax), b, v);
              } else {
                v = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(sv[t][e], r, bias), b, v);
              }
            }
            zsum = __builtin_amdgcn_sad_u8(v, 0u, zsum);
            pop[t][q] = (int)(v ^ a.pflip);
          }
        const float ps = dp * a.inv_qmax;        // s_p
        const float pm = pmin + a.poff_f * ps;   // m~_p
        const float pz = ps * (float)(xh_sum_i((int)zsum) - a.poff * PI);  // s_p * sum p~'
        const u32x4 rb = row_rank(half ? pm : fmaf((float)PI, pm, pz));
        const u32x4 sb = row_scale(ps, half);

        // ---------------- O^T += V'^T P'^T with Eq. 4 (lane: row, channels 32 j + acc_row) ----------------
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int ch = 32 * j + col;  // channel of this lane's A-operand row
          v4i vx[NT];
          load_codes<BITS, C::BYTES, NT>(st.v + ch * C::VROW + half * C::VHALF, vx);
          o[j] = mfma_bf16(st.vr[half][ch], rb, o[j]);
          const v16f sc = mfma_bf16(st.vs[ch], sb, zero16());
          v16i ci;
#pragma unroll
          for (int i = 0; i < 16; ++i) ci[i] = 0;
#pragma unroll
          for (int t = 0; t < NT; ++t) ci = mfma_i8(vx[t], pop[t], ci);
#pragma unroll
          for (int i = 0; i < 16; ++i) o[j][i] = fmaf(sc[i], (float)ci[i], o[j][i]);
        }
      } else {
        // fp16 open block: O[row][ch] += sum_{t < T} p[row][t] v_t[ch] with unquantized p as
        // three fp16 pieces under a factor 2^7 (p <= 2^8): exact to 2^-32 of p's scale.
        // One tile's pieces at a time, and V rows by clamped index: the pieces of four tiles
        // (partition 128) do not fit beside O, and a branch around each load made its wave wait
        // for the load before (64 prompts of 60 tokens, 4 bits, partition 64: 63.7 -> 45.8 us;
        // 100 tokens, 2 bits, 128: 29.3 -> 21.8).
        // An infinite V value enters once, times whether the row gives the token weight: a
        // piece of p may be zero where p is not, and infinity times that would be NaN.
        const __half* vt = c.v_tail + (((int64_t)s * c.kv_heads + hkv) * PI) * D;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (16 * t >= T) break;
          u32x4 pb[2][3];
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                float x = sv[t][8 * g + 2 * i + e] * 128.0f;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                  const __half h = __float2half_rn(x);
                  x -= __half2float(h);
                  w[k] |= (uint32_t)__half_as_ushort(h) << (16 * e);
                }
              }
#pragma unroll
              for (int k = 0; k < 3; ++k) pb[g][k][i] = w[k];
            }
#pragma unroll 1
          for (int jj = 0; jj < 4; ++jj) {
            u32x4 av[2];
            uint32_t nonzero = 0u;  // sum of 0 v: zero unless some v is infinite
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              const int tk = half * (PI / 2) + 16 * t + 8 * g;
              av[g] = u32x4{0u, 0u, 0u, 0u};
              if (16 * t + 8 * g < T) {
                uint32_t x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = __half_as_ushort(vt[min(tk + i, T - 1) * D + 32 * jj + col]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  av[g][i] = (tk + 2 * i < T ? x[2 * i] : 0u) | (tk + 2 * i + 1 < T ? x[2 * i + 1] << 16 : 0u);
                  asm volatile("v_pk_fma_f16 %0, %1, 0, %0" : "+v"(nonzero) : "v"(av[g][i]));
                }
              }
            }
            v16f acc = zero16();
            if (__builtin_amdgcn_ballot_w64(nonzero != 0u) != 0) {
#pragma unroll
              for (int g = 0; g < 2; ++g) {
                u32x4 inf, one;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const uint32_t w = av[g][i];
                  const uint32_t m = ((w & 0x7C00u) == 0x7C00u ? 0xFFFFu : 0u) |
                                     ((w & 0x7C000000u) == 0x7C000000u ? 0xFFFF0000u : 0u);
                  inf[i] = w & m;
                  av[g][i] = w & ~m;
                  one[i] = (sv[t][8 * g + 2 * i] > 0.0f ? 0x3C00u : 0u) |
                           (sv[t][8 * g + 2 * i + 1] > 0.0f ? 0x3C000000u : 0u);
                }
                acc = mfma_f16(inf, one, acc);
              }
            }
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
              for (int k = 2; k >= 0; --k) acc = mfma_f16(av[g], pb[g][k], acc);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (j == jj) {
#pragma unroll
                for (int i = 0; i < 16; ++i) o[j][i] = fmaf(acc[i], 0x1p-7f, o[j][i]);
              }
          }
        }
      }
    }
  };
  const int nq = min(nblk, F), iters = (nblk + KG - 1) / KG;
#pragma unroll 1
  for (int it = 0; it < iters; ++it) {
    const int kb = KG * it + kg;
    const bool next = kb + KG < nblk;
    if (next) {
      stage_load(sr, kb + KG, next_page);
      if (kb + 2 * KG < nblk) next_page = page_entry(kb + 2 * KG);
    }
    if (kb < nq) block(kb, stages[it & 1], std::false_type{});
    if (next) sr.store(stages[(it + 1) & 1]);
    __syncthreads();  // stage of iteration it + 1 complete; stage of it free for it + 2
  }
  // the open block is some group's block of the last iteration, in a stage still intact
  if (nblk > nq && (KG == 1 || nq % KG == kg)) block(nq, stages[(iters - 1) & 1], std::true_type{});

  float lsum = xh_sum(l_run);
  if constexpr (KG > 1) {
    // merge: group 1 leaves (max, sum, O) per lane in LDS, group 0 weighs the two.  A group
    // without a block has max -inf and sum 0.
    static_assert(KG <= 2, "one group's records fit");
    float* rec = reinterpret_cast<float*>(all_stages) + wave * (66 * 64) + lane;
    __syncthreads();  // every group is done with its stages
    if (kg == 1) {
      rec[0] = m_ref;
      rec[64] = lsum;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) rec[(2 + 16 * j + i) * 64] = o[j][i];
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = rec[0], m = fmaxf(m_ref, m1);
    const float w0 = m_ref > -INFINITY ? __builtin_amdgcn_exp2f(m_ref - m) : 0.0f;
    const float w1 = m1 > -INFINITY ? __builtin_amdgcn_exp2f(m1 - m) : 0.0f;
    lsum = fmaf(lsum, w0, rec[64] * w1);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[j][i] = fmaf(o[j][i], w0, rec[(2 + 16 * j + i) * 64] * w1);
  }
  // ---- normalize and write O[row][32 j + acc_row] ----
  if (live && row < L) {
    const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
    float* dst = a.out + (((int64_t)s * a.num_q_heads + hq) * L + row) * D;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<float4*>(dst + 32 * j + acc_row(4 * i, half)) =
            float4{o[j][4 * i] * inv, o[j][4 * i + 1] * inv, o[j][4 * i + 2] * inv, o[j][4 * i + 3] * inv};
  }
}

template <int BITS, int PI>
static hipError_t prefill_impl(PrefillArgs& a, bool stochastic, hipStream_t stream) {
  const PrefillGrid g =
      prefill_grid(a.nqb, a.c.kv_heads * a.head_groups, a.batch, a.len, PI, a.causal != 0, stochastic);
  // at least 768 bytes of queries and outputs each: the count stays far below 2^31
  if (g.workgroups > 0x7FFFFFFF) return hipErrorInvalidValue;
  a.grid_x = (int)g.x;
  a.workgroups = (int)g.workgroups;
  const dim3 grid((unsigned)g.x, (unsigned)g.y);
  const bool two = g.groups == 2;
  const dim3 threads(kGroupThreads * (two ? 2 : 1));
  if (stochastic) {
    if (two) hipLaunchKernelGGL((prefill_kernel<BITS, PI, true, 2>), grid, threads, 0, stream, a);
    else hipLaunchKernelGGL((prefill_kernel<BITS, PI, true, 1>), grid, threads, 0, stream, a);
  } else {
    if (two) hipLaunchKernelGGL((prefill_kernel<BITS, PI, false, 2>), grid, threads, 0, stream, a);
    else hipLaunchKernelGGL((prefill_kernel<BITS, PI, false, 1>), grid, threads, 0, stream, a);
  }
  return hipGetLastError();
}

hipError_t launch_prefill(const hack_kv_layout& lay, const CacheView& c, const __half* q, int num_q_heads,
                          int batch, int len, int causal, float* out, hipStream_t stream) {
  PrefillArgs a;
  a.c = c;
  a.q = q;
  a.out = out;
  a.num_q_heads = num_q_heads;
  a.group = num_q_heads / lay.num_kv_heads;
  // four heads to a workgroup where the kv group has them (they share its K and V), fewer
  // heads and more rows of each otherwise
  a.hw_log2 = a.group >= 3 ? 2 : (a.group == 2 ? 1 : 0);
  const int hw = 1 << a.hw_log2, wg_rows = kWaveRows * (4 / hw);
  a.head_groups = (a.group + hw - 1) / hw;
  a.batch = batch;
  a.len = len;
  a.causal = causal;
  a.nqb = (len + wg_rows - 1) / wg_rows;
  a.key_q = lay.seed ^ (3ull << 56);
  a.key_p = lay.seed ^ (4ull << 56);
  const bool sr = lay.rounding == HACK_ROUND_STOCHASTIC;
  a.qmax = (float)((1 << lay.qp_bits) - 1);
  a.inv_qmax = 1.0f / a.qmax;
  a.qoff = 1 << (lay.qp_bits - 1);
  a.qoff_f = (float)a.qoff;
  a.poff = lay.qp_bits == 8 ? 128 : 0;
  a.poff_f = (float)a.poff;
  a.pflip = lay.qp_bits == 8 ? 0x80808080u : 0u;
  switch (lay.kv_bits * 1000 + lay.partition) {
    case 2032: return prefill_impl<2, 32>(a, sr, stream);
    case 2064: return prefill_impl<2, 64>(a, sr, stream);
    case 4032: return prefill_impl<4, 32>(a, sr, stream);
    case 4064: return prefill_impl<4, 64>(a, sr, stream);
    case 2128: return prefill_impl<2, 128>(a, sr, stream);
    case 4128: return prefill_impl<4, 128>(a, sr, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hack
