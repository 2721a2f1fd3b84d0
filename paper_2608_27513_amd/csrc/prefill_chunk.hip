// Prefill at d = 128 on the matrix cores (App. A.5, prefill path; section 3.1
// Eq. (1)): the recurrence of a chunk of C = 16 tokens in matrix form, with
// fp32 accuracy.
//
// For tokens t = 0 .. C - 1 of a chunk with incoming state S0 and decays a_t,
// let G_t = a_0 ... a_t and L_ts = a_{s+1} ... a_t. Eq. (1) unrolls to
//   delta_t = v_t - G_t S0^T k_t - sum_{s<t} A_ts delta_s,  A_ts = L_ts beta_s k_t.k_s
//   o_t     = G_t S0^T q_t + sum_{s<=t} B_ts delta_s,       B_ts = L_ts beta_s q_t.k_s
//   S_C     = G_C S0 + sum_s k_s (L_{C-1,s} beta_s delta_s)^T
// so with R = V - diag(G) K S0 and T = (I + A)^-1 (unit lower triangular,
// by forward substitution):
//   [U; O'] = [diag(E) T; B T] R,  E_s = L_{C-1,s} beta_s
//   O = diag(G) Q S0 + O',  S_C = G_C S0 + K^T U.
// T and B T do not depend on the state: they are formed for several chunks at
// once, before the chunks run.
//
// Precision. Every fp32 operand x of a product enters the bf16 matrix cores
// as x = hi + mid + lo, three bf16 numbers (exact: 24 bits), and products
// accumulate in fp32. q and k are bf16 already, so K S0, Q S0, K K^T, Q K^T
// and K^T U have one factor exact and take three products; a product of two
// split factors takes the six whose weight is above 2^-26. Decay ratios are
// running products as in the sequential form, never exponentials of sums.
// A zero in a product does not hide a factor that is not finite, so a value out
// of range at one token would reach the tokens before it: a chunk whose inputs,
// decay products, T or B T are not all finite, and a wave whose R is not, run
// token by token in fp32 (run_tokens).
//
// KDA's decay is per key channel, so k and q carry it: with the reference
// token r = 7 of a chunk and rho_t the product of a channel's decays between
// tokens r and t (1 at r),
//   k~_t = k_t rho_t, q~_t = q_t rho_t, k^_s = k_s / rho_s
// and, with S0' = diag(a_0 ... a_7) S0, the same formulas hold with L = G = 1:
//   A_ts = beta_s k~_t.k^_s, S_C = diag(a_8 ... a_15) (S0' + K^^T U).
// The products on either side of r must stay in [2^-80, 2^80]. A channel whose
// decays leave it on one side (a zero decay included) is steep in this chunk:
// k~.k^ then lacks its share between two tokens of that side, k_t k_s times the
// product of the decays between them, which the wave that stages them sums by
// itself, and its rows for the products with the state take the chunk's ends as
// references, where no inverse is needed: k_t G_t with S0, k_s L_{15,s} with U,
// and S0 takes G_15 between the two. A chunk runs token by token if a product
// passes 2^80, if its k, q, v or beta reaches 2^32, 2^32, 2^32, 2^16 or a column
// of its v or a pair of channels of its q is below 2^-24 but not zero: so k^ and
// k^ U stay finite, and the third parts of S0', R and q~ stay above the smallest
// normal number, below which the products drop them. Nor may |A| pass 2^7 (it is
// looked at where k, beta or a decay is above one): so T, whose entries reach
// (1 + |A|)^14, stays finite.
// One channel at g = -9 in every head, FP32 state, token by token and in this
// form: B = 32, 250 tokens 835 -> 372 us (334 with none), B = 8, 1024 tokens
// 1433 -> 421 (307), B = 256, 64 tokens 1530 -> 706 (667). Every channel: 785 ->
// 565, 1433 -> 843, 1536 -> 1002.
//
// Mapping. A workgroup of four waves owns one (request, value head) tile;
// wave w holds columns 32 w .. 32 w + 31 of the state for all 128 channels, in
// natural channel order, as the accumulators of 32 x 32 matrix instructions
// (64 registers a lane). The rows of an accumulator block are assigned so
// that eight consecutive accumulator registers of a lane are eight consecutive
// channels (or tokens): exactly the lane's part of the right-hand operand of
// the next product, which is therefore split in registers, without any
// exchange between lanes. The left-hand operands are read from LDS: rows of
// k and q (16-byte pieces xor-swizzled by the row, so that the lanes of a
// read hit distinct banks), and for K^T U the same rows through the
// transposing LDS read. The stored tile passes through LDS once on the way in
// and once on the way out, half its columns at a time, and takes its channel
// permutation there, so that k, q and g are read as whole rows.
//
// What bounds it: the issue of vector instructions, about 800 per wave and
// chunk besides 42 matrix instructions (GDN; KDA 1000 and 78), of which the
// three-way splits are half. A wave alone issues one in 5 cycles, and a matrix
// instruction keeps the SIMD's vector unit from others' use for about 22 of
// its 32 cycles, so the kernel is held to 168 registers and 51 200 bytes of
// LDS: three workgroups a CU. KDA's four-wave form waits as much as it issues
// (39% of its wave cycles): it stages a single chunk, behind barriers at which
// only some waves have work. While there are no more tiles than CUs, a workgroup
// has four more waves that stage the next chunks meanwhile (SPLIT). A register
// that spills costs more than it looks (its reload waits for every load and
// store before it: 336 -> 440 us with some ten in the loop), hence opaque() and
// the scheduling barriers. Chunks of 16: the products within a chunk and T grow
// with its square.
// Measured against the token-by-token fp32 kernel before it (two FMAs per
// value and token for the read-outs, one for the update), GDN, B = 256, 32
// heads, 64 tokens: 805 -> 309 us; KDA, B = 32, 250 tokens: 498 -> 264 us; GDN,
// two requests of 1024 tokens: 722 -> 134 us; 2 tokens at B = 256: 154 -> 139 us
// (GDN), 167 -> 164 us (KDA).
#include <atomic>
#include <cfloat>
#include <cstdint>

#include "device.hpp"
#include "internal.hpp"
#include "prefill.hpp"

namespace damp {
namespace {

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef short s4v __attribute__((ext_vector_type(4)));

constexpr int kC = 16;    // tokens of a chunk
constexpr int kD = 128;
constexpr int kRow = 256;  // bytes of a row of 128 bf16
constexpr int kPitch = 68;  // floats of a row of half the tile's columns in transit
constexpr float kRhoMin = 0x1p-80f, kRhoMax = 0x1p80f;
constexpr float kBetaMax = 0x1p16f, kKeysMax = 0x1p7f;  // KDA's matrix form (see above)

__device__ __forceinline__ f16v mfma32(u4v a, u4v b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8v, a),
                                                 __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
}
__device__ __forceinline__ f4v mfma16(u4v a, u4v b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a),
                                                 __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
}

// x = hi + mid + lo of two values, packed.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& hi, uint32_t& mid,
                                       uint32_t& lo) {
  hi = pack_bf16x2(x0, x1);
  const float r0 = x0 - bf16_lo(hi), r1 = x1 - bf16_hi(hi);
  mid = pack_bf16x2(r0, r1);
  lo = pack_bf16x2(r0 - bf16_lo(mid), r1 - bf16_hi(mid));
}

// Hides how x was formed, so that the few instructions of an address are
// repeated where it is used instead of every address of the token loop being
// kept in registers.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The same by truncation, one vector cycle in ten less: for products whose
// three parts all count (the rounded parts are smaller, so that the three
// dropped products of two split factors are).
__device__ __forceinline__ void split2_cut(float x0, float x1, uint32_t& hi, uint32_t& mid,
                                           uint32_t& lo) {
  constexpr uint32_t kTop = 0xffff0000u, kPair = 0x07060302u;  // the upper halves of two words
  const float r0 = x0 - __uint_as_float(__float_as_uint(x0) & kTop);
  const float r1 = x1 - __uint_as_float(__float_as_uint(x1) & kTop);
  const float l0 = r0 - __uint_as_float(__float_as_uint(r0) & kTop);
  const float l1 = r1 - __uint_as_float(__float_as_uint(r1) & kTop);
  hi = __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), kPair);
  mid = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), kPair);
  lo = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), kPair);
}

struct Split8 {
  u4v part[3];  // hi, mid, lo of eight values
};
template <bool CUT = false>
__device__ __forceinline__ Split8 split8(const float* x) {
  Split8 s;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t hi, mid, lo;
    if (CUT) split2_cut(x[2 * j], x[2 * j + 1], hi, mid, lo);
    else split2(x[2 * j], x[2 * j + 1], hi, mid, lo);
    s.part[0][j] = hi;
    s.part[1][j] = mid;
    s.part[2][j] = lo;
  }
  return s;
}

// big + small + a b over split factors, the product of the leading parts into
// big and the others into small (three in all when a is exact, NA = 1, else the
// six above 2^-26 of the largest), so that big is rounded once per call.
template <int NA>
__device__ __forceinline__ void mfma32_split(const u4v* a, const Split8& b, f16v& big,
                                             f16v& small) {
  if constexpr (NA == 1) {
    small = mfma32(a[0], b.part[2], small);
    small = mfma32(a[0], b.part[1], small);
  } else {
    small = mfma32(a[2], b.part[0], small);
    small = mfma32(a[0], b.part[2], small);
    small = mfma32(a[1], b.part[1], small);
    small = mfma32(a[1], b.part[0], small);
    small = mfma32(a[0], b.part[1], small);
  }
  big = mfma32(a[0], b.part[0], big);
}
// c + a b into one accumulator, smallest products first.
template <int NA>
__device__ __forceinline__ f16v mfma32_split(const u4v* a, const Split8& b, f16v c) {
  f16v s = c;
  if constexpr (NA == 1) {
    s = mfma32(a[0], b.part[2], s);
    s = mfma32(a[0], b.part[1], s);
  } else {
    s = mfma32(a[2], b.part[0], s);
    s = mfma32(a[0], b.part[2], s);
    s = mfma32(a[1], b.part[1], s);
    s = mfma32(a[1], b.part[0], s);
    s = mfma32(a[0], b.part[1], s);
  }
  return mfma32(a[0], b.part[0], s);
}

// The value N lanes before in the row of 16 lanes, 1 where there is none or the
// lane's bank of four is not in BANKS.
template <int N, int BANKS>
__device__ __forceinline__ float lanes_before(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(1.0f), __float_as_int(x),
                                                    0x110 + N, 0xf, BANKS, false));
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// 16-byte piece ck of row r of a swizzled [rows][128] bf16 array.
__device__ __forceinline__ int row_at(int r, int ck) { return r * kRow + ((ck ^ (r & 15)) << 4); }

// Non-zero if a bf16 half of w is an infinity or a NaN.
__device__ __forceinline__ uint32_t nonfinite(uint32_t w) {
  return ((w & 0x7f807f80u) + 0x00800080u) & 0x80008000u;
}
// The bits of the largest magnitude among bf16 pairs.
struct MaxBits {
  typedef uint16_t us2 __attribute__((ext_vector_type(2)));
  us2 pair = {0, 0};
  __device__ __forceinline__ void add(uint32_t w) {
    pair = __builtin_elementwise_max(pair, __builtin_bit_cast(us2, w & 0x7fff7fffu));
  }
  __device__ __forceinline__ uint32_t bits() const { return pair.x > pair.y ? pair.x : pair.y; }
};
constexpr uint32_t bf16_pow2(int e) { return static_cast<uint32_t>(127 + e) << 7; }
// Of the bits of a bf16 magnitude: not zero, and outside [2^-24, 2^32).
__device__ __forceinline__ bool out_of_scale(uint32_t bits) {
  return bits != 0u && bits - bf16_pow2(-24) >= bf16_pow2(32) - bf16_pow2(-24);
}

// `n` rows of `bytes` bytes, `step` bytes apart, as a raw buffer that ends with
// the last row: reads past it return zero and writes are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* base, int step, int bytes,
                                                            int n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (n - 1) * step + bytes,
                                           0x00020000);
}

// How a chunk is run, if not in the plain matrix form (a bit set).
constexpr int kTokens = 1;  // token by token
constexpr int kSteep = 2;   // KDA: channels in steep form beside the others
constexpr int kKeys = 4;    // KDA: |A| may be large and is looked at
constexpr int kSteepBatch = 8;  // steep channels that a staging wave takes at a time

// LDS of one chunk's operands. GDN: kq holds the 16 rows of k, then of q, and
// tm [U rows; O rows] as three bf16 parts. KDA: kq holds k~ and q~ in three
// parts, kh k^ in three parts, tm the fp32 values (split when read).
template <bool KDA>
struct ChunkLds;
template <>
struct alignas(16) ChunkLds<false> {
  uint8_t kq[1][32 * kRow];
  uint16_t tm[3][32][kC];
  float G[kC], a[kC], beta[kC];
  int32_t flag;
};
template <>
struct alignas(16) ChunkLds<true> {
  uint8_t kq[3][32 * kRow];
  uint8_t kh[3][16 * kRow];
  float tm[32][kC];
  alignas(16) float pre[kD], fin[kD];
  float beta[kC];
  int32_t flag[4];  // what each staging wave found
  // steep channels, by staging wave: a bit per pair of channels (even, odd
  // channels); some of them at its tokens (k, q, a); their sums for A and B
  // between its tokens s and t, at 8 s + t; and for all, the factors that take
  // the place of pre and fin
  uint32_t steep[4][2];
  float4 row[4][kSteepBatch][8];
  float2 sum[4][64];
  alignas(16) float pre_s[kD], mid_s[kD], fin_s[kD];
  int32_t grows;  // with kKeys: 0, or kTokens if A is out of range
};

// SPLIT: eight waves a workgroup, four of which stage the next chunks into a
// second buffer while the others run these.
template <bool KDA, bool SPLIT>
struct Prefill {
  static constexpr int NT = SPLIT ? 512 : 256;
  static constexpr int NC = KDA ? 1 : 4;  // chunks staged together
  static constexpr int NA = KDA ? 3 : 1;
  using Chunk = ChunkLds<KDA>;
  static constexpr size_t kTransit = sizeof(float) * kD * kPitch;
  static constexpr size_t kStaged = (SPLIT ? 2 : 1) * NC * sizeof(Chunk);
  static constexpr size_t kBytes =
      SPLIT ? kStaged + kTransit : (kStaged > kTransit ? kStaged : kTransit);
};
static_assert(Prefill<true, false>::kBytes <= 51200 && Prefill<false, false>::kBytes <= 51200,
              "three workgroups share a CU's LDS");
static_assert(Prefill<true, true>::kBytes <= 160 * 1024 && Prefill<false, true>::kBytes <= 160 * 1024,
              "LDS of a CU");

// (I + A)^-1 by forward substitution, one column per lane (c = lane % 16, the
// four lanes of a column alike), and the rows of [diag(E) T; B T] for a chunk
// of n tokens (the rows of four tokens past the end are left out). ab: A rows
// 0..15 and B rows 16..31, fp32, zero where s >= t (A) or s > t (B). On return
// um[i] and om[i] hold rows 4 (lane / 16) + i of the two halves.
__device__ __forceinline__ void solve_chunk(const float (*ab)[kC], int lane, int n,
                                            const float (&e4)[4], float (&um)[4],
                                            float (&om)[4]) {
  const int c = opaque(lane & 15), quad = lane >> 4;
  float T[kC];
#pragma unroll
  for (int i = 0; i < 4; ++i) um[i] = om[i] = 0.0f;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) T[4 * g + i] = 0.0f;
    if (4 * g < n) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = 4 * g + i;
        float acc = t == c ? 1.0f : 0.0f;
#pragma unroll
        for (int s4 = 0; s4 < (t + 3) / 4; ++s4) {
          const float4 a4 = *reinterpret_cast<const float4*>(&ab[t][4 * s4]);
          const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
          for (int m = 0; m < 4; ++m)
            if (4 * s4 + m < t) acc = fmaf(-av[m], T[4 * s4 + m], acc);
        }
        T[t] = acc;
        um[i] = quad == g ? acc : um[i];  // the lane's own rows
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // four rows at a time: registers
  }
#pragma unroll
  for (int s4 = 0; s4 < 4; ++s4) {
    if (4 * s4 < n) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 b4 = *reinterpret_cast<const float4*>(&ab[16 + 4 * quad + i][4 * s4]);
        om[i] = fmaf(b4.x, T[4 * s4], om[i]);
        om[i] = fmaf(b4.y, T[4 * s4 + 1], om[i]);
        om[i] = fmaf(b4.z, T[4 * s4 + 2], om[i]);
        om[i] = fmaf(b4.w, T[4 * s4 + 3], om[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) um[i] *= e4[i];
  __builtin_amdgcn_sched_barrier(0);
}

template <int KIND, bool KDA, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 512 : 256, SPLIT ? 2 : 3) void prefill_chunk128(
    const PrefillParams p) {
  using P = Prefill<KDA, SPLIT>;
  constexpr int NC = P::NC, NA = P::NA, CPT = 16, TPR = 8;
  __shared__ __attribute__((aligned(16))) uint8_t lds_raw[P::kBytes];
  typename P::Chunk* L = reinterpret_cast<typename P::Chunk*>(lds_raw);
  float(*tbuf)[kPitch] = reinterpret_cast<float(*)[kPitch]>(lds_raw + (SPLIT ? P::kStaged : 0));

  const int t = threadIdx.x & 255, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool stages = SPLIT && __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) != 0;
  const int ph = lane >> 5, l32 = lane & 31;  // half: tokens (or channels) 8 ph ..
  // Workgroups go to the eight XCDs in turn. The value heads that share a key
  // head read the same k and q: of each 8 rep consecutive workgroups, rep
  // neighbouring heads go to one XCD, whose L2 then serves all but the first
  // (GDN, B = 256, 64 tokens, two heads a key head, with v no longer touched
  // ahead: 764 -> 446 MB fetched, 320 -> 316 us; a few tiles gain nothing).
  int h = blockIdx.x, b = blockIdx.y;
  const int rep = p.HV / p.HK;
  if (!KDA && !SPLIT && rep > 1 && gridDim.x * gridDim.y % (8u * rep) == 0) {
    const unsigned id = blockIdx.y * gridDim.x + blockIdx.x, span = 8u * rep;
    const unsigned in = id % span, tile_id = id - in + (in & 7) * rep + (in >> 3);
    b = tile_id / gridDim.x;
    h = tile_id % gridDim.x;
  }
  const int T = p.T;
  const int hk = h / rep;
  const int col = 32 * wave + l32;  // this lane's state column
  const size_t o_esize = p.o_bf16 ? 2 : 4;
  const size_t o_step = static_cast<size_t>(p.HV) * kD * o_esize;
  uint8_t* const o_col = static_cast<uint8_t*>(p.o) +
                         ((static_cast<size_t>(b) * T * p.HV + h) * kD + col) * o_esize;
  auto write_o = [&](int tok, float val) __attribute__((always_inline)) {
    uint8_t* at = o_col + static_cast<size_t>(tok) * o_step;
    if (p.o_bf16) *reinterpret_cast<uint16_t*>(at) = f32_to_bf16(val);
    else *reinterpret_cast<float*>(at) = val;
  };

  const int slot = __builtin_amdgcn_readfirstlane(p.slot_idx[b]);
  if (slot < 0 || slot >= p.num_slots) {  // padded request: o = 0, state untouched
    if (p.o && !stages)
      for (int tok = ph; tok < T; tok += 2) write_o(tok, 0.0f);
    return;
  }
  uint8_t* tile = p.layer_base + static_cast<size_t>(slot) * p.slot_stride +
                  static_cast<size_t>(h) * p.tile_stride;
  const int k_hi = KIND == kFp32 ? kD : p.k_hi;
  uint8_t* codes = tile + static_cast<size_t>(k_hi) * kD * 2;
  uint8_t* meta_bytes = codes + static_cast<size_t>(kD - k_hi) * code_row_bytes<KIND, kD>();
  const bool had = p.had != 0;

  // rows of the inputs: token tok of this request and head
  const size_t tok0 = static_cast<size_t>(b) * p.t_pitch + p.t0;
  auto k_row = [&](int tok) __attribute__((always_inline)) { return ((tok0 + tok) * p.HK + hk) * kD; };
  auto v_row = [&](int tok) __attribute__((always_inline)) { return (tok0 + tok) * p.HV + h; };

  // ---- inputs of NC chunks, through buffer resources that end with the last
  // token: later tokens read zeros
  constexpr int NL = 4;
  struct Ahead {
    u4v k[KDA ? 1 : NL], q[KDA ? 1 : NL];
    uint32_t kp[KDA ? NL : 1], qp[KDA ? NL : 1], gp[KDA ? NL : 1];
    uint32_t v[KDA ? 8 : 1];
    uint32_t g, beta;
  } in;
  const int kq_step = p.HK * kRow, v_step = p.HV * kRow;
  // buffer loads of a word and more need a word's alignment: k, q and KDA's g
  // that do not have it are read by halves
  const bool by_halves = ((reinterpret_cast<uintptr_t>(p.k) | reinterpret_cast<uintptr_t>(p.q) |
                           (KDA ? reinterpret_cast<uintptr_t>(p.g) : 0)) & 2) != 0;
  auto load_halves = [&](const auto& rsrc, int at) __attribute__((always_inline)) -> uint32_t {
    const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(rsrc, at, 0, 0);
    const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(rsrc, at + 2, 0, 0);
    return lo | hi << 16;
  };
  auto load_inputs = [&](int tb0) __attribute__((always_inline)) {
    const int lane = opaque(t) & 63, ph = lane >> 5, l32 = lane & 31, col = 32 * wave + l32;
    const int ntok = T - tb0 < NC * kC ? T - tb0 : NC * kC;
    const size_t row = tok0 + tb0;
    const auto rk = rows_rsrc(p.k + (row * p.HK + hk) * kD, kq_step, kRow, ntok);
    const auto rq = rows_rsrc(p.q + (row * p.HK + hk) * kD, kq_step, kRow, ntok);
    const auto rb = rows_rsrc(p.beta + row * p.HV + h, 2 * p.HV, 2, ntok);
    if constexpr (!KDA) {  // wave w: chunk w; 16 bytes of four rows per load
      const auto rg = rows_rsrc(p.g + row * p.HV + h, 2 * p.HV, 2, ntok);
      const int tt = opaque(kC * wave + (lane >> 4));
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int kq = (tt + 4 * i) * kq_step + 16 * (lane & 15);
        if (__builtin_expect(by_halves, 0)) {
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            in.k[i][w] = load_halves(rk, kq + 4 * w);
            in.q[i][w] = load_halves(rq, kq + 4 * w);
          }
          continue;
        }
        in.k[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, kq, 0, 0);
        in.q[i] = __builtin_amdgcn_raw_buffer_load_b128(rq, kq, 0, 0);
      }
      const int ts = (kC * wave + (lane & 15)) * 2 * p.HV;
      in.g = __builtin_amdgcn_raw_buffer_load_b16(rg, ts, 0, 0);
      in.beta = __builtin_amdgcn_raw_buffer_load_b16(rb, ts, 0, 0);
    } else {  // wave w: tokens 8 (w / 2) + 4 (lane / 32) .. + 3, two channels per lane
      const auto rg = rows_rsrc(p.g + (row * p.HV + h) * kD, v_step, kRow, ntok);
      const auto rv = rows_rsrc(p.v + (row * p.HV + h) * kD, v_step, kRow, ntok);
      const int tt = 8 * (wave >> 1) + 4 * ph, at = 128 * (wave & 1) + 4 * l32;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int kq = (tt + i) * kq_step + at, gv = (tt + i) * v_step + at;
        if (__builtin_expect(by_halves, 0)) {
          in.kp[i] = load_halves(rk, kq);
          in.qp[i] = load_halves(rq, kq);
          in.gp[i] = load_halves(rg, gv);
          continue;
        }
        in.kp[i] = __builtin_amdgcn_raw_buffer_load_b32(rk, kq, 0, 0);
        in.qp[i] = __builtin_amdgcn_raw_buffer_load_b32(rq, kq, 0, 0);
        in.gp[i] = __builtin_amdgcn_raw_buffer_load_b32(rg, gv, 0, 0);
      }
      in.beta = __builtin_amdgcn_raw_buffer_load_b16(rb, (lane & 15) * 2 * p.HV, 0, 0);
      const int v_at = 8 * ph * v_step + 2 * col;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        in.v[KDA ? e : 0] = __builtin_amdgcn_raw_buffer_load_b16(rv, e * v_step + v_at, 0, 0);
    }
  };
  // one load per 128-byte line of the rows of the NC chunks from token tb0, so
  // that load_inputs finds them in the L2; the caller drops the values
  auto touch = [&](int tb0, uint32_t& x0, uint32_t& x1) __attribute__((always_inline)) {
    const int t = opaque(threadIdx.x & 255);
    const int ntok = T - tb0 < NC * kC ? T - tb0 : NC * kC;
    const size_t row = tok0 + tb0;
    const auto rk = rows_rsrc(p.k + (row * p.HK + hk) * kD, kq_step, kRow, ntok);
    const auto rq = rows_rsrc(p.q + (row * p.HK + hk) * kD, kq_step, kRow, ntok);
    const auto rv = rows_rsrc(p.v + (row * p.HV + h) * kD, v_step, kRow, ntok);
    if constexpr (!KDA) {
      const int tt = (t >> 1) & 63, line = 128 * (t & 1);
      x0 = t < 128 ? __builtin_amdgcn_raw_buffer_load_b16(rk, tt * kq_step + line, 0, 0)
                   : __builtin_amdgcn_raw_buffer_load_b16(rq, tt * kq_step + line, 0, 0);
      // v only ahead of the staging waves: before a whole round of chunks it
      // would be out of the L2 again when it is read
      x1 = SPLIT && t < 128 ? __builtin_amdgcn_raw_buffer_load_b16(rv, tt * v_step + line, 0, 0) : 0u;
    } else {
      const auto rg = rows_rsrc(p.g + (row * p.HV + h) * kD, v_step, kRow, ntok);
      const int tt = (t >> 1) & 15, line = 128 * (t & 1);
      x0 = wave == 0   ? __builtin_amdgcn_raw_buffer_load_b16(rk, tt * kq_step + line, 0, 0)
           : wave == 1 ? __builtin_amdgcn_raw_buffer_load_b16(rq, tt * kq_step + line, 0, 0)
           : wave == 2 ? __builtin_amdgcn_raw_buffer_load_b16(rv, tt * v_step + line, 0, 0)
                       : __builtin_amdgcn_raw_buffer_load_b16(rg, tt * v_step + line, 0, 0);
      x1 = 0u;
    }
  };

  // the lane id, formed anew in each phase (see opaque)
  auto lane_now = [&]() __attribute__((always_inline)) { return opaque(t) & 63; };

  // 0, or what a chunk's staging found
  auto form_of = [&](const typename P::Chunk& ck) __attribute__((always_inline)) -> int {
    int f;
    if constexpr (KDA)
      f = ck.flag[0] | ck.flag[1] | ck.flag[2] | ck.flag[3];
    else
      f = ck.flag;
    return __builtin_amdgcn_readfirstlane(f);
  };
  // KDA: the same once the products are there
  auto with_grows = [&](const typename P::Chunk& ck, int form) __attribute__((always_inline)) -> int {
    if constexpr (KDA) {
      if (__builtin_expect((form & kKeys) != 0, 0))
        form |= __builtin_amdgcn_readfirstlane(ck.grows);
    }
    return form;
  };

  // ---- GDN staging, wave-local: wave w stages chunk w
  auto stage_gdn = [&](typename P::Chunk& ck, int tb) __attribute__((always_inline)) {
    if constexpr (!KDA) {
      if (tb >= T) return;
      const int lane = lane_now();
      uint32_t bad = 0u;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int row = (lane >> 4) + 4 * i;
        *reinterpret_cast<u4v*>(ck.kq[0] + row_at(row, lane & 15)) = in.k[i];
        *reinterpret_cast<u4v*>(ck.kq[0] + row_at(16 + row, lane & 15)) = in.q[i];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          bad |= nonfinite(in.k[i][j]) | nonfinite(in.q[i][j]);
      }
      const float a = __expf(bf16_to_f32(static_cast<uint16_t>(in.g)));  // 1 past the end
      const float beta = bf16_to_f32(static_cast<uint16_t>(in.beta));
      if (!(a <= FLT_MAX) || !(fabsf(beta) <= FLT_MAX)) bad = 1u;
      if (lane < kC) {
        ck.a[lane] = a;
        ck.beta[lane] = beta;
      }
      // decay ratios: this lane's column s, rows t = 4 quad + i
      const int s = lane & 15, quad = lane >> 4;
      float Lr[4] = {0.0f, 0.0f, 0.0f, 0.0f}, G = 1.0f, run = 1.0f, Gs = 1.0f;
#pragma unroll
      for (int tt = 0; tt < kC; ++tt) {
        const float at = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), tt));
        G *= at;
        if (s == tt) Gs = G;
        run = tt <= s ? 1.0f : run * at;
        if (quad == (tt >> 2)) Lr[tt & 3] = run;
      }
      if (lane < kC) ck.G[lane] = Gs;
      const float E = run * beta;  // L_{15,s} beta_s
      // an overflow of G or of a ratio is in the last one too
      if (!(G <= FLT_MAX) || !(fabsf(E) <= FLT_MAX)) bad = 1u;
      const bool any = __builtin_amdgcn_ballot_w64(bad != 0u) != 0;
      if (lane == 0) ck.flag = any ? 1 : 0;
      if (any) return;
      wave_sync();
      f4v kk = {0.0f, 0.0f, 0.0f, 0.0f}, qk = kk;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const u4v fk = *reinterpret_cast<const u4v*>(ck.kq[0] + row_at(s, 4 * ks + quad));
        const u4v fq = *reinterpret_cast<const u4v*>(ck.kq[0] + row_at(16 + s, 4 * ks + quad));
        kk = mfma16(fk, fk, kk);
        qk = mfma16(fq, fk, qk);
      }
      float(*ab)[kC] = reinterpret_cast<float(*)[kC]>(ck.tm);
      float e4[4], um[4], om[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tt = 4 * quad + i;
        const float f = Lr[i] * beta;
        ab[tt][s] = s < tt ? f * kk[i] : 0.0f;
        ab[16 + tt][s] = s <= tt ? f * qk[i] : 0.0f;
        e4[i] = __shfl(E, tt, 64);
      }
      wave_sync();
      solve_chunk(ab, lane, T - tb, e4, um, om);
      // keys that amplify the state out of range within the chunk
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += fabsf(um[i]) + fabsf(om[i]);
      if (__builtin_amdgcn_ballot_w64(!(sum <= FLT_MAX)) != 0 && lane == 0) ck.flag = 1;
      wave_sync();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t hi, mid, lo;
        split2(um[i], om[i], hi, mid, lo);
        const int tt = 4 * quad + i;
        ck.tm[0][tt][s] = static_cast<uint16_t>(hi);
        ck.tm[1][tt][s] = static_cast<uint16_t>(mid);
        ck.tm[2][tt][s] = static_cast<uint16_t>(lo);
        ck.tm[0][16 + tt][s] = static_cast<uint16_t>(hi >> 16);
        ck.tm[1][16 + tt][s] = static_cast<uint16_t>(mid >> 16);
        ck.tm[2][16 + tt][s] = static_cast<uint16_t>(lo >> 16);
      }
    }
  };

  // ---- KDA staging by four waves in three steps, a barrier after each: waves
  // 0 and 1 take the first eight tokens, waves 2 and 3 the others
  auto kda_operands = [&](typename P::Chunk& ck) __attribute__((always_inline)) {
    if constexpr (KDA) {
      const int half = wave >> 1;
      const int lane = lane_now(), ph = lane >> 5, l32 = lane & 31;
      // cum[i]: the channel's product between token 7 and token i of the lane's four
      float cum[2][4], a[2][4];
      MaxBits kmax, qmax;
      float amax = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[0][i] = __expf(bf16_lo(in.gp[i]));
        a[1][i] = __expf(bf16_hi(in.gp[i]));
        amax = fmaxf(fmaxf(a[0][i], a[1][i]), amax);
        kmax.add(in.kp[i]);
        qmax.add(in.qp[i]);
      }
      float whole[2];
      uint64_t low[2];  // the lanes of steep channels
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const float mine = (a[m][0] * a[m][1]) * (a[m][2] * a[m][3]);
        const float other = __shfl_xor(mine, 32, 64);
        float run = (half == 0) == (ph == 0) ? other : 1.0f;  // the four tokens nearer to token 7
        if (half == 0) {
#pragma unroll
          for (int i = 3; i >= 0; --i) {
            cum[m][i] = run;
            run *= a[m][i];
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            run *= a[m][i];
            cum[m][i] = run;
          }
        }
        float least = kRhoMax;
#pragma unroll
        for (int i = 0; i < 4; ++i) least = fminf(least, cum[m][i]);
        low[m] = __builtin_amdgcn_ballot_w64(least < kRhoMin);
        whole[m] = run;  // a NaN in cum is in it too
      }
      const float beta = bf16_to_f32(static_cast<uint16_t>(in.beta));
      const uint32_t kbits = kmax.bits();
      uint32_t vmax = 0u;  // of this wave's columns
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t av = in.v[KDA ? e : 0] & 0x7fffu;
        vmax = av > vmax ? av : vmax;
      }
      bool bad = out_of_scale(qmax.bits()) || out_of_scale(vmax) || !(whole[0] <= FLT_MAX) ||
                 !(whole[1] <= FLT_MAX);
      int form = 0;
      // |k|, |beta| and the decays at most 1: |A| <= 128 = kKeysMax
      const bool wide = kbits > bf16_pow2(0) || !(fabsf(beta) <= 1.0f) || amax > 1.0f;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(wide) != 0, 0)) {
        form = kKeys;
        float top = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) top = fmaxf(fmaxf(cum[0][i], cum[1][i]), top);
        bad = bad || kbits >= bf16_pow2(32) || !(fabsf(beta) <= kBetaMax) || top > kRhoMax;
      }
      if (__builtin_amdgcn_ballot_w64(bad) != 0) form |= kTokens;
      if (__builtin_expect((low[0] | low[1]) != 0, 0)) {
        uint32_t steep[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          steep[m] = static_cast<uint32_t>(low[m]) | static_cast<uint32_t>(low[m] >> 32);
          if (lane == 0) ck.steep[wave][m] = steep[m];
        }
        form |= kSteep;
      }
      if (lane == 0) ck.flag[wave] = form;
      if (wave == 0 && lane < kC) ck.beta[lane] = beta;
      // the lanes of a channel's far tokens hold the product of all eight
      if ((half == 0) == (ph == 0))
        *reinterpret_cast<float2*>(&(half == 0 ? ck.pre : ck.fin)[64 * (wave & 1) + 2 * l32]) =
            make_float2(whole[0], whole[1]);
      // row 8 half + 4 ph + i: (at ^ 16 i) + i rows; q 16 rows after k
      const int first = 8 * half + 4 * ph;
      const int at = row_at(first, 8 * (wave & 1) + (l32 >> 2)) + 4 * (l32 & 3);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = (at ^ (i << 4)) + i * kRow;
        const float i0 = refined_rcp(cum[0][i]), i1 = refined_rcp(cum[1][i]);
        const float f0 = half == 0 ? i0 : cum[0][i], f1 = half == 0 ? i1 : cum[1][i];
        const float n0 = half == 0 ? cum[0][i] : i0, n1 = half == 0 ? cum[1][i] : i1;
        const float k0 = bf16_lo(in.kp[i]), k1 = bf16_hi(in.kp[i]);
        uint32_t s3[3];
        split2(k0 * f0, k1 * f1, s3[0], s3[1], s3[2]);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          *reinterpret_cast<uint32_t*>(ck.kq[KDA ? j : 0] + row) = s3[j];
        split2(bf16_lo(in.qp[i]) * f0, bf16_hi(in.qp[i]) * f1, s3[0], s3[1], s3[2]);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          *reinterpret_cast<uint32_t*>(ck.kq[KDA ? j : 0] + row + 16 * kRow) = s3[j];
        split2(k0 * n0, k1 * n1, s3[0], s3[1], s3[2]);
#pragma unroll
        for (int j = 0; j < 3; ++j) *reinterpret_cast<uint32_t*>(ck.kh[j] + row) = s3[j];
      }
      if (__builtin_expect((form & (kSteep | kTokens)) != kSteep, 1)) return;
      // steep channels: the side of 1 / rho leaves the products (zero); what
      // they lack there is summed here, token s = lane / 8 with t = lane % 8
      uint32_t steep[2];
      int rank[2], total = 0;  // of the lane's channels, -1: not steep
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        steep[m] = static_cast<uint32_t>(low[m]) | static_cast<uint32_t>(low[m] >> 32);
        const bool own = (steep[m] >> l32 & 1u) != 0u;
        rank[m] = own ? total + __builtin_popcount(steep[m] & ((1u << l32) - 1u)) : -1;
        total += __builtin_popcount(steep[m]);
        if (!own) continue;
        const uint32_t keep = m ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = (at ^ (i << 4)) + i * kRow;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            if (half == 0) {
              *reinterpret_cast<uint32_t*>(ck.kq[KDA ? j : 0] + row) &= keep;
              *reinterpret_cast<uint32_t*>(ck.kq[KDA ? j : 0] + row + 16 * kRow) &= keep;
            } else {
              *reinterpret_cast<uint32_t*>(ck.kh[j] + row) &= keep;
            }
          }
        }
      }
      const int ts = lane >> 3, tt = lane & 7;
      float2 sum = make_float2(0.0f, 0.0f);
#pragma unroll 1
      for (int first_c = 0; first_c < total; first_c += kSteepBatch) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int c = rank[m] - first_c;
          if (rank[m] < first_c || c >= kSteepBatch) continue;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            ck.row[wave][c][4 * ph + i] = make_float4(m ? bf16_hi(in.kp[i]) : bf16_lo(in.kp[i]),
                                                      m ? bf16_hi(in.qp[i]) : bf16_lo(in.qp[i]),
                                                      a[m][i], 0.0f);
        }
        wave_sync();
        const int n = total - first_c < kSteepBatch ? total - first_c : kSteepBatch;
#pragma unroll 2
        for (int c = 0; c < n; ++c) {
          const float4 kqa = ck.row[wave][c][tt];
          const float ks = ck.row[wave][c][ts].x;
          // the product of the decays of the tokens s + 1 .. t, over eight lanes
          float run = tt > ts ? kqa.z : 1.0f;
          const float by1 = lanes_before<1, 0xf>(run);
          run *= tt >= 1 ? by1 : 1.0f;
          const float by2 = lanes_before<2, 0xf>(run);
          run *= tt >= 2 ? by2 : 1.0f;
          run *= lanes_before<4, 0xa>(run);
          const float f = run * ks;
          sum.x = fmaf(f, kqa.x, sum.x);
          sum.y = fmaf(f, kqa.y, sum.y);
        }
        wave_sync();
      }
      ck.sum[wave][lane] = sum;
    }
  };
  // one wave of each half of the rows: A = beta_s k~_t.k^_s, B = beta_s q~_t.k^_s
  auto kda_products = [&](typename P::Chunk& ck, int form, int who) __attribute__((always_inline)) {
    if constexpr (KDA) {
      if ((form & kTokens) != 0) return;
      const int lane = lane_now();
      if (((wave ^ who) & 2) != 0) return;
      const int s = lane & 15, quad = lane >> 4, rows = (wave ^ who) & 1;
      f4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
      const int at_b = row_at(s, quad), at_a = at_b + 16 * rows * kRow;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        u4v fa[3], fb[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          fa[j] = *reinterpret_cast<const u4v*>(ck.kq[KDA ? j : 0] + (at_a ^ (ks << 6)));
          fb[j] = *reinterpret_cast<const u4v*>(ck.kh[j] + (at_b ^ (ks << 6)));
        }
        acc = mfma16(fa[2], fb[0], acc);
        acc = mfma16(fa[0], fb[2], acc);
        acc = mfma16(fa[1], fb[1], acc);
        acc = mfma16(fa[1], fb[0], acc);
        acc = mfma16(fa[0], fb[1], acc);
        acc = mfma16(fa[0], fb[0], acc);
      }
      if (__builtin_expect((form & kSteep) != 0, 0)) {
        const int half = quad >> 1;
#pragma unroll
        for (int w = 2 * half; w < 2 * half + 2; ++w) {
          if ((s >> 3) != half || (ck.flag[w] & kSteep) == 0) continue;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float2 x = ck.sum[w][8 * (s & 7) + 4 * (quad & 1) + i];
            acc[i] += rows == 0 ? x.x : x.y;
          }
        }
      }
      const float bs = ck.beta[s];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tt = 4 * quad + i;
        const bool in_tri = rows == 0 ? s < tt : s <= tt;
        acc[i] = in_tri ? bs * acc[i] : 0.0f;
        ck.tm[16 * rows + tt][s] = acc[i];
      }
      if (__builtin_expect((form & kKeys) != 0, 0) && rows == 0) {
        const float sum = (fabsf(acc[0]) + fabsf(acc[1])) + (fabsf(acc[2]) + fabsf(acc[3]));
        const bool grows = __builtin_amdgcn_ballot_w64(!(sum <= kKeysMax)) != 0;
        if (lane == 0) ck.grows = grows ? kTokens : 0;
      }
    }
  };
  // a chunk that is not in the plain form, after its products. Token by token:
  // k and q themselves in the first part, the decays of even and odd channels in
  // the second. Else the steep channels' rows for the products with the state,
  // referred to the chunk's two ends
  auto kda_restage = [&](typename P::Chunk& ck, int form) __attribute__((always_inline)) {
    if constexpr (KDA) {
      if ((form & (kTokens | kSteep)) == 0) return;
      const int lane = lane_now(), half = wave >> 1, ph = lane >> 5, l32 = lane & 31;
      const int first = 8 * half + 4 * ph, ch = 64 * (wave & 1) + 2 * l32;
      const int at = row_at(first, 8 * (wave & 1) + (l32 >> 2)) + 4 * (l32 & 3);
      float a[2][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[0][i] = __expf(bf16_lo(in.gp[i]));
        a[1][i] = __expf(bf16_hi(in.gp[i]));
      }
      if ((form & kTokens) != 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint8_t* row = ck.kq[0] + (at ^ (i << 4)) + i * kRow;
          *reinterpret_cast<uint32_t*>(row) = in.kp[i];
          *reinterpret_cast<uint32_t*>(row + 16 * kRow) = in.qp[i];
          row += sizeof(ck.kq[0]);
          *reinterpret_cast<uint32_t*>(row) = __float_as_uint(a[0][i]);
          *reinterpret_cast<uint32_t*>(row + 16 * kRow) = __float_as_uint(a[1][i]);
        }
        return;
      }
      float G[2][4], E[2][4];  // products from the chunk's start to a token, from there to its end
      uint32_t keep = 0u;      // the halves of a word whose channel is not steep
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const float pre = ck.pre[ch + m], fin = ck.fin[ch + m];
        const float mine = (a[m][0] * a[m][1]) * (a[m][2] * a[m][3]);
        const float other = __shfl_xor(mine, 32, 64);
        float run = (half ? pre : 1.0f) * (ph ? other : 1.0f);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          run *= a[m][i];
          G[m][i] = run;
        }
        run = (half ? 1.0f : fin) * (ph ? 1.0f : other);
#pragma unroll
        for (int i = 3; i >= 0; --i) {
          E[m][i] = run;
          run *= a[m][i];
        }
        bool steep = false;
#pragma unroll
        for (int w = wave & 1; w < 4; w += 2)
          if ((ck.flag[w] & kSteep) != 0) steep = steep || (ck.steep[w][m] >> l32 & 1u) != 0u;
        if (!steep) keep |= 0xffffu << (16 * m);
        if (half == 0 && ph == 0) {
          ck.pre_s[ch + m] = steep ? 1.0f : pre;
          ck.mid_s[ch + m] = steep ? pre * fin : 1.0f;
          ck.fin_s[ch + m] = steep ? 1.0f : fin;
        }
      }
      if (keep == ~0u) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = (at ^ (i << 4)) + i * kRow;
        const float k0 = bf16_lo(in.kp[i]), k1 = bf16_hi(in.kp[i]);
        auto put = [&](uint8_t* base, const uint32_t (&s3)[3], int step) {
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            uint32_t* w = reinterpret_cast<uint32_t*>(base + j * step);
            *w = (*w & keep) | (s3[j] & ~keep);
          }
        };
        uint32_t s3[3];
        split2(k0 * G[0][i], k1 * G[1][i], s3[0], s3[1], s3[2]);
        put(ck.kq[0] + row, s3, sizeof(ck.kq[0]));
        split2(bf16_lo(in.qp[i]) * G[0][i], bf16_hi(in.qp[i]) * G[1][i], s3[0], s3[1], s3[2]);
        put(ck.kq[0] + row + 16 * kRow, s3, sizeof(ck.kq[0]));
        split2(k0 * E[0][i], k1 * E[1][i], s3[0], s3[1], s3[2]);
        put(ck.kh[0] + row, s3, sizeof(ck.kh[0]));
      }
    }
  };
  auto kda_solve = [&](typename P::Chunk& ck, int form, int tb,
                       int who) __attribute__((always_inline)) {
    if constexpr (KDA) {
      if (wave != who || (form & kTokens) != 0) return;
      const int lane = lane_now(), s = lane & 15, quad = lane >> 4;
      float e4[4], um[4], om[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) e4[i] = ck.beta[4 * quad + i];
      solve_chunk(ck.tm, lane, T - tb, e4, um, om);
      wave_sync();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ck.tm[4 * quad + i][s] = um[i];
        ck.tm[16 + 4 * quad + i][s] = om[i];
      }
    }
  };

  auto stage = [&](typename P::Chunk* buf, int tb0) __attribute__((always_inline)) {
    load_inputs(tb0);
    if constexpr (!KDA) stage_gdn(buf[wave], tb0 + kC * wave);
  };
  constexpr int kStep = NC * kC;
  uint32_t seen0, seen1;
  touch(0, seen0, seen1);
  // ---- SPLIT: the staging waves. They meet every barrier of the others: four
  // while the tile passes through LDS, those of the chunks, and those of the
  // way out
  if (stages) {
    auto staged = [&](int tb0) __attribute__((always_inline)) {
      typename P::Chunk* buf = L + (tb0 / kStep & 1) * NC;
      if (tb0 < T) {
        asm volatile("" ::"v"(seen0), "v"(seen1));
        stage(buf, tb0);
        if (tb0 + kStep < T) touch(tb0 + kStep, seen0, seen1);
      }
      if constexpr (KDA) {
        const int who = (tb0 / kC + h) & 3;
        if (tb0 < T) kda_operands(buf[0]);
        __syncthreads();
        int form = 0;
        if (tb0 < T) {
          form = form_of(buf[0]);
          kda_products(buf[0], form, who);
        }
        __syncthreads();
        if (tb0 < T) {
          form = with_grows(buf[0], form);
          kda_solve(buf[0], form, tb0, who);
          if (__builtin_expect(form != 0, 0)) kda_restage(buf[0], form);
        }
        __syncthreads();
      }
    };
    staged(0);
    for (int i = 0; i < (KDA ? 1 : 4); ++i) __syncthreads();
#pragma unroll 1
    for (int tb0 = 0; tb0 < T; tb0 += kStep) {
      if constexpr (!KDA) __syncthreads();
      staged(tb0 + kStep);
    }
    for (int i = 0; i < (KIND == kNvfp4 ? 6 : 4); ++i) __syncthreads();
    return;
  }

  // ---- the tile, row slices through LDS into natural channel order: thread
  // t moves columns 16 cg .. + 15 of tile rows t / 8 + 32 i
  const int cg = t & 7, col0 = cg * CPT, rr = t >> 3;
  int u_of[4];
  f16v S[4];
  {
    RowSlice<KIND, CPT> raw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      raw[i] = load_row<KIND, kD, CPT>(tile, codes, meta_bytes, rr + 32 * i, k_hi, col0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = rr + 32 * i;
      u_of[i] = p.perm ? (static_cast<int>(p.perm[static_cast<size_t>(h) * kD + r]) & (kD - 1)) : r;
    }
    float x[4][CPT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      decode_slice<KIND, kD, CPT>(raw[i], tile, codes, meta_bytes, rr + 32 * i, k_hi, cg, col0, had,
                                  x[i]);
    // half the columns at a time: those of waves 2 hf and 2 hf + 1
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if ((cg >> 2) == hf) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q4 = 0; q4 < CPT / 4; ++q4)
            *reinterpret_cast<float4*>(&tbuf[u_of[i]][(col0 & 63) + 4 * q4]) =
                make_float4(x[i][4 * q4], x[i][4 * q4 + 1], x[i][4 * q4 + 2], x[i][4 * q4 + 3]);
      }
      __syncthreads();
      // accumulator register 8 cc + e of block bb: channel 32 bb + 16 cc + 8 ph + e
      if ((wave >> 1) == hf) {
#pragma unroll
        for (int bb = 0; bb < 4; ++bb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            S[bb][i] = tbuf[32 * bb + 16 * (i >> 3) + 8 * ph + (i & 7)][col & 63];
      }
      __syncthreads();
    }
  }

  // ---- one flagged chunk token by token in fp32 (n tokens from token tb):
  // rows of k and q in bf16 and KDA's decays in fp32 from LDS
  auto run_tokens = [&](const typename P::Chunk& ck, int tb, int n) __attribute__((always_inline)) {
    const uint8_t* kq = ck.kq[0];
    const int lane = lane_now(), ph = lane >> 5, col = 32 * wave + (lane & 31);
#pragma unroll 1
    for (int tok = 0; tok < n; ++tok) {
      float w = 0.0f, pq = 0.0f, qk = 0.0f;
      const int at = opaque(row_at(tok, ph));  // of k; q 16 rows on
#pragma unroll
      for (int bb = 0; bb < 4; ++bb)
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          const uint8_t* row = kq + (at ^ ((4 * bb + 2 * cc) << 4));
          const u4v k8 = *reinterpret_cast<const u4v*>(row);
          const u4v q8 = *reinterpret_cast<const u4v*>(row + 16 * kRow);
          float a8[8];
          if constexpr (KDA) {
            const u4v a0 = *reinterpret_cast<const u4v*>(row + sizeof(ck.kq[0]));
            const u4v a1 = *reinterpret_cast<const u4v*>(row + sizeof(ck.kq[0]) + 16 * kRow);
#pragma unroll
            for (int e = 0; e < 8; ++e) a8[e] = __uint_as_float(e & 1 ? a1[e >> 1] : a0[e >> 1]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) a8[e] = ck.a[tok];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float kf = e & 1 ? bf16_hi(k8[e >> 1]) : bf16_lo(k8[e >> 1]);
            const float qf = e & 1 ? bf16_hi(q8[e >> 1]) : bf16_lo(q8[e >> 1]);
            const float x = S[bb][8 * cc + e] * a8[e];
            S[bb][8 * cc + e] = x;
            w = fmaf(kf, x, w);
            pq = fmaf(qf, x, pq);
            qk = fmaf(qf, kf, qk);
          }
        }
      w += __shfl_xor(w, 32, 64);
      pq += __shfl_xor(pq, 32, 64);
      qk += __shfl_xor(qk, 32, 64);
      const float vf = bf16_to_f32(p.v[v_row(tb + tok) * kD + col]);
      const float beta = ck.beta[tok], delta = vf - w;
      if (p.o && ph == 0) write_o(tb + tok, p.scale * fmaf(beta * qk, delta, pq));
      const float bd = beta * delta;
#pragma unroll
      for (int bb = 0; bb < 4; ++bb)
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          const u4v k8 = *reinterpret_cast<const u4v*>(kq + (at ^ ((4 * bb + 2 * cc) << 4)));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float kf = e & 1 ? bf16_hi(k8[e >> 1]) : bf16_lo(k8[e >> 1]);
            S[bb][8 * cc + e] = fmaf(kf, bd, S[bb][8 * cc + e]);
          }
        }
    }
  };


  // ---- one chunk of up to 16 tokens from token tb on this wave's columns
  // (vr: v of tokens 8 ph + e, this lane's column); false, and nothing done, if
  // some R of this wave's columns is not finite (GDN; KDA's flags have v)
  auto run_chunk = [&](const typename P::Chunk& ck, int tb, bool steep,
                       const uint32_t (&vr)[8]) __attribute__((always_inline)) -> bool {
    const int lane = lane_now(), ph = lane >> 5, l32 = lane & 31, col = 32 * wave + l32;
    // rows of the left-hand operands: lane l32 is row m of the 32; m % 16 bits
    // (r, p, i) stand for token (p, r, i), so that a lane's accumulators 0..7
    // (8..15) are tokens 8 ph .. 8 ph + 7 of the first (second) 16 rows
    const int m_tok = 8 * ((l32 >> 2) & 1) + 4 * ((l32 >> 3) & 1) + (l32 & 3);
    const int m_row = (l32 & 16) + m_tok;
    // transposing read of K^T: lane l32 of half ph asks for row s = 8 ph + 4 x + (l32 % 16) / 4,
    // channels 32 bb + 16 (l32 / 16) + 8 p' + 4 r0 with l32 % 4 = 2 r0 + p'
    const int tr_s = 8 * ph + ((l32 >> 2) & 3);
    const int tr_ck = 2 * (l32 >> 4) + (l32 & 1), tr_half = ((l32 >> 1) & 1) * 8;
    auto scale_rows = [&](const float* by) __attribute__((always_inline)) {
#pragma unroll
      for (int bb = 0; bb < 4; ++bb)
#pragma unroll
        for (int c2 = 0; c2 < 4; ++c2) {
          const float4 f = *reinterpret_cast<const float4*>(
              &by[32 * bb + 16 * (c2 >> 1) + 8 * ph + 4 * (c2 & 1)]);
          S[bb][4 * c2] *= f.x;
          S[bb][4 * c2 + 1] *= f.y;
          S[bb][4 * c2 + 2] *= f.z;
          S[bb][4 * c2 + 3] *= f.w;
        }
    };
    // with three workgroups a CU the factors' reads are kept together: mixed
    // with the splits they took one register group in turn (297 -> 292 us at
    // B = 32, 250 tokens); alone on its SIMD a wave is better with the mix
    if constexpr (KDA) scale_rows(steep ? ck.pre_s : ck.pre);
    if constexpr (KDA && !SPLIT) __builtin_amdgcn_sched_barrier(0);
    // [K; Q] S0: accumulators 0..7 are rows k_t, 8..15 rows q_t, t = 8 ph + e
    f16v acc, low;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = low[i] = 0.0f;
    const int a_at = row_at(m_row, ph);  // piece 2 ks + ph: bits 5 and up xor 2 ks
    Split8 sb;
    u4v fa[NA];
    auto step_operands = [&](int ks) __attribute__((always_inline)) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = S[ks >> 1][8 * (ks & 1) + e];
      sb = split8<!KDA>(x);
#pragma unroll
      for (int j = 0; j < NA; ++j)
        fa[j] = *reinterpret_cast<const u4v*>(ck.kq[j] + (a_at ^ (ks << 5)));
    };
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      step_operands(ks);
      mfma32_split<NA>(fa, sb, acc, low);
      // the operands of one step (GDN: two) at a time: registers
      if (KDA || (ks & 1)) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (KDA) {
      if (__builtin_expect(steep, 0)) scale_rows(ck.mid_s);
    }
    if constexpr (KDA) __syncthreads();  // tm is there (SPLIT: the other waves' first step is done)
    // R = V - G K S0; G Q S0 stays in acc[8 + e]
    float R[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float w = acc[e] + low[e];
      acc[8 + e] += low[8 + e];
      if constexpr (KDA) {
        R[e] = bf16_lo(vr[e]) - w;
      } else {
        const float G = ck.G[8 * ph + e];
        R[e] = fmaf(-G, w, bf16_lo(vr[e]));
        acc[8 + e] *= G;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) low[i] = 0.0f;
    {
      const Split8 sr = split8(R);
      Split8 tm;
      if constexpr (KDA) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = ck.tm[m_row][8 * ph + e];
        tm = split8(x);
      } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
          tm.part[j] = *reinterpret_cast<const u4v*>(&ck.tm[j][m_row][8 * ph]);
      }
      low = mfma32_split<3>(tm.part, sr, low);
    }
    // [diag(E) T; B T] is finite, so the first row's product is not finite
    // if any R of the column is not: v is not finite, or K S0 overflows
    if constexpr (!KDA) {
      const bool out = !(fabsf(low[0]) <= FLT_MAX);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(out) != 0, 0)) return false;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      acc[8 + e] += low[8 + e];
      acc[e] = low[e];
    }
    if (p.o) {
      const int o_row = kD * static_cast<int>(o_esize), step = p.HV * o_row;
      const auto ro = rows_rsrc(static_cast<uint8_t*>(p.o) +
                                    ((static_cast<size_t>(b) * T + tb) * p.HV + h) * o_row,
                                step, o_row, T - tb < kC ? T - tb : kC);
      const int at = 8 * ph * step + col * static_cast<int>(o_esize);
      if (p.o_bf16) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(p.scale * acc[8 + e]), ro, at + e * step,
                                                0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(p.scale * acc[8 + e]), ro,
                                                at + e * step, 0, 0);
      }
    }
    if constexpr (KDA && SPLIT) __syncthreads();
    // S = G_C S0 + K^T U
    float U[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) U[e] = acc[e];
    const Split8 su = split8<!KDA>(U);
    float gc = 1.0f;
    if constexpr (!KDA) gc = ck.G[kC - 1];
    typedef __attribute__((address_space(3))) s4v* lds_s4;
    const int tr_at0 = row_at(tr_s, tr_ck) + tr_half, tr_at1 = row_at(tr_s + 4, tr_ck) + tr_half;
#pragma unroll
    for (int bb = 0; bb < 4; ++bb) {
      if constexpr (!KDA) {
#pragma unroll
        for (int i = 0; i < 16; ++i) S[bb][i] *= gc;
      }
      u4v fa[NA];
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const uint8_t* rows;
        if constexpr (KDA) rows = ck.kh[j];
        else rows = ck.kq[0];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const s4v v4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s4)(rows + ((x ? tr_at1 : tr_at0) ^ (bb << 6))));
          const uint2 w2 = __builtin_bit_cast(uint2, v4);
          fa[j][2 * x] = w2.x;
          fa[j][2 * x + 1] = w2.y;
        }
      }
      S[bb] = mfma32_split<NA>(fa, su, S[bb]);
    }
    if constexpr (KDA && !SPLIT) __builtin_amdgcn_sched_barrier(0);
    if constexpr (KDA) scale_rows(steep ? ck.fin_s : ck.fin);
    return true;
  };

  auto load_v = [&](int tb, uint32_t (&vr)[8]) __attribute__((always_inline)) {
    const auto rv = rows_rsrc(p.v + ((tok0 + tb) * p.HV + h) * kD, v_step, kRow,
                              T - tb < kC ? T - tb : kC);
    const int lane = lane_now(), v_at = 8 * (lane >> 5) * v_step + 2 * (32 * wave + (lane & 31));
#pragma unroll
    for (int e = 0; e < 8; ++e)
      vr[e] = __builtin_amdgcn_raw_buffer_load_b16(rv, e * v_step + v_at, 0, 0);
  };
  auto run = [&](const typename P::Chunk* buf, int tb0) __attribute__((always_inline)) {
#pragma unroll 1
    for (int c = 0; c < NC && tb0 + kC * c < T; ++c) {
      const int tb = tb0 + kC * c, n = T - tb < kC ? T - tb : kC;
      uint32_t vr[8];
      if constexpr (KDA && !SPLIT) {
#pragma unroll
        for (int e = 0; e < 8; ++e) vr[e] = in.v[KDA ? e : 0];
      } else {
        load_v(tb, vr);
      }
      bool done = false;
      const int form = with_grows(buf[c], form_of(buf[c]));
      if ((form & kTokens) == 0) done = run_chunk(buf[c], tb, (form & kSteep) != 0, vr);
      if (__builtin_expect(!__builtin_amdgcn_readfirstlane(done ? 1 : 0), 0)) {
        run_tokens(buf[c], tb, n);
        if constexpr (KDA && SPLIT) {  // those of run_chunk
          __syncthreads();
          __syncthreads();
        }
      }
    }
  };
  if constexpr (!SPLIT) {
#pragma unroll 1
    for (int tb0 = 0; tb0 < T; tb0 += kStep) {
      asm volatile("" ::"v"(seen0), "v"(seen1));
      stage(L, tb0);
      if constexpr (KDA) {
        const int who = (tb0 / kC + h) & 3;
        kda_operands(L[0]);
        __syncthreads();
        int form = form_of(L[0]);
        kda_products(L[0], form, who);
        __syncthreads();
        if (__builtin_expect(form != 0, 0)) {
          form = with_grows(L[0], form);
          kda_restage(L[0], form);
          __syncthreads();
        }
        kda_solve(L[0], form, tb0, who);  // the other waves start on the chunk
      } else {
        __syncthreads();
      }
      if (tb0 + kStep < T) touch(tb0 + kStep, seen0, seen1);
      run(L, tb0);
      __syncthreads();
    }
  } else {
#pragma unroll 1
    for (int tb0 = 0; tb0 < T; tb0 += kStep) {
      if constexpr (!KDA) __syncthreads();  // staged
      run(L + (tb0 / kStep & 1) * NC, tb0);
      if constexpr (KDA) __syncthreads();
    }
  }

  // ---- store the final state per its tier, as it came
  const int rs = opaque(rr), cs = opaque(cg), ps = opaque(ph);
  float x[4][CPT];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    if ((wave >> 1) == hf) {
#pragma unroll
      for (int bb = 0; bb < 4; ++bb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          tbuf[32 * bb + 16 * (i >> 3) + 8 * ps + (i & 7)][col & 63] = S[bb][i];
    }
    __syncthreads();
    if ((cs >> 2) == hf) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q4 = 0; q4 < CPT / 4; ++q4) {
          const float4 v4 =
              *reinterpret_cast<const float4*>(&tbuf[u_of[i]][16 * (cs & 3) + 4 * q4]);
          x[i][4 * q4] = v4.x;
          x[i][4 * q4 + 1] = v4.y;
          x[i][4 * q4 + 2] = v4.z;
          x[i][4 * q4 + 3] = v4.w;
        }
    }
    __syncthreads();
  }
  float s_g = 1.0f;
  if constexpr (KIND == kNvfp4) {  // the global scale of the final low tier
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (rs + 32 * i >= k_hi)
#pragma unroll
        for (int j = 0; j < CPT; ++j) amax = fmaxf(amax, fabsf(x[i][j]));
    s_g = nvfp4_global(block_max<256>(amax));
    if (t == 0) store_global_scale<kD>(meta_bytes, k_hi, s_g);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    encode_row<KIND, kD, CPT, TPR>(x[i], rs + 32 * i, k_hi, cs, 16 * cs, tile, codes, meta_bytes, had,
                                   s_g);
}

// A CU (256 of them, fewer in a partition of the device) holds one eight-wave
// workgroup or three of four waves. While every tile has a CU to itself, a
// wave's own instruction rate is what counts (one in 5 cycles, whatever else the
// CU could do), so staging beside the chunks pays; with more tiles the second
// round it costs does not. One to eight requests of 32 heads (up to 256 tiles),
// 1024 tokens: GDN 181-186 -> 135-137 us, KDA 402-404 -> 280-283; 8 tokens:
// 10.3-11.4 -> 10.3-10.5 and 12.2-13.3 -> 11.4-12.5 (the first chunks are staged
// while the tile arrives). Twelve requests (384 tiles), 250 tokens: GDN 71 ->
// 84, KDA 136 -> 152.
bool split_waves(int64_t tiles) {
  static std::atomic<int> cus_of[16];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return false;
  int cus = cus_of[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return false;
    cus_of[dev].store(cus, std::memory_order_relaxed);
  }
  return tiles <= cus;
}

template <int KIND, bool KDA>
void launch_kind(const PrefillParams& p, int B, hipStream_t stream) {
  const dim3 grid(p.HV, B);
  if (split_waves(static_cast<int64_t>(B) * p.HV))
    hipLaunchKernelGGL((prefill_chunk128<KIND, KDA, true>), grid, dim3(512), 0, stream, p);
  else
    hipLaunchKernelGGL((prefill_chunk128<KIND, KDA, false>), grid, dim3(256), 0, stream, p);
}
template <int KIND>
void launch_kind(bool kda, const PrefillParams& p, int B, hipStream_t stream) {
  if (kda) launch_kind<KIND, true>(p, B, stream);
  else launch_kind<KIND, false>(p, B, stream);
}

}  // namespace

void launch_prefill_chunk128(int codec, bool kda, const PrefillParams& p, int B,
                             hipStream_t stream) {
  switch (codec) {
    case kCodecFp32: launch_kind<kFp32>(kda, p, B, stream); break;
    case kCodecPaper: launch_kind<kPaper>(kda, p, B, stream); break;
    case kCodecInt4: launch_kind<kInt4>(kda, p, B, stream); break;
    case kCodecFp8: launch_kind<kFp8>(kda, p, B, stream); break;
    case kCodecNvfp4: launch_kind<kNvfp4>(kda, p, B, stream); break;
    default: launch_kind<kMixed>(kda, p, B, stream); break;
  }
}

}  // namespace damp
