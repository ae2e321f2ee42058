// Matrix products staged through registers (gfx950): the fp32 products, and
// the bf16 ones whose operands the direct kernel cannot load (rows that are
// not whole aligned 16-byte chunks, operands still in fp32).
//
//     C[M,N] = sum_k A(m,k) B(n,k),  fp32 result
//
// Both use the bf16 matrix instruction; bf16 products round their operands
// (RNE) into one plane, fp32 products split theirs into three.
//
// The fp32 matrix instruction (v_mfma_f32_32x32x2_f32) runs at a sixteenth
// of the bf16 one's rate.  An fp32 value is exactly the sum of three bf16
// values: a = a1 + a2 + a3 with a1 = bf16(a), a2 = bf16(a - a1),
// a3 = a - a1 - a2 (24 significant bits in three signed parts of 8; both
// differences are exact).  A product then takes six bf16 matrix
// instructions:
//     a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + O(2^-24 |a b|)
// each an exact product of 8-bit significands summed in fp32.  The terms left
// out, a2 b3 + a3 b2 + a3 b3, are at most 2^-24 |a b| (|a2| <= 2^-8 |a|, |a3|
// <= 2^-17 |a|), as much as rounding a b to fp32, and a quarter of that as a
// mean square over normal values (0.10 against 0.42 of 2^-24); a 16-k slab is
// rounded into the accumulator 6 times instead of 8.
//
// The matrix instruction rounds to nearest, but where its products exceed
// the accumulator it drops the accumulator's low bits, always downwards: a
// sum comes out about 1e-8 of its scale too small, a tenth of its rounding
// error but with the same sign in every element, which sums over many
// elements carry (the v gradients over 12,800 tokens: 3.3e-6 off instead of
// 8.5e-7).  So each row of A, and with it the row's results, is negated or
// not, at random as far as the remainder is concerned, which then does not
// add up.  For a K-contiguous A 16 values decide, by the parity of their bits:
// four groups of four spread evenly over the row, so that leading features
// that are constant, or zero, do not give every row one sign (with the first
// four values alone, and those zero in every row, the mean error over 12,800
// rows of 1000 values was 15 standard errors from zero; eight groups instead
// of four cost 2 % more of a product).  The row's values
// alone decide: its results, where K is not split, are the same bits wherever
// it stands, however a sequence is cut into calls.  For a row-contiguous A (a
// sum over tokens) the row's index decides.
//
// The parts are formed once per tile, between the global loads and LDS: the
// tile's three planes lie in LDS as bf16 [rows][BK + 8], so a fragment of a
// plane is one 16-byte read.
//
// Bound by the matrix units where tiles fill the chip (1.3 PFLOP/s of bf16
// products, what the library's large bf16 products reach), by the latency of
// a step (load, split, LDS, six dependent products) where they do not.
// Against the fp32 instruction on 128 x 128 tiles: 16384 x 3072 x 1024 takes 905 -> 475 us,
// 3072 x 1024 over 16384 tokens 940 -> 516 us with its split sum, 2048 x 768
// x 256 24.7 -> 13.6 us.
//
// Every fp32 value is a multiple of 2^-149, but bf16's smallest is 2^-133 and
// its smallest normal value 2^-126: below 2^-110 the parts would lose bits
// (2.7e-3 of a product of values around 1e-38).  So both operands are
// multiplied by 2^24, which makes every part a normal number, and the results
// by 2^-48, both exact but for results below 2^-126, which round once.  (The
// row's sign rides on A's factor; the multiplication costs 0 to 3 % of a
// product: 16384 x 3072 x 1024 467 us with and without, 4096 x 3072 x 1024
// 147 -> 150 us.)
//
// A value that is not finite after this (infinities, NaN, magnitudes above
// 2^103 = 1e31) turns its second part, and so every result it enters, into
// NaN, and results above 2^79 may overflow.  A wave that finds a result that
// is not finite therefore computes the 32 rows that hold one again with the
// fp32 matrix instruction, and writes these results alone: they are fp32
// arithmetic's own, and the finite ones beside them keep their bits.
#include <algorithm>

#include "sru_gemm_tile.h"
#include "sru_internal.h"

namespace sru {
namespace {

// Loads of the operands: buffer loads of whole aligned chunks of four
// elements, buffer loads of single elements (any alignment and extent), or
// plain loads with 64-bit offsets (panels beyond the buffer offsets' 2 GiB).
enum LoadMode { kChunk, kSingle, kPlain };

// NP: bf16 planes per operand (3: fp32 products, 1: bf16 products).
template <int NP_, int BM_, int BN_, int BK_, int WAVES_M_, int WAVES_N_, int D_>
struct FCfg {
  static constexpr int NP = NP_, BM = BM_, BN = BN_, BK = BK_, D = D_;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, WAVES = WAVES_M * WAVES_N;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int FM = WM / 32, FN = WN / 32;
  static constexpr int THREADS = WAVES * 64;
  // bytes of an LDS row.  16 bytes of padding keep the 16 rows of a fragment
  // read on distinct banks.
  static constexpr int ROWB = 2 * BK + 16;
  static constexpr int A_PLANE = BM * ROWB, B_PLANE = BN * ROWB;
  static constexpr int STAGE = NP * (A_PLANE + B_PLANE);
  static constexpr int LDS = 2 * STAGE;  // two buffers
  static_assert(LDS <= 160 * 1024 && BK % 16 == 0 && WM % 32 == 0 && WN % 32 == 0, "tile");
};

constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;  // factors of the operands, the results

// x, negated where r has an odd number of bits.  Row r of a row-contiguous A:
// the Thue-Morse sequence.
__device__ __forceinline__ float signed_by(float x, unsigned r) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) ^
                                       ((unsigned)__builtin_popcount(r) << 31));
}

// Two values' parts, packed per plane.  Three parts: of the values times f.
template <int NP>
__device__ __forceinline__ void split_pair(float x, float y, float f, unsigned (&p)[NP]) {
  if constexpr (NP == 3) {
    x *= f;
    y *= f;
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    p[i] = pack_bf16(x, y);
    if (i < NP - 1) {
      x -= __builtin_bit_cast(float, p[i] << 16);
      y -= __builtin_bit_cast(float, p[i] & 0xFFFF0000u);
    }
  }
}

// The elements of one chunk of four (element e is valid when e < valid), as
// loaded: fp32 one per register; bf16 two per register (kChunk) or one.
template <int MODE, class S>
__device__ __forceinline__ u32x4 load_chunk(__amdgpu_buffer_rsrc_t rs, const S* src,
                                            long long idx, unsigned off, int valid) {
  u32x4 v;
  if constexpr (MODE == kChunk && sizeof(S) == 4) {
    v = buf_load16(rs, valid > 0 ? off : kOOB);
  } else if constexpr (MODE == kChunk) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, valid > 0 ? off : kOOB, 0, 0);
    v[0] = w[0];
    v[1] = w[1];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = e < valid;
      if constexpr (MODE == kPlain)
        v[e] = ok ? __builtin_bit_cast(
                        std::conditional_t<sizeof(S) == 4, unsigned, uint16_t>, src[ok ? idx + e : 0])
                  : 0u;
      else if constexpr (sizeof(S) == 4)
        v[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, ok ? off + 4u * e : kOOB, 0, 0);
      else
        v[e] = __builtin_amdgcn_raw_buffer_load_b16(rs, ok ? off + 2u * e : kOOB, 0, 0);
    }
  }
  return v;
}

// Element e of a loaded chunk as fp32.
template <int MODE, class S>
__device__ __forceinline__ float elem(const u32x4& v, int e) {
  if constexpr (sizeof(S) == 4) {
    return f32_of(v, e);
  } else if constexpr (MODE == kChunk) {
    const unsigned w = v[e >> 1];
    return __builtin_bit_cast(float, e & 1 ? w & 0xFFFF0000u : w << 16);
  } else {
    const unsigned w = v[e];
    return __builtin_bit_cast(float, w << 16);
  }
}

// K-contiguous operand: element (r, k) at src[r*ld + k].  A thread owns
// chunks of four k of one row.
template <class C, int R, int MODE, class S>
struct FLoadKC {
  static constexpr int ES = sizeof(S);
  static constexpr int CPR = C::BK / 4;
  static constexpr int PER = R * CPR / C::THREADS;
  static_assert(R * CPR % C::THREADS == 0, "tile splits evenly over the threads");
  struct Regs {
    u32x4 v[PER];
  };
  unsigned off[PER];  // bytes from (row r0, the stage's k); rows clamped to the last
  float factor[PER];   // kUp with the sign of the chunk's row (signs())
  int r0, rows;
  long long ld, bytes;
  const S* src;

  __device__ __forceinline__ void init(const S* s, long long ld_, int r0_, int rows_, int K,
                                       int tid) {
    src = s;
    ld = ld_;
    r0 = r0_;
    rows = rows_;
    bytes = ES * ((long long)(rows - 1) * ld + K);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      const int r = min(c / CPR, rows - 1 - r0);
      off[i] = (unsigned)(((long long)r * ld + (c % CPR) * 4) * ES);
    }
  }
  // The rows' signs, on the factors of the split and (table) the results: of
  // the 4 sampled chunks of a row each of its threads loads one.
  __device__ __forceinline__ void signs(float* table, int K, int tid) {
    static_assert(CPR % 4 == 0 && 64 % CPR == 0, "a row's threads are neighbours in a wave");
    const long long base = ES * (long long)r0 * ld;
    const __amdgpu_buffer_rsrc_t rs = panel_rsrc(src, base, bytes);
    const int step = K >= 16 ? (K + 3) / 4 / 4 : 1;  // chunks from one sample to the next
    u32x4 v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      const int k = (c % 4) * step * 4;
      v[i] = load_chunk<MODE, S>(rs, src, (long long)min(r0 + c / CPR, rows - 1) * ld + k,
                                 off[i] + (unsigned)((k - (c % CPR) * 4) * ES), K - k);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      unsigned bits = v[i][0] ^ v[i][1] ^ v[i][2] ^ v[i][3];
      bits ^= __shfl_xor(bits, 1);
      bits ^= __shfl_xor(bits, 2);
      factor[i] = signed_by(kUp, bits);
      if (c % CPR == 0) table[c / CPR] = signed_by(kDown, bits);
    }
  }
  __device__ __forceinline__ void load(Regs& g, int k0, int kend, int tid) const {
    const long long base = ES * ((long long)r0 * ld + k0);
    const __amdgpu_buffer_rsrc_t rs = panel_rsrc(src, base, max(bytes, base));
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      const int k = k0 + (c % CPR) * 4;
      const long long idx = (long long)min(r0 + c / CPR, rows - 1) * ld + k;
      g.v[i] = load_chunk<MODE, S>(rs, src, idx, off[i], kend - k);
    }
  }
  // SIGN: the rows take their signs.
  template <bool SIGN>
  __device__ __forceinline__ void store(const Regs& g, unsigned char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      unsigned char* dst = lds + (c / CPR) * C::ROWB + (c % CPR) * 8;
      unsigned p[2][C::NP];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        split_pair(elem<MODE, S>(g.v[i], 2 * h), elem<MODE, S>(g.v[i], 2 * h + 1),
                   SIGN ? factor[i] : kUp, p[h]);
#pragma unroll
      for (int q = 0; q < C::NP; ++q) {
        u32x2 w;
        w[0] = p[0][q];
        w[1] = p[1][q];
        *reinterpret_cast<u32x2*>(dst + q * R * C::ROWB) = w;
      }
    }
  }
};

// Row-contiguous operand: element (r, k) at src[k*ld + r].  A thread owns KB
// k-rows of four rows and transposes them on the way into LDS; consecutive
// threads take consecutive k-blocks of the same rows.
template <class C, int R, int MODE, class S>
struct FLoadRC {
  static constexpr int ES = sizeof(S);
  static constexpr int KB = R * C::BK / 16 >= C::THREADS ? 4 : 2;
  static constexpr int NKB = C::BK / KB;
  static constexpr int PER = (R / 4) * NKB / C::THREADS;
  static_assert((R / 4) * NKB % C::THREADS == 0 && PER > 0, "tile splits evenly over the threads");
  struct Regs {
    u32x4 v[PER][KB];
  };
  unsigned off[PER];  // bytes from (row r0, the stage's k)
  float factor[PER];   // kUp with the sign of the block's first row (signs())
  int r0, rows;
  long long ld, bytes;
  const S* src;

  __device__ __forceinline__ void init(const S* s, long long ld_, int r0_, int rows_, int K,
                                       int tid) {
    src = s;
    ld = ld_;
    r0 = r0_;
    rows = rows_;
    bytes = ES * ((long long)(K - 1) * ld + rows);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      off[i] = (unsigned)(((long long)(c % NKB) * KB * ld + (c / NKB) * 4) * ES);
    }
  }
  __device__ __forceinline__ void signs(float* table, int, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      factor[i] = signed_by(kUp, r0 + (tid + i * C::THREADS) / NKB * 4);
    if (tid < R) table[tid] = signed_by(kDown, r0 + tid);
  }
  __device__ __forceinline__ void load(Regs& g, int k0, int kend, int tid) const {
    const long long base = ES * ((long long)k0 * ld + r0);
    const __amdgpu_buffer_rsrc_t rs = panel_rsrc(src, base, max(bytes, base));
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
      const int r = r0 + (c / NKB) * 4;
#pragma unroll
      for (int kk = 0; kk < KB; ++kk) {
        const int k = k0 + (c % NKB) * KB + kk;
        g.v[i][kk] = load_chunk<MODE, S>(rs, src, (long long)k * ld + r,
                                      off[i] + (unsigned)(kk * ld * ES), k < kend ? rows - r : 0);
      }
    }
  }
  // SIGN: the rows take their signs.
  template <bool SIGN>
  __device__ __forceinline__ void store(const Regs& g, unsigned char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = tid + i * C::THREADS;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        unsigned char* dst = lds + ((c / NKB) * 4 + e) * C::ROWB + (c % NKB) * 2 * KB;
        unsigned p[KB / 2][C::NP];
#pragma unroll
        for (int h = 0; h < KB / 2; ++h)  // (r0 and the block are multiples of 4)
          split_pair(elem<MODE, S>(g.v[i][2 * h], e), elem<MODE, S>(g.v[i][2 * h + 1], e),
                     SIGN ? signed_by(factor[i], e) : kUp, p[h]);
#pragma unroll
        for (int q = 0; q < C::NP; ++q) {
          if constexpr (KB == 4) {
            u32x2 w;
            w[0] = p[0][q];
            w[1] = p[1][q];
            *reinterpret_cast<u32x2*>(dst + q * R * C::ROWB) = w;
          } else {
            *reinterpret_cast<unsigned*>(dst + q * R * C::ROWB) = p[0][q];
          }
        }
      }
    }
  }
};

// Workgroup barrier that waits for this wave's LDS accesses only: the fence
// of __syncthreads would also drain the loads of the stages ahead.
__device__ __forceinline__ void lds_only_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) (vmcnt 63, expcnt 7)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The FN 32 x 32 blocks of results from (m0, n0) on, already written, over k in
// [kbeg, kend) on the fp32 instruction, put where the results are not finite.
// One wave; operands straight from memory, 16 k in flight.  (No result
// finite, 16384 x 3072 x 1024: 1.7 ms; block by block 5.8, whole tiles through
// LDS 1.2.  One row: 0.67 ms, of 0.83 with whole tiles.)
template <bool A_KC, bool B_KC, int FN>
__device__ __forceinline__ void fp32_blocks(const KernelArgs& g, int m0, int n0, int kbeg,
                                            int kend, int lane, int split) {
  float* out = g.out + (long long)split * g.split_stride;
  const int n = n0 + (lane & 31), mb = m0 + (lane >> 5) * 4;
  auto row = [&](int e) { return mb + (e >> 2) * 8 + (e & 3); };
  auto finite = [](float x) { return x * 0.f == 0.f; };
  bool bad = false;
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (row(e) < g.M && n + 32 * j < g.N)
        bad |= !finite(out[(long long)row(e) * g.ldo + n + 32 * j]);
  if (__ballot(bad) == 0) return;
  // rows and columns past the end repeat the last: their results are not used
  const long long ar = min(m0 + (lane & 31), g.M - 1);
  const float* ap = static_cast<const float*>(g.A) + (A_KC ? ar * g.lda : ar);
  const float* bp[FN];
  floatx16 acc[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const long long br = min(n + 32 * j, g.N - 1);
    bp[j] = static_cast<const float*>(g.B) + (B_KC ? br * g.ldb : br);
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
  }
  // a half wave takes 8 consecutive k of 16
  auto step = [&](auto whole, int k0) {
    constexpr bool WHOLE = decltype(whole)::value;
    float af[8], bf[FN][8];
    const int kl = k0 + (lane >> 5) * 8;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const long long k = WHOLE ? kl + s : min(kl + s, kend - 1);
      const bool in = WHOLE || kl + s < kend;
      const float x = ap[A_KC ? k : k * g.lda];
      af[s] = in ? x : 0.f;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const float y = bp[j][B_KC ? k : k * g.ldb];
        bf[j][s] = in ? y : 0.f;
      }
    }
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[s], bf[j][s], acc[j], 0, 0, 0);
  };
  int k0 = kbeg;
  for (; k0 + 16 <= kend; k0 += 16) step(std::true_type{}, k0);
  if (k0 < kend) step(std::false_type{}, k0);
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = row(e), nj = n + 32 * j;
      if (m < g.M && nj < g.N) {
        float* o = out + (long long)m * g.ldo + nj;
        const float* add = g.add + (long long)m * g.add_ld + nj;
        float v = acc[j][e];
        if (g.add_count > 0) v += add[0];
        if (g.add_count > 1) v += add[g.add_off];
        if (!finite(*o)) *o = v;
      }
    }
}

// Workgroup w of a product's nwg.  smem: C::LDS bytes; row_factors: C::BM words
// (fp32 products).
template <class C, bool A_KC, bool B_KC, int MODE, class S>
__device__ __forceinline__ void staged_tile(const KernelArgs& g, int w, int nwg,
                                            unsigned char* smem, float* row_factors) {
  const TileIdx ti = tile_of(g, w, nwg);
  const int m0 = ti.tm * C::BM;
  const int n0 = ti.tn * C::BN;
  const int kbeg = ti.split * g.k_per_split;
  const int kend = min(g.K, kbeg + g.k_per_split);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm0 = (wave / C::WAVES_N) * C::WM;
  const int wn0 = (wave % C::WAVES_N) * C::WN;

  using LA = std::conditional_t<A_KC, FLoadKC<C, C::BM, MODE, S>, FLoadRC<C, C::BM, MODE, S>>;
  using LB = std::conditional_t<B_KC, FLoadKC<C, C::BN, MODE, S>, FLoadRC<C, C::BN, MODE, S>>;
  LA la;
  LB lb;
  la.init(static_cast<const S*>(g.A), g.lda, m0, g.M, g.K, tid);
  lb.init(static_cast<const S*>(g.B), g.ldb, n0, g.N, g.K, tid);

  // low: a second accumulator for the five small terms in the sums over
  // tokens where registers allow (one MFMA tile per wave): a slab then rounds
  // the sum once instead of 6 times.  (Not in the other products, whose
  // results are the same bits in every tile.)
  constexpr bool F32 = C::NP == 3;
  constexpr bool LOW = F32 && C::FM * C::FN == 1 && !A_KC;
  floatx16 acc[C::FM][C::FN], low;
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    if constexpr (LOW) low = acc[0][0];
  };
  clear();

  // Pipeline: the loads of stages k + 1 .. k + D are in flight (D register
  // sets) while the matrix instructions run stage k from one LDS buffer;
  // stage k + 1 is then split into the other.  Stages past the end load
  // zeros (out-of-range offsets), so no branch separates the loads.
  typename LA::Regs ra[C::D];
  typename LB::Regs rb[C::D];
  const int nk = (kend - kbeg + C::BK - 1) / C::BK;
  auto load = [&](int p, int kt) {
    la.load(ra[p], kbeg + kt * C::BK, kend, tid);
    lb.load(rb[p], kbeg + kt * C::BK, kend, tid);
  };
  auto store = [&](int p, int kt) {
    unsigned char* s = smem + (kt & 1) * C::STAGE;
    la.template store<F32>(ra[p], s, tid);
    lb.template store<false>(rb[p], s + C::NP * C::A_PLANE, tid);
  };
  auto compute = [&](int kt) {
    const unsigned char* As = smem + (kt & 1) * C::STAGE;
    const unsigned char* Bs = As + C::NP * C::A_PLANE;
#pragma unroll
    for (int ks = 0; ks < C::BK; ks += 16) {
      const int ko = (ks + (lane >> 5) * 8) * 2;
      bf16x8 af[C::FM][C::NP], bf[C::FN][C::NP];
#pragma unroll
      for (int q = 0; q < C::NP; ++q) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
          af[i][q] = *reinterpret_cast<const bf16x8*>(
              As + q * C::A_PLANE + (wm0 + i * 32 + (lane & 31)) * C::ROWB + ko);
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
          bf[j][q] = *reinterpret_cast<const bf16x8*>(
              Bs + q * C::B_PLANE + (wn0 + j * 32 + (lane & 31)) * C::ROWB + ko);
      }
      // the small terms first
      constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
      for (int q = F32 ? 0 : 5; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
          for (int j = 0; j < C::FN; ++j) {
            floatx16& c = LOW && q < 5 ? low : acc[i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i][PA[q]], bf[j][PB[q]], c, 0, 0, 0);
          }
    }
  };

#pragma unroll
  for (int p = 0; p < C::D; ++p) load(p, p);
  if constexpr (F32) la.signs(row_factors, g.K, tid);
  store(0, 0);
  lds_only_barrier();
  for (int k0 = 0; k0 < nk; k0 += C::D) {
#pragma unroll
    for (int p = 0; p < C::D; ++p) {
      const int kt = k0 + p;
      if (kt < nk) {
        load(p, kt + C::D);
        __builtin_amdgcn_sched_barrier(0);
        compute(kt);
        store((p + 1) % C::D, kt + 1);
        lds_only_barrier();
      }
    }
  }

  if constexpr (F32) {
    if constexpr (LOW) acc[0][0] += low;
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float f = row_factors[wm0 + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)];
#pragma unroll
        for (int j = 0; j < C::FN; ++j) acc[i][j][e] *= f;
      }
  }
  float z = 0.f;  // NaN where a result is not finite
  if constexpr (F32) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) z = fmaf(acc[i][j][e], 0.f, z);
  }
  if (g.add_count == 0) write_tile_add<C, 0>(g, acc, m0, n0, wm0, wn0, lane, ti.split);
  else if (g.add_count == 1) write_tile_add<C, 1>(g, acc, m0, n0, wm0, wn0, lane, ti.split);
  else write_tile_add<C, 2>(g, acc, m0, n0, wm0, wn0, lane, ti.split);
  if constexpr (F32) {
    if (__ballot(!(z == 0.f)) != 0) {
      for (int i = 0; i < C::FM; ++i)
        fp32_blocks<A_KC, B_KC, C::FN>(g, m0 + wm0 + i * 32, n0 + wn0, kbeg, kend, lane, ti.split);
    }
  }
}

template <class C, bool A_KC, bool B_KC, int MODE, class S>
__global__ __launch_bounds__(C::THREADS, 2) void gemm_staged_kernel(KernelArgs g) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::LDS];
  __shared__ float row_factors[C::NP == 3 ? C::BM : 1];
  staged_tile<C, A_KC, B_KC, MODE, S>(g, blockIdx.x, gridDim.x, smem, row_factors);
}

// dX (n1 workgroups; W read as it lies, row-contiguous, so bf16 needs no
// transposed copy) and dW (n2) in one launch, the one of longer workgroups
// first.
template <class C, class S>
__global__ __launch_bounds__(C::THREADS, 2) void gemm_staged_pair_kernel(KernelArgs g1, int n1,
                                                                         KernelArgs g2, int n2,
                                                                         bool dw_first) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::LDS];
  __shared__ float row_factors[C::NP == 3 ? C::BM : 1];
  const PairIdx p = pair_index(n1, n2, dw_first);
  if (p.dx) staged_tile<C, true, false, kChunk, S>(g1, p.w, n1, smem, row_factors);
  else staged_tile<C, false, false, kChunk, S>(g2, p.w, n2, smem, row_factors);
}

// Tiles.  Big: 8 waves of 64 x 128, one workgroup per CU; fewest bytes and
// LDS reads per operation.  Mid: 4 waves of 64 x 64, two workgroups per CU.
// Small: 4 waves of 32 x 32, two per CU, for products of few tiles.
template <int NP>
using FBig = FCfg<NP, 256, 256, NP == 3 ? 16 : 32, 4, 2, 2>;
template <int NP>
using FMid = FCfg<NP, 128, 128, NP == 3 ? 16 : 32, 2, 2, 2>;
template <int NP>
using FSmall = FCfg<NP, 64, 64, NP == 3 ? 32 : 64, 2, 2, 2>;

// The tile for loads of single elements.  They take a register each, also in
// bf16: with two stages in flight the big bf16 tile spilled 138 to 240 of them
// to memory, so there one stage is in flight.  8733 x 7792 x 209 368 -> 182
// us, 16384 x 903 x 301 116 -> 48, 7792 x 209 over 8733 tokens 205 -> 141.
template <class C>
using SingleCfg = FCfg<C::NP, C::BM, C::BN, C::BK, C::WAVES_M, C::WAVES_N,
                       C::NP == 1 && C::BM == 256 ? 1 : C::D>;

// Time of a product in us: per 16 k, one time for a workgroup alone on its CU
// and one for each of several, and what a workgroup's start and end add; a
// split adds its partials' traffic and the launch that sums them.  From times
// measured over K 128 .. 16384, M 128 .. 16384.  fp32: 16384 x 3072 x 1024
// runs at 217 TFLOP/s on Big, 182 on Mid, 129 on Small (the fp32
// instruction: 114); 2048 x 768 x 256 takes 35, 18.5 and 13.6 us (24); 128 x
// 384 x 128 24, 12 and 6.4 us (14.3).  bf16 (before: one 256 x 256 tile,
// element-wise loads where rows were no whole 16-byte chunks): 1001 x 1600 x
// 300 9.1 us (31.5 with fp32 operands, 92 with bf16 ones), 12800 x 900 x 300
// 27 (35), 4000 x 771 x 257 21 (80), 16384 x 3072 x 1024 143 (208).
struct TileCost {
  int bm, bn, bk;
  double base_alone, alone, base_shared, shared;
};
constexpr TileCost kTilesF32[3] = {{256, 256, FBig<3>::BK, 7.0, 2.35, 7.0, 2.4},
                                   {128, 128, FMid<3>::BK, 4.0, 0.90, 2.0, 0.74},
                                   {64, 64, FSmall<3>::BK, 3.0, 0.33, 1.5, 0.25}};
constexpr TileCost kTilesBf16[3] = {{256, 256, FBig<1>::BK, 7.0, 0.80, 7.0, 0.80},
                                    {128, 128, FMid<1>::BK, 4.0, 0.30, 2.0, 0.25},
                                    {64, 64, FSmall<1>::BK, 3.0, 0.15, 1.5, 0.10}};
// Loads of single elements, on every tile the bound of a step: by precision and
// layout of A.  Of 58 sizes each (rows of 16 to 1,500 odd elements, up to
// 30,000 tokens) every tile's times lie within 4 to 7 % of these (Small at few
// steps 20 %).  With the chunk loads' times above the plan put sums over tokens
// on Small tiles, whose element loads cost most: 3612 x 301 over 2048 tokens in
// bf16 166 us, now 49 and 10 more for the split sum; 9264 x 186 over 2884 245
// and 11, now 70 and 25; 7064 x 405 over 670 in fp32 113, now 48 and 20 more.
constexpr TileCost kTilesSingle[2][2][3] = {
    {{{256, 256, FBig<3>::BK, 9.5, 2.4, 6.0, 2.45},   // fp32, row-contiguous A
      {128, 128, FMid<3>::BK, 6.5, 1.05, 2.5, 0.83},
      {64, 64, FSmall<3>::BK, 2.3, 0.76, 1.5, 0.63}},
     {{256, 256, FBig<3>::BK, 12.5, 2.8, 9.7, 3.1},   // K-contiguous
      {128, 128, FMid<3>::BK, 7.5, 1.5, 3.0, 1.24},
      {64, 64, FSmall<3>::BK, 4.8, 0.54, 2.5, 0.41}}},
    {{{256, 256, FBig<1>::BK, 7.8, 1.58, 4.5, 1.58},  // bf16
      {128, 128, FMid<1>::BK, 4.8, 0.70, 1.0, 0.65},
      {64, 64, FSmall<1>::BK, 2.0, 0.65, 1.5, 0.61}},
     {{256, 256, FBig<1>::BK, 11.2, 1.41, 9.7, 1.57},
      {128, 128, FMid<1>::BK, 7.7, 0.70, 3.0, 0.66},
      {64, 64, FSmall<1>::BK, 3.5, 0.28, 1.9, 0.23}}}};
const TileCost& tile_cost(const GemmDesc& g, int t) { return (g.bf16 ? kTilesBf16 : kTilesF32)[t]; }
// ... with the loads that the extents ask for (pitches and alignments are not
// known when a workspace is sized)
const TileCost& load_cost(const GemmDesc& g, int t) {
  const bool chunks = (g.a_kc ? g.K : g.M) % 4 == 0 && (g.b_kc ? g.K : g.N) % 4 == 0;
  return chunks ? tile_cost(g, t) : kTilesSingle[g.bf16][g.a_kc][t];
}
constexpr double kSumLaunch = 4.0, kBytesPerUs = 4.5e6;

struct Plan {
  int tile, splits;
};

// The product over all tokens (row-contiguous A) is split, for fp32 into
// chains of at most 2048 terms, and others where the caller gives room for partials
// (kc_split).  The fp32 Big and Mid tiles round 6 times per 16 k, so on few
// output tiles, where the sum has many short chains anyway, they keep to
// chains of about 1/380 of the terms times the 128 x 128 tiles; Small rounds
// once.  The choice depends on the sizes alone, so a workspace sized from it
// fits whatever the pointers and pitches are.
//
// A K-contiguous product is split only where its 128 x 128 tiles fill at most
// a quarter of the CUs, and only dX asks for it: U does not depend on M, so
// that a sequence cut into calls gives one call's bits.
struct SplitRange {
  int lo, hi;
};
SplitRange split_range(const GemmDesc& g, int t) {
  const int mid_tiles = (int)std::min<long long>(
      ((g.M + 127LL) / 128) * ((g.N + 127LL) / 128), 1 << 20);
  int lo = 1, hi = 1;
  if (!g.a_kc && !g.bf16) {
    lo = (g.K + 2047) / 2048;
    if (t < 2) lo = std::max(lo, std::min({48, g.K / 128, (384 + mid_tiles - 1) / mid_tiles}));
  }
  if (!g.a_kc || (g.kc_split && mid_tiles <= 64))
    hi = std::max(lo, std::min(64, (g.K + tile_cost(g, t).bk - 1) / tile_cost(g, t).bk / 4));
  return {lo, hi};
}
// every count up to 6, then steps of a third or less
int next_split(int s) { return s + std::max(1, s / 6); }

// What a product is on tile t in s splits: workgroups, 16-k steps of each,
// the time its partials' traffic takes.
struct Shape {
  long long wg;
  double steps, traffic;
};
Shape shape_of(const GemmDesc& g, int t, int s) {
  const TileCost& c = tile_cost(g, t);
  const long long tiles = (long long)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn);
  const int kt = (g.K + c.bk - 1) / c.bk;
  return {tiles * s, (double)((kt + s - 1) / s) * c.bk / 16,
          s > 1 ? (2 * s + 1) * 4.0 * g.M * g.N / kBytesPerUs : 0.0};
}
// the real number of splits, each of whole K steps
int real_splits(const GemmDesc& g, int t, int s) {
  const int bk = tile_cost(g, t).bk, kt = (g.K + bk - 1) / bk, per = (kt + s - 1) / s;
  return (kt + per - 1) / per;
}

Plan plan_staged(const GemmDesc& g, double* time = nullptr) {
  if (g.plan_splits > 0) return {g.plan_tile, g.plan_splits};
  Plan best{0, 1};
  double best_cost = -1.0;
  for (int t = 0; t < 3; ++t) {
    const TileCost& c = load_cost(g, t);
    const SplitRange r = split_range(g, t);
    for (int s = r.lo; s <= r.hi; s = next_split(s)) {
      const Shape h = shape_of(g, t, s);
      const long long per_cu = (h.wg + 255) / 256;
      double cost = per_cu == 1 ? c.base_alone + h.steps * c.alone
                                : per_cu * (c.base_shared + h.steps * c.shared);
      if (s > 1) cost += kSumLaunch + h.traffic;
      if (best_cost < 0 || cost < best_cost) {
        best = {t, s};
        best_cost = cost;
      }
    }
  }
  best.splits = real_splits(g, best.tile, best.splits);
  if (time) *time = best_cost;
  return best;
}

// Chunk loads need chunks that are wholly inside or outside the operand and
// aligned; buffer offsets need a panel (a tile's rows, or a stage's k-rows)
// below 2 GiB.
LoadMode load_mode(const GemmDesc& g, int bm, int bn, int bk) {
  const long long es = g.a_bf16 ? 2 : 4;
  auto whole = [&](const void* p, long long ld, int extent) {
    return reinterpret_cast<uintptr_t>(p) % (4 * es) == 0 && ld % 4 == 0 && extent % 4 == 0;
  };
  auto fits = [&](bool kc, long long ld, int rows) {
    return es * ((kc ? rows : bk) * ld + std::max(rows, bk)) < (long long)kOOB;
  };
  if (!fits(g.a_kc, g.lda, bm) || !fits(g.b_kc, g.ldb, bn)) return kPlain;
  return whole(g.A, g.lda, g.a_kc ? g.K : g.M) && whole(g.B, g.ldb, g.b_kc ? g.K : g.N) ? kChunk
                                                                                        : kSingle;
}

template <class C, bool A_KC, bool B_KC, class S>
hipError_t launch_staged(const GemmDesc& g, const KernelArgs& a, hipStream_t st) {
  const dim3 grid(a.tiles_m * a.tiles_n * a.splits), block(C::THREADS);
  const LoadMode mode = load_mode(g, C::BM, C::BN, C::BK);
  if (mode == kChunk)
    hipLaunchKernelGGL((gemm_staged_kernel<C, A_KC, B_KC, kChunk, S>), grid, block, 0, st, a);
  else if (mode == kSingle)
    hipLaunchKernelGGL((gemm_staged_kernel<SingleCfg<C>, A_KC, B_KC, kSingle, S>), grid, block, 0,
                       st, a);
  else
    hipLaunchKernelGGL((gemm_staged_kernel<C, A_KC, B_KC, kPlain, S>), grid, block, 0, st, a);
  return hipGetLastError();
}

// The operand types and layouts that occur: fp32 operands in every layout in
// both precisions; bf16 operands as the layer's products read them (U = X
// W^T and dX = dU (W^T)^T K-contiguous, dW = dU^T X row-contiguous).
template <class C>
hipError_t launch_layout(const GemmDesc& g, const KernelArgs& a, hipStream_t st) {
  if (g.a_bf16 != g.b_bf16 || (!g.a_kc && g.b_kc)) return hipErrorInvalidValue;
  if constexpr (C::NP == 1) {
    if (g.a_bf16) {
      if (g.b_kc) return launch_staged<C, true, true, uint16_t>(g, a, st);
      if (!g.a_kc) return launch_staged<C, false, false, uint16_t>(g, a, st);
      return hipErrorInvalidValue;
    }
  }
  if (g.a_bf16) return hipErrorInvalidValue;
  if (g.b_kc) return launch_staged<C, true, true, float>(g, a, st);
  if (g.a_kc) return launch_staged<C, true, false, float>(g, a, st);
  return launch_staged<C, false, false, float>(g, a, st);
}

template <int NP>
hipError_t launch_tile(int tile, const GemmDesc& g, const KernelArgs& a, hipStream_t st) {
  return tile == 0   ? launch_layout<FBig<NP>>(g, a, st)
         : tile == 1 ? launch_layout<FMid<NP>>(g, a, st)
                     : launch_layout<FSmall<NP>>(g, a, st);
}

KernelArgs staged_args(const GemmDesc& g, const Plan& p) {
  const TileCost& c = tile_cost(g, p.tile);
  const int kt = (g.K + c.bk - 1) / c.bk;
  KernelArgs a{};
  a.A = g.A;
  a.B = g.B;
  a.lda = g.lda;
  a.ldb = g.ldb;
  a.M = g.M;
  a.N = g.N;
  a.K = g.K;
  a.k_per_split = ((kt + p.splits - 1) / p.splits) * c.bk;
  a.tiles_m = (g.M + c.bm - 1) / c.bm;
  a.tiles_n = (g.N + c.bn - 1) / c.bn;
  a.splits = p.splits;
  if (p.splits > 1) {
    a.out = g.partials;
    a.ldo = g.N;
    a.split_stride = (long long)g.M * g.N;
  } else {
    a.out = g.C;
    a.ldo = g.ldc;
    a.add = g.add;
    a.add_count = g.add_count;
    a.add_ld = g.add_ld;
    a.add_off = g.add_off;
  }
  return a;
}

template <class C, class S>
void launch_pair(const KernelArgs& ax, const KernelArgs& aw, hipStream_t st) {
  const int n1 = ax.tiles_m * ax.tiles_n * ax.splits, n2 = aw.tiles_m * aw.tiles_n * aw.splits;
  hipLaunchKernelGGL((gemm_staged_pair_kernel<C, S>), dim3(n1 + n2), dim3(C::THREADS), 0, st, ax,
                     n1, aw, n2, aw.k_per_split > ax.k_per_split);
}

}  // namespace

int gemm_staged_splits(const GemmDesc& g) { return plan_staged(g).splits; }

double gemm_staged_time(const GemmDesc& g) {
  double t;
  plan_staged(g, &t);
  return t;
}

hipError_t gemm_staged_launch(const GemmDesc& g, hipStream_t st) {
  const Plan p = plan_staged(g);
  const KernelArgs a = staged_args(g, p);
  timing_before(gemm_label(g), st);
  const hipError_t e = g.bf16 ? launch_tile<1>(p.tile, g, a, st) : launch_tile<3>(p.tile, g, a, st);
  timing_after(st);
  return e;
}

// The pair is built for chunk loads: by the sizes here, by the pointers too at
// the launch.
static bool pair_loads(const GemmDesc& gx, const GemmDesc& gw, const TileCost& c) {
  return load_mode(gx, c.bm, c.bn, c.bk) == kChunk && load_mode(gw, c.bm, c.bn, c.bk) == kChunk;
}

// Mid or Small tiles for both (Big ones fill the chip by themselves), where
// pair_time beats the two plans one after the other.  L 64, B 32, d 256 fp32
// (Small tiles): 21 us against 15 + 15.  Shapes
// that fill the chip one by one gain nothing (L 400, B 32, 256 -> 128 units in
// both directions, Mid: 106 us against 68 + 47, the step no faster).
GemmPair gemm_staged_pair_plan(const GemmDesc& gx, const GemmDesc& gw, double time) {
  GemmPair best{0, 0, 0};
  if (gx.bf16 != gw.bf16 || gx.a_bf16 != gw.a_bf16 || !gx.a_kc || gx.b_kc || gw.a_kc || gw.b_kc ||
      gx.a_bf16 != gx.bf16)
    return best;
  double best_cost = time;
  for (int t = 1; t < 3; ++t) {
    const TileCost& c = tile_cost(gx, t);
    if (!pair_loads(gx, gw, c)) continue;
    const SplitRange rx = split_range(gx, t), rw = split_range(gw, t);
    for (int sx = rx.lo; sx <= rx.hi; sx = next_split(sx)) {
      const Shape x = shape_of(gx, t, sx);
      for (int sw = rw.lo; sw <= rw.hi; sw = next_split(sw)) {
        const Shape w = shape_of(gw, t, sw);
        const double cost =
            c.base_alone +
            pair_time(x.wg, x.steps, c.alone, w.wg, w.steps, c.alone, c.base_shared, c.shared) +
            x.traffic + w.traffic + (sx > 1 || sw > 1 ? kSumLaunch : 0.0);
        if (cost < best_cost) {
          best = {t, real_splits(gx, t, sx), real_splits(gw, t, sw)};
          best_cost = cost;
        }
      }
    }
  }
  return best;
}

bool gemm_staged_pair_launch(const GemmDesc& gx, const GemmDesc& gw, hipStream_t st) {
  const TileCost& c = tile_cost(gx, gx.plan_tile);
  if (!pair_loads(gx, gw, c)) return false;
  const KernelArgs ax = staged_args(gx, plan_staged(gx)), aw = staged_args(gw, plan_staged(gw));
  timing_before("gemm_dx_dw", st);
  if (gx.bf16) {
    if (gx.plan_tile == 1) launch_pair<FMid<1>, uint16_t>(ax, aw, st);
    else launch_pair<FSmall<1>, uint16_t>(ax, aw, st);
  } else {
    if (gx.plan_tile == 1) launch_pair<FMid<3>, float>(ax, aw, st);
    else launch_pair<FSmall<3>, float>(ax, aw, st);
  }
  timing_after(st);
  return true;
}

}  // namespace sru
