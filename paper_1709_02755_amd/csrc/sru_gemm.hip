// bf16 matrix products of the SRU layer on the gfx950 matrix cores (MFMA),
// the conversions to bf16 they read, the sums of split products, and the
// fused projection + scan.  The products whose operands the direct kernel
// cannot load, and the fp32 ones, are in sru_gemm_staged.hip.
//
// The forward projection of Sec. 3.1 (U = X [W; W_f; W_r]^T over all L*B
// tokens at once) and the two products of the backward pass (dX = dU W and
// dW = dU^T X) are one kernel template:
//     C[M,N] = sum_k A(m,k) B(n,k)
// with each operand either K-contiguous ("KC": row-major [rows, K]) or
// row-contiguous ("RC": [K, rows]).
// Work mapping: one workgroup per output tile (and K split).  Workgroups are
// dispatched round-robin over the 8 XCDs, so the linear tile order is
// remapped to give each XCD a contiguous run of tiles that share A panels in
// its own L2.
#include <algorithm>
#include <type_traits>

#include "sru_device.h"
#include "sru_gemm_tile.h"
#include "sru_internal.h"

namespace sru {
namespace {

// Epilogue of the direct kernel, whose MFMAs take the B-operand fragment
// first and so accumulate the transposed tile: element e of lane l is row
// l%32, column 8*(e/4) + 4*(l/32) + e%4 of the 32x32 output tile.  Each
// group of four elements is four consecutive columns of one row, written
// (and its addend read) as one 16-byte access when the tile lies wholly
// inside the output and vec_out holds (16-byte aligned rows).
// OB: also (or, when g.out is null, only) write the bf16 rounding of the
// result to g.outb (four columns as one 8-byte store); no addend then.
template <class C, int ADD, bool OB = false>
__device__ __forceinline__ void write_tile_rows(const KernelArgs& g,
                                                const floatx16 (&acc)[C::FM][C::FN], int m0,
                                                int n0, int wm0, int wn0, int lane, int split) {
  static_assert(!OB || ADD == 0, "the bf16 result takes no addend");
  float* out = g.out ? g.out + (long long)split * g.split_stride : nullptr;
  const int cl = 4 * (lane >> 5);
  if constexpr (OB) {
    if (g.vec_out && m0 + C::BM <= g.M && n0 + C::BN <= g.N) {
#pragma unroll
      for (int i = 0; i < C::FM; ++i) {
        const int m = m0 + wm0 + i * 32 + (lane & 31);
        const long long col = n0 + wn0 + cl;
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float a0 = acc[i][j][4 * q], a1 = acc[i][j][4 * q + 1];
            const float a2 = acc[i][j][4 * q + 2], a3 = acc[i][j][4 * q + 3];
            u32x2 w;
            w[0] = pack_bf16(a0, a1);
            w[1] = pack_bf16(a2, a3);
            *reinterpret_cast<u32x2*>(g.outb + m * g.ldob + col + j * 32 + 8 * q) = w;
            if (out) {
              floatx4 v;
              v[0] = a0;
              v[1] = a1;
              v[2] = a2;
              v[3] = a3;
              *reinterpret_cast<floatx4*>(out + m * g.ldo + col + j * 32 + 8 * q) = v;
            }
          }
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int j = 0; j < C::FN; ++j) {
        const int m = m0 + wm0 + i * 32 + (lane & 31);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int n = n0 + wn0 + j * 32 + 8 * (e >> 2) + cl + (e & 3);
          if (m < g.M && n < g.N) {
            const float v = acc[i][j][e];
            g.outb[(long long)m * g.ldob + n] = __builtin_bit_cast(uint16_t, (__bf16)v);
            if (out) out[(long long)m * g.ldo + n] = v;
          }
        }
      }
    return;
  }
  if constexpr (ADD > 0) {
    if (g.vec_out && m0 + C::BM <= g.M && n0 + C::BN <= g.N) {
      // Addends of one row of MFMA tiles are loaded one row ahead, before
      // the stores of the current row: the loads never wait behind stores
      // (which the compiler would otherwise keep in program order, since
      // it cannot rule out aliasing), so a wave has one exposed memory
      // round trip instead of one per MFMA tile.
      constexpr int NA = C::FN * 4;  // 16-byte addend chunks per tile row
      floatx4 buf[2][ADD][NA];
      auto load_row = [&](int i, floatx4 (&a)[ADD][NA]) {
        const int m = m0 + wm0 + i * 32 + (lane & 31);
        const float* arow = g.add + (long long)m * g.add_ld + n0 + wn0 + cl;
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            a[0][j * 4 + q] = *reinterpret_cast<const floatx4*>(arow + j * 32 + 8 * q);
            if constexpr (ADD > 1)
              a[1][j * 4 + q] =
                  *reinterpret_cast<const floatx4*>(arow + g.add_off + j * 32 + 8 * q);
          }
      };
      load_row(0, buf[0]);
#pragma unroll
      for (int i = 0; i < C::FM; ++i) {
        floatx4 v[NA];
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j * 4 + q][e] = acc[i][j][4 * q + e];
            v[j * 4 + q] += buf[i & 1][0][j * 4 + q];
            if constexpr (ADD > 1) v[j * 4 + q] += buf[i & 1][1][j * 4 + q];
          }
        if (i + 1 < C::FM) load_row(i + 1, buf[(i + 1) & 1]);
        const int m = m0 + wm0 + i * 32 + (lane & 31);
        float* orow = out + (long long)m * g.ldo + n0 + wn0 + cl;
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<floatx4*>(orow + j * 32 + 8 * q) = v[j * 4 + q];
      }
      return;
    }
  }
  if (ADD == 0 && g.vec_out && m0 + C::BM <= g.M && n0 + C::BN <= g.N) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
      const int m = m0 + wm0 + i * 32 + (lane & 31);
      float* orow = out + (long long)m * g.ldo + n0 + wn0 + cl;
      const float* arow = ADD > 0 ? g.add + (long long)m * g.add_ld + n0 + wn0 + cl : nullptr;
#pragma unroll
      for (int j = 0; j < C::FN; ++j) {
        floatx4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[q][e] = acc[i][j][4 * q + e];
        if constexpr (ADD > 0) {
          floatx4 a0[4], a1[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            a0[q] = *reinterpret_cast<const floatx4*>(arow + j * 32 + 8 * q);
            if constexpr (ADD > 1)
              a1[q] = *reinterpret_cast<const floatx4*>(arow + g.add_off + j * 32 + 8 * q);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            v[q] += a0[q];
            if constexpr (ADD > 1) v[q] += a1[q];
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<floatx4*>(orow + j * 32 + 8 * q) = v[q];
      }
    }
    return;
  }
  // edge tiles (or unaligned rows): element by element, inside the bounds
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const int m = m0 + wm0 + i * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int n = n0 + wn0 + j * 32 + 8 * (e >> 2) + cl + (e & 3);
        if (m < g.M && n < g.N) {
          float v = acc[i][j][e];
          if constexpr (ADD > 0) {
            const float* ar = g.add + (long long)m * g.add_ld + n;
            v += ar[0];
            if constexpr (ADD > 1) v += ar[g.add_off];
          }
          out[(long long)m * g.ldo + n] = v;
        }
      }
    }
}

// fp32 epilogue of a whole tile through LDS.  The accumulator layout makes a
// direct store write 32 rows x 32 bytes; here each wave moves one row of
// MFMA tiles (32 x WN) at a time through its own LDS block and reads it back
// row by row, so that a store instruction writes 4 rows x 256 bytes, i.e.
// whole 128-byte lines, and the addends are read the same way.  The caller
// has ended every wave's reads of the operand stages (barrier).
constexpr int kStagePitch = 68;  // floats per staged row: 64 + 4 keeps 16-byte writes conflict-free
template <class C, int ADD>
__device__ __forceinline__ void write_tile_staged(const KernelArgs& g,
                                                  const floatx16 (&acc)[C::FM][C::FN],
                                                  unsigned char* smem, int m0, int n0, int wm0,
                                                  int wn0, int lane, int wave, int split) {
  static_assert(C::WN == 64, "staged rows of 64 columns");
  float* out = g.out + (long long)split * g.split_stride;
  const int cl = 4 * (lane >> 5);
  static_assert(C::WAVES * 32 * kStagePitch * 4 <= C::LDS, "staging fits the operand stages");
  float* blk = reinterpret_cast<float*>(smem) + wave * 32 * kStagePitch;
  const int rr = lane >> 4, cc = 4 * (lane & 15);  // read-back: rows rr + 4 s, columns cc..cc+3
#pragma unroll
  for (int i = 0; i < C::FM; ++i) {
    const long long mrow = m0 + wm0 + i * 32 + rr;  // row of read-back s = 0
    floatx4 ad[ADD > 0 ? ADD : 1][8];
    if constexpr (ADD > 0) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float* ar = g.add + (mrow + 4 * s) * g.add_ld + n0 + wn0 + cc;
        ad[0][s] = *reinterpret_cast<const floatx4*>(ar);
        if constexpr (ADD > 1) ad[1][s] = *reinterpret_cast<const floatx4*>(ar + g.add_off);
      }
    }
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e];
        *reinterpret_cast<floatx4*>(blk + (lane & 31) * kStagePitch + j * 32 + 8 * q + cl) = v;
      }
    // one wave's LDS accesses run in order: the reads below see the writes,
    // and the next row group's writes come after these reads
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      floatx4 v = *reinterpret_cast<const floatx4*>(blk + (rr + 4 * s) * kStagePitch + cc);
      if constexpr (ADD > 0) v += ad[0][s];
      if constexpr (ADD > 1) v += ad[1][s];
      *reinterpret_cast<floatx4*>(out + (mrow + 4 * s) * g.ldo + n0 + wn0 + cc) = v;
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 x bf16 products with global -> LDS loads that bypass registers.
// Buffer loads with the LDS flag write each lane's 16 bytes straight into
// LDS at (wave-uniform base + 16 * lane); a ring of two tiles lets the loads
// run a K step ahead of the MFMAs (A, in a third slot, two) at no register
// cost.  Both
// operands have the same layout, selected by RC:
//
// K-contiguous (RC = false; U = X W^T and dX = dU W as dU (W^T)^T):
//   row r of a tile holds BK k (2*BK bytes) at r*2*BK, its 16-byte k-chunks
//   permuted as slot = chunk ^ swz(r), which keeps the 16 rows of one
//   ds_read_b128 phase on distinct banks.  BK = 64 makes each row one whole
//   128-byte line of the operand: a wave load (8 rows, lane l: row l/8,
//   slot l%8) then touches 8 lines instead of 16 half lines, which is what
//   bounds the load rate.  A fragment is one ds_read_b128.
// Row-contiguous (RC = true; dW = dU^T X, both operands [K, rows]):
//   the tile is kept as loaded, k-row s at s*2R bytes (R rows of bf16), its
//   R/8 16-byte row-chunks permuted as slot = chunk ^ 4*(s & 3).  A wave
//   load fills 512/R k-rows.  A fragment (8 consecutive k of one row) is two
//   ds_read_b64_tr_b16: within each group of 16 lanes, input lane 4s+q names
//   k-row s, rows 4q..4q+3 of the group's 16 rows, and output lane i
//   receives that k-run of row i.  A k-row is a multiple of 256 bytes, so
//   its slot p sits on banks 4p..4p+3 (mod 64) whatever s is; the two groups
//   of a half wave read chunks c..c+3 (c a multiple of 4) of the same four
//   k-rows, and the XOR by 4*(s & 3) puts those 16 chunks on 16 distinct
//   slots mod 16, i.e. all 64 banks once.  (An XOR by 2*(s & 3) put both
//   groups on the same 8 slots: a two-way conflict on every read.)
//
// Each wave of a big tile owns a 128 x 64 block of it (4 x 2 MFMA tiles of 32
// x 32, 128 accumulator registers per lane); two waves share each SIMD, so
// one's LDS reads and barrier waits hide behind the other's MFMAs.  A 256 x
// 256 tile loads half the bytes per flop of a 128 x 128 one, which its loads
// bound, not the MFMAs.
template <int BM_, int BN_, int BK_, int WAVES_M_, int WAVES_N_, int STAGES_, int SA_ = STAGES_>
struct DCfg {
  // STAGES: slots of the B operand's ring; SA: slots of the A operand's
  // ring (STAGES or STAGES + 1: A then loads one K step further ahead)
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_, SA = SA_;
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int FM = WM / 32, FN = WN / 32;
  static constexpr int KSLAB = 16, SLABS = BK / KSLAB;
  static constexpr int A_OPB = BM * BK * 2, B_OPB = BN * BK * 2;  // bytes per stage
  static constexpr int STB = A_OPB + B_OPB;
  static constexpr int A_BPW = A_OPB / 1024 / WAVES, B_BPW = B_OPB / 1024 / WAVES;
  static constexpr int IPS = A_BPW + B_BPW;  // load instructions per stage per wave
  static constexpr int LDS = SA * A_OPB + STAGES * B_OPB;  // A slots, then B slots
  static constexpr int OCC = LDS <= 80 * 1024 ? 2 : 1;  // workgroups per CU
  static_assert(SA == STAGES || SA == STAGES + 1, "A ring depth");
  static_assert(STAGES == 2 && BK == 64, "ring and k per stage");
  static_assert((WM == 128 && WN == 64) || (WM == 64 && (WN == 64 || WN == 96 || WN == 128)),
                "wave block");
  static_assert(A_BPW * 1024 * WAVES == A_OPB && B_BPW * 1024 * WAVES == B_OPB,
                "whole 1 KiB load blocks per wave");
  static_assert(LDS <= 160 * 1024 && IPS * (SA - 1) < 64, "LDS and vmcnt");
};
// Big tiles: 8 waves of 128 x 64, one workgroup per CU.  K-contiguous
// operands load A two K steps ahead (160 KiB).
using CfgBigKC = DCfg<256, 256, 64, 2, 4, 2, 3>;
using CfgBigRC = DCfg<256, 256, 64, 2, 4, 2>;
// Mid tiles, for products of few big ones: 4 waves of 64 x 64, two
// workgroups per CU, so that one's loads and epilogue run beside the other's
// MFMAs.  Against 256 x 128 tiles of 4 waves (one wave per SIMD), us:
// 2048 x 3072 x 1024 24.1 -> 20.3, 2048 x 1024 x 3072 in two splits 30.4 ->
// 21.2, 16384 x 512 x 1024 25.7 -> 23.3, 512 x 3072 x 1024 19.7 -> 12.6; 3072
// x 1024 over 2048 tokens 25.0 (big, 5 splits) -> 21.4 (2 splits).
using CfgMidKC = DCfg<128, 128, 64, 2, 2, 2, 3>;
using CfgMidRC = DCfg<128, 128, 64, 2, 2, 2>;

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_t;
typedef __attribute__((address_space(3))) v4i16 lds_v4;

// s_waitcnt immediate waiting for vmcnt <= n only (expcnt 7, lgkmcnt 15)
constexpr int vm_wait(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// One operand's part of the direct loads: R tile rows, this wave's BPW
// 1 KiB blocks.  off: byte offset at k0 = 0 from the panel's base (init:
// row r0 of a K-contiguous operand, k-row kbase of a row-contiguous one, see
// issue; init_rows: the operand's start); kk: k (within a stage) of the
// lane's data; oob: out-of-range bit for rows past the end (RC).
template <int R, bool RC, int BPW, int BK>
struct DirectOperand {
  static constexpr int LPR = BK / 8;    // KC: 16-byte chunks (lanes) per row
  static constexpr int RPB = 64 / LPR;  // KC: rows per 1 KiB block
  unsigned off[BPW], oob[BPW];
  int kk[BPW];

  __device__ __forceinline__ static int swz(int r) {
    return (r >> 1) & 7;
  }
  __device__ __forceinline__ void init(int wave, int lane, int r0, int rows, long long ld) {
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
      const int blk = wave * BPW + j;
      if constexpr (!RC) {
        const int r = blk * RPB + lane / LPR;
        const int chunk = (lane % LPR) ^ swz(r);
        kk[j] = chunk * 8;
        off[j] = (unsigned)(((long long)(min(r0 + r, rows - 1) - r0) * ld + chunk * 8) * 2);
        oob[j] = 0;  // rows past the end are clamped: they feed discarded outputs
      } else {
        constexpr int CPK = R / 8;  // 16-byte chunks per k-row
        static_assert(CPK >= 16, "the k-row swizzle XORs chunk indices with up to 12");
        const int srow = blk * (512 / R) + lane / CPK;
        const int chunk = (lane % CPK) ^ (4 * (srow & 3));
        const int r = r0 + chunk * 8;
        kk[j] = srow;
        off[j] = (unsigned)(((long long)srow * ld + min(r, rows - 8)) * 2);
        oob[j] = (unsigned)(r >= rows) << 31;  // rows % 8 == 0: chunks are whole
      }
    }
  }
  // K-contiguous operand whose tile row r is row row_of(r) of the operand,
  // or a row of zeros where row_of(r) < 0 (no memory is read for it).
  template <class F>
  __device__ __forceinline__ void init_rows(int wave, int lane, F row_of, long long ld) {
    static_assert(!RC, "row maps are for K-contiguous operands");
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
      const int blk = wave * BPW + j;
      const int r = blk * RPB + lane / LPR;
      const int chunk = (lane % LPR) ^ swz(r);
      const long long gr = row_of(r);
      kk[j] = chunk * 8;
      off[j] = gr >= 0 ? (unsigned)((gr * ld + chunk * 8) * 2) : 0u;
      oob[j] = gr >= 0 ? 0u : kOOB;
    }
  }
  // Loads of the stage at k0 (RC: k-rows from kbase on lie at the panel's
  // base; KC: the base holds k = 0).
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, unsigned char* lds, int wave,
                                        int k0, int kend, long long ld, int kbase) const {
    const unsigned dk = RC ? (unsigned)((long long)(k0 - kbase) * ld * 2) : (unsigned)(k0 * 2);
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
      // past the end of K: an out-of-range offset, for which the hardware
      // writes zeros
      const unsigned kob = (unsigned)(k0 + kk[j] >= kend) << 31;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_t*)(lds + (wave * BPW + j) * 1024), 16,
                                               (off[j] + dk) | kob | oob[j], 0, 0, 0);
    }
  }
  // 16-byte MFMA fragment: k-chunk c (8 k) of tile row `row`
  __device__ __forceinline__ static floatx4 frag(const unsigned char* base, int row, int c,
                                                 int lane) {
    if constexpr (!RC) {
      return *reinterpret_cast<const floatx4*>(base + row * (2 * BK) + ((c ^ swz(row)) << 4));
    } else {
      // this lane's role in its 16-lane group: k-row s, rows 4q..4q+3
      const int gl = lane & 15;
      const int r = (row & ~15) + 4 * (gl & 3);
      const int kr = c * 8 + (gl >> 2);
      auto addr = [&](int k) {
        return base + k * (2 * R) + (((r >> 3) ^ (4 * (k & 3))) << 4) + (r & 7) * 2;
      };
      const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(addr(kr)));
      const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(addr(kr + 4)));
      floatx4 f;
      f[0] = __builtin_bit_cast(float, __builtin_shufflevector(lo, lo, 0, 1));
      f[1] = __builtin_bit_cast(float, __builtin_shufflevector(lo, lo, 2, 3));
      f[2] = __builtin_bit_cast(float, __builtin_shufflevector(hi, hi, 0, 1));
      f[3] = __builtin_bit_cast(float, __builtin_shufflevector(hi, hi, 2, 3));
      return f;
    }
  }
};

// The main loop of the direct products: the tile whose operand loads la and
// lb were set up, accumulated over k in [kbeg, kend) into acc.  TRANS: the
// MFMAs take B first, so acc holds the transposed tile (lane l: tile row
// l % 32 of each 32 x 32 block); else lane l holds tile column l % 32, rows
// 8 (e / 4) + 4 (l / 32) + e % 4 of element e.
template <class C, bool TRANS = true, class OpA, class OpB>
__device__ __forceinline__ void direct_mainloop(unsigned char* smem, const OpA& la,
                                                const OpB& lb, __amdgpu_buffer_rsrc_t ra,
                                                __amdgpu_buffer_rsrc_t rb, long long lda,
                                                long long ldb, int kbeg, int kend, int wave,
                                                int lane, int wm0, int wn0,
                                                floatx16 (&acc)[C::FM][C::FN]) {
  constexpr int STAGES = C::STAGES, SA = C::SA;
  constexpr bool ALEAD = SA > STAGES;  // A loads one K step further ahead than B
  const int nk = (kend - kbeg + C::BK - 1) / C::BK;
  auto a_slot = [&](int kt) { return smem + (kt % SA) * C::A_OPB; };
  auto b_slot = [&](int kt) { return smem + SA * C::A_OPB + (kt % STAGES) * C::B_OPB; };
  auto issue_a = [&](int kt) {
    la.issue(ra, a_slot(kt), wave, kbeg + kt * C::BK, kend, lda, kbeg);
  };
  auto issue_b = [&](int kt) {
    lb.issue(rb, b_slot(kt), wave, kbeg + kt * C::BK, kend, ldb, kbeg);
  };
  auto issue = [&](int kt) {
    issue_a(kt);
    issue_b(kt);
  };

#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s);
  // the A ring's extra slot: A of step STAGES - 1 goes out with the prologue
  if constexpr (ALEAD)
    if (STAGES - 1 < nk) issue_a(STAGES - 1);

  // Wait until this wave's part of stage kt has landed.  With the deeper A
  // ring the loads go out in the order A(kt+1) ... B(kt) A(kt+1) B(kt+1)
  // A(kt+2), so A of step kt + 1 may stay in flight.
  auto wait_stage = [&](int kt) {
    if (ALEAD && kt + 1 < nk) __builtin_amdgcn_s_waitcnt(vm_wait(C::A_BPW));
    else __builtin_amdgcn_s_waitcnt(vm_wait(0));
  };
  // Workgroup barrier without the release fence of __syncthreads (which
  // would wait for every outstanding vector memory operation, i.e. drain the
  // prefetched stages): this wave's LDS reads are waited for explicitly, the
  // stage's loads by wait_stage, and the memory clobbers keep the compiler
  // from moving LDS accesses across it.
  auto barrier = [] {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only (vmcnt 63, expcnt 7)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  struct Frags {
    floatx4 a[C::FM], b[C::FN];
  };
  auto load_frags = [&](Frags& f, int kt, int sl) {
    const unsigned char* As = a_slot(kt);
    const unsigned char* Bs = b_slot(kt);
    const int c = 2 * sl + (lane >> 5);
#pragma unroll
    for (int i = 0; i < C::FM; ++i) f.a[i] = OpA::frag(As, wm0 + i * 32 + (lane & 31), c, lane);
#pragma unroll
    for (int j = 0; j < C::FN; ++j) f.b[j] = OpB::frag(Bs, wn0 + j * 32 + (lane & 31), c, lane);
  };
  auto mfmas = [&](const Frags& f) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
        acc[i][j] = TRANS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, f.b[j]),
                                __builtin_bit_cast(bf16x8, f.a[i]), acc[i][j], 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, f.a[i]),
                                __builtin_bit_cast(bf16x8, f.b[j]), acc[i][j], 0, 0, 0);
  };

  // Software pipeline over the SLABS fragment slabs (16 k each) of a stage:
  // a slab's fragments are read from LDS before the MFMAs of the previous
  // slab are issued (f[0] and f[1] alternate; SLABS is even, so slab 0 of
  // every stage is f[0]).  The barrier that publishes stage kt+1 sits before
  // the MFMAs of the last slab of stage kt; it also ends every wave's reads
  // of stage kt, which frees that slot for the loads issued at the top of
  // the next iteration.  The last stage is peeled off so that no branch
  // separates the reads of the next f[0] from the MFMAs of the last slab: at
  // a join the compiler would count those newer reads into the wait.  A
  // scheduling barrier after each slab's reads keeps the compiler from
  // sinking them next to the MFMAs that consume them.
  Frags f[2];
  if (nk > 0) {
    wait_stage(0);
    barrier();
    load_frags(f[0], 0, 0);
    for (int kt = 0; kt + 1 < nk; ++kt) {
      if constexpr (ALEAD) {
        // slots of stage kt-1, free: B of the next step, then A of the one after
        if (kt + 1 < nk) issue_b(kt + 1);
        if (kt + 2 < nk) issue_a(kt + 2);
      } else {
        if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1);  // slot of stage kt-1, free
      }
#pragma unroll
      for (int sl = 0; sl + 1 < C::SLABS; ++sl) {
        load_frags(f[(sl + 1) & 1], kt, sl + 1);
        __builtin_amdgcn_sched_barrier(0);  // reads of the next slab stay ahead
        mfmas(f[sl & 1]);
      }
      wait_stage(kt + 1);
      barrier();
      load_frags(f[0], kt + 1, 0);
      __builtin_amdgcn_sched_barrier(0);  // reads of the next slab stay ahead
      mfmas(f[1]);
    }
#pragma unroll
    for (int sl = 0; sl < C::SLABS; ++sl) {
      if (sl + 1 < C::SLABS) load_frags(f[(sl + 1) & 1], nk - 1, sl + 1);
      __builtin_amdgcn_sched_barrier(0);  // reads of the next slab stay ahead
      mfmas(f[sl & 1]);
    }
  }
}

// Workgroup w of a product's nwg.  smem: C::LDS bytes.
template <class C, int ADD, bool A_RC, bool B_RC, bool OB>
__device__ __forceinline__ void direct_tile(const KernelArgs& g, int w, int nwg,
                                            unsigned char* smem) {
#ifdef __HIP_DEVICE_COMPILE__  // (the host pass fails to instantiate the main loop twice)
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
  // Buffer resources based at this workgroup's panels: a K-contiguous
  // operand at the tile's first row, a row-contiguous one at the split's
  // first k-row.  The loaders' offsets count from there, so they stay below
  // kOOB however large the operand is (the plan bounds the panels).
  const __amdgpu_buffer_rsrc_t ra =
      panel_rsrc(g.A, 2LL * (A_RC ? kbeg : m0) * g.lda, g.a_bytes);
  const __amdgpu_buffer_rsrc_t rb =
      panel_rsrc(g.B, 2LL * (B_RC ? kbeg : n0) * g.ldb, g.b_bytes);

  using OpA = DirectOperand<C::BM, A_RC, C::A_BPW, C::BK>;
  using OpB = DirectOperand<C::BN, B_RC, C::B_BPW, C::BK>;
  OpA la;
  OpB lb;
  la.init(wave, lane, m0, g.M, g.lda);
  lb.init(wave, lane, n0, g.N, g.ldb);
  floatx16 acc[C::FM][C::FN];
  direct_mainloop<C>(smem, la, lb, ra, rb, g.lda, g.ldb, kbeg, kend, wave, lane, wm0, wn0,
                     acc);
  if constexpr (!OB) {
    if (g.vec_out && m0 + C::BM <= g.M && n0 + C::BN <= g.N) {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // this wave's LDS reads (lgkmcnt 0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();  // every wave is done with the operand stages
      asm volatile("" ::: "memory");
      write_tile_staged<C, ADD>(g, acc, smem, m0, n0, wm0, wn0, lane, wave, ti.split);
      return;
    }
  }
  write_tile_rows<C, ADD, OB>(g, acc, m0, n0, wm0, wn0, lane, ti.split);
#endif
}

template <class C, int ADD, bool A_RC, bool B_RC, bool OB>
__global__ __launch_bounds__(C::THREADS, C::OCC) void gemm_direct_kernel(KernelArgs g) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS];
  direct_tile<C, ADD, A_RC, B_RC, OB>(g, blockIdx.x, gridDim.x, smem);
}

// dX (n1 workgroups) and dW (n2) on mid tiles in one launch, the one of longer
// workgroups first.
template <int ADD>
__global__ __launch_bounds__(CfgMidKC::THREADS, 2) void gemm_direct_pair_kernel(KernelArgs g1, int n1,
                                                                                KernelArgs g2, int n2,
                                                                                bool dw_first) {
  static_assert(CfgMidKC::THREADS == CfgMidRC::THREADS, "one block size");
  __shared__ __attribute__((aligned(1024))) unsigned char
      smem[CfgMidKC::LDS > CfgMidRC::LDS ? CfgMidKC::LDS : CfgMidRC::LDS];
  const PairIdx p = pair_index(n1, n2, dw_first);
  if (p.dx) direct_tile<CfgMidKC, ADD, false, false, false>(g1, p.w, n1, smem);
  else direct_tile<CfgMidRC, 0, true, true, false>(g2, p.w, n2, smem);
}
template __global__ void gemm_direct_pair_kernel<0>(KernelArgs, int, KernelArgs, int, bool);
template __global__ void gemm_direct_pair_kernel<1>(KernelArgs, int, KernelArgs, int, bool);
template __global__ void gemm_direct_pair_kernel<2>(KernelArgs, int, KernelArgs, int, bool);

// ---- fused projection + forward scan (inference: neither U nor C kept) ----
// One workgroup per (direction, group of 64 hidden units, group of bb
// sequences), bb = 2, 4 or 8.  Per time block of 256 / bb steps it computes
// the tile of U whose 256 rows are the block's (step, sequence) pairs and
// whose 64 k columns are the k gate blocks of the 64 units (k = 4: block 3
// is the highway input x_hat; k = 3 reads x_t from X).  The MFMAs leave the
// tile untransposed on 64 x 32k wave blocks, and the operand rows are mapped
// so that a lane's accumulators are the scan's inputs: lane l of wave
// (wm, wn) holds column l % 32 of each of its k 32-column MFMA blocks, i.e.
// the gates of unit 64 g + 32 wn + l % 32, and rows of one sequence (l / 32
// picks one of the wave's two), 16 consecutive steps per 32-row block, so 32
// steps in all.  The lane then runs Eq. 1-4 over those steps from its own
// registers: U is neither written to memory nor staged.  A block's 256 / bb
// steps lie in 8 / bb waves (time chunks of 32 steps), which scan one after
// the other and hand c over through LDS; c carries over from block to block
// the same way.  The scan arithmetic is the forward scan kernel's, in the
// same order, so H equals the unfused path's bit for bit.
// 8 waves of 64 x 32k, A two K steps ahead (a type of its own per k: two
// kernels instantiating the main loop on one configuration type trip the
// host compilation pass)
template <int KB>
struct FusedCfg : DCfg<256, 64 * KB, 64, 4, 2, 2, 3> {};

template <bool B_>
struct BoolC {
  static constexpr bool value = B_;
};

template <int KB>
__global__ __launch_bounds__(512, 1) void proj_scan_fwd_kernel(FusedFwdArgs a) {
  using C = FusedCfg<KB>;
  static_assert(C::THREADS == 512, "8 waves");
  static_assert(C::FM == 2 && C::FN == KB, "a lane: 2 row blocks, one column block per gate");
  static_assert(C::WAVES_M == 4 && C::WAVES_N == 2, "wave rows and columns");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::LDS];

  // workgroup -> (direction, unit group, sequence group); XCD-aware, so the
  // workgroups of one XCD share the Wcat rows of a unit group
  const int nwg = gridDim.x, w = blockIdx.x;
  const int q8 = nwg / 8, rmd = nwg % 8, x8 = w % 8;
  const int wu = x8 * q8 + (x8 < rmd ? x8 : rmd) + w / 8;
  const int bg = wu % a.nbgroups;
  const int dg = wu / a.nbgroups;
  const int dir = dg / a.ngroups, g = dg % a.ngroups;
  const int nchunk = 8 / a.bb;  // time chunks of 32 steps per tile
  const int b0 = bg * a.bb;
  const bool rev = a.direction == 1 || (a.direction == 2 && dir == 1);
  const int L = a.L, Bs = a.B, d = a.d;
  const long long nfeat = (long long)a.ndir * d;

  // wave -> (time chunk, sequence pair, column half wn): the waves of one
  // chunk are consecutive, so they sit on different SIMDs (with two chunks,
  // waves 0-3 scan the first and waves 4-7 the second)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave & 1;
  const int pairs = 4 / nchunk;
  const int q2 = (wave >> 1) / pairs;
  const int pair = (wave >> 1) % pairs;
  const int wm = pair * nchunk + q2;  // the wave's 64-row block of the tile
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.Xb, a.a_bytes);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(a.Wb, a.b_bytes);
  using OpA = DirectOperand<C::BM, false, C::A_BPW, C::BK>;
  using OpB = DirectOperand<C::BN, false, C::B_BPW, C::BK>;
  // tile column 32 k cw + 32 gate + u: gate block `gate` of unit 64 g + 32 cw + u
  OpB lb;
  lb.init_rows(
      wave, lane,
      [&](int col) -> long long {
        const int cw = col / (32 * KB), gate = (col >> 5) % KB;
        return (long long)(dir * KB + gate) * d + g * 64 + cw * 32 + (col & 31);
      },
      a.d_in);
  // this lane's scan: sequence sb, unit 64 g + 32 wn + lane % 32, time chunk
  // q2 of every block; c carries over from block to block
  const int sb = b0 + 2 * pair + (lane >> 5);
  const bool live = sb < Bs;
  const int unit = g * 64 + wn * 32 + (lane & 31);
  const long long fidx = (long long)dir * d + unit;
  float vf = 0.f, vr = 0.f, bf = 0.f, br = 0.f, c = 0.f;
  if (live) {
    if (!a.linear) {
      vf = a.v_f[fidx];
      vr = a.v_r[fidx];
    }
    bf = a.b_f[fidx];
    br = a.b_r[fidx];
    c = a.c0 ? a.c0[(long long)sb * nfeat + fidx] : 0.f;
  }
  // gate parameters scaled by -log2(e), as in the forward scan
  const float vfs = vf * kNegLog2e, vrs = vr * kNegLog2e;
  const float bfs = bf * kNegLog2e, brs = br * kNegLog2e;
  const float alpha = a.alpha;
  const bool rn = a.reset_new != 0;
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // this wave's LDS accesses (lgkmcnt 0) only
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // hand-over of c between the waves of consecutive chunks, in LDS, which is
  // free between a block's product and the next block's
  float* cx = reinterpret_cast<float*>(smem) + (pair * C::WAVES_N + wn) * 64 + lane;

  const int TB = 32 * nchunk;  // steps per block
  const int nblk = (L + TB - 1) / TB;
  int prev = -1;  // the time chunk scanned last (-1: none yet)
  for (int ib = 0; ib < nblk; ++ib) {
    const int t0 = (rev ? nblk - 1 - ib : ib) * TB;  // blocks in the direction's order
    // tile row r: wave row r / 64 = (sequence pair, time chunk); in a 32-row
    // block, row rr is sequence (rr / 4) % 2 of the pair at step
    // 4 (rr / 8) + rr % 4 of the block's 16 (the MFMA's row of element e)
    OpA la;
    la.init_rows(
        wave, lane,
        [&](int r) -> long long {
          const int wr = r >> 6, rr = r & 31;
          const int b = b0 + 2 * (wr / nchunk) + ((rr >> 2) & 1);
          const int t =
              t0 + 32 * (wr % nchunk) + 16 * ((r >> 5) & 1) + 4 * (rr >> 3) + (rr & 3);
          return t < L && b < Bs ? (long long)t * Bs + b : -1;
        },
        a.d_in);
    floatx16 acc[C::FM][C::FN];
    direct_mainloop<C, false>(smem, la, lb, ra, rb, a.d_in, a.d_in, 0, a.d_in, wave, lane,
                              wm * C::WM, wn * C::WN, acc);
    // k = 3: the highway input x_t of the wave's chunk, loaded now so that it
    // arrives while earlier chunks scan (steps past L re-read step L - 1)
    float xr[32];
    if constexpr (KB == 3) {
      if (live) {
        const float* xp = a.X + (long long)sb * a.d_in + unit;
        const long long xs = (long long)Bs * a.d_in;
#pragma unroll
        for (int tt = 0; tt < 32; ++tt) xr[tt] = xp[min(t0 + 32 * q2 + tt, L - 1) * xs];
      }
    }
    (void)xr;
    barrier();  // every wave is done with the operand stages

    // the 32 steps of the chunk from step tb (scan order: backward for a
    // reverse direction); steps at or past L are not computed.  A whole
    // chunk runs without a branch between its steps, so the compiler can
    // overlap one step's output (reset gate, h, stores) with the next step's
    // chain.
    auto scan_chunk = [&](auto rev_c, auto whole_c, auto hb_c, int tb) {
      constexpr bool RV = decltype(rev_c)::value, WHOLE = decltype(whole_c)::value;
      constexpr bool HB = decltype(hb_c)::value;
      const int nv = min(32, L - tb);
      // padding bits of the chunk's steps: lane u of each half reads step
      // tb + u of its sequence, and the ballot hands each half its 32 bits
      unsigned mbits = 0;
      if (a.mask) {
        const int tm = tb + (lane & 31);
        const bool pad = live && tm < L && a.mask[(long long)tm * Bs + sb] != 0;
        mbits = (unsigned)(__ballot(pad) >> (32 * (lane >> 5)));
      }
      if (!live) return;
      // output offset at the chunk's first step in scan order, moved one
      // step at a time (the empty asm keeps the compiler from precomputing
      // every step's offset)
      const int tt0 = RV ? (WHOLE ? 31 : nv - 1) : 0;
      long long o = ((long long)(tb + tt0) * Bs + sb) * nfeat + fidx;
      const long long dstep = (RV ? -1LL : 1LL) * Bs * nfeat;
      // A step carries c forward first (Eq. 1-2) and then finishes the
      // previous step's output (Eq. 3-4, the store), which no longer lies on
      // the chain from one c to the next.
      float p_cn = 0.f, p_rin = 0.f, p_zr = 0.f, p_xh = 0.f;
      bool p_pad = false, pend = false;
      auto emit = [&]() {
        const float r = sigmoid_scaled(fmaf(vrs, p_rin, p_zr));        // Eq. 3
        float h = fmaf(r, p_cn, (1.0f - r) * (alpha * p_xh));          // Eq. 4 (Sec. 3.2)
        h = p_pad ? 0.0f : h;
        __builtin_nontemporal_store(h, a.H + o);
        if constexpr (HB)
          __builtin_nontemporal_store(__builtin_bit_cast(uint16_t, (__bf16)h), a.Hb + o);
        o += dstep;
        asm volatile("" : "+v"(o));
      };
#pragma unroll
      for (int s = 0; s < 32; ++s) {
        const int tt = RV ? 31 - s : s;
        if (WHOLE || tt < nv) {
          const float u0 = acc[tt >> 4][0][tt & 15], u1 = acc[tt >> 4][1][tt & 15];
          const float u2 = acc[tt >> 4][2][tt & 15];
          float xh;
          if constexpr (KB == 4) xh = acc[tt >> 4][3][tt & 15];
          else xh = xr[tt];
          const float f = sigmoid_scaled(fmaf(vfs, c, fmaf(u1, kNegLog2e, bfs)));  // Eq. 1
          const float cn = fmaf(f, c, fmaf(-f, u0, u0));                           // Eq. 2
          const float rin = rn ? cn : c;
          const bool pad = (mbits >> tt) & 1u;
          c = pad ? c : cn;
          if (WHOLE ? s > 0 : pend) emit();
          p_cn = cn;
          p_rin = rin;
          p_zr = fmaf(u2, kNegLog2e, brs);
          p_xh = xh;
          p_pad = pad;
          pend = true;
        }
      }
      if (pend) emit();
    };
    // one instantiation per (direction of time, whole chunk, bf16 copy of H)
    auto scan_any = [&](auto rev_c, int tb) {
      const bool whole = L - tb >= 32;
      if (whole) {
        if (a.Hb) scan_chunk(rev_c, BoolC<true>{}, BoolC<true>{}, tb);
        else scan_chunk(rev_c, BoolC<true>{}, BoolC<false>{}, tb);
      } else {
        if (a.Hb) scan_chunk(rev_c, BoolC<false>{}, BoolC<true>{}, tb);
        else scan_chunk(rev_c, BoolC<false>{}, BoolC<false>{}, tb);
      }
    };
    for (int i = 0; i < nchunk; ++i) {
      const int q = rev ? nchunk - 1 - i : i;  // the chunk scanned now
      if (nchunk > 1 && prev >= 0) {
        // the wave of the previous chunk (of this block or the one before)
        // hands its c over
        if (q2 == prev) *cx = c;
        barrier();
        if (q2 == q) c = *cx;
      }
      if (q2 == q) {
        if (rev) scan_any(BoolC<true>{}, t0 + 32 * q);
        else scan_any(BoolC<false>{}, t0 + 32 * q);
      }
      prev = q;
    }
    barrier();  // the hand-over's LDS reads are done before the next block's loads
  }
  if (live && a.c_last && q2 == prev) a.c_last[(long long)sb * nfeat + fidx] = c;
}

template <class C, int ADD, bool A_RC, bool B_RC, bool OB = false>
void launch_direct(const KernelArgs& a, int nwg, hipStream_t st) {
  hipLaunchKernelGGL((gemm_direct_kernel<C, ADD, A_RC, B_RC, OB>), dim3(nwg), dim3(C::THREADS), 0, st,
                     a);
}

// Sum of split partials in split order, plus the optional addend.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part,
                                                            int splits, int M, int N,
                                                            float* C, long long ldc,
                                                            const float* add, long long add_ld,
                                                            long long add_off, int add_count) {
  const long long total = (long long)M * N;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (long long)gridDim.x * 256) {
    const int m = (int)(i / N);
    const int n = (int)(i - (long long)m * N);
    float s = 0.f;
    for (int z = 0; z < splits; ++z) s += part[(long long)z * total + i];
    if (add_count > 0) {
      const float* ar = add + (long long)m * add_ld + n;
      s += ar[0];
      if (add_count > 1) s += ar[add_off];
    }
    C[(long long)m * ldc + n] = s;
  }
}

// The same for rows of 16-byte aligned groups of 4 (N % 4 == 0): one group
// per thread, the partials read as 16-byte loads.  The per-element sum is
// the same sequence of additions, so the result is bit-identical.  Blocks
// from `main_blocks` on run the v/b sums of the backward pass instead
// (vb_sum_block: the same bits as their own launch).
__device__ __forceinline__ void split_sum4_block(const SplitSum& j, unsigned blk) {
  const long long total = (long long)j.M * j.N;
  const long long i = ((long long)blk * 256 + threadIdx.x) * 4;
  if (i >= total) return;
  const int m = (int)(i / j.N);
  const int n = (int)(i - (long long)m * j.N);
  floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int z = 0; z < j.splits; ++z)
    s += *reinterpret_cast<const floatx4*>(j.part + z * total + i);
  if (j.add_count > 0) {
    const float* ar = j.add + (long long)m * j.add_ld + n;
    s += *reinterpret_cast<const floatx4*>(ar);
    if (j.add_count > 1) s += *reinterpret_cast<const floatx4*>(ar + j.add_off);
  }
  *reinterpret_cast<floatx4*>(j.C + (long long)m * j.ldc + n) = s;
}

// Blocks [0, n1) sum j1, [n1, n1 + n2) sum j2 (another product's deferred
// split sum: one launch instead of two), the rest the v/b sums.
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(SplitSum j1, unsigned n1,
                                                             SplitSum j2, unsigned n2,
                                                             VbSum vb) {
  const unsigned b = blockIdx.x;
  if (b < n1) {
    split_sum4_block(j1, b);
  } else if (b < n1 + n2) {
    split_sum4_block(j2, b - n1);
  } else {
    __shared__ float red[256];
    vb_sum_block(vb.partial, vb.rows, vb.nfeat, vb.qlo, vb.out, b - n1 - n2, red);
  }
}

bool split_sum_vec(const SplitSum& j) {
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return j.N % 4 == 0 && j.ldc % 4 == 0 && al16(j.part) && al16(j.C) &&
         (j.add_count == 0 || (j.add_ld % 4 == 0 && j.add_off % 4 == 0 && al16(j.add)));
}

// Split sum j (if j.part), the deferred split sum `extra` (if extra.part) and
// the v/b sums (if vb.partial), in one launch where the rows allow 16-byte
// accesses.
hipError_t launch_splitk_reduce(const SplitSum& j, const SplitSum& extra, const VbSum& vb,
                                hipStream_t st) {
  const bool vec = (!j.part || split_sum_vec(j)) && (!extra.part || split_sum_vec(extra));
  if (!vec) {
    // one element per thread, each sum in its own launch
    for (const SplitSum* q : {&extra, &j}) {
      if (!q->part) continue;
      const long long total = (long long)q->M * q->N;
      const int grid = (int)std::min<long long>((total + 255) / 256, 8192);
      timing_before("splitk_reduce", st);
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3(grid), dim3(256), 0, st, q->part, q->splits,
                         q->M, q->N, q->C, q->ldc, q->add, q->add_ld, q->add_off, q->add_count);
      timing_after(st);
      if (hipError_t e = hipGetLastError()) return e;
    }
    return vb.partial ? vb_sum_launch(vb, st) : hipSuccess;
  }
  auto blocks = [](const SplitSum& q) {
    return q.part ? (unsigned)(((long long)q.M * q.N / 4 + 255) / 256) : 0u;
  };
  const unsigned n1 = blocks(j), n2 = blocks(extra);
  const unsigned nv = vb.partial ? (unsigned)vb_sum_blocks(vb) : 0u;
  if (n1 + n2 + nv == 0) return hipSuccess;
  timing_before(n1 + n2 > 0 ? "splitk_reduce" : "reduce_vb", st);
  hipLaunchKernelGGL(splitk_reduce4_kernel, dim3(n1 + n2 + nv), dim3(256), 0, st, j, n1, extra,
                     n2, vb);
  timing_after(st);
  return hipGetLastError();
}

SplitSum split_sum_of(const GemmDesc& g, int splits) {
  SplitSum j;
  j.part = g.partials;
  j.splits = splits;
  j.M = g.M;
  j.N = g.N;
  j.C = g.C;
  j.ldc = g.ldc;
  j.add = g.add;
  j.add_ld = g.add_ld;
  j.add_off = g.add_off;
  j.add_count = g.add_count;
  return j;
}

// After a product: its split sum (unless deferred), the deferred split sum
// of an earlier product, and the v/b sums, in one launch.
hipError_t finish_product(const GemmDesc& g, int splits, hipStream_t st) {
  if (splits > 1 && g.defer_sum) return hipSuccess;
  const SplitSum own = splits > 1 ? split_sum_of(g, splits) : SplitSum{};
  return launch_splitk_reduce(own, g.extra, g.vb, st);
}

// fp32 -> bf16 conversions (RNE).  Plain copy: 8 elements per thread (two
// 16-byte loads, one 16-byte store).
__global__ __launch_bounds__(256) void to_bf16_kernel(const float* __restrict__ src,
                                                      long long n, uint16_t* __restrict__ dst) {
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i + 7 < n) {
    const floatx4 v0 = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(src + i));
    const floatx4 v1 = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(src + i + 4));
    u32x4 w;
    w[0] = pack_bf16(v0[0], v0[1]);
    w[1] = pack_bf16(v0[2], v0[3]);
    w[2] = pack_bf16(v1[0], v1[1]);
    w[3] = pack_bf16(v1[2], v1[3]);
    *reinterpret_cast<u32x4*>(dst + i) = w;
  } else {
    for (long long j = i; j < n; ++j)
      dst[j] = __builtin_bit_cast(uint16_t, (__bf16)src[j]);
  }
}

// Source element as fp32: fp32 as is, bf16 (raw bits) widened exactly.
__device__ __forceinline__ float src_f32(float v) { return v; }
__device__ __forceinline__ float src_f32(uint16_t v) {
  return __builtin_bit_cast(float, (unsigned)v << 16);
}

// Transposed: dst[c*rows + r] = bf16(src[r*cols + c]) through a 64x64 LDS tile.
// Few workgroups at the sizes it meets, so bound by latency: a thread's 16
// loads are all in flight before the first is used (8.6 us one by one at 1600 x
// 300; the backward of L 77, B 13, 304 -> 200 in both directions 42.1 -> 38.3
// us).  Rows and columns past the edge load the last one's.
template <class S>
__global__ __launch_bounds__(256) void to_bf16_t_kernel(const S* __restrict__ src, int rows,
                                                        int cols, uint16_t* __restrict__ dst) {
  __shared__ float tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  S v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = min(r0 + ty + 4 * k, rows - 1), c = min(c0 + tx, cols - 1);
    v[k] = src[(long long)r * cols + c];
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) tile[ty + 4 * k][tx] = src_f32(v[k]);
  __syncthreads();
#pragma unroll
  for (int i = ty; i < 64; i += 4) {
    const int c = c0 + i, r = r0 + tx;
    if (c < cols && r < rows)
      dst[(long long)c * rows + r] = __builtin_bit_cast(uint16_t, (__bf16)tile[tx][i]);
  }
}

// The same for whole 64 x 64 tiles with 16-byte accesses on both sides: each
// lane loads 16 bytes of a source row (4 fp32 or 8 bf16 elements) into the
// LDS tile, then packs 8 elements of a tile column into one 16-byte segment
// of an output row.  With the row pitch of 65 floats both the row writes and
// the column reads of the tile hit 64 distinct banks.
template <class S>
__global__ __launch_bounds__(256) void to_bf16_t_tiled_kernel(const S* __restrict__ src, int rows,
                                                              int cols, uint16_t* __restrict__ dst) {
  __shared__ float tile[64][65];
  constexpr int E = 16 / (int)sizeof(S);  // source elements per 16-byte load
  constexpr int TPR = 64 / E;             // lanes per tile row
  constexpr int RPR = 256 / TPR;          // tile rows per pass
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int t = threadIdx.x;
  const int lc = (t % TPR) * E;
  for (int i = t / TPR; i < 64; i += RPR) {
    const S* row = src + (long long)(r0 + i) * cols + c0 + lc;
    if constexpr (sizeof(S) == 4) {
      // loaded as floats: a bit cast of a vector element would read element 0
      const floatx4 v = *reinterpret_cast<const floatx4*>(row);
#pragma unroll
      for (int w = 0; w < 4; ++w) tile[i][lc + w] = v[w];
    } else {
      const u32x4 v = *reinterpret_cast<const u32x4*>(row);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const unsigned x = v[w];
        tile[i][lc + 2 * w] = __builtin_bit_cast(float, x << 16);
        tile[i][lc + 2 * w + 1] = __builtin_bit_cast(float, x & 0xFFFF0000u);
      }
    }
  }
  __syncthreads();
  const int q = t & 7;  // 8-element segment of the output row
  for (int c = t >> 3; c < 64; c += 32) {
    u32x4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = pack_bf16(tile[8 * q + 2 * j][c], tile[8 * q + 2 * j + 1][c]);
    *reinterpret_cast<u32x4*>(dst + (long long)(c0 + c) * rows + r0 + 8 * q) = w;
  }
}

// Direct loads need 16-byte aligned chunks that are either wholly inside or
// wholly outside the operand, i.e. the contiguous extent (K for KC, the row
// count for RC) and the leading dimension are multiples of 8 elements.
bool whole_chunks(const void* p, long long ld, int contiguous_extent) {
  return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 8 == 0 && contiguous_extent % 8 == 0;
}

// ---- the direct path: plan (shared by workspace sizing and launch) ----
long long operand_bytes(bool kc, int rows, int K, long long ld, int esz) {
  return (long long)esz * (kc ? (long long)(rows - 1) * ld + K : (long long)(K - 1) * ld + rows);
}

// The direct kernel addresses each operand from its workgroup's panel (a
// tile's 256 rows of a K-contiguous operand, a split's k-rows of a
// row-contiguous one) with 32-bit offsets below kOOB.  Bytes a panel spans:
long long panel_bytes(bool kc, int rows, int K, long long ld, long long k_rows) {
  return 2 * (kc ? (long long)(min(rows, 256) - 1) * ld + K : (k_rows - 1) * ld + rows);
}
// The largest K range (whole 64-k stages) whose row-contiguous panel fits;
// 0 if not even one stage does.
long long rc_max_k(int rows, long long ld) {
  const long long room = (long long)kOOB - 1 - 2LL * rows;  // bytes for (k_rows - 1) * 2 ld
  if (room < 0) return 0;
  return ((room / (2 * ld) + 1) / 64) * 64;
}
bool split_allowed(const GemmDesc& g) { return !g.Cb && (!g.a_kc || g.kc_split); }

// bf16 x bf16 operands whose 16-byte chunks are whole (the contiguous
// extent and leading dimension are multiples of 8 elements) and whose
// panels fit the 32-bit offsets: a K-contiguous operand's 256 rows, a
// row-contiguous one's whole K when the product is not split, else one
// 64-k stage (the split count then keeps each split's panel in range, see
// plan_direct).  Layouts: both K-contiguous or both row-contiguous.
bool direct_ok(const GemmDesc& g) {
  if (!g.bf16 || !g.a_bf16 || !g.b_bf16 || g.a_kc != g.b_kc) return false;
  auto fits = [&](bool kc, int rows, long long ld) {
    if (kc) return panel_bytes(true, rows, g.K, ld, 0) < (long long)kOOB;
    return split_allowed(g) ? rc_max_k(rows, ld) >= 64 : rc_max_k(rows, ld) >= g.K;
  };
  return whole_chunks(g.A, g.lda, g.a_kc ? g.K : g.M) &&
         whole_chunks(g.B, g.ldb, g.b_kc ? g.K : g.N) && g.M > 0 && g.N > 0 &&
         g.K > 0 && fits(g.a_kc, g.M, g.lda) && fits(g.b_kc, g.N, g.ldb);
}

// Time in us of wg workgroups of st K steps (64 k) each, from times measured
// over 32 to 3072 workgroups and 8 to 128 steps.  Big: rounds of one per CU,
// whose steps slow down as the chip fills (shared caches and clock).  Mid: two
// per CU run at half speed each; an odd one left over runs alone.
double direct_cost(bool mid, bool rc, long long wg, double st) {
  const long long n = (wg + 255) / 256;
  if (!mid) return n * (8.0 + st * (1.2 + 0.5 * std::min(1.0, wg / 256.0)));
  return 3.0 + (n / 2) * 2 * (1.4 + 0.51 * st) + (n % 2) * (2.0 + (rc ? 0.85 : 0.62) * st);
}

// Tile and split count of a direct product: the least modelled time, K-contiguous
// ones of fewer than kBigMinSteps K steps on mid tiles.  (There a product is its
// output, which the one workgroup of a CU writes while nothing else runs: 4653 x
// 2784 x 32 35 us on big tiles, 15.6 on mid; 1520 x 5472 x 88 36 and 19; 10640 x
// 1376 x 176 29 and 24; in 130 sizes of at most 5 steps big ones were never ahead
// by more than 3 %: 1626 x 7168 x 64 17.0 and 17.6.)  The
// K = tokens product (row-contiguous operands) may be cut over K, and so may
// a K-contiguous product whose caller asks for it (kc_split: dX of a small
// batch, whose few tiles would leave most CUs idle), with at least 6 K steps
// per split; the split sum reads the partials at about 6.5 TB/s.  A bf16
// result (Cb) is never split.  E.g. 3072 x 1024 over 16384 tokens: big tiles
// in 5 splits (240 workgroups of 52 steps, 101 us and 12 for the sum); over
// 2048: mid tiles in 2 (21 and 6 us; big ones in 5: 25 and 12).
constexpr int kBigMinSteps = 6;
struct DirectPlan {
  bool mid;
  int splits;
};
struct DirectRange {
  int lo, hi;
};
DirectRange direct_range(const GemmDesc& g) {
  const int kt = (g.K + 63) / 64;
  if (!split_allowed(g)) return {1, 1};
  // fewest splits whose row-contiguous panels fit (direct_ok: one stage does)
  long long kmax = kt;
  if (!g.a_kc)
    kmax = std::max(1LL, std::min({kmax, rc_max_k(g.M, g.lda) / 64, rc_max_k(g.N, g.ldb) / 64}));
  const int lo = (int)((kt + kmax - 1) / kmax);
  return {lo, std::max(lo, kt / 6)};
}
// every count up to 8, then steps of a quarter or less
int next_direct_split(int s) { return s + std::max(1, s / 8); }
long long direct_tiles(const GemmDesc& g, int b) {
  return (long long)((g.M + b - 1) / b) * ((g.N + b - 1) / b);
}
double sum_traffic(const GemmDesc& g, int s) {
  return s > 1 ? (s + 1) * 4.0 * g.M * g.N / 6.5e6 : 0.0;
}
// the real number of splits, each of whole K steps
int real_direct_splits(const GemmDesc& g, int s) {
  const int kt = (g.K + 63) / 64, per = (kt + s - 1) / s;
  return (kt + per - 1) / per;
}

DirectPlan plan_direct(const GemmDesc& g, double* time = nullptr) {
  if (g.plan_splits > 0) return {g.plan_tile != 0, g.plan_splits};
  const int kt = (g.K + 63) / 64;
  const DirectRange r = direct_range(g);
  DirectPlan best{false, r.lo};
  double best_cost = -1.0;
  for (int m = g.a_kc && kt < kBigMinSteps; m < 2; ++m) {
    const long long tiles = direct_tiles(g, m ? 128 : 256);
    for (int s = r.lo; s <= r.hi; s = next_direct_split(s)) {
      const double cost = direct_cost(m, !g.a_kc, tiles * s, (kt + s - 1) / s) +
                          (s > 1 ? 2.0 + sum_traffic(g, s) : 0.0);
      if (best_cost < 0 || cost < best_cost) {
        best = {m != 0, s};
        best_cost = cost;
      }
    }
  }
  best.splits = real_direct_splits(g, best.splits);
  if (time) *time = best_cost;
  return best;
}

// dX and dW together on mid tiles, where pair_time beats the two plans one
// after the other.  L 256, B 8, d 1024: dX in 2 splits
// and dW whole, 40 us and 6 for the sum, against 21 + 21 us and 12 (each in 2
// splits).
GemmPair direct_pair_plan(const GemmDesc& gx, const GemmDesc& gw, double& best_cost) {
  GemmPair best{0, 0, 0};
  double tx, tw;
  plan_direct(gx, &tx);
  plan_direct(gw, &tw);
  best_cost = tx + tw;
  const int kx = (gx.K + 63) / 64, kw = (gw.K + 63) / 64;
  const DirectRange rx = direct_range(gx), rw = direct_range(gw);
  const long long nx = direct_tiles(gx, 128), nw = direct_tiles(gw, 128);
  for (int sx = rx.lo; sx <= rx.hi; sx = next_direct_split(sx)) {
    const int stx = (kx + sx - 1) / sx;
    for (int sw = rw.lo; sw <= rw.hi; sw = next_direct_split(sw)) {
      const int stw = (kw + sw - 1) / sw;
      const double cost = 3.0 + pair_time(nx * sx, stx, 0.62, nw * sw, stw, 0.85, 1.4, 0.51) +
                          sum_traffic(gx, sx) + sum_traffic(gw, sw) +
                          (sx > 1 || sw > 1 ? 2.0 : 0.0);
      if (cost < best_cost) {
        best = {1, real_direct_splits(gx, sx), real_direct_splits(gw, sw)};
        best_cost = cost;
      }
    }
  }
  return best;
}

// Explicit instantiations: the host pass did not emit the launch stubs of
// every specialisation referenced through launch_direct_cfg.
#define SRU_DIRECT_INST(CFG, ADD, ARC, BRC, OB) \
  template __global__ void gemm_direct_kernel<CFG, ADD, ARC, BRC, OB>(KernelArgs);
SRU_DIRECT_INST(CfgBigKC, 0, false, false, false)
SRU_DIRECT_INST(CfgBigKC, 1, false, false, false)
SRU_DIRECT_INST(CfgBigKC, 2, false, false, false)
SRU_DIRECT_INST(CfgBigKC, 0, false, false, true)
SRU_DIRECT_INST(CfgMidKC, 0, false, false, false)
SRU_DIRECT_INST(CfgMidKC, 1, false, false, false)
SRU_DIRECT_INST(CfgMidKC, 2, false, false, false)
SRU_DIRECT_INST(CfgMidKC, 0, false, false, true)
SRU_DIRECT_INST(CfgBigRC, 0, true, true, false)
SRU_DIRECT_INST(CfgMidRC, 0, true, true, false)
#undef SRU_DIRECT_INST

template <class C, bool OB = false>
KernelArgs direct_args(const GemmDesc& g, int splits) {
  static_assert(C::BK == 64, "the plan counts 64-k steps");
  const int kt = (g.K + C::BK - 1) / C::BK;
  const int kps = ((kt + splits - 1) / splits) * C::BK;
  KernelArgs a{};
  a.A = g.A;
  a.B = g.B;
  a.lda = g.lda;
  a.ldb = g.ldb;
  a.M = g.M;
  a.N = g.N;
  a.K = g.K;
  a.a_bytes = operand_bytes(g.a_kc, g.M, g.K, g.lda, 2);
  a.b_bytes = operand_bytes(g.b_kc, g.N, g.K, g.ldb, 2);
  a.k_per_split = kps;
  a.tiles_m = (g.M + C::BM - 1) / C::BM;
  a.tiles_n = (g.N + C::BN - 1) / C::BN;
  a.splits = splits;
  if (splits > 1) {
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
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  a.outb = g.Cb;
  a.ldob = g.ldcb;
  a.vec_out = a.ldo % 4 == 0 && a.split_stride % 4 == 0 && (!a.out || al16(a.out)) &&
              (a.add_count == 0 || (a.add_ld % 4 == 0 && a.add_off % 4 == 0 && al16(a.add))) &&
              (!OB || (a.ldob % 4 == 0 && ((uintptr_t)a.outb & 7) == 0));
  return a;
}

template <class C, bool RC, bool OB = false>
hipError_t launch_direct_cfg(const GemmDesc& g, int splits, hipStream_t st) {
  const KernelArgs a = direct_args<C, OB>(g, splits);
  const int nwg = a.tiles_m * a.tiles_n * splits;
  timing_before(gemm_label(g), st);
  if constexpr (OB) launch_direct<C, 0, RC, RC, true>(a, nwg, st);
  else if constexpr (RC) launch_direct<C, 0, RC, RC>(a, nwg, st);  // no addend
  else if (a.add_count == 2) launch_direct<C, 2, RC, RC>(a, nwg, st);
  else if (a.add_count == 1) launch_direct<C, 1, RC, RC>(a, nwg, st);
  else launch_direct<C, 0, RC, RC>(a, nwg, st);
  timing_after(st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return finish_product(g, splits, st);
}

}  // namespace

bool gemm_is_direct(const GemmDesc& g) { return direct_ok(g); }

int gemm_splits(const GemmDesc& g) {
  if (direct_ok(g)) return plan_direct(g).splits;
  return gemm_staged_splits(g);
}

SplitSum gemm_split_sum(const GemmDesc& g) { return split_sum_of(g, gemm_splits(g)); }

size_t gemm_partial_bytes(int M, int N, int splits) {
  return splits > 1 ? sizeof(float) * (size_t)splits * (size_t)M * (size_t)N : 0;
}

hipError_t gemm_launch(const GemmDesc& g, hipStream_t st) {
  if ((g.a_bf16 || g.b_bf16) && !g.bf16) return hipErrorInvalidValue;
  if (direct_ok(g)) {
    const DirectPlan p = plan_direct(g);
    if (g.Cb) {
      // bf16 result: K-contiguous operands, no addend (never split)
      if (!g.a_kc || g.add_count != 0) return hipErrorInvalidValue;
      return p.mid ? launch_direct_cfg<CfgMidKC, false, true>(g, 1, st)
                   : launch_direct_cfg<CfgBigKC, false, true>(g, 1, st);
    }
    if (!g.a_kc) {
      if (g.add_count != 0) return hipErrorInvalidValue;
      return p.mid ? launch_direct_cfg<CfgMidRC, true>(g, p.splits, st)
                   : launch_direct_cfg<CfgBigRC, true>(g, p.splits, st);
    }
    return p.mid ? launch_direct_cfg<CfgMidKC, false>(g, p.splits, st)
                 : launch_direct_cfg<CfgBigKC, false>(g, p.splits, st);
  }
  if (g.Cb) return hipErrorInvalidValue;  // a bf16 result needs the direct path
  if (hipError_t e = gemm_staged_launch(g, st)) return e;
  return finish_product(g, gemm_staged_splits(g), st);
}

// A dW that cannot run direct (ragged rows) takes dX along on staged tiles
// where that beats the two: L 77, B 13, 300 -> 200 units in both directions,
// 18 us against 8.6 for W^T, 13.5 and 16.6 us and one more split sum (the whole
// backward 54.2 -> 33.6 us); 20,000 tokens of 612 columns are left as they were.
// Two that could run direct do so too at the smallest sizes, whose 64 x 64 tiles
// are several where 128 x 128 is one: the backward of L 20, B 4, d 64 27.0 ->
// 13.1 us, L 32, B 4, d 96 30.3 -> 15.2 us; from L 64, B 32, d 256 the direct
// plans stay ahead.
GemmPairPlan gemm_pair_plan(const GemmDesc& gx, const GemmDesc& gx_nn, const GemmDesc& gw) {
  const bool dx = direct_ok(gx), dw = direct_ok(gw);
  if (gx.Cb || gw.Cb || gw.add_count != 0 || (dw && !dx)) return {};
  GemmPairPlan p{};
  double time;  // to beat
  if (dw) {
    static_cast<GemmPair&>(p) = direct_pair_plan(gx, gw, time);
  } else {
    if (dx) plan_direct(gx, &time);
    else time = gemm_staged_time(gx);
    time += gemm_staged_time(gw);
  }
  const GemmPair staged = gemm_staged_pair_plan(gx_nn, gw, time);
  return staged.splits_x > 0 ? GemmPairPlan{staged, true} : p;
}

hipError_t gemm_pair_launch(const GemmDesc& gx, const GemmDesc& gw, hipStream_t st) {
  const bool dx = direct_ok(gx) && direct_ok(gw);
  if (!dx && (gx.b_kc || !gemm_staged_pair_launch(gx, gw, st))) {
    // operands that need other loads than the plan assumed: fp32 ones of a
    // caller, on 4 bytes (bf16 ones are in the workspace or on 16 bytes)
    if (gx.bf16) return hipErrorInvalidValue;
    if (hipError_t e = gemm_launch(gx, st)) return e;
    return gemm_launch(gw, st);
  }
  if (dx) {
    const KernelArgs a = direct_args<CfgMidKC>(gx, gx.plan_splits);
    const KernelArgs b = direct_args<CfgMidRC>(gw, gw.plan_splits);
    const int n1 = a.tiles_m * a.tiles_n * a.splits, n2 = b.tiles_m * b.tiles_n * b.splits;
    const dim3 grid(n1 + n2), block(CfgMidKC::THREADS);
    const bool dwf = b.k_per_split > a.k_per_split;
    timing_before("gemm_dx_dw", st);
    if (a.add_count == 2)
      hipLaunchKernelGGL(gemm_direct_pair_kernel<2>, grid, block, 0, st, a, n1, b, n2, dwf);
    else if (a.add_count == 1)
      hipLaunchKernelGGL(gemm_direct_pair_kernel<1>, grid, block, 0, st, a, n1, b, n2, dwf);
    else
      hipLaunchKernelGGL(gemm_direct_pair_kernel<0>, grid, block, 0, st, a, n1, b, n2, dwf);
    timing_after(st);
  }
  if (hipError_t e = hipGetLastError()) return e;
  // both split sums and the v/b sums in one launch
  return launch_splitk_reduce(gw.plan_splits > 1 ? split_sum_of(gw, gw.plan_splits) : SplitSum{},
                              gx.plan_splits > 1 ? split_sum_of(gx, gx.plan_splits) : SplitSum{},
                              gw.vb, st);
}

template <class S>
void launch_transpose(const S* src, int rows, int cols, uint16_t* dst, hipStream_t st) {
  const dim3 grid((cols + 63) / 64, (rows + 63) / 64);
  const bool tiled = rows % 64 == 0 && cols % 64 == 0 &&
                     (reinterpret_cast<uintptr_t>(src) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
  if (tiled)
    hipLaunchKernelGGL(to_bf16_t_tiled_kernel<S>, grid, dim3(256), 0, st, src, rows, cols, dst);
  else
    hipLaunchKernelGGL(to_bf16_t_kernel<S>, grid, dim3(256), 0, st, src, rows, cols, dst);
}

hipError_t to_bf16_t_launch(const void* src, bool src_bf16, int rows, int cols, uint16_t* dst,
                            hipStream_t st, const char* label) {
  timing_before(label, st);
  if (src_bf16) launch_transpose(static_cast<const uint16_t*>(src), rows, cols, dst, st);
  else launch_transpose(static_cast<const float*>(src), rows, cols, dst, st);
  timing_after(st);
  return hipGetLastError();
}

void launch_copy(const float* src, long long n, uint16_t* dst, hipStream_t st) {
  const long long threads = (n + 7) / 8;
  hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                     src, n, dst);
}

hipError_t to_bf16_launch(const float* src, int rows, int cols, uint16_t* dst, bool transpose,
                          hipStream_t st, const char* label) {
  timing_before(label, st);
  if (transpose) {
    launch_transpose(src, rows, cols, dst, st);
  } else {
    launch_copy(src, (long long)rows * cols, dst, st);
  }
  timing_after(st);
  return hipGetLastError();
}

hipError_t proj_scan_forward_launch(const FusedFwdArgs& a, hipStream_t st) {
  // a tile holds 256 / bb steps of bb sequences, in time chunks of 32 steps;
  // k = 3 reads x_t from X (d_in = d)
  if ((a.bb != 2 && a.bb != 4 && a.bb != 8) || (a.k != 3 && a.k != 4) ||
      (a.k == 3 && (!a.X || a.d_in != a.d)))
    return hipErrorInvalidValue;
  const int grid = a.ndir * a.ngroups * a.nbgroups;
  timing_before("proj_scan_fwd", st);
  if (a.k == 3)
    hipLaunchKernelGGL((proj_scan_fwd_kernel<3>), dim3(grid), dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL((proj_scan_fwd_kernel<4>), dim3(grid), dim3(512), 0, st, a);
  timing_after(st);
  return hipGetLastError();
}

hipError_t to_bf16_n_launch(const float* src, long long n, uint16_t* dst, hipStream_t st,
                            const char* label) {
  timing_before(label, st);
  launch_copy(src, n, dst, st);
  timing_after(st);
  return hipGetLastError();
}

}  // namespace sru
