// Projection and forward scan of a few tokens in one kernel (gfx950): the
// decode step of inference with bf16 products, and short chunks.  Neither U
// nor C is kept.
//
// With at most 128 tokens the layer is one pass over Wcat: what counts is how
// many CUs read it at once and how soon, not the matrix units.  A workgroup
// is one wave and owns 8 hidden units of one direction: their k gate rows of
// Wcat are the 32 columns of one 32-column MFMA block (k = 3: 24 and zeros),
// the tokens its rows (FM blocks of 32).  d = 1024 then takes 128 CUs, and
// each reads 48 KiB (k = 3; 64 for k = 4).  Both operands go straight from memory into registers in
// the MFMA's layout, 16 bytes a lane, two sets of S slabs (16 k) in flight;
// X is rounded on the way (RNE) where that beats a launch that rounds it first
// (step_rounds_x), unless the caller holds it in bf16.  The slabs accumulate in the order of
// the other products, so U has their bits; it passes through LDS, where the
// scan gives each lane one (sequence, unit).
//
// One step (L 1) of B 8, d 1024: 21.9 us on the tiled kernel, whose 256-row
// tiles give 64 CUs one tile of 16 serial stages each, and 2.5 us for rounding
// X; 8.0 us here, most of it two round trips to memory and the launch.
#include "sru_device.h"
#include "sru_gemm_tile.h"
#include "sru_internal.h"

namespace sru {
namespace {

constexpr int kStepUnits = 8;  // hidden units per workgroup

template <int KB, int FM, bool XB>
__global__ __launch_bounds__(64, 1) void few_tokens_fwd_kernel(FusedFwdArgs a) {
  constexpr int S = FM == 1 ? 16 : FM == 2 ? 8 : 4;  // slabs per register set
  __shared__ float u[FM * 32][33];

  const int lane = threadIdx.x;
  const int d = a.d, d_in = a.d_in, Bs = a.B, L = a.L;
  const int groups = d / kStepUnits;
  const int dir = blockIdx.x / groups;
  const int unit0 = (blockIdx.x - dir * groups) * kStepUnits;
  const bool rev = a.direction == 1 || (a.direction == 2 && dir == 1);
  const int M = L * Bs;

  const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.Wb, a.b_bytes);
  const __amdgpu_buffer_rsrc_t rx =
      XB ? make_rsrc(a.Xb, a.a_bytes) : make_rsrc(a.X, 2 * a.a_bytes);
  constexpr unsigned XE = XB ? 2 : 4;
  const int h8 = (lane >> 5) * 8;  // the lane's k within a slab
  const int gate = (lane & 31) >> 3;
  // offsets at slab 0; rows past the end read zeros (no memory)
  const unsigned woff =
      gate < KB ? (unsigned)((((long long)dir * KB + gate) * d + unit0 + (lane & 7)) * d_in + h8) * 2u
                : kOOB;
  unsigned xoff[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = i * 32 + (lane & 31);
    xoff[i] = m < M ? (unsigned)(m * d_in + h8) * XE : kOOB;
  }

  struct Set {
    u32x4 w[S], x[S][FM][XB ? 1 : 2];
  };
  auto load = [&](Set& g, int s0) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = (s0 + s) * 16;
      const unsigned oob = (unsigned)(k + h8 >= d_in) << 31;
      g.w[s] = buf_load16(rw, (woff + (unsigned)k * 2u) | oob);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const unsigned o = (xoff[i] + (unsigned)k * XE) | oob;
        g.x[s][i][0] = buf_load16(rx, o);
        if constexpr (!XB) g.x[s][i][1] = buf_load16(rx, o + 16u);
      }
    }
  };
  floatx16 acc[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  auto compute = [&](const Set& g) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        u32x4 x;
        if constexpr (XB) {
          x = g.x[s][i][0];
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            x[q] = pack_bf16(f32_of(g.x[s][i][q >> 1], 2 * (q & 1)),
                             f32_of(g.x[s][i][q >> 1], 2 * (q & 1) + 1));
        }
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, g.w[s]), acc[i], 0, 0, 0);
      }
  };
  const int nslab = (d_in + 15) / 16;
  Set g0, g1;
  load(g0, 0);
  load(g1, S);
  for (int s = 0; s < nslab; s += 2 * S) {  // slabs past the end are zeros
    compute(g0);
    load(g0, s + 2 * S);
    __builtin_amdgcn_sched_barrier(0);
    compute(g1);
    load(g1, s + 3 * S);
    __builtin_amdgcn_sched_barrier(0);
  }

#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e)
      u[i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)][lane & 31] = acc[i][e];
  __syncthreads();

  // Eq. 1-4, the forward scan's arithmetic in its order
  const long long nfeat = (long long)a.ndir * d;
  for (int p = lane; p < Bs * kStepUnits; p += 64) {
    const int b = p / kStepUnits, uu = p % kStepUnits;
    const long long fidx = (long long)dir * d + unit0 + uu;
    const float vfs = (a.linear ? 0.f : a.v_f[fidx]) * kNegLog2e;
    const float vrs = (a.linear ? 0.f : a.v_r[fidx]) * kNegLog2e;
    const float bfs = a.b_f[fidx] * kNegLog2e, brs = a.b_r[fidx] * kNegLog2e;
    float c = a.c0 ? a.c0[b * nfeat + fidx] : 0.f;
    for (int s = 0; s < L; ++s) {
      const int t = rev ? L - 1 - s : s;
      const int m = t * Bs + b;
      const float u0 = u[m][uu], u1 = u[m][8 + uu], u2 = u[m][16 + uu];
      const float xh = KB == 4 ? u[m][24 + uu] : a.X[(long long)m * d_in + unit0 + uu];
      const bool pad = a.mask && a.mask[m] != 0;
      const float f = sigmoid_scaled(fmaf(vfs, c, fmaf(u1, kNegLog2e, bfs)));
      const float cn = fmaf(f, c, fmaf(-f, u0, u0));
      const float r = sigmoid_scaled(fmaf(vrs, a.reset_new ? cn : c, fmaf(u2, kNegLog2e, brs)));
      float h = fmaf(r, cn, (1.0f - r) * (a.alpha * xh));
      h = pad ? 0.f : h;
      c = pad ? c : cn;
      a.H[m * nfeat + fidx] = h;
      if (a.Hb) a.Hb[m * nfeat + fidx] = __builtin_bit_cast(uint16_t, (__bf16)h);
    }
    if (a.c_last) a.c_last[b * nfeat + fidx] = c;
  }
}

template <int KB, int FM>
void launch_step(const FusedFwdArgs& a, hipStream_t st) {
  const dim3 grid(a.ndir * (a.d / kStepUnits));
  if (a.Xb) hipLaunchKernelGGL((few_tokens_fwd_kernel<KB, FM, true>), grid, dim3(64), 0, st, a);
  else hipLaunchKernelGGL((few_tokens_fwd_kernel<KB, FM, false>), grid, dim3(64), 0, st, a);
}

template <int KB>
void launch_step_rows(const FusedFwdArgs& a, hipStream_t st) {
  const int M = a.L * a.B;
  if (M <= 32) launch_step<KB, 1>(a, st);
  else if (M <= 64) launch_step<KB, 2>(a, st);
  else launch_step<KB, 4>(a, st);
}

}  // namespace

hipError_t step_forward_launch(const FusedFwdArgs& a, hipStream_t st) {
  const long long tokens = (long long)a.L * a.B, nfeat = (long long)a.ndir * a.d;
  if ((a.k != 3 && a.k != 4) || !step_few_tokens(tokens, a.L, nfeat) || a.d % kStepUnits != 0 ||
      !a.X || (a.k == 3 && a.d_in != a.d) || (!a.Xb && !step_rounds_x(tokens, a.d_in, nfeat)))
    return hipErrorInvalidValue;
  timing_before("proj_scan_fwd", st);
  if (a.k == 3) launch_step_rows<3>(a, st);
  else launch_step_rows<4>(a, st);
  timing_after(st);
  return hipGetLastError();
}

}  // namespace sru
