// Two time steps per launch for wide 2-D stencils (radius 4 .. 7, 16-bit carry, sparse
// engine).
//
// One step per launch moves a 10240^2 fp16 grid through memory in 88 us at the rate of a
// large copy, and its 15 instructions per 16 x 16 outputs (r = 7) take 60: with two
// waves per SIMD neither hides under the other (114 us).  Two steps share the
// operands and the line walk of one wave: the first step's lines go to the second through
// one LDS line, rounded to the carry as a stored grid would be and zero outside the grid,
// and memory is passed once for both.  Fp16, 10240^2, us per step, one step and two: r = 4
// 102 and 63, r = 5 105 and 71, r = 6 109 and 82, r = 7 114 and 93, where the matrix
// instructions are the largest bound (the pipe is busy 68 % of a launch by its counter).
//
// Registers decide the shape: 15 operand rows and 2 x 15 accumulators are 188 of the 256
// that two waves per SIMD leave, so input lines are staged a third of a turn at a time
// (five lines, five lines ahead) instead of a whole one, and outputs are stored as they
// complete.  The sums are those of two launches of one step bit for bit: strips start at
// x = 8 mod 16 in both, and every line's products are added in the order of the lines.
// (Of finite values; infinities and NaN of the line between the steps reach the strip from
// the columns that it computes only, whereas single steps multiply whole chunks.)
#include <hip/hip_runtime.h>

#include "band_common.h"
#include "kernels.h"

namespace spider_impl {

template <int R, int OP, bool ALIGNED>
__device__ __forceinline__ void band2d_wide2_body(const BandGrid& g, int w, uint32_t* lds) {
  constexpr int RR = 2 * R + 1;
  constexpr int GS = (RR + 2) / 3;  // lines staged together (the last third may be shorter)
  const int lane = threadIdx.x;
  const int strip = w % g.nstrips, seg = w / g.nstrips;
  const int x0 = strip * kStripW2_host, y0 = seg * g.seg_h;
  const int hrows = min(g.seg_h, g.ny - y0);
  // the second step runs one line behind the first: output i completes with input i + 4R + 1
  const int nin = (hrows + 4 * R + 1 + RR - 1) / RR * RR;
  const int nx = g.nx, ny = g.ny;

  u32x4 A[RR];
  uint32_t I[(RR + 1) / 2];
#pragma unroll
  for (int a = 0; a < RR; ++a) A[a] = reinterpret_cast<const u32x4*>(g.apack)[a * 64 + lane];
#pragma unroll
  for (int a = 0; a < (RR + 1) / 2; ++a) I[a] = g.ipack[a * 64 + lane];
  __builtin_amdgcn_s_waitcnt(0);

  int p1, p2;
  band_gather_offsets(lane, &p1, &p2);
  // a staged line covers [x0 - 16, x0 + 256); either step computes [x0 - 8, x0 + 248)
  const OddTail tail(ALIGNED ? 0 : nx, x0 - 16, 8 * kRowChunks);
  const uint32_t lvoff = tail.voff(chunk_voffset(x0 - 8, lane), lane, nx);
  const int xl = x0 - 8 + 16 * (lane & 15) + 4 * (lane >> 4);  // this lane's four columns
  const uint32_t ovoff = xl >= x0 && xl < x0 + kStripW2_host ? (uint32_t)(xl * 2) : kOffNone;
  const int odd = ALIGNED ? 0 : odd_store(nx, x0, x0 + kStripW2_host);
  const uint32_t ooff = odd_store_off(nx, xl);
  const uint32_t xm0 = (xl >= 0 && xl < nx ? 0x0000ffffu : 0u) | (xl + 1 >= 0 && xl + 1 < nx ? 0xffff0000u : 0u);
  const uint32_t xm1 = (xl + 2 >= 0 && xl + 2 < nx ? 0x0000ffffu : 0u) | (xl + 3 >= 0 && xl + 3 < nx ? 0xffff0000u : 0u);
  const int lw = lds_phys(4 * (lane < kRowChunks ? lane : 0));
  // the line between the steps; the eight columns on either side that no lane writes
  // feed only columns that are not stored
  uint32_t* mid = lds + GS * kLdsRowDw;
  const int mw = lds_phys(4 + 8 * (lane & 15) + 2 * (lane >> 4));
  for (int i = lane; i < kLdsRowDw; i += 64) mid[i] = 0u;

  LineWalk lin(g.in, y0 - 2 * R, max(0, y0 - 2 * R), min(ny, y0 + hrows + 2 * R), nx * 2);
  LineWalk lout(g.out, y0 - 4 * R - 1, y0, y0 + hrows, nx * 2);
  u32x4 stg[GS];
  auto load = [&](auto n) {
#pragma unroll
    for (int q = 0; q < n.value; ++q) stg[q] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
  };
  auto stage = [&](auto n) {
    if (lane < kRowChunks) {
#pragma unroll
      for (int q = 0; q < n.value; ++q) store_chunk_lds(lds, lw + q * kLdsRowDw, stg[q]);
    }
    if constexpr (!ALIGNED) {
#pragma unroll
      for (int q = 0; q < n.value; ++q) tail.put(lds + q * kLdsRowDw, lds_phys(tail.at >> 1), lane, stg[q]);
    }
  };
  using First = std::integral_constant<int, GS>;
  using Last = std::integral_constant<int, RR - 2 * GS>;
  load(First{});
  stage(First{});
  load(First{});
  wave_lds_sync();
  u32x4 b = {lds[p1], lds[p1 + 10], lds[p2], lds[p2 + 10]};
  u32x4 b2 = {0u, 0u, 0u, 0u};
  f32x4 acc1[RR], acc2[RR];
#pragma unroll
  for (int s = 0; s < RR; ++s) acc1[s] = acc2[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
  int ym = y0 - 3 * R;  // grid row of the line between the steps that line j completes

  for (int jb = 0; jb < nin; jb += RR) {
#pragma unroll
    for (int q = 0; q < RR; ++q) {
      auto mma = [&](f32x4* acc, int a, const u32x4& v) {
        const int slot = ((q - a) % RR + RR) % RR;
        const u32x4 none = {0u, 0u, 0u, 0u};
        if (a & 1)
          acc[slot] = band_mma<OP, 1, 1>(acc[slot], A[a], none, none, I[a / 2], v);
        else
          acc[slot] = band_mma<OP, 1, 0>(acc[slot], A[a], none, none, I[a / 2], v);
      };
      const int fs = (q + 1) % RR;
      // the lines that complete with this one first, so that their rounding, the LDS round
      // trip to the next line's second step and the store lie under the other instructions
      mma(acc1, 2 * R, b);
      mma(acc2, 2 * R, b2);
#pragma unroll
      for (int a = 0; a < R; ++a) mma(acc2, a, b2);
      {
        const uint2 pv = pack_out<OP>(acc1[fs]);
        const bool rok = (uint32_t)ym < (uint32_t)ny;
        ++ym;
        wave_lds_sync();
        *reinterpret_cast<uint2*>(mid + mw) = make_uint2(rok ? (pv.x & xm0) : 0u, rok ? (pv.y & xm1) : 0u);
        acc1[fs] = (f32x4){0.f, 0.f, 0.f, 0.f};
        store_row_packed<ALIGNED>(lout.next(), ovoff, ooff, odd, pack_out<OP>(acc2[fs]));
        acc2[fs] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
      // the next third of a turn
      if (q + 1 == GS) {
        stage(First{});
        load(Last{});
      } else if (q + 1 == 2 * GS) {
        stage(Last{});
        load(First{});
      } else if (q + 1 == RR) {
        stage(First{});
        load(First{});
      }
      wave_lds_sync();
      const uint32_t* lrow = lds + (q + 1 == RR ? 0 : (q + 1) % GS) * kLdsRowDw;
      const u32x4 nb = {lrow[p1], lrow[p1 + 10], lrow[p2], lrow[p2 + 10]};
      const u32x4 nb2 = {mid[p1], mid[p1 + 10], mid[p2], mid[p2 + 10]};
#pragma unroll
      for (int a = R; a < 2 * R; ++a) mma(acc2, a, b2);
#pragma unroll
      for (int a = 0; a < 2 * R; ++a) mma(acc1, a, b);
      b = nb;
      b2 = nb2;
    }
  }
}

template <int R, int OP, bool ALIGNED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void band2d_wide2_kernel(BandGrid g) {
  __shared__ uint32_t lds[((2 * R + 3) / 3 + 1) * kLdsRowDw];
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  if (ALIGNED || (w % g.nstrips) * kStripW2_host + 256 <= g.nx)
    band2d_wide2_body<R, OP, true>(g, w, lds);
  else
    band2d_wide2_body<R, OP, ALIGNED>(g, w, lds);
}

namespace {
template <int OP, bool AL>
hipError_t dispatch_wide2(int r, const BandGrid& g, hipStream_t s) {
  const dim3 grid(g.nblocks), block(64);
  switch (r) {
    case 4: hipLaunchKernelGGL((band2d_wide2_kernel<4, OP, AL>), grid, block, 0, s, g); break;
    case 5: hipLaunchKernelGGL((band2d_wide2_kernel<5, OP, AL>), grid, block, 0, s, g); break;
    case 6: hipLaunchKernelGGL((band2d_wide2_kernel<6, OP, AL>), grid, block, 0, s, g); break;
    case 7: hipLaunchKernelGGL((band2d_wide2_kernel<7, OP, AL>), grid, block, 0, s, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_band2d_wide2(int r, int operand, const BandGrid& g, hipStream_t s) {
  const bool al = (g.nx % 8) == 0;
  if (operand == 2) return al ? dispatch_wide2<2, true>(r, g, s) : dispatch_wide2<2, false>(r, g, s);
  if (operand == 3) return al ? dispatch_wide2<3, true>(r, g, s) : dispatch_wide2<3, false>(r, g, s);
  return hipErrorInvalidValue;
}

}  // namespace spider_impl
