// 1-D lines (r <= 3) advanced many steps per launch inside LDS.
//
// What bounds the step-by-step and the four-step kernels on a line is not the
// matrix pipe (one instruction per 256 points and step) but the launches and, in
// a launch, the round trips of a short stream.  A line needs a halo of only T r
// points for T steps, so here a wave loads one contiguous section of NB blocks of
// 256 points, advances it T steps in place in its own LDS rows and stores the
// points that are still exact; the grid crosses HBM once per launch.  A step of
// one block is two (four with the lo rows) ds_read2_b32, one (two) matrix
// instructions, the conversions and one (two) ds_write_b64 per lane; vector issue
// and LDS bound it about equally (28 vector instructions per block with the lo
// rows = 112 of a SIMD's cycles, 112 LDS cycles per four blocks of a CU; by counters LDS is
// busy 66 % of a launch's cycles, vector issue 56 % and the matrix pipe 22 %), the
// matrix pipe needs 32.  Small sections win although their halo is larger, because
// more waves are in flight: sections of 2 / 4 / 8 / 16 / 24 blocks take
// 152 / 139 / 147 / 219 / 285 us for 48 steps of a 10 240 000-point line (fp16,
// split 3, r = 1) and 51 / 40 / 52 / 115 / 167 us on 2 500 001 points (fp32, r = 2).
// Against the four-step kernel: 827 -> 261 us for 100 steps of the long line,
// 319 -> 52 us for 60 steps of the other.
//
// A section starts at x = 8 mod 16, so its 16-point chunks are those of the
// single-step kernel and every value is summed in the same order: the result
// equals single steps (or, for a 16-bit grid with split 3, launches that round
// the grid at the same steps) bit for bit, as long as values are finite.  An infinity
// or NaN spreads over whole chunks in single steps (zero taps of a chunk's window times
// infinity), up to 24 points per step; a section sees T r + 8 points beyond those it
// stores, so from further off it takes only what the stencil itself reaches.  (To see
// all, a section would need 16 points per step on either side: 1280 of the 1024 points of
// a section of four blocks at 40 steps.)
//
// In-place update: the operands of up to four blocks are gathered before the
// group in front of them is written, so a block's window (8 points beyond either
// end) is read before its neighbours change.  One wave owns the section, its LDS
// operations execute in order, and no barrier is needed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "band_common.h"
#include "band_f32_common.h"
#include "kernels.h"

namespace spider_impl {

namespace {

// LDS dwords of one row of a section of nb blocks: 8 points beyond either end.
__host__ __device__ constexpr int line_row_dw(int nb) { return 160 * nb + 10; }

// The section of wave w: nb blocks computed from x = w width - lead, points
// [w width, w width + width) stored.  Both are multiples of 8 (lead: 8 mod 16).
struct LineGeom {
  int lead, width;
};
__host__ __device__ constexpr LineGeom line_geom(int nb, int halo) {
  const int lead = halo <= 8 ? 8 : ((halo - 8 + 15) / 16) * 16 + 8;
  return {lead, ((256 * nb - lead - halo) / 16) * 16};
}

// EDGE: sections that reach beyond the line (values outside it are kept zero), or
// any section of a grid whose base is not 16-byte aligned; their loads and stores
// go element by element where a whole 16-byte access could leave the line.
template <int OP, int ENG, bool IO16, bool XLO, int NB, bool EDGE>
__device__ __forceinline__ void line_deep_body(const LineDeep& g, int w, uint32_t* lds) {
  constexpr int ES = IO16 ? 2 : 4;  // bytes per grid element
  constexpr int G = NB < 4 ? NB : 4;  // blocks per group
  constexpr int ROWDW = line_row_dw(NB);
  const int lane = threadIdx.x;
  const int nx = g.nx;
  const LineGeom geo = line_geom(NB, g.halo);
  const int a = w * geo.width - geo.lead;  // first computed point
  const int x_lo = w * geo.width, x_hi = min(nx, x_lo + geo.width);

  const u32x4 A0 = (ENG == 1) ? reinterpret_cast<const u32x4*>(g.apack)[lane] : (u32x4){0, 0, 0, 0};
  const u32x4 Dh = (ENG == 1) ? (u32x4){0, 0, 0, 0} : reinterpret_cast<const u32x4*>(g.dpack)[lane * 2 + 0];
  const u32x4 Dl = (ENG == 1) ? (u32x4){0, 0, 0, 0} : reinterpret_cast<const u32x4*>(g.dpack)[lane * 2 + 1];
  const uint32_t I0 = (ENG == 1) ? g.ipack[lane] : 0u;
  const __amdgpu_buffer_rsrc_t rin =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.in), (short)0, nx * ES, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(g.out, (short)0, nx * ES, kRsrcWord3);

  // ---- load: chunk c holds the 8 points from a - 8 + 8 c; 32 NB + 2 chunks
  auto put = [&](int c, const u32x4* v) {
    const int u = lds_phys(4 * c);
    if constexpr (IO16) {
      store_chunk_lds(lds, u, v[0]);
      if constexpr (XLO) store_chunk_lds(lds + ROWDW, u, (u32x4){0, 0, 0, 0});
    } else {
      u32x4 h, l;
      uint32_t t0, t1;
      split2<OP, XLO>(v[0].x, v[0].y, &t0, &t1), h.x = t0, l.x = t1;
      split2<OP, XLO>(v[0].z, v[0].w, &t0, &t1), h.y = t0, l.y = t1;
      split2<OP, XLO>(v[1].x, v[1].y, &t0, &t1), h.z = t0, l.z = t1;
      split2<OP, XLO>(v[1].z, v[1].w, &t0, &t1), h.w = t0, l.w = t1;
      store_chunk_lds(lds, u, h);
      if constexpr (XLO) store_chunk_lds(lds + ROWDW, u, l);
    }
  };
  auto get = [&](int c, u32x4* v) {  // points outside the line read as zero (a negative x wraps out of range)
    const uint32_t off = (uint32_t)((a - 8 + 8 * c) * ES);
    if constexpr (IO16) {
      v[0] = load_chunk<!EDGE>(rin, off);
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if constexpr (EDGE)
          v[q] = (u32x4){__builtin_amdgcn_raw_buffer_load_b32(rin, off + 16 * q, 0, 0),
                         __builtin_amdgcn_raw_buffer_load_b32(rin, off + 16 * q + 4, 0, 0),
                         __builtin_amdgcn_raw_buffer_load_b32(rin, off + 16 * q + 8, 0, 0),
                         __builtin_amdgcn_raw_buffer_load_b32(rin, off + 16 * q + 12, 0, 0)};
        else
          v[q] = __builtin_amdgcn_raw_buffer_load_b128(rin, off + 16 * q, 0, 0);
      }
    }
  };
  {
    constexpr int NV = IO16 ? 1 : 2, NC = NB / 2;  // whole rounds of 64 chunks, then two more chunks
    u32x4 v[NC][NV], t[NV];
#pragma unroll
    for (int i = 0; i < NC; ++i) get(64 * i + lane, v[i]);
    if (lane < 2) get(64 * NC + lane, t);
#pragma unroll
    for (int i = 0; i < NC; ++i) put(64 * i + lane, v[i]);
    if (lane < 2) put(64 * NC + lane, t);
  }

  // gather offsets of every second block, kept in registers: the two reads of a block
  // and of the next one reach 170 dwords on, within a ds_read2_b32's offsets
  int p1, p2;
  band_gather_offsets(lane, &p1, &p2);
  constexpr int NS = XLO ? 2 : 1;
  int o1[NS][NB / 2], o2[NS][NB / 2];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int k = 0; k < NB / 2; ++k) {
      o1[s][k] = p1 + 320 * k + s * ROWDW;
      o2[s][k] = p2 + 320 * k + s * ROWDW;
      asm volatile("" : "+v"(o1[s][k]), "+v"(o2[s][k]));
    }
  const int n = lane & 15, h = lane >> 4;
  uint32_t* const wr = lds + lds_phys(4 + 8 * n + 2 * h);  // this lane's 4 outputs of block 0: points 16 n + 4 h ..
  const int ox = a + 16 * n + 4 * h;

  struct Ops {
    u32x4 v[NS][G];
  };
  auto gather = [&](int k0, Ops& o) {
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const uint32_t* r1 = lds + o1[s][(k0 + q) / 2] + 160 * ((k0 + q) & 1);
        const uint32_t* r2 = lds + o2[s][(k0 + q) / 2] + 160 * ((k0 + q) & 1);
        o.v[s][q] = (u32x4){r1[0], r1[10], r2[0], r2[10]};
      }
  };
  // the group's products; the sums replace the group's rows, or (LAST) go to the grid
  auto finish = [&](int k0, const Ops& o, auto round16, auto last) {
    f32x4 acc[G];
#pragma unroll
    for (int q = 0; q < G; ++q)
      acc[q] = band_mma<OP, ENG, 0>((f32x4){0.f, 0.f, 0.f, 0.f}, A0, Dh, Dl, I0, o.v[0][q]);
    if constexpr (XLO) {
#pragma unroll
      for (int q = 0; q < G; ++q) acc[q] = band_mma<OP, ENG, 0>(acc[q], A0, Dh, Dl, I0, o.v[1][q]);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const int x = ox + 256 * (k0 + q);
      if constexpr (decltype(last)::value) {
        // x_lo and width are multiples of 16, so a quad is stored or not as a whole up to x_hi = nx
        const uint32_t off = (x >= x_lo && x < x_hi) ? (uint32_t)(x * ES) : kOffNone;
        if constexpr (IO16)
          store_packed<!EDGE>(rout, off, pack_out<OP>(acc[q]));
        else
          store_f32x4<!EDGE>(rout, off, acc[q]);
      } else {
        // (the whole vector is cast first: element-wise casts of a float vector have
        // been seen to compile to four copies of element 0)
        u32x4 v = __builtin_bit_cast(u32x4, acc[q]);
        if constexpr (EDGE) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (x + e < 0 || x + e >= nx) v[e] = 0u;
        }
        constexpr bool LO = XLO && !decltype(round16)::value;  // a step that rounds the grid keeps no lo part
        uint32_t h0, l0, h1, l1;
        split2<OP, LO>(v.x, v.y, &h0, &l0);
        split2<OP, LO>(v.z, v.w, &h1, &l1);
        *reinterpret_cast<uint2*>(wr + 160 * (k0 + q)) = make_uint2(h0, h1);
        if constexpr (XLO) *reinterpret_cast<uint2*>(wr + ROWDW + 160 * (k0 + q)) = make_uint2(l0, l1);
      }
    }
  };
  auto step = [&](auto round16, auto last) {
    Ops o[NB / G];
    wave_lds_sync();
    gather(0, o[0]);
#pragma unroll
    for (int k = 0; k < NB / G; ++k) {
      if (k + 1 < NB / G) gather((k + 1) * G, o[k + 1]);
      wave_lds_sync();
      finish(k * G, o[k], round16, last);
    }
  };
  for (int s = 1; s < g.T; ++s) {
    if (IO16 && XLO && ((g.rounds >> (s - 1)) & 1))
      step(std::true_type{}, std::false_type{});
    else
      step(std::false_type{}, std::false_type{});
  }
  step(std::false_type{}, std::true_type{});
}

template <int OP, int ENG, bool IO16, bool XLO, int NB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(XLO ? 3 : 4))) void line_deep_kernel(LineDeep g) {
  __shared__ uint32_t lds[line_row_dw(NB) * (XLO ? 2 : 1)];
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const LineGeom geo = line_geom(NB, g.halo);
  const int a = w * geo.width - geo.lead;
  // interior sections: every point loaded, computed or stored lies inside the line
  if (g.aligned && a - 8 >= 0 && (int64_t)a + 256 * NB + 8 <= g.nx)
    line_deep_body<OP, ENG, IO16, XLO, NB, false>(g, w, lds);
  else
    line_deep_body<OP, ENG, IO16, XLO, NB, true>(g, w, lds);
}

template <int OP, int ENG, int NB>
hipError_t dispatch_line_nb(bool io16, bool xlo, const LineDeep& g, int sections, hipStream_t s) {
  const dim3 grid(sections), block(64);
  if (io16 && xlo)
    hipLaunchKernelGGL((line_deep_kernel<OP, ENG, true, true, NB>), grid, block, 0, s, g);
  else if (io16)
    hipLaunchKernelGGL((line_deep_kernel<OP, ENG, true, false, NB>), grid, block, 0, s, g);
  else if (xlo)
    hipLaunchKernelGGL((line_deep_kernel<OP, ENG, false, true, NB>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((line_deep_kernel<OP, ENG, false, false, NB>), grid, block, 0, s, g);
  return hipGetLastError();
}

template <int OP, int ENG>
hipError_t dispatch_line(bool io16, bool xlo, int nb, const LineDeep& g, int sections, hipStream_t s) {
  return nb == 2   ? dispatch_line_nb<OP, ENG, 2>(io16, xlo, g, sections, s)
         : nb == 4 ? dispatch_line_nb<OP, ENG, 4>(io16, xlo, g, sections, s)
                   : dispatch_line_nb<OP, ENG, 8>(io16, xlo, g, sections, s);
}

}  // namespace

// Blocks per section: a step of a lone section takes about 75 ns per block (36
// without the lo rows), a CU full of sections 17 ns (8) per block, 6 % more at
// eight blocks than at four (measured); fewer blocks mean more sections in flight
// on a short line and more halo on a long one.
LineChoice line_deep_choice(int nx, int r, int T, int ncu) {
  LineChoice best;
  double best_cost = 1e30;
  for (int nb : {2, 4, 8}) {
    const int width = line_geom(nb, T * r).width;
    if (width < 64) continue;
    const long long sections = ((long long)nx + width - 1) / width;
    const long long per_cu = (sections + ncu - 1) / ncu;
    const double cost = nb * std::max((nb == 8 ? 17.0 * 1.06 : 17.0) * (double)per_cu, 75.0);
    if (cost < best_cost) {
      best_cost = cost;
      best.nb = nb;
      best.sections = (int)sections;
    }
  }
  return best;
}

hipError_t launch_line_deep(int operand, int engine, bool io16, bool xlo, int r, int T, uint64_t rounds,
                            const LineChoice& c, const BandGrid& b, hipStream_t s) {
  if (T < 1 || T > kLineDeepMaxSteps || r < 1 || r > 3 || (c.nb != 2 && c.nb != 4 && c.nb != 8) || c.sections < 1)
    return hipErrorInvalidValue;
  if (line_geom(c.nb, T * r).width < 16) return hipErrorInvalidValue;
  LineDeep g;
  g.in = b.in;
  g.out = b.out;
  g.apack = b.apack;
  g.ipack = b.ipack;
  g.dpack = b.dpack;
  g.nx = b.nx;
  g.T = T;
  g.halo = T * r;
  g.rounds = rounds;
  g.aligned = ((reinterpret_cast<uintptr_t>(b.in) | reinterpret_cast<uintptr_t>(b.out)) & 15) == 0;
  if (operand == 2 && engine == 1) return dispatch_line<2, 1>(io16, xlo, c.nb, g, c.sections, s);
  if (operand == 2 && engine == 2) return dispatch_line<2, 2>(io16, xlo, c.nb, g, c.sections, s);
  if (operand == 3 && engine == 1) return dispatch_line<3, 1>(io16, xlo, c.nb, g, c.sections, s);
  if (operand == 3 && engine == 2) return dispatch_line<3, 2>(io16, xlo, c.nb, g, c.sections, s);
  return hipErrorInvalidValue;
}

}  // namespace spider_impl
