// Direct neighbour-sum engine, several steps per launch on large 2-D grids.
//
// A single step reads and writes the grid once and is bound by that: Star-2D13P on
// 8192^2 in fp32 ran 119 us per step, 4.5 of the 4.8 TB/s a copy reaches.  Here one
// wave owns a strip of 256 columns (four per lane) and streams lines through T
// levels held in registers: level t keeps the partial sums of its 2R + 1 output
// lines in flight, and a line it finishes is at once the next input line of level
// t + 1, so the T - 1 lines between never leave the wave.  The x neighbours come
// from the adjacent lanes by DPP wave shifts: no LDS, no barrier, no wait but for
// the prefetched input lines.  Values are exact on a window that shrinks by R per
// level on either side; the wave stores the columns that remain after T levels.
// Each point sums its taps in the single-step kernel's order (kernel rows, then
// taps along x, one fused multiply-add each), so the result is that of single
// steps bit for bit.
// us per step, single steps before / now: Star-2D13P (r = 3) fp32 8192^2 124 / 44,
// 2048 x 2051 26.7 / 6.7; 9 points fp32 8192^2 121 / 25 (eight levels), 4096^2
// 26.7 / 8.6 (four); fp64 6000^2 133 / 38 (r = 1, four levels), 136 / 70 (star r = 3,
// two).  At four levels of Star-2D13P the vector ALUs are the bound (52 multiply-adds
// and 6 shifts per lane, line and level; 70 % of a launch's cycles by their counter), at
// r = 1 still the memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "direct_stream.h"

namespace spider_impl {

namespace {

constexpr int kRsrc3 = 0x00020000;
constexpr uint32_t kOff = 0xffffff00u;  // beyond every line's range
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <typename E>
__device__ __forceinline__ E fma_e(E a, E b, E c) {
  if constexpr (sizeof(E) == 4)
    return __builtin_fmaf(a, b, c);
  else
    return __builtin_fma(a, b, c);
}

// The value of the lane before (UP) or after this one; zero beyond the wave's ends.
template <bool UP>
__device__ __forceinline__ uint32_t lane_shift(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, UP ? 0x138 : 0x130, 0xf, 0xf, true);
}
template <bool UP, typename E>
__device__ __forceinline__ E shift_e(E v) {
  if constexpr (sizeof(E) == 4) {
    return __builtin_bit_cast(E, lane_shift<UP>(__builtin_bit_cast(uint32_t, v)));
  } else {
    const u32x2 u = __builtin_bit_cast(u32x2, v);
    return __builtin_bit_cast(E, (u32x2){lane_shift<UP>(u.x), lane_shift<UP>(u.y)});
  }
}

// Columns lost on either side: T R, as whole 16-byte pieces of fp32.
constexpr int stream_margin(int T, int R) { return (T * R + 3) / 4 * 4; }
constexpr int stream_width(int T, int R) { return 256 - 2 * stream_margin(T, R); }

template <typename E>
struct Quad {
  E v[4];
};

// A lane's four values of a line.  The range check works on dwords: a straddling
// piece reads its values inside the line and zeros beyond it.
template <typename E>
__device__ __forceinline__ Quad<E> load_quad(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  Quad<E> q;
  if constexpr (sizeof(E) == 4) {
    const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    __builtin_memcpy(&q, &c, 16);
  } else {
    const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    const u32x4 d = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0);
    __builtin_memcpy(&q.v[0], &c, 16);
    __builtin_memcpy(&q.v[2], &d, 16);
  }
  return q;
}

// off[]: byte offsets of the four values (EDGE), or off[0] for all of them.
template <typename E, bool EDGE>
__device__ __forceinline__ void store_quad(__amdgpu_buffer_rsrc_t rs, const uint32_t* off, const Quad<E>& q) {
  if constexpr (!EDGE) {
    u32x4 c;
    __builtin_memcpy(&c, &q.v[0], 16);
    __builtin_amdgcn_raw_buffer_store_b128(c, rs, off[0], 0, 0);
    if constexpr (sizeof(E) == 8) {
      __builtin_memcpy(&c, &q.v[2], 16);
      __builtin_amdgcn_raw_buffer_store_b128(c, rs, off[0] + 16, 0, 0);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (sizeof(E) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, q.v[e]), rs, off[e], 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, q.v[e]), rs, off[e], 0, 0);
    }
  }
}

// EDGE: waves that reach beyond the grid; levels between are zeroed outside it.
template <typename E, int R, bool STAR, int T, bool EDGE>
__device__ __forceinline__ void stream_body(const E* __restrict__ in, E* __restrict__ out, int ny, int nx,
                                            const E* __restrict__ w, int seg_h, int strip, int seg) {
  constexpr int RR = 2 * R + 1, M = stream_margin(T, R), SW = stream_width(T, R), ES = sizeof(E);
  // lines per turn of the loop (accumulators rotate without copies), all loaded a turn ahead
  constexpr int U = R == 1 ? 2 * RR : RR;
  const int lane = threadIdx.x;
  const int x = strip * SW - M + 4 * lane;  // this lane's first column
  const int y0 = seg * seg_h, hrows = min(seg_h, ny - y0);
  const int nin = hrows + 2 * T * R;
  const uint32_t voff = EDGE && x < 0 ? kOff : (uint32_t)(x * ES);
  uint32_t soff[4];
  bool xin[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bool st = 4 * lane >= M && 4 * lane < M + SW;
    xin[e] = x + e >= 0 && x + e < nx;
    soff[e] = st && xin[e] ? (uint32_t)((x + e) * ES) : kOff;
  }
  const int64_t pitch = (int64_t)nx * ES;
  const char* src = reinterpret_cast<const char*>(in) + (y0 - T * R) * pitch;
  char* dst = reinterpret_cast<char*>(out) + (y0 - 2 * T * R) * pitch;
  auto load = [&](int j) {  // input line y0 - T R + j
    const int y = y0 - T * R + j;
    const bool ok = EDGE ? (unsigned)y < (unsigned)ny && j < nin : j < nin;
    return load_quad<E>(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src + (ok ? j * pitch : 0)), (short)0,
                                                          ok ? (int)pitch : 0, kRsrc3),
                        voff);
  };
  Quad<E> acc[T][RR];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int m = 0; m < RR; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][m].v[e] = E(0);
  Quad<E> pf[U];
#pragma unroll
  for (int j = 0; j < U; ++j) pf[j] = load(j);

  for (int jb = 0; jb < nin; jb += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = jb + u;
      if (j >= nin) break;
      Quad<E> cur = pf[u];
      pf[u] = load(j + U);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        // level t's line y0 - T R + j - t R; its output lines are of use from j = 2 t R on
        if (t > 0 && j < 2 * t * R) break;
        E v[4 + 2 * R];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[R + e] = cur.v[e];
#pragma unroll
        for (int e = 0; e < R; ++e) {
          v[e] = shift_e<true>(cur.v[4 - R + e]);
          v[R + 4 + e] = shift_e<false>(cur.v[e]);
        }
#pragma unroll
        for (int a = 0; a < RR; ++a) {
          // row a of the output line R - a lines further on (slots by line number)
          Quad<E>& d = acc[t][((u - t * R + R - a) % RR + 2 * RR * T) % RR];
#pragma unroll
          for (int k = 0; k < RR; ++k) {
            if (STAR && a != R && k != R) continue;
            const E c = w[a * RR + k];
            const bool first = a == 0 && k == (STAR ? R : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) d.v[e] = fma_e<E>(c, v[k + e], first ? E(0) : d.v[e]);
          }
        }
        cur = acc[t][((u - t * R - R) % RR + 2 * RR * T) % RR];  // line j - (t + 1) R of the next level is complete
        if constexpr (EDGE) {
          if (t + 1 < T) {
            const bool yin = (unsigned)(y0 - T * R + j - (t + 1) * R) < (unsigned)ny;
#pragma unroll
            for (int e = 0; e < 4; ++e) cur.v[e] = yin && xin[e] ? cur.v[e] : E(0);
          }
        }
        if (t + 1 == T) {
          const bool ok = j >= 2 * T * R;
          store_quad<E, EDGE>(__builtin_amdgcn_make_buffer_rsrc(dst + (ok ? j * pitch : 0), (short)0,
                                                                ok ? (int)pitch : 0, kRsrc3),
                              soff, cur);
        }
      }
    }
  }
}

template <typename E, int R, bool STAR, int T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void direct2d_stream_kernel(
    const E* __restrict__ in, E* __restrict__ out, int ny, int nx, const E* __restrict__ w, int seg_h, int nstrips) {
  constexpr int M = stream_margin(T, R), SW = stream_width(T, R);
  // neighbouring strips share halo columns: hand them to one XCD's L2
  const int total = gridDim.x, per = total / 8, extra = total % 8, xcd = blockIdx.x % 8;
  const int wv = xcd * per + min(xcd, extra) + (int)(blockIdx.x / 8);
  const int strip = wv % nstrips, seg = wv / nstrips;
  const int y0 = seg * seg_h, hrows = min(seg_h, ny - y0);
  const bool inside = strip * SW - M >= 0 && strip * SW - M + 256 <= nx && y0 - T * R >= 0 && y0 + hrows + T * R <= ny;
  if (inside)
    stream_body<E, R, STAR, T, false>(in, out, ny, nx, w, seg_h, strip, seg);
  else
    stream_body<E, R, STAR, T, true>(in, out, ny, nx, w, seg_h, strip, seg);
}

// The deepest launch.  A level costs the same vector work at any depth, so depth
// pays while the single step waits for memory and stops where the vector ALUs are
// the bound (us per step on 4096^2 / 8192^2 fp32, best heights: box r = 2 at 1 / 2 /
// 4 levels 24.7 / 20.3 / 24.6 and 115 / 68 / 65; box r = 3 at 1 / 2 levels 39 / 51 and
// 129 / 132), or where a wave's sums no longer fit its registers.
constexpr int max_steps(int elem, int R, bool star) {
  if (elem == 4) return R == 1 ? 8 : star ? 4 : R == 2 ? 2 : 1;
  return R == 1 ? 4 : R == 2 || star ? 2 : 1;
}

template <typename E, int R, bool STAR, int T>
struct Stream {
  static hipError_t launch(const E* in, E* out, int ny, int nx, const E* w, int seg_h, hipStream_t s) {
    const int nstrips = (nx + stream_width(T, R) - 1) / stream_width(T, R);
    const long long n = (long long)nstrips * ((ny + seg_h - 1) / seg_h);
    if (n > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((direct2d_stream_kernel<E, R, STAR, T>), dim3((unsigned)n), dim3(64), 0, s, in, out, ny, nx, w,
                       seg_h, nstrips);
    return hipGetLastError();
  }
};

// f(Stream<...>{}) for the instance of these run-time values; `none` if there is none.
template <typename E, int R, bool STAR, typename F, typename V>
V pick_t(int T, F f, V none) {
  constexpr int m = max_steps(sizeof(E), R, STAR);
  if (T == 1) return f(Stream<E, R, STAR, 1>{});
  if constexpr (m >= 2)
    if (T == 2) return f(Stream<E, R, STAR, 2>{});
  if constexpr (m >= 4)
    if (T == 4) return f(Stream<E, R, STAR, 4>{});
  if constexpr (m >= 8)
    if (T == 8) return f(Stream<E, R, STAR, 8>{});
  return none;
}
template <typename E, int R, typename F, typename V>
V pick_z(int zm, int T, F f, V none) {
  switch (zm) {
    case 0: return pick_t<E, R, false>(T, f, none);
    case 2: return pick_t<E, R, true>(T, f, none);
    default: return none;
  }
}
template <typename E, typename F, typename V>
V pick(int r, int zm, int T, F f, V none) {
  switch (r) {
    case 1: return pick_z<E, 1>(zm, T, f, none);
    case 2: return pick_z<E, 2>(zm, T, f, none);
    case 3: return pick_z<E, 3>(zm, T, f, none);
    default: return none;
  }
}

}  // namespace

int direct2d_stream_max_steps(int r, int dtype, int zero_taps, long long points) {
  if (r < 1 || r > 3 || (dtype != 0 && dtype != 1) || zero_taps == 1) return 0;
  const int m = max_steps(dtype == 0 ? 8 : 4, r, zero_taps == 2);
  // eight levels where the grid no longer fits the last-level cache (8192^2: 25 us per
  // step against 33 at four), four below (4096^2: 8.5 against 9.6)
  return m == 8 && points < (1LL << 25) ? 4 : m;
}

// Rows per wave.  With k waves per SIMD a launch takes about k (h + 1.2 T r) line
// times (the levels of the first 2 T r lines start one after the other, so about
// half of them is spent), and a lone wave or two leave latency uncovered (35 and 10
// per cent); k is the best of 1 .. 8.  Star r = 3, us per step: 2048^2 6.4 at the 19 rows
// chosen for T = 4 (64 rows 13.1), 4096^2 13.6 at 37 (128 rows 23.2).
int direct2d_stream_rows(int r, int T, int ny, int nx, int ncu) {
  const long long nstrips = (nx + stream_width(T, r) - 1) / stream_width(T, r);
  int best = ny;
  double best_cost = 1e300;
  for (int k = 1; k <= 8; ++k) {
    const long long segs = std::max<long long>(1, (long long)k * 4 * ncu / nstrips);
    const int h = (int)((ny + segs - 1) / segs);
    const double waves = (double)(nstrips * ((ny + h - 1) / h)) / (4.0 * ncu);
    const double cost = std::max(1.0, waves) * (h + 1.2 * T * r) * (k == 1 ? 1.35 : k == 2 ? 1.1 : 1.0);
    if (cost < best_cost) {
      best_cost = cost;
      best = h;
    }
  }
  return best;
}

hipError_t launch_direct2d_stream(int r, int dtype, int zero_taps, int T, const void* in, void* out, int ny, int nx,
                                  const void* coeffs_dev, int seg_h, hipStream_t s) {
  if (ny < 1 || nx < 1 || seg_h < 1) return hipErrorInvalidValue;
  auto go = [&](auto e, auto st) {
    using E = decltype(e);
    return st.launch(static_cast<const E*>(in), static_cast<E*>(out), ny, nx, static_cast<const E*>(coeffs_dev), seg_h, s);
  };
  if (dtype == 0) return pick<double>(r, zero_taps, T, [&](auto st) { return go(0.0, st); }, hipErrorInvalidValue);
  if (dtype == 1) return pick<float>(r, zero_taps, T, [&](auto st) { return go(0.0f, st); }, hipErrorInvalidValue);
  return hipErrorInvalidValue;
}

}  // namespace spider_impl
