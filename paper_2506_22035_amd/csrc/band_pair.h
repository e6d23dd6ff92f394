// Device code of the paired-line band (2-D, r <= 3) shared by its kernels and
// the batched kernel: LDS layout, gather, operand product, stores, the one- and
// two-step bodies of even radii and the dense engine, and the bodies of odd radii
// on the sparse engine at any depth (quads, at the end).  See kernels_band_pair.hip
// for the scheme.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "band_common.h"
#include "kernels.h"

namespace spider_impl {

constexpr int kPairChunks = 33;               // 16-byte chunks per staged line
constexpr int kPairRowDw = 6 * kPairChunks;   // LDS dwords per staged line
constexpr int kPairHalfDw = 6 * 16;           // LDS offset of the second half's windows

// Per-lane LDS dword offsets of the gather: lane (n = lane % 16, h = lane / 16)
// feeds chunk n and K slots 8 (h & 1) .. + 7 of both lines of the pair; slots
// 0..7 are the 2:4 groups joining window pairs (0, 4) and (1, 5), slots 8..15
// the groups (3, 7) and (2, 6).  Window pair w of chunk n is data dword 4n + w,
// stored at 6n + w + 2 (w >= 4), so the partner pair is always 6 dwords on.
__device__ __forceinline__ void pair_gather_offsets(int lane, int* p1, int* p2) {
  const int n = lane & 15, odd = (lane >> 4) & 1;
  *p1 = 6 * n + (odd ? 3 : 0);
  *p2 = 6 * n + (odd ? 2 : 1);
}

__device__ __forceinline__ u32x4 pair_gather(const uint32_t* line, int p1, int p2) {
  return (u32x4){line[p1], line[p1 + 6], line[p2], line[p2 + 6]};
}

// Sequential walk over output line pairs: pair (y, y + 1), lines in [lo, hi) valid.
struct PairWalk {
  uint64_t addr;
  int rel;      // y - lo
  int span;     // hi - lo
  int nbytes;   // bytes per line
  __device__ __forceinline__ PairWalk(const void* base, int y, int lo, int hi, int nbytes_)
      : addr(reinterpret_cast<uint64_t>(base) + (int64_t)y * nbytes_), rel(y - lo), span(hi - lo), nbytes(nbytes_) {}
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t next() {
    const int left = span - rel;
    const int nv = (rel < 0 || left <= 0) ? 0 : (left >= 2 ? 2 : 1);
    // the size is wave-uniform; say so, so the resource stays in scalar registers
    const int nrec = __builtin_amdgcn_readfirstlane(nv * nbytes);
    __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(addr), (short)0, nrec, kRsrcWord3);
    addr += (uint64_t)(2 * (int64_t)nbytes);
    rel += 2;
    return rs;
  }
};

// One paired-band instruction: acc += A x [X_j; X_j; X_j+1; X_j+1].
//   sparse: v_smfmac_f32_16x16x64 with the compressed A of instruction k
//   dense:  two v_mfma_f32_16x16x32, A over line j then over line j + 1
template <int OP, int ENG, int ABID>
__device__ __forceinline__ f32x4 pair_mma(f32x4 acc, u32x4 a, u32x4 d0, u32x4 d1, uint32_t idx, u32x4 b0, u32x4 b1) {
  if constexpr (ENG == 1) {
    const u32x8 bb = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    if constexpr (OP == 2)
      return __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x16, bb),
                                                      acc, (int)idx, 0, ABID);
    else
      return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x16, bb), acc, (int)idx, 0, ABID);
  } else {
    if constexpr (OP == 2) {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, d0), __builtin_bit_cast(f16x8, b0), acc,
                                                   0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, d1), __builtin_bit_cast(f16x8, b1), acc,
                                                    0, 0, 0);
    } else {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d0), __builtin_bit_cast(bf16x8, b0),
                                                    acc, 0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d1), __builtin_bit_cast(bf16x8, b1),
                                                     acc, 0, 0, 0);
    }
  }
}

// A lane's place in the output pair: byte offset of its 4 outputs from the pair's
// first line (the lane's line and column folded in), out of range where it stores
// nothing; on ragged widths the one quad of either line that straddles the end of
// its line (a whole store would reach into the pair's second line) has an offset of
// its own.
template <bool ALIGNED>
struct PairStore {
  uint32_t off;
  bool whole, part;  // this lane stores a whole quad / is the straddling one
  int rem;  // wave-uniform: elements of the straddling quad, 0 where this wave has none
  // the lane's column x and line; columns [lo, hi) stored; the wave's quads are at [w0, w0 + 128)
  __device__ __forceinline__ PairStore(int x, int line_off, int lo, int hi, int nx, int w0, int es) {
    const bool in = x >= lo && x < hi;
    whole = in && (ALIGNED || x + 4 <= nx);
    part = in && !whole;
    off = ALIGNED && !in ? kOffNone : (uint32_t)((x + line_off) * es);
    rem = !ALIGNED && (nx & 3) && (nx & ~3) >= w0 && (nx & ~3) < w0 + 128 && (nx & ~3) < hi ? (nx & 3) : 0;
  }
  __device__ __forceinline__ uint32_t full_off() const { return ALIGNED || whole ? off : kOffNone; }
  __device__ __forceinline__ uint32_t part_off() const { return part ? off : kOffNone; }
};

template <bool ALIGNED>
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t rs, const PairStore<ALIGNED>& o, uint2 w) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64((u32x2){w.x, w.y}, rs, o.full_off(), 0, kStoreNT);
  if constexpr (!ALIGNED) {
    if (o.rem) {
      if (o.rem & 2) __builtin_amdgcn_raw_buffer_store_b32(w.x, rs, o.part_off(), 0, 0);
      if (o.rem & 1)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)((o.rem & 2) ? w.y : w.x), rs, o.part_off() + 2 * (o.rem & 2), 0, 0);
    }
  }
}

// Strips of `width` columns: every column the wave stages (264 from strip width -
// lead - kPairWinLead on) lies inside the lines' end.
__device__ __forceinline__ bool pair_inside(const BandGrid& g, int w, int width, int lead) {
  return (w % g.nstrips) * width - lead + 260 <= g.nx;
}

// Dword of element i of a staged line.
__device__ __forceinline__ int pair_dword(int i) { return 6 * (i >> 3) + ((i >> 1) & 3); }

template <int R, int OP, int ENG, bool ALIGNED>
__device__ __forceinline__ void band2d_pair_body(const BandGrid& g, int w, uint32_t* lds) {
  constexpr int NP = R + 1;                   // instructions per input pair = live output pairs
  constexpr int UP = (NP >= 3) ? NP : 2 * NP;  // input pairs per body (multiple of NP)
  constexpr int NL = 2 * UP;                  // staged lines per body
  const int lane = threadIdx.x;
  const int strip = w % g.nstrips, seg = w / g.nstrips;
  const int xs = strip * kStripWPair - kPairWinLead;  // first output column of the strip
  const int y0 = seg * g.seg_h;                       // seg_h is even: pairs start on even rows
  const int hrows = min(g.seg_h, g.ny - y0);
  const int npin = (hrows + 1) / 2 + R;               // input pairs needed
  const int nbody = (npin + UP - 1) / UP;
  const int nx = g.nx, ny = g.ny;

  u32x4 A[NP], D0[NP], D1[NP];
  uint32_t I[(NP + 1) / 2];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if constexpr (ENG == 1) {
      A[k] = reinterpret_cast<const u32x4*>(g.apack)[k * 64 + lane];
      D0[k] = D1[k] = (u32x4){0, 0, 0, 0};
    } else {
      A[k] = (u32x4){0, 0, 0, 0};
      D0[k] = reinterpret_cast<const u32x4*>(g.dpack)[(k * 64 + lane) * 2 + 0];
      D1[k] = reinterpret_cast<const u32x4*>(g.dpack)[(k * 64 + lane) * 2 + 1];
    }
  }
#pragma unroll
  for (int k = 0; k < (NP + 1) / 2; ++k) I[k] = (ENG == 1) ? g.ipack[k * 64 + lane] : 0u;
  __builtin_amdgcn_s_waitcnt(0);

  int p1, p2;
  pair_gather_offsets(lane, &p1, &p2);
  // loads: lane c < 33 holds the 8 inputs at xs - 4 + 8c (half h's chunk n window = data dwords 64h + 4n ..+7)
  const bool stager = lane < kPairChunks;
  const OddTail tail(ALIGNED ? 0 : nx, xs - kPairWinLead, 8 * kPairChunks);
  const uint32_t lvoff =
      tail.voff(stager ? (uint32_t)((xs - kPairWinLead + 8 * lane) * 2) : kOffNone, lane, nx);
  const int lw = 6 * lane;
  // stores: lane (n, h) holds outputs x = xs + 128 half + 8n + 4 (h & 1) + e of line i + (h >> 1)
  const int xo = xs + 8 * (lane & 15) + 4 * ((lane >> 4) & 1);
  const int line_off = (lane >> 5) * nx;
  const PairStore<ALIGNED> ova(xo, line_off, 0, nx, nx, xs, 2), ovb(xo + 128, line_off, 0, nx, nx, xs + 128, 2);

  LineWalk lin(g.in, y0 - R, max(0, y0 - R), min(ny, y0 + hrows + R), nx * 2);
  PairWalk pout(g.out, y0 - 2 * R, y0, y0 + hrows, nx * 2);
  u32x4 stg[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) stg[l] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
  f32x4 acc_a[NP], acc_b[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) acc_a[s] = acc_b[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
  uint2 done_a[UP], done_b[UP];

  for (int b = 0; b < nbody; ++b) {
    wave_lds_sync();
    if (stager) {
#pragma unroll
      for (int l = 0; l < NL; ++l) store_chunk_lds(lds, lw + l * kPairRowDw, stg[l]);
    }
    if constexpr (!ALIGNED) {
#pragma unroll
      for (int l = 0; l < NL; ++l) tail.put(lds + l * kPairRowDw, pair_dword(tail.at), lane, stg[l]);
    }
    if (b > 0) {
#pragma unroll
      for (int q = 0; q < UP; ++q) {
        const __amdgpu_buffer_rsrc_t rs = pout.next();
        store_pair<ALIGNED>(rs, ova, done_a[q]);
        store_pair<ALIGNED>(rs, ovb, done_b[q]);
      }
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) stg[l] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < UP; ++q) {
      const uint32_t* l0 = lds + (2 * q) * kPairRowDw;
      const uint32_t* l1 = l0 + kPairRowDw;
      // input pair P feeds output pair P - k through instruction k; slot (P - k) mod NP
      {
        const u32x4 b0 = pair_gather(l0, p1, p2), b1 = pair_gather(l1, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            acc_a[slot] = pair_mma<OP, ENG, 1>(acc_a[slot], A[k], D0[k], D1[k], I[k / 2], b0, b1);
          else
            acc_a[slot] = pair_mma<OP, ENG, 0>(acc_a[slot], A[k], D0[k], D1[k], I[k / 2], b0, b1);
        }
      }
      {
        const u32x4 b0 = pair_gather(l0 + kPairHalfDw, p1, p2), b1 = pair_gather(l1 + kPairHalfDw, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            acc_b[slot] = pair_mma<OP, ENG, 1>(acc_b[slot], A[k], D0[k], D1[k], I[k / 2], b0, b1);
          else
            acc_b[slot] = pair_mma<OP, ENG, 0>(acc_b[slot], A[k], D0[k], D1[k], I[k / 2], b0, b1);
        }
      }
      // output pair P - R is complete: slot (P - R) mod NP = (q + 1) mod NP
      const int fs = (q + 1) % NP;
      done_a[q] = pack_out<OP>(acc_a[fs]);
      done_b[q] = pack_out<OP>(acc_b[fs]);
      acc_a[fs] = acc_b[fs] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  }
#pragma unroll
  for (int q = 0; q < UP; ++q) {
    const __amdgpu_buffer_rsrc_t rs = pout.next();
    store_pair<ALIGNED>(rs, ova, done_a[q]);
    store_pair<ALIGNED>(rs, ovb, done_b[q]);
  }
}

// ----------------------------------------------------------------------------- two fused steps
// Two time steps per launch on paired-line bands.  The first pass treats the
// intermediate step's line pairs as its outputs, aligned so that they are
// exactly the input pairs the second pass needs (rows y0 - r + 2m, m >= 0);
// every finished intermediate pair is rounded to the carry type, zeroed outside
// the grid, written to an LDS line pair in the staged-line layout and multiplied
// again one input pair later (software-pipelined) into a second set of
// accumulators.  The wave computes 256 columns per pass and stores the 240 in
// [240 s, 240 s + 240): the intermediate values it lacks beyond its strip only
// reach outputs it does not store.  For odd r the intermediate pairs start on
// odd rows, unlike the one-step kernel's output pairs, so the fused result
// agrees with two single steps to rounding, not bit for bit; it never depends
// on the tiling.
// EDGE = false: every row and column the wave computes lies inside the grid, so
// the intermediate values need no zero-halo masking.
template <int R, int OP, int ENG, bool ALIGNED, bool EDGE>
__device__ __forceinline__ void band2d_pair_tb2_body(const BandGrid& g, int w, uint32_t* lds) {
  constexpr int NP = R + 1;
  constexpr int UP = (NP >= 3) ? NP : 2 * NP;
  constexpr int NL = 2 * UP;
  const int lane = threadIdx.x;
  const int strip = w % g.nstrips, seg = w / g.nstrips;
  const int xp = strip * kStripWPair2 - kPairWinLead;  // first column of both passes
  const int y0 = seg * g.seg_h;
  const int hrows = min(g.seg_h, g.ny - y0);
  const int npin = (hrows + 1) / 2 + 2 * R + 1;       // input pairs streamed
  const int nbody = (npin + UP - 1) / UP;
  const int nx = g.nx, ny = g.ny;

  u32x4 A[NP], D0[NP], D1[NP];
  uint32_t I[(NP + 1) / 2];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if constexpr (ENG == 1) {
      A[k] = reinterpret_cast<const u32x4*>(g.apack)[k * 64 + lane];
      D0[k] = D1[k] = (u32x4){0, 0, 0, 0};
    } else {
      A[k] = (u32x4){0, 0, 0, 0};
      D0[k] = reinterpret_cast<const u32x4*>(g.dpack)[(k * 64 + lane) * 2 + 0];
      D1[k] = reinterpret_cast<const u32x4*>(g.dpack)[(k * 64 + lane) * 2 + 1];
    }
  }
#pragma unroll
  for (int k = 0; k < (NP + 1) / 2; ++k) I[k] = (ENG == 1) ? g.ipack[k * 64 + lane] : 0u;
  __builtin_amdgcn_s_waitcnt(0);

  int p1, p2;
  pair_gather_offsets(lane, &p1, &p2);
  const bool stager = lane < kPairChunks;
  const OddTail tail(ALIGNED ? 0 : nx, xp - kPairWinLead, 8 * kPairChunks);
  const uint32_t lvoff =
      tail.voff(stager ? (uint32_t)((xp - kPairWinLead + 8 * lane) * 2) : kOffNone, lane, nx);
  const int lw = 6 * lane;
  // this lane's 4 values of either pass: columns xo + e (half a) and xo + 128 + e (half b)
  // of line 2m + (lane >> 5) of the pair
  const int xo = xp + 8 * (lane & 15) + 4 * ((lane >> 4) & 1);
  const int phi = lane >> 5;
  const int line_off = phi * nx;
  const int x_lo = strip * kStripWPair2, x_hi = min(nx, x_lo + kStripWPair2);  // stored columns
  const PairStore<ALIGNED> ova(xo, line_off, x_lo, x_hi, nx, xp, 2), ovb(xo + 128, line_off, x_lo, x_hi, nx, xp + 128, 2);
  uint32_t ma0 = 0, ma1 = 0, mb0 = 0, mb1 = 0;  // 16-bit lanes of the intermediate values inside the grid
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t half = (e & 1) ? 0xffff0000u : 0x0000ffffu;
    const int ya = xo + e, yb = xo + 128 + e;
    if (ya >= 0 && ya < nx) (e < 2 ? ma0 : ma1) |= half;
    if (yb >= 0 && yb < nx) (e < 2 ? mb0 : mb1) |= half;
  }
  // intermediate LDS line pairs (two, alternating): this lane's 2 dwords of half a
  // sit at data dword 4n + 2 + 2 (h & 1) of line phi; half b 96 dwords further
  uint32_t* mid = lds + NL * kPairRowDw;
  const int mw = 6 * (lane & 15) + (((lane >> 4) & 1) ? 6 : 2) + phi * kPairRowDw;
  for (int i = lane; i < 4 * kPairRowDw; i += 64) mid[i] = 0u;

  LineWalk lin(g.in, y0 - 2 * R, max(0, y0 - 2 * R), min(ny, y0 + hrows + 2 * R), nx * 2);
  PairWalk pout(g.out, y0 - 2 * (2 * R + 1), y0, y0 + hrows, nx * 2);
  u32x4 stg[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) stg[l] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
  f32x4 a1[NP], b1[NP], a2[NP], b2[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) a1[s] = b1[s] = a2[s] = b2[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
  uint2 done_a[UP], done_b[UP];
  // row of this lane's line in intermediate pair m: y0 - R + 2m + phi
  const int mrow0 = y0 - R + phi;

  for (int b = 0; b < nbody; ++b) {
    wave_lds_sync();
    if (stager) {
#pragma unroll
      for (int l = 0; l < NL; ++l) store_chunk_lds(lds, lw + l * kPairRowDw, stg[l]);
    }
    if constexpr (!ALIGNED) {
#pragma unroll
      for (int l = 0; l < NL; ++l) tail.put(lds + l * kPairRowDw, pair_dword(tail.at), lane, stg[l]);
    }
    if (b > 0) {
#pragma unroll
      for (int q = 0; q < UP; ++q) {
        const __amdgpu_buffer_rsrc_t rs = pout.next();
        store_pair<ALIGNED>(rs, ova, done_a[q]);
        store_pair<ALIGNED>(rs, ovb, done_b[q]);
      }
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) stg[l] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
#pragma unroll
    for (int q = 0; q < UP; ++q) {
      const int P = b * UP + q;
      wave_lds_sync();  // the intermediate pair written last iteration is visible
      const uint32_t* l0 = lds + (2 * q) * kPairRowDw;
      const uint32_t* l1 = l0 + kPairRowDw;
      const uint32_t* m0 = mid + ((P + 1) & 1) * 2 * kPairRowDw;  // intermediate pair P - 1 - R
      const uint32_t* m1 = m0 + kPairRowDw;
      // first pass: input pair P -> intermediate pair P - k
      {
        const u32x4 x0 = pair_gather(l0, p1, p2), x1 = pair_gather(l1, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            a1[slot] = pair_mma<OP, ENG, 1>(a1[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
          else
            a1[slot] = pair_mma<OP, ENG, 0>(a1[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
        }
      }
      {
        const u32x4 x0 = pair_gather(l0 + kPairHalfDw, p1, p2), x1 = pair_gather(l1 + kPairHalfDw, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            b1[slot] = pair_mma<OP, ENG, 1>(b1[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
          else
            b1[slot] = pair_mma<OP, ENG, 0>(b1[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
        }
      }
      // second pass: intermediate pair P - 1 - R -> output pair P - 1 - R - k, slot (q - k) mod NP
      {
        const u32x4 x0 = pair_gather(m0, p1, p2), x1 = pair_gather(m1, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            a2[slot] = pair_mma<OP, ENG, 1>(a2[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
          else
            a2[slot] = pair_mma<OP, ENG, 0>(a2[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
        }
      }
      {
        const u32x4 x0 = pair_gather(m0 + kPairHalfDw, p1, p2), x1 = pair_gather(m1 + kPairHalfDw, p1, p2);
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          const int slot = ((q - k) % NP + NP) % NP;
          if (k & 1)
            b2[slot] = pair_mma<OP, ENG, 1>(b2[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
          else
            b2[slot] = pair_mma<OP, ENG, 0>(b2[slot], A[k], D0[k], D1[k], I[k / 2], x0, x1);
        }
      }
      const int fs = (q + 1) % NP;
      // output pair P - 1 - 2R is complete
      done_a[q] = pack_out<OP>(a2[fs]);
      done_b[q] = pack_out<OP>(b2[fs]);
      a2[fs] = b2[fs] = (f32x4){0.f, 0.f, 0.f, 0.f};
      // intermediate pair P - R is complete: round, zero outside the grid, keep for the next iteration
      const uint2 va = pack_out<OP>(a1[fs]), vb = pack_out<OP>(b1[fs]);
      uint32_t* mc = mid + (P & 1) * 2 * kPairRowDw;
      if constexpr (!EDGE) {
        *reinterpret_cast<uint2*>(mc + mw) = va;
        *reinterpret_cast<uint2*>(mc + mw + kPairHalfDw) = vb;
      } else {
        const int mrow = mrow0 + 2 * (P - R);
        const bool rok = mrow >= 0 && mrow < ny;
        *reinterpret_cast<uint2*>(mc + mw) = make_uint2(rok ? (va.x & ma0) : 0u, rok ? (va.y & ma1) : 0u);
        *reinterpret_cast<uint2*>(mc + mw + kPairHalfDw) =
            make_uint2(rok ? (vb.x & mb0) : 0u, rok ? (vb.y & mb1) : 0u);
      }
      a1[fs] = b1[fs] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  }
#pragma unroll
  for (int q = 0; q < UP; ++q) {
    const __amdgpu_buffer_rsrc_t rs = pout.next();
    store_pair<ALIGNED>(rs, ova, done_a[q]);
    store_pair<ALIGNED>(rs, ovb, done_b[q]);
  }
}

// ----------------------------------------------------------------------------- odd radii: four input lines
// One sparse instruction on four input lines, two consecutive pairs, one copy of
// each line's window per lane half (the planner's pack_quad).  Compared with a hi
// and a lo copy of two lines in K, every line pair is gathered once instead of
// twice, the operand of pair j (registers of the older pair kept, those of the one
// before it replaced) is ready before the matrix instructions start, and only
// (r - 1) / 2 + 1 output pairs per level are in flight instead of r + 1.  The
// instructions per output are the same r + 1.  Box-2D49P 10240^2, us per step: fp16,
// four steps per launch, 39.3 before and 35.4 now; fp32 carry, three, 82.3 and 76.9.

// The coefficient operands: instruction k for operands whose lower half is the older
// pair (a[0]) or the newer one (a[1]: the same with its K halves exchanged).
template <int R>
struct QuadA {
  u32x4 a[2][R + 1];
  uint32_t i[2][(R + 1) / 2];
  __device__ __forceinline__ void load(const BandGrid& g, int lane) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int la = lane ^ (32 * v);
#pragma unroll
      for (int k = 0; k <= R; ++k) a[v][k] = reinterpret_cast<const u32x4*>(g.apack)[k * 64 + la];
#pragma unroll
      for (int k = 0; k < (R + 1) / 2; ++k) i[v][k] = g.ipack[k * 64 + la];
    }
  }
};

// The operand of two line pairs.  Which half holds which pair decides the order an
// instruction sums them in, so it follows the pair's row in the grid, not its place
// in the stream: the pair that starts at row y is in half floor(y / 2) % 2, and
// results do not depend on segment heights or on how many steps a launch fuses.
struct QuadB {
  u32x4 p[2];
};

// acc += A_k x quad, newest pair in half NEW.
// (NEW is a constant once the loops over levels unroll)
template <int OP, int R, int K>
__device__ __forceinline__ f32x4 quad_mma(int NEW, f32x4 acc, const QuadA<R>& A, const QuadB& b) {
  return pair_mma<OP, 1, (K & 1)>(acc, A.a[1 - NEW][K], (u32x4){0, 0, 0, 0}, (u32x4){0, 0, 0, 0}, A.i[1 - NEW][K / 2],
                                  b.p[0], b.p[1]);
}

// floor(y / 2) % 2 of the level-t pairs, less that of stream iteration P: they start
// at row y0 - (T - t) R + 2 j, y0 a multiple of 4, j of P's parity.
template <int R, int T>
constexpr int quad_parity(int t) {
  return (((T - t) * R + 1) / 2) & 1;
}

// Live output pairs of one level and half.  Pair j has arrived in half NEW of the
// operand: quad (j - 1, j) completes output pair j - R and starts output pair
// j - 1, which takes over its place (r = 1: they are the same, nothing is carried).
template <int R>
struct QuadAcc {
  f32x4 s[R == 3 ? 2 : 1];
  __device__ __forceinline__ void zero() { s[0] = s[R == 3 ? 1 : 0] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
};

// T = 2 .. 4 steps per launch.  The stream of band2d_pair_tbt_body (kernels_band_pair.hip)
// with quads: level t (0 = input, T = output) has its line pairs start at row y0 -
// (T - t) r; at stream iteration P pass t multiplies the level-t pair P - t (r + 1),
// staged (t = 0) or written by pass t - 1 in iteration P - 1.  An iteration completes
// its output pairs first, writes them, and only then starts the next ones (r = 3),
// gathering the next iteration's lines between those instructions: the LDS round
// trip is covered by matrix work, and one pair per level is all the LDS holds.  T >= 2
// steps store pair_tb_width columns (240 at T = 2).  A launch of one step (fp32 carry, split 3) has
// no level between and stores the 256 columns it computes.
constexpr int quad_width(int T, int R) {
  return T == 1 ? kStripWPair : T == 2 ? kStripWPair2 : pair_tb_width(T, R);
}
constexpr int quad_margin(int T, int R) { return T <= 2 ? kPairWinLead : pair_tb_margin(T, R); }
// LDS: one line pair of the input and of every level between.
template <int T>
constexpr int quad_lds_dw() {
  return 2 * T * kPairRowDw;
}

// What a wave computes beyond the grid: nothing (0), columns (1), or rows and perhaps
// columns (2); values there are the zero halo of the next step.
template <int R, int T>
__device__ __forceinline__ int quad_edge(const BandGrid& g, int w, bool aligned) {
  if (T == 1) return 0;  // no step in between
  const int strip = w % g.nstrips, seg = w / g.nstrips;
  const int xp = strip * quad_width(T, R) - quad_margin(T, R);
  const int y0 = seg * g.seg_h, hrows = min(g.seg_h, g.ny - y0);
  if ((y0 & ~3) - T * R < 0 || y0 + hrows + T * R + 2 > g.ny) return 2;
  return xp >= 0 && xp + (aligned ? 256 : 260) <= g.nx ? 0 : 1;
}

template <int R, int OP, bool ALIGNED, int T, int EDGE>
__device__ __forceinline__ void band2d_quad_body(const BandGrid& g, int w, uint32_t* lds) {
  constexpr int PAIR = 2 * kPairRowDw;
  constexpr int MARGIN = quad_margin(T, R), WIDTH = quad_width(T, R);
  const int lane = threadIdx.x;
  const int strip = w % g.nstrips, seg = w / g.nstrips;
  const int xp = strip * WIDTH - MARGIN;                // first computed column of every pass (4 mod 8)
  const int x_lo = strip * WIDTH;                       // stored columns
  // a segment that starts at row 2 mod 4 streams from the pair of rows before it
  const int ys = seg * g.seg_h, y0 = ys & ~3;
  const int hrows = min(g.seg_h, g.ny - ys) + (ys - y0);
  const int npin = (hrows + 1) / 2 + T * R + (T - 1);  // input pairs streamed, in whole bodies of four
  const int nit = (npin + 3) / 4 * 4;
  const int nx = g.nx, ny = g.ny;
  const int x_hi = min(nx, x_lo + WIDTH);

  QuadA<R> A;
  A.load(g, lane);
  __builtin_amdgcn_s_waitcnt(0);

  int p1, p2;
  pair_gather_offsets(lane, &p1, &p2);
  p1 += (lane >> 5) * kPairRowDw;  // lanes 32..63 feed the pair's second line
  p2 += (lane >> 5) * kPairRowDw;
  const bool stager = lane < kPairChunks;
  const OddTail tail(ALIGNED ? 0 : nx, xp - kPairWinLead, 8 * kPairChunks);
  const uint32_t lvoff =
      tail.voff(stager ? (uint32_t)((xp - kPairWinLead + 8 * lane) * 2) : kOffNone, lane, nx);
  const int lw = 6 * lane;
  // this lane's 4 values of every pass: columns xo + e (half a) and xo + 128 + e (half b)
  // of line 2m + (lane >> 5) of the pair
  const int xo = xp + 8 * (lane & 15) + 4 * ((lane >> 4) & 1);
  const int phi = lane >> 5;
  const int line_off = phi * nx;
  const PairStore<ALIGNED> ova(xo, line_off, x_lo, x_hi, nx, xp, 2), ovb(xo + 128, line_off, x_lo, x_hi, nx, xp + 128, 2);
  // ragged widths: 16-bit lanes of the intermediate values inside the grid
  uint32_t ma0 = 0, ma1 = 0, mb0 = 0, mb1 = 0;
  if constexpr (!ALIGNED) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t half = (e & 1) ? 0xffff0000u : 0x0000ffffu;
      const int ya = xo + e, yb = xo + 128 + e;
      if (ya >= 0 && ya < nx) (e < 2 ? ma0 : ma1) |= half;
      if (yb >= 0 && yb < nx) (e < 2 ? mb0 : mb1) |= half;
    }
  }
  // the input and the intermediate levels 1 .. T-1, an LDS line pair each; this lane's 2 dwords of half a sit at data dword 4n + 2 + 2 (h & 1) of line phi,
  // half b 96 further.  Quads outside the grid's columns go to the pad dwords behind
  // their chunk instead (their own place keeps the zeros it starts with), so the waves
  // at the grid's sides do no more than the others: masking their values took 20 %
  // longer, and a launch lasts as long as its slowest wave.
  const int odd_chunk = (lane >> 4) & 1;
  const int mw = 6 * (lane & 15) + (odd_chunk ? 6 : 2) + phi * kPairRowDw;
  int mwa = mw, mwb = mw + kPairHalfDw;
  if constexpr (EDGE != 0) {
    const int pad = odd_chunk ? 4 : 2;
    if (xo + 4 <= 0 || xo >= nx) mwa += pad;
    if (xo + 132 <= 0 || xo + 128 >= nx) mwb += pad;
  }
  for (int i = lane; i < (T - 1) * PAIR; i += 64) lds[PAIR + i] = 0u;

  LineWalk lin(g.in, y0 - T * R, max(0, y0 - T * R), min(ny, y0 + hrows + T * R), nx * 2);
  // output pair P - (T - 1)(R + 1) - R is finished at iteration P
  PairWalk pout(g.out, y0 - 2 * ((T - 1) * (R + 1) + R), ys, y0 + hrows, nx * 2);
  // input pairs P + 1 and P + 2 are in registers or on their way when iteration P begins
  u32x4 stg[2][2];
  auto load = [&](u32x4* v) {
    v[0] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
    v[1] = load_row_chunk<ALIGNED>(lin.next(), lvoff, nx);
  };
  auto stage = [&](uint32_t* d, const u32x4* v) {
    if (stager) {
      store_chunk_lds(d, lw, v[0]);
      store_chunk_lds(d + kPairRowDw, lw, v[1]);
    }
    if constexpr (!ALIGNED) {
      tail.put(d, pair_dword(tail.at), lane, v[0]);
      tail.put(d + kPairRowDw, pair_dword(tail.at), lane, v[1]);
    }
  };
  load(stg[0]);
  load(stg[1]);
  stage(lds, stg[0]);
  load(stg[0]);
  QuadAcc<R> acc_a[T], acc_b[T];
  QuadB ba[T], bb[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    acc_a[t].zero();
    acc_b[t].zero();
    ba[t].p[0] = ba[t].p[1] = bb[t].p[0] = bb[t].p[1] = (u32x4){0u, 0u, 0u, 0u};
  }

  // pass t's next line pair, into half NEW of its operands
  auto gather = [&](int t, int NEW) {
    ba[t].p[NEW ^ quad_parity<R, T>(t)] = pair_gather(lds + t * PAIR, p1, p2);
    bb[t].p[NEW ^ quad_parity<R, T>(t)] = pair_gather(lds + t * PAIR + kPairHalfDw, p1, p2);
  };
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < T; ++t) gather(t, 0);

  auto iter = [&](int P, auto nc) {
    constexpr int NEW = decltype(nc)::value, S = 1 - NEW;  // P % 2; the place of the pairs completed now
    uint2 fa[T], fb[T];
    if constexpr (R == 1) {
      f32x4 sa[T], sb[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        sa[t] = quad_mma<OP, R, 0>(NEW ^ quad_parity<R, T>(t), (f32x4){0.f, 0.f, 0.f, 0.f}, A, ba[t]);
        sb[t] = quad_mma<OP, R, 0>(NEW ^ quad_parity<R, T>(t), (f32x4){0.f, 0.f, 0.f, 0.f}, A, bb[t]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        sa[t] = quad_mma<OP, R, 1>(NEW ^ quad_parity<R, T>(t), sa[t], A, ba[t]);
        sb[t] = quad_mma<OP, R, 1>(NEW ^ quad_parity<R, T>(t), sb[t], A, bb[t]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        fa[t] = pack_out<OP>(sa[t]);
        fb[t] = pack_out<OP>(sb[t]);
      }
    } else {
      // the chains of the levels and halves are independent: one instruction of each in turn
#pragma unroll
      for (int t = 0; t < T; ++t) {
        acc_a[t].s[S] = quad_mma<OP, R, 2>(NEW ^ quad_parity<R, T>(t), acc_a[t].s[S], A, ba[t]);
        acc_b[t].s[S] = quad_mma<OP, R, 2>(NEW ^ quad_parity<R, T>(t), acc_b[t].s[S], A, bb[t]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        acc_a[t].s[S] = quad_mma<OP, R, 3>(NEW ^ quad_parity<R, T>(t), acc_a[t].s[S], A, ba[t]);
        acc_b[t].s[S] = quad_mma<OP, R, 3>(NEW ^ quad_parity<R, T>(t), acc_b[t].s[S], A, bb[t]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        fa[t] = pack_out<OP>(acc_a[t].s[S]);
        fb[t] = pack_out<OP>(acc_b[t].s[S]);
      }
    }
    // level-(t + 1) pair P - t (R + 1) - R is complete: round, zero outside the grid,
    // keep it for pass t + 1 at the next iteration
#pragma unroll
    for (int t = 0; t + 1 < T; ++t) {
      const int mrow0 = y0 - (T - 1 - t) * R + 2 * (P - t * (R + 1) - R);  // the phi = 0 row
      uint32_t* mc = lds + (t + 1) * PAIR;
      uint2 oa = fa[t], ob = fb[t];
      if constexpr (!ALIGNED) {
        oa = make_uint2(oa.x & ma0, oa.y & ma1);
        ob = make_uint2(ob.x & mb0, ob.y & mb1);
      }
      if constexpr (EDGE == 2) {
        // (a branch over the few pairs that need it would cut the loop body in pieces, at
        // the price of copies of the sums)
        const uint32_t m = (unsigned)(mrow0 + phi) < (unsigned)ny ? 0xffffffffu : 0u;
        oa = make_uint2(oa.x & m, oa.y & m);
        ob = make_uint2(ob.x & m, ob.y & m);
      }
      *reinterpret_cast<uint2*>(mc + (EDGE == 0 ? mw : mwa)) = oa;
      *reinterpret_cast<uint2*>(mc + (EDGE == 0 ? mw + kPairHalfDw : mwb)) = ob;
    }
    stage(lds, stg[1 - NEW]);  // input pair P + 1
    load(stg[1 - NEW]);        // input pair P + 3
    const __amdgpu_buffer_rsrc_t rs = pout.next();
    store_pair<ALIGNED>(rs, ova, fa[T - 1]);
    store_pair<ALIGNED>(rs, ovb, fb[T - 1]);
    wave_lds_sync();  // the pairs written are visible
    if constexpr (R == 3) {
      // each level's lines of the next iteration replace the older pair of its operands as
      // soon as its last instruction has been issued
#pragma unroll
      for (int t = 0; t < T; ++t) {
        acc_a[t].s[S] = quad_mma<OP, R, 0>(NEW ^ quad_parity<R, T>(t), (f32x4){0.f, 0.f, 0.f, 0.f}, A, ba[t]);
        acc_b[t].s[S] = quad_mma<OP, R, 0>(NEW ^ quad_parity<R, T>(t), (f32x4){0.f, 0.f, 0.f, 0.f}, A, bb[t]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        acc_a[t].s[S] = quad_mma<OP, R, 1>(NEW ^ quad_parity<R, T>(t), acc_a[t].s[S], A, ba[t]);
        acc_b[t].s[S] = quad_mma<OP, R, 1>(NEW ^ quad_parity<R, T>(t), acc_b[t].s[S], A, bb[t]);
        gather(t, 1 - NEW);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * T, 0);
#pragma unroll
      for (int i = 0; i < 2 * T; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
    } else {
#pragma unroll
      for (int t = 0; t < T; ++t) gather(t, 1 - NEW);
    }
    wave_lds_sync();
  };
  for (int P = 0; P < nit; P += 2) {
    iter(P, std::integral_constant<int, 0>{});
    iter(P + 1, std::integral_constant<int, 1>{});
  }
}

// The quad body for what wave w computes beyond the grid.  ALIGNED = false: some widths
// are not multiples of 8, and the waves at the end of such lines run the ragged body.
template <int R, int OP, bool ALIGNED, int T>
__device__ __forceinline__ void quad_bodies(const BandGrid& g, int w, uint32_t* lds) {
  const int edge = quad_edge<R, T>(g, w, true);
  if (!ALIGNED && g.nx % 8 != 0 && !pair_inside(g, w, quad_width(T, R), quad_margin(T, R)))
    band2d_quad_body<R, OP, ALIGNED, T, 2>(g, w, lds);
  else if (edge == 0)
    band2d_quad_body<R, OP, true, T, 0>(g, w, lds);
  else if (edge == 1)
    band2d_quad_body<R, OP, true, T, 1>(g, w, lds);
  else
    band2d_quad_body<R, OP, true, T, 2>(g, w, lds);
}

// Whether a launch of T steps at radius R runs quads.  A single step gains nothing from
// them: it waits for memory, and the paired body loads and multiplies 2 (r + 1) lines
// between two waits for LDS where quads take two (fp16, us per step, quads and pairs:
// r = 3 3000 x 3008 11.4 and 9.0, 4096^2 20.0 and 17.8, r = 1 10.8 and 9.7).  Only the
// fp32 carry's input split keeps them, whose sums they round less often (see
// band2d_quad_f32_body; 19.2 and 19.2 on 3000 x 3008, r = 3).
template <int R, int ENG, int T, bool XLO = false>
constexpr bool use_quad() {
  return ENG == 1 && R != 2 && (T > 1 || XLO);
}

}  // namespace spider_impl
