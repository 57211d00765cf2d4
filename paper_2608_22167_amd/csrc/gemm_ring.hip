// Grouped GEMM whose operands reach LDS by direct loads through rings of 64-wide
// reduction slices (gfx950, bf16 activations, bf16 or MXFP4 weights): the MXFP4
// experts from 8 rows in all and bf16 experts from 56 rows each, where the launch
// repays its start, and the dense projections between about a thousand and ten
// thousand rows (bf16 as far as the pipelined kernel does not take them).
//
// A workgroup owns a BM x BN output tile (token rows x weight rows): WM x WN
// wavefronts multiply, and PX + PW producer wavefronts only request slices, by
// 16-byte buffer loads straight into LDS (a load fills 1 KB, lane l at byte
// 16 l), and wait for them; one barrier per slice hands slices over. Loads
// return in order, so wavefronts that load for themselves wait for the weights'
// HBM latency whenever they need the activations, which come from L2; with
// producers of their own the weights run up to seven slices ahead. (One
// producer issuing 16 loads a slice is the bound at few rows: two for the
// activations, 98 -> 80 us at 16 tokens; at over 512 rows per expert one is
// faster, 1.62 -> 1.52 ms at 14,000 tokens.) The workgroups are persistent, one
// per CU: the producers load the next tile's first slices during an epilogue.
//
// MXFP4 weights stay codes until the fragment: a slice of 256 rows is 8 KB of
// LDS instead of 32, a lane reads its 16 codes of a slice (indices 16 g ..
// 16 g + 15 for lane group g, eight per product, the activation fragments
// taking the same indices) and decodes them with the packed e2m1 -> bf16
// conversion that applies the block scale (exact for the accepted scales). On
// gfx950 a product blocks the vector pipe for one issue slot only, so the
// conversions run beside the other wavefront's products; work per code that
// does not (checking scales, masking) is done once per tile. Codes are loaded
// 64 bytes of a row at a time (32-byte pieces: 121 -> 110 us at 512 tokens).
//
// Measured (32 experts, 2880 x 5760 gate/up and 2880 x 2880 down, both
// projections together, before -> after; before: weight slabs up to 96 rows per
// expert, 128 x 128 or 256 x 256 tiles that decode into LDS above): 8 tokens
// 105 -> 83 us, 64 155 -> 124, 300 195 -> 142, 512 213 -> 166, 1888 574 -> 427,
// 14,008 3.78 -> 2.42 ms (1.19 PFLOP/s gate/up). Up to about 300 tokens the
// bound is the stream of codes (283 + 141 MB, 3.5 TB/s); at 512 tokens counters
// show no one pipe full: 3.1 TB/s from HBM, L2 channels 83% busy, matrix cores 34%,
// three vector instructions per product, one item per CU and a rest.
//
// LDS layouts. Rows of 128 B (activations, row-major bf16 weights): 16-byte
// piece c of row r in slot c ^ (r & 7). Code rows of 64 B (two slices): piece c
// of row r in slot c ^ ((r >> 2) & 3). Streaming-order weights: whole 1 KB fragments,
// row r of block b at r ^ 4 (b & 3). All fragment reads then spread over the
// banks; the direct loads keep LDS linear and permute their source instead.
//
// Products put weight rows on the accumulator's row axis, so which weight row
// a fragment row holds decides which output columns a lane ends up with
// (piece_row): gate/up tiles give a lane adjacent columns, the projection both
// halves of its rotary pairs, and the epilogues run from the registers with
// no pass through LDS and no barrier.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace mcpu {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int RK = 64;                   // reduction indices per slice
constexpr int RBUF_D3 = 0x00020000;      // raw buffer descriptor word 3 (gfx9 family)
constexpr int RING_MAX_KB = 96;          // MXFP4: scale blocks per weight row that the LDS plan holds
constexpr int RING_DENSE_TILES = 300;    // bf16 matrices: 128 x 128 tiles from which the ring is taken
constexpr int RING_MIN_ROWS = 56;        // bf16 experts: rows per group
constexpr int RING_MIN_WORK = 65536;     // ... and tiles (rows even over the groups) times reduction
constexpr int RXROW = RK * 2;            // bytes of a staged activation row

__device__ __forceinline__ u32x4 lds16(const uint8_t* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ u32x2 lds8(const uint8_t* p) { return *reinterpret_cast<const u32x2*>(p); }
__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                  0, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ring_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7FFFFFFF, RBUF_D3);
}

// 16 bytes per lane to LDS, lane l at byte 16 l
__device__ __forceinline__ void to_lds16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t vo, int so) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(dst), 16, vo, so, 0, 0);
}

// Weight row, within a wavefront's piece of 16 NT rows, that fragment nb holds
// in its row i. Accumulator lane group g, register r is fragment row 4 g + r,
// so: gate/up pieces give lane group g the 4 NT consecutive columns 4 NT g ..;
// projection pieces (NT = 4) dims j0 .. j0 + 7 (fragments 0, 1) and
// d/2 + j0 .. (2, 3) of one head; the others keep the natural order, whose
// fp32 stores cover 64 bytes of a row per fragment.
template <int EPI, int NT>
__device__ __forceinline__ int piece_row(const Gemm& P, int nb, int i) {
  if constexpr (EPI == EPI_SWIGLU) {
    return 4 * NT * (i >> 2) + 4 * nb + (i & 3);
  } else if constexpr (EPI == EPI_QKV) {
    const int D = P.head_dim, half = D / 2, j = 8 * (i >> 2);
    return (j / half) * D + j % half + 4 * (nb & 1) + (i & 3) + (nb >> 1) * half;
  } else {
    return 16 * nb + i;
  }
}

// A group's tiles, one group per lane: its first row, row count and the
// exclusive prefix of m-tiles (each wavefront holds its own copy, so finding a
// work item takes neither LDS nor a barrier).
struct RingGroups {
  int r0, rows, start, total;
};
template <int BM>
__device__ __forceinline__ RingGroups ring_groups(const Gemm& P, int lane) {
  RingGroups q{0, 0, 0, 0};
  if (P.group_off) {
    if (lane < P.n_groups) {
      q.r0 = P.group_off[lane];
      q.rows = max(P.group_off[lane + 1] - q.r0, 0);
    }
  } else if (lane == 0) {
    q.rows = P.n_rows;
  }
  const int cnt = (q.rows + BM - 1) / BM, incl = wave_incl_scan(cnt);
  q.start = incl - cnt;
  q.total = __builtin_amdgcn_readlane(incl, 63);
  return q;
}

// PX, PW: producer wavefronts for activations and weights; XS, CS: LDS stages
// of each (powers of two, XS <= CS)
template <int BM, int BN, int WM, int WN, int XS, int CS, int PX, int PW, int EPI, int WF, bool WP>
__global__ __launch_bounds__((WM * WN + PX + PW) * 64) void gemm_ring_kernel(Gemm P) {
  constexpr int NW = WM * WN;
  constexpr int MT = BM / 16 / WM, NT = BN / 16 / WN;  // 16-row fragments per wavefront
  static_assert(!WP || WF == 0, "streaming-order copies are bf16");
  static_assert(EPI != EPI_QKV || NT == 4, "a projection piece is 64 rows");
  constexpr int SPU = WF ? 2 : 1, WROW = WF ? RK : RK * 2;    // slices per weight stage, bytes of its rows
  constexpr int XB = BM * RXROW, WB = BN * WROW;              // bytes of a stage
  constexpr int XJ = XB / 1024 / PX, WJ = WB / 1024 / PW;     // direct loads per producer and slice
  constexpr int WOFF = XS * XB, SOFF = WOFF + CS * WB;        // LDS: activations, weights, scales
  constexpr int SCL = WF ? BN * RING_MAX_KB : 0;
  static_assert(XB % (1024 * PX) == 0 && WB % (1024 * PW) == 0, "whole loads");
  static_assert(XS >= 4 && XS <= CS * SPU && (XS & (XS - 1)) == 0 && (CS & (CS - 1)) == 0, "stages");
  static_assert(SOFF + SCL <= 160 * 1024, "LDS");
  constexpr int UN = CS * SPU;                              // slices per unrolled round
  constexpr int GM = BM == 64 ? 8 : BM == 128 ? 4 : 2;  // m-tiles per band
  __shared__ __align__(1024) uint8_t lds[SOFF + SCL];
  __shared__ int rejected;  // MXFP4: the last item with a rejected scale
  uint8_t* scl = lds + SOFF;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int nk = P.k / RK, kb = P.k / 32, nkp = (nk + UN - 1) / UN * UN;

  // ---- work items: this workgroup's share of its XCD's range -------------------
  const RingGroups q = ring_groups<BM>(P, lane);
  const int n_tn = (P.n + BN - 1) / BN, total = q.total * n_tn, chunk = (total + 7) >> 3;
  int idx = uniform((int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3));
  const int step = (int)gridDim.x >> 3, end = uniform(min(((int)(blockIdx.x & 7) + 1) * chunk, total));
  if (idx >= end) return;
  struct Item {
    int grp, m0, mrows, n0;
  };
  auto item_of = [&](int i) __attribute__((always_inline)) {
    Item t;
    t.grp = uniform(__popcll(__ballot(lane < P.n_groups && q.start * n_tn <= i)) - 1);
    const int start = __builtin_amdgcn_readlane(q.start, t.grp), rows = __builtin_amdgcn_readlane(q.rows, t.grp);
    int mt, tn;
    band_order<GM>(i - start * n_tn, (rows + BM - 1) / BM, n_tn, mt, tn);
    t.m0 = uniform(__builtin_amdgcn_readlane(q.r0, t.grp) + mt * BM);
    t.mrows = uniform(min(BM, rows - mt * BM));
    t.n0 = uniform(tn * BN);
    return t;
  };
  // weight row of item t held by LDS row `slot` of the tile; rows past n repeat
  // the last one (their columns are dropped)
  auto wrow_of = [&](const Item& t, int slot) __attribute__((always_inline)) {
    const int piece = slot / (16 * NT), s = slot % (16 * NT);
    return min(t.n0 + piece * 16 * NT + piece_row<EPI, NT>(P, s >> 4, s & 15), P.n - 1);
  };
  auto xswz = [&](int r) __attribute__((always_inline)) { return WF ? ((r >> 1) & 1) | (r & 4) : r & 7; };
  // the workgroup's barrier; the empty asm keeps LDS accesses on their side
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- producers -----------------------------------------------------------------
  // A producer fills the LDS stages in units of SPU slices, L units ahead of
  // the multiplying wavefronts: in the first slot of unit u of an item it
  // requests unit u + L (of the next item past the padded end; units past k
  // re-read the last one and are not used) into the stage that unit u - 1 left,
  // and in every slot t it waits until only the units behind slice t + 2 are in
  // flight and meets the barrier that publishes that slice.
  if (wave >= NW) {
    auto produce = [&](auto SPU_, auto L_, auto aim, auto request, auto wait, auto scales) __attribute__((always_inline)) {
      constexpr int SPU = decltype(SPU_)::value, L = decltype(L_)::value;
      const int units = (nk + SPU - 1) / SPU, pad = nkp / SPU;
      auto slots = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < SPU; ++s) {
          wait();
          meet();
        }
      };
      Item cur = item_of(idx);
      aim(cur);
      for (int u = 0; u < L; ++u) request(min(u, units - 1), u);
      scales(cur);
      while (true) {
        __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0): the item's first units and scales (during the last epilogue)
        meet();
        meet();  // scales checked
        const bool more = idx + step < end;
        const Item next = more ? item_of(idx + step) : cur;
        int u = 0;
        for (; u < pad - L; ++u) {
          request(min(u + L, units - 1), u + L);
          slots();
        }
        aim(next);
        for (; u < pad; ++u) {
          request(min(u + L - pad, units - 1), u + L);  // pad is a multiple of the stages
          slots();
        }
        if (!more) break;
        scales(next);
        cur = next;
        idx += step;
      }
      __builtin_amdgcn_s_waitcnt(0);  // no load into LDS may outlive the workgroup
    };
    if (wave < NW + PX) {
      // activations: piece p of a slice is tile rows 8 p + [0, 8), lane l in row
      // l / 8, slot l % 8; rows past the tile's end repeat its last row
      // (dropped), and fragments that hold no rows are out of the buffer's range
      // (no memory access)
      const int p0 = XJ * (wave - NW);
      __amdgpu_buffer_rsrc_t xr;
      uint32_t vo[XJ];
      auto aim = [&](const Item& t) __attribute__((always_inline)) {
        xr = ring_rsrc(reinterpret_cast<const uint8_t*>(P.x) + (P.row_src ? 0 : (int64_t)t.m0 * P.k * 2));
        const int used = (t.mrows + 16 * WM - 1) / (16 * WM) * (16 * WM);  // rows the multiplied fragments read
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
          const int row = 8 * (p0 + j) + (lane >> 3), r = min(row, t.mrows - 1);
          const int src = P.row_src ? P.row_src[t.m0 + r] : r;
          vo[j] = row < used ? (uint32_t)src * (uint32_t)(P.k * 2) + 16u * ((lane & 7) ^ xswz(lane >> 3)) : 0x80000000u;
        }
      };
      auto request = [&](int ks, int slot) __attribute__((always_inline)) {
        uint8_t* dst = lds + (slot % XS) * XB + 1024 * p0;
#pragma unroll
        for (int j = 0; j < XJ; ++j) to_lds16(xr, dst + 1024 * j, vo[j], uniform(ks * (RK * 2)));
      };
      auto wait = [&]() __attribute__((always_inline)) {
        constexpr int N = (XS - 3) * XJ;
        static_assert(N < 64, "vmcnt");
        __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));  // vmcnt(N)
      };
      produce(std::integral_constant<int, 1>{}, std::integral_constant<int, XS - 1>{}, aim, request, wait, [](const Item&) {});
    } else {
      const int p0 = WJ * (wave - NW - PX);
      const int wchunks = (P.k + 127) / 128;  // streaming order: 4 KB per 16-row block and 128 columns
      __amdgpu_buffer_rsrc_t wr;
      uint32_t vo[WJ];
      auto aim = [&](const Item& t) __attribute__((always_inline)) {
        const uint8_t* base = WP ? reinterpret_cast<const uint8_t*>(P.w_packed) + (int64_t)t.grp * (P.n / 16) * wchunks * 4096
                                 : reinterpret_cast<const uint8_t*>(P.w) + (int64_t)t.grp * P.w_group_stride * (WF ? 1 : 2);
        // MXFP4: a half last unit reads on into the next row, past the group's end zeros
        wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, WF ? P.n * (P.k / 2) : 0x7FFFFFFF, RBUF_D3);
#pragma unroll
        for (int j = 0; j < WJ; ++j) {
          const int p = p0 + j;
          if constexpr (WP) {  // product p % 2 of the slice of block p / 2
            const int b = p >> 1;
            vo[j] = (uint32_t)min(t.n0 / 16 + b, P.n / 16 - 1) * (uint32_t)(wchunks * 4096) + 1024u * (p & 1) +
                    16u * (lane ^ (4 * (b & 3)));
          } else if constexpr (WF == 0) {
            vo[j] = (uint32_t)wrow_of(t, 8 * p + (lane >> 3)) * (uint32_t)(P.k * 2) + 16u * ((lane & 7) ^ (lane >> 3));
          } else {
            vo[j] = (uint32_t)wrow_of(t, 16 * p + (lane >> 2)) * (uint32_t)(P.k / 2) + 16u * ((lane & 3) ^ (lane >> 4));
          }
        }
      };
      auto request = [&](int ks, int slot) __attribute__((always_inline)) {
        uint8_t* dst = lds + WOFF + (slot % CS) * WB + 1024 * p0;
        const int so = uniform(ks * (WP ? 2048 : WROW));
#pragma unroll
        for (int j = 0; j < WJ; ++j) to_lds16(wr, dst + 1024 * j, vo[j], so);
      };
      // MXFP4: an item's E8M0 scales, [row][k / 32], are staged whole, once the
      // item before is multiplied: their rows are consecutive in memory, so that
      // is a few whole-line loads, where byte loads per slice and fragment (four
      // rows per address quad) took longer than the products
      auto scales = [&](const Item& t) __attribute__((always_inline)) {
        if constexpr (WF == 1) {
          const int bytes = min(BN, P.n - t.n0) * kb;
          const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc(
              const_cast<uint8_t*>(P.w_scales) + t.grp * (P.w_group_stride / 16) + (int64_t)t.n0 * kb, 0, bytes, RBUF_D3);
          for (int p = wave - NW - PX; p * 1024 < bytes; p += PW) to_lds16(sr, scl + 1024 * p, 1024u * p + 16u * lane, 0);
        }
      };
      // in flight behind slice t + 2: units (t + 2) / SPU + 1 .. t / SPU + L
      auto wait = [&]() __attribute__((always_inline)) {
        constexpr int L = CS - 1, N = (SPU == 1 ? L - 2 : L - 1) * WJ;
        static_assert(N >= 0 && N < 64, "vmcnt");
        __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));  // vmcnt(N)
      };
      produce(std::integral_constant<int, SPU>{}, std::integral_constant<int, CS - 1>{}, aim, request, wait, scales);
    }
    return;
  }

  // ---- multiplying wavefronts ------------------------------------------------------
  // wavefront (wm, wn): token rows 16 (WM s + wm) + [0, 16), s < MT (dealt in
  // turn, so a short tile is shared evenly), weight rows 16 NT wn + [0, 16 NT).
  // Product c of a slice: indices 32 c + 8 g .. + 7 (MXFP4: 16 g + 8 c ..) for
  // lane group g.
  const int fr = lane & 15, g = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const uint32_t xo = (16 * wm + fr) * RXROW + 16 * ((WF ? 2 * g : g) ^ xswz(fr));
  const uint32_t xo1 = xo ^ (WF ? 16u : 64u);
  auto xread = [&](int stage, int c, int s) __attribute__((always_inline)) {
    return lds16(lds + (c ? xo1 : xo) + stage * XB + s * (16 * WM * RXROW));
  };
  uint32_t wo[NT];  // LDS offset of this lane's part of weight fragment nb
#pragma unroll
  for (int nb = 0; nb < NT; ++nb) {
    const int slot = 16 * (NT * wn + nb) + fr;
    if constexpr (WP) {
      const int rho = piece_row<EPI, NT>(P, nb, fr), b = NT * wn + (rho >> 4);
      wo[nb] = WOFF + 2048 * b + 16 * (((rho & 15) ^ (4 * (b & 3))) + 16 * g);
    } else if constexpr (WF == 0) {
      wo[nb] = WOFF + slot * WROW + 16 * (g ^ (fr & 7));
    } else {
      wo[nb] = WOFF + slot * WROW + 16 * ((g >> 1) ^ (fr >> 2)) + 8 * (g & 1);
    }
  }
  auto wread = [&](int stage, int c, int nb) __attribute__((always_inline)) {
    return lds16(lds + (WP ? wo[nb] + 1024u * c : wo[nb] ^ (64u * c)) + stage * WB);
  };
  uint32_t so[WF ? NT : 1];  // MXFP4: this lane's scale bytes of the item (block g / 2 of slice 0)
  // a slice's codes and scale factors
  struct Codes {
    u32x2 w[NT];
    float s[NT];
  };
  // Scales outside [2, 252] raise the error bit, once per item and outside the
  // reduction; the block contributes zero: its scale is staged as 0 and the
  // item's reduction takes the form that clears such blocks' codes (its own
  // form, so that the others carry no mask).
  auto check_scales = [&](const Item& t, int item) __attribute__((always_inline)) {
    if constexpr (WF == 1) {
      const int pieces = min(BN, P.n - t.n0) * kb / 16;  // whole: n is a multiple of 16, k of 64
      for (int p = tid; p < pieces; p += NW * 64) {
        u32x4 w = *reinterpret_cast<const u32x4*>(scl + 16 * p);
        uint32_t bad = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // any byte below 2, or above 252 (a carry can only come from one below 2)
          const uint32_t lo = w[j] & 0xFEFEFEFEu, hi = (~w[j] + 0x01010101u) & 0xFCFCFCFCu;
          bad |= ((lo - 0x01010101u) & ~lo) | ((hi - 0x01010101u) & ~hi);
        }
        if (bad & 0x80808080u) {
          bool any = false;
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < 32; b += 8)
              if (((w[j] >> b) & 255u) - 2u > 250u) {
                w[j] &= ~(255u << b);
                any = true;
              }
          if (any) {
            *reinterpret_cast<u32x4*>(scl + 16 * p) = w;
            rejected = item;
            set_error(P.err, 16);
          }
        }
      }
      __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (3 << 14));  // lgkmcnt(0): a replaced scale is visible
    }
  };
  auto decode = [&](const Codes& k, int c, int nb) __attribute__((always_inline)) {
    const uint32_t w = k.w[nb][c];
    const float s = k.s[nb];
    return u32x4{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s, 0)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s, 1)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s, 2)),
                 __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, s, 3))};
  };
  f32x4 acc[NT][MT];

  // The reduction of an item with MV of the MT token fragments (those that hold
  // rows), nkp slots. While slice i is multiplied, the head of slice i + 1 (its
  // first weight fragments or codes and two token fragments) is read into the
  // other of two register sets.
  auto reduce = [&](auto MV_, auto CLEAR_) __attribute__((always_inline)) {
    constexpr int MV = decltype(MV_)::value, U = 2 * MV;  // U steps of NT products per slice
    constexpr bool CLEAR = decltype(CLEAR_)::value;       // MXFP4: clear the codes of rejected blocks
    auto codes = [&](Codes& k, int nb, const uint8_t* at, uint32_t scale) __attribute__((always_inline)) {
      k.w[nb] = lds8(at);
      if constexpr (CLEAR) k.w[nb] &= scale ? ~0u : 0u;
      k.s[nb] = __uint_as_float((CLEAR && !scale ? 127u : scale) << 23);
    };
    u32x4 bh[2][2], ah[2][NT];
    Codes kc[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) bh[0][u] = xread(0, u / MV, u % MV);
    if constexpr (WF == 1) {
#pragma unroll
      for (int nb = 0; nb < NT; ++nb) codes(kc[0], nb, lds + wo[nb], scl[so[nb]]);
    } else {
#pragma unroll
      for (int nb = 0; nb < NT; ++nb) ah[0][nb] = wread(0, 0, nb);
    }
    auto multiply = [&](auto J_, int i) __attribute__((always_inline)) {
      constexpr int J = decltype(J_)::value, H = J % 2, XC = J % XS, XN = (J + 1) % XS, WC = J / SPU % CS, WN_ = (J + 1) / SPU % CS;
      u32x4 b[U], a0[NT], a1[NT];
      const int sn = 2 * min(i + 1, nk - 1);  // the next slice's first block
      b[0] = bh[H][0];
      b[1] = bh[H][1];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = u / MV, s = u % MV;
        if (u + 2 < U) b[u + 2] = xread(XC, (u + 2) / MV, (u + 2) % MV);
        else bh[H ^ 1][u + 2 - U] = xread(XN, (u + 2 - U) / MV, (u + 2 - U) % MV);
        // weights: product 1's fragments during product 0, the next slice's
        // head during product 1 (codes and scales during product 0)
#pragma unroll
        for (int nb = 0; nb < NT; ++nb)
          if (nb * MV / NT == s) {
            if constexpr (WF == 0) {
              if (c == 0) a1[nb] = wread(WC, 1, nb);
              else ah[H ^ 1][nb] = wread(WN_, 0, nb);
            } else {
              if (c == 0)  // the slice's half of the rows
                codes(kc[H ^ 1], nb, lds + (wo[nb] ^ (32u * (H ^ 1))) + WN_ * WB, scl[so[nb] + sn]);
            }
          }
        if (s == 0) {
#pragma unroll
          for (int nb = 0; nb < NT; ++nb) {
            if constexpr (WF == 0) a0[nb] = c == 0 ? ah[H][nb] : a1[nb];
            else a0[nb] = decode(kc[H], c, nb);
          }
        }
#pragma unroll
        for (int nb = 0; nb < NT; ++nb) acc[nb][s] = mfma(a0[nb], b[u], acc[nb][s]);
      }
    };
    auto full = [&](auto J_, int i) __attribute__((always_inline)) {
      multiply(J_, i + decltype(J_)::value);
      meet();
    };
    auto last = [&](auto J_, int i) __attribute__((always_inline)) {
      if (i + decltype(J_)::value < nk) multiply(J_, i + decltype(J_)::value);
      meet();
    };
    int i = 0;
    for (; i + UN <= nk; i += UN) {
      full(std::integral_constant<int, 0>{}, i);
      full(std::integral_constant<int, 1>{}, i);
      full(std::integral_constant<int, 2>{}, i);
      full(std::integral_constant<int, 3>{}, i);
      if constexpr (UN > 4) {
        full(std::integral_constant<int, 4>{}, i);
        full(std::integral_constant<int, 5>{}, i);
        full(std::integral_constant<int, 6>{}, i);
        full(std::integral_constant<int, 7>{}, i);
      }
    }
    if (i < nk) {
      last(std::integral_constant<int, 0>{}, i);
      last(std::integral_constant<int, 1>{}, i);
      last(std::integral_constant<int, 2>{}, i);
      last(std::integral_constant<int, 3>{}, i);
      if constexpr (UN > 4) {
        last(std::integral_constant<int, 4>{}, i);
        last(std::integral_constant<int, 5>{}, i);
        last(std::integral_constant<int, 6>{}, i);
        last(std::integral_constant<int, 7>{}, i);
      }
    }
  };

  Item cur = item_of(idx);
  if constexpr (WF == 1) {
    if (tid == 0) rejected = -1;
    __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (3 << 14));  // lgkmcnt(0)
  }
  while (true) {
    meet();  // the item's first slices and its scales have landed
    check_scales(cur, idx);
    meet();
    if constexpr (WF == 1) {
#pragma unroll
      for (int nb = 0; nb < NT; ++nb)
        so[nb] = (uint32_t)(wrow_of(cur, 16 * (NT * wn + nb) + fr) - cur.n0) * (uint32_t)kb + (g >> 1);
    }
#pragma unroll
    for (int nb = 0; nb < NT; ++nb)
#pragma unroll
      for (int mb = 0; mb < MT; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // token fragments in use per wavefront: the same for all, so every
    // wavefront meets the same barriers
    const int m0 = cur.m0, mrows = cur.mrows, n0 = cur.n0;
    const int mv = uniform((mrows + 16 * WM - 1) / (16 * WM));
    constexpr std::false_type keep{};
    bool clear = false;
    if constexpr (WF == 1) clear = uniform(rejected) == idx;
    if (WF == 1 && __builtin_expect(clear, 0)) {  // all fragments, also those without rows (their sums are dropped)
      if constexpr (WF == 1) reduce(std::integral_constant<int, MT>{}, std::true_type{});
    } else if constexpr (MT == 4) {
      if (mv == 1) reduce(std::integral_constant<int, 1>{}, keep);
      else if (mv == 2) reduce(std::integral_constant<int, 2>{}, keep);
      else if (mv == 3) reduce(std::integral_constant<int, 3>{}, keep);
      else reduce(std::integral_constant<int, 4>{}, keep);
    } else {
      static_assert(MT == 2, "two or four token fragments per wavefront");
      if (mv == 1) reduce(std::integral_constant<int, 1>{}, keep);
      else reduce(std::integral_constant<int, 2>{}, keep);
    }

    // ---- epilogue, straight from the accumulators -----------------------------
    // acc[nb][mb][r] = C[row m0 + 16 (WM mb + wm) + fr][piece_row(nb, 4 g + r)];
    // the next item's first slices land meanwhile
    const int p0 = n0 + 16 * NT * wn;  // first column of the piece
    const float* bias = P.bias + (int64_t)cur.grp * P.bias_group_stride;
    float bv[4 * NT];
#pragma unroll
    for (int nb = 0; nb < NT; ++nb) {
      const int c = min(p0 + piece_row<EPI, NT>(P, nb, 4 * g), P.n - 4);
      *reinterpret_cast<float4*>(bv + 4 * nb) = *reinterpret_cast<const float4*>(bias + c);
    }
    if constexpr (EPI == EPI_SWIGLU) {
      const int c0 = p0 + 4 * NT * g;  // n is a multiple of 16: a lane's columns are in or out together
      bf16* out = reinterpret_cast<bf16*>(P.out) + c0 / 2;
#pragma unroll
      for (int mb = 0; mb < MT; ++mb) {
        const int m = 16 * (WM * mb + wm) + fr;
        if (m >= mrows || c0 >= P.n) continue;
        uint32_t o[NT];
#pragma unroll
        for (int nb = 0; nb < NT; ++nb) {
          const float y0 = swiglu(acc[nb][mb][0] + bv[4 * nb], acc[nb][mb][1] + bv[4 * nb + 1], P.swiglu_alpha,
                                  P.swiglu_limit, P.swiglu_beta);
          const float y1 = swiglu(acc[nb][mb][2] + bv[4 * nb + 2], acc[nb][mb][3] + bv[4 * nb + 3], P.swiglu_alpha,
                                  P.swiglu_limit, P.swiglu_beta);
          o[nb] = pack_bf16(y0, y1);
        }
        bf16* p = out + (int64_t)(m0 + m) * (P.n / 2);
        if constexpr (NT == 4) *reinterpret_cast<u32x4*>(p) = u32x4{o[0], o[1], o[2], o[3]};
        else *reinterpret_cast<u32x2*>(p) = u32x2{o[0], o[1]};
      }
    } else if constexpr (EPI == EPI_QKV) {
      const int D = P.head_dim, f0 = p0 + piece_row<EPI, NT>(P, 0, 4 * g);
#pragma unroll
      for (int mb = 0; mb < MT; ++mb) {
        const int m = 16 * (WM * mb + wm) + fr;
        if (m >= mrows || p0 >= P.n) continue;  // n is a multiple of 64 here: whole pieces
        float lo[8], hi[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lo[r] = acc[0][mb][r] + bv[r];
          lo[4 + r] = acc[1][mb][r] + bv[4 + r];
          hi[r] = acc[2][mb][r] + bv[8 + r];
          hi[4 + r] = acc[3][mb][r] + bv[12 + r];
        }
        qkv_store<bf16>(P, m0 + m, f0 / D, f0 % D, lo, hi);
      }
    } else {  // EPI_RESIDUAL, EPI_BIAS
      float* out = reinterpret_cast<float*>(P.out);
#pragma unroll
      for (int nb = 0; nb < NT; ++nb) {
        const int c0 = p0 + 16 * nb + 4 * g;
        if (p0 + 16 * nb >= P.n) continue;
        float4 res[MT];
        if constexpr (EPI == EPI_RESIDUAL) {  // the residual rows requested together, before a store
#pragma unroll
          for (int mb = 0; mb < MT; ++mb)
            res[mb] = *reinterpret_cast<const float4*>(P.residual + (int64_t)(m0 + min(16 * (WM * mb + wm) + fr, mrows - 1)) * P.n + c0);
        }
#pragma unroll
        for (int mb = 0; mb < MT; ++mb) {
          const int m = 16 * (WM * mb + wm) + fr;
          if (m >= mrows) continue;
          float4 v = make_float4(acc[nb][mb][0] + bv[4 * nb], acc[nb][mb][1] + bv[4 * nb + 1], acc[nb][mb][2] + bv[4 * nb + 2],
                                 acc[nb][mb][3] + bv[4 * nb + 3]);
          if constexpr (EPI == EPI_RESIDUAL) {
            v.x += res[mb].x; v.y += res[mb].y; v.z += res[mb].z; v.w += res[mb].w;
          }
          *reinterpret_cast<float4*>(out + (int64_t)(m0 + m) * P.n + c0) = v;
        }
      }
    }
    idx += step;
    if (idx >= end) break;
    cur = item_of(idx);
  }
}

template <int BM, int BN, int WM, int WN, int XS, int CS, int PX, int PW, int WF, bool WP>
hipError_t ring_launch(const Gemm& g, hipStream_t s) {
  // one persistent workgroup per CU, eight XCDs
  dim3 gd((unsigned)std::min<int64_t>(tile_grid(g, BM, BN), 256)), bd((WM * WN + PX + PW) * 64);
#define RING(E) hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WM, WN, XS, CS, PX, PW, E, WF, WP>), gd, bd, 0, s, g)
  constexpr int NT = BN / 16 / WN;
  if constexpr (NT == 4 && WF == 0) {  // one matrix: the projections
    if (g.epi == EPI_QKV) RING(EPI_QKV);
    else if (g.epi == EPI_RESIDUAL) RING(EPI_RESIDUAL);
    else return hipErrorNotSupported;
  } else {
    if (g.epi == EPI_BIAS) {
      RING(EPI_BIAS);
    } else {
      if constexpr (NT == 3) return hipErrorNotSupported;  // 192-wide tiles are the down projection's
      else if (g.epi == EPI_SWIGLU) RING(EPI_SWIGLU);
      else return hipErrorNotSupported;
    }
  }
#undef RING
  return hipGetLastError();
}

}  // namespace

// m-tiles of `bm` rows if the rows fall evenly on the groups (by chance where there are few)
static double even_m_tiles(const Gemm& g, int bm) {
  const double G = g.n_groups, avg = g.n_rows / G;
  return avg < 4 ? G * (1 - std::pow(1 - 1 / G, g.n_rows)) : G * std::ceil(avg / bm);
}

// MXFP4: whether the launch has enough work to repay the ring's start and its
// wide tiles, by its 256-wide tiles and, where those are few, their reduction.
// Against weight slabs (up to SLAB_MAX_ROWS_FP4 rows per group): gate/up of short
// groups needs more than 128 tiles, as up to there slabs, half as wide, still find
// a CU each (slab -> ring: 45 tiles of 64 experts 15 -> 19 us, 103 of 16 experts 16
// -> 20, 165 of 32 experts 28 -> 25); from 12 rows, and for the down projection, only
// tiny launches do not pay (8 experts of 576 x 640 8 -> 10 us, of 1024 x 2048 even).
// Against the register-loading tiles above: 8 experts of 512 x 1024 at 128 rows
// 13 -> 16 us, at 500 24 -> 17; of 1024 x 2048 at 128 23 -> 22.
static bool mxfp4_ring_pays(const Gemm& g) {
  const double avg = (double)g.n_rows / g.n_groups;
  const double tiles = even_m_tiles(g, avg <= 40 ? 64 : 128) * ((g.n + 255) / 256), work = tiles * g.k;
  if (avg > SLAB_MAX_ROWS_FP4) return work >= 65536;
  return work >= 16384 && (g.epi == EPI_BIAS || avg >= 12 || tiles > 128);
}

// Whether the ring takes a launch. MXFP4 experts from 8 rows in all (both
// projections, slabs -> ring: one token 38 -> 41 us, two 58 -> 51). bf16 experts
// from RING_MIN_ROWS rows each, as far as the pipelined kernel does not take them
// (32 experts, 2880 x 5760 and 2880 x 2880 together, 64-row tiles -> ring, rows even
// / Zipf: 48 rows 306 -> 317 / 345 -> 384 us, 52 306 -> 323 / 370 -> 376, 56 334 ->
// 326 / 396 -> 393, 64 390 -> 334 / 410 -> 382, 125 504 -> 457 / 523 -> 485), if the
// launch has enough work to repay the ring's start (RING_MIN_WORK: 128-wide tiles
// times reduction; 8 experts of 512 x 1024 at 100 rows 9 -> 10 us, of 1024 x 2048
// 16 -> 14; where few tiles a CU meet uneven rows either side can win, 16 experts
// of 2048 x 4096 at 56 rows 65 -> 56 / 65 -> 73). One matrix
// from 300 tiles of 128 x 128 (QKV of 1408 rows 84 -> 71 us, of 3008 175 -> 119;
// O of 1888 99 -> 77, of 5008 213 -> 146; fewer tiles leave CUs idle: QKV of 512
// rows 38 -> 46).
bool ring_gemm_applies(int dtype, int expert_fmt, const Gemm& g) {
  if (dtype != 1 || expert_fmt > 1 || g.epi == EPI_LOGITS || g.k <= 0 || g.k % RK || g.n % 16 || g.n_groups > 64) return false;
  // 32-bit buffer offsets: token rows from x itself when gathered (else from
  // the tile), weights within one group
  const int64_t xr = g.row_src ? (g.x_rows > 0 ? g.x_rows : g.n_rows) : 128;
  if (xr * g.k * 2 >= (1LL << 31) || (int64_t)g.n * g.k * 2 >= (1LL << 31)) return false;
  if (expert_fmt != 0)  // the tile's scales are staged whole, 16 bytes at a time
    return g.n_rows >= 8 && g.k <= 32 * RING_MAX_KB && g.w_scales && (uintptr_t)g.w_scales % 16 == 0 &&
           (uintptr_t)g.w % 16 == 0 && (g.epi == EPI_SWIGLU || g.epi == EPI_BIAS) && mxfp4_ring_pays(g);
  if (g.w_packed && (int64_t)(g.n / 16) * ((g.k + 127) / 128) * 4096 >= (1LL << 31)) return false;
  // 16-byte direct loads to LDS are used on 16-byte aligned matrices only (token
  // rows come from the workspace); others keep the kernels that load to registers
  if ((uintptr_t)g.w % 16 || (uintptr_t)g.w_packed % 16) return false;
  if (g.epi == EPI_QKV && (g.n % 64 || (g.head_dim != 32 && g.head_dim != 64))) return false;
  if (pipe_gemm_applies(dtype, g)) return false;
  const int64_t groups = g.group_off ? g.n_groups : 1, tiles = ((int64_t)g.n_rows + 127) / 128 * ((g.n + 127) / 128);
  if (g.group_off) {
    const int64_t even = groups * ((g.n_rows + 128 * groups - 1) / (128 * groups)) * ((g.n + 127) / 128);
    return g.n_rows >= RING_MIN_ROWS * groups && even * g.k >= RING_MIN_WORK;
  }
  return tiles >= RING_DENSE_TILES;
}

hipError_t launch_gemm_ring(int expert_fmt, const Gemm& g, hipStream_t s) {
  if (expert_fmt != 0) {
    const double avg = (double)g.n_rows / g.n_groups;
    // 256-wide n-tiles, or 192-wide where the last round of 256 workgroups is
    // then better filled
    auto narrow = [&](int bm) {
      auto cost = [&](int bn) { return std::ceil(even_m_tiles(g, bm) * ((g.n + bn - 1) / bn) / 256) * bn; };
      return g.epi == EPI_BIAS && 10 * cost(192) < 9 * cost(256);
    };
    if (avg <= 40)
      return narrow(64) ? ring_launch<64, 192, 2, 4, 4, 4, 2, 1, 1, false>(g, s) : ring_launch<64, 256, 2, 4, 4, 4, 2, 1, 1, false>(g, s);
    if (avg <= 512)
      return narrow(128) ? ring_launch<128, 192, 2, 4, 4, 4, 2, 1, 1, false>(g, s) : ring_launch<128, 256, 2, 4, 4, 4, 2, 1, 1, false>(g, s);
    return ring_launch<128, 256, 2, 4, 4, 4, 1, 1, 1, false>(g, s);
  }
  if (g.group_off)
    return g.w_packed ? ring_launch<128, 128, 2, 4, 4, 4, 2, 2, 0, true>(g, s) : ring_launch<128, 128, 2, 4, 4, 4, 2, 2, 0, false>(g, s);
  return g.w_packed ? ring_launch<128, 128, 2, 2, 4, 4, 2, 2, 0, true>(g, s) : ring_launch<128, 128, 2, 2, 4, 4, 2, 2, 0, false>(g, s);
}

}  // namespace mcpu
