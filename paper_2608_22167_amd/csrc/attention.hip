// Paged GQA attention with per-head sinks for gfx950.
//
// The step's attention (every new token attends to its sequence's cached keys,
// plus the sink logit of its head) is split three ways:
//   plan    one workgroup maps tokens to (sequence, position) and cuts each
//           token's visible page range into splits of `pps` pages;
//   split   one wavefront per (split, KV head) streams the split's K and V
//           pages and keeps a running max / sum / weighted value sum for the
//           G = Hq / Hkv query heads that share the KV head;
//   combine a wavefront per (token, query head) merges the splits and adds the
//           sink to the normaliser.
// The score and value products run on the matrix cores: with keys as rows
// and the G query heads as columns (padded to 16), S^T = K q^T is one 16x16
// tile per page, and O^T += V^T P^T consumes it without any lane shuffle
// because the score tile's lane layout is exactly the value product's B
// operand layout. The page format (include/mcpu.h) makes every K and V
// fragment load a contiguous 512 B - 1 KiB segment per wavefront.
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace mcpu {

constexpr float LOG2E = 1.4426950408889634f;

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------

__device__ __forceinline__ int token_splits(int pos, int window, int pps) {
  int lo = window > 0 ? max(0, pos - window + 1) : 0;
  int pages = pos / PAGE - lo / PAGE + 1;
  return (pages + pps - 1) / pps;
}

__device__ __forceinline__ int seq_of_token(const int32_t* cu_q, int batch, int t) {
  // last b with cu_q[b] <= t
  int lo = 0, hi = batch - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (cu_q[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ bool is_prefill(const AttnPlan& P, int b) {
  return P.cu_q && P.prefill_min_q > 0 && P.cu_q[b + 1] - P.cu_q[b] >= P.prefill_min_q;
}

// Exclusive prefix of `local` over the 1024 threads of the block, and the total.
__device__ int block_exclusive_scan(int local, int* sums, int& total) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int incl = wave_incl_scan(local);
  const int wave = tid >> 6, lane = tid & 63;
  if (lane == 63) sums[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int w = lane < (nt >> 6) ? sums[lane] : 0;
    const int wi = wave_incl_scan(w);
    if (lane < (nt >> 6)) sums[64 + lane] = wi - w;  // exclusive prefix of wave totals
    if (lane == (nt >> 6) - 1) sums[128] = wi;       // grand total
  }
  __syncthreads();
  const int excl = sums[64 + wave] + incl - local;
  total = sums[128];
  __syncthreads();  // sums is reused by the next scan
  return excl;
}

constexpr int PLAN_SEQS = 2048;  // cu_q of up to this many sequences is searched in LDS
constexpr int PLAN_TILE = 4;     // from this many tiles of one token per thread on, four per thread
constexpr int PLAN_OWN = 8;      // up to this many splits a token's lane writes them itself

// The token part of the plan by one workgroup, in tiles of V consecutive tokens
// per thread: positions, the running split count and the splits' descriptors.
// Where no token of a wavefront has more than PLAN_OWN splits each lane writes
// its own token's (one each: 5.2 us, 5.6 together); where one has more, the
// wavefront writes them together (lane j the tile's j-th split). Returns their
// number.
// One tile costs a scan of the workgroup (three barriers), so many tokens take
// four per thread; with few, one per thread spreads the descriptors over more
// wavefronts. Bound by latency. Against a contiguous run of tokens per thread with a
// search in memory and a serial loop over descriptors: one token with 16 K keys
// 10.5 -> 5.5 us, 31 K tokens 184 -> 164 us (the norm beside it moves 540 MB).
template <int V>
__device__ int plan_tokens(const AttnPlan& P, const int32_t* cu, int* sums) {
  const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
  int base = 0;
  for (int tile = 0; tile < P.n_tokens; tile += V * nt) {
    const int t0 = tile + V * tid;
    int seq[V], pos[V], ns[V], local = 0;
    int b = cu ? seq_of_token(cu, P.batch, min(t0, P.n_tokens - 1)) : 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int t = t0 + i;
      seq[i] = pos[i] = ns[i] = 0;
      if (t >= P.n_tokens) continue;
      if (cu) {
        while (b < P.batch - 1 && cu[b + 1] <= t) ++b;
      } else {
        b = t;
      }
      seq[i] = b;
      pos[i] = P.seq_lens[b] + (cu ? t - cu[b] : 0);
      const bool pre = cu && P.prefill_min_q > 0 && cu[b + 1] - cu[b] >= P.prefill_min_q;
      ns[i] = pre ? 0 : token_splits(pos[i], P.window, P.pps);
      local += ns[i];
    }
    int total = 0;
    int run = base + block_exclusive_scan(local, sums, total);
    int start[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      start[i] = run;
      run += ns[i];
      if (t0 + i < P.n_tokens) {
        P.tok_seq[t0 + i] = seq[i];
        P.tok_pos[t0 + i] = pos[i];
        P.split_start[t0 + i] = start[i];
      }
    }
    // split k of token t's n: its splits share its np pages evenly (sizes differ by at most one)
    auto describe = [&](auto OWN_, int at, int t, int b, int p, int k, int n) __attribute__((always_inline)) {
      if ((unsigned)at >= (unsigned)max(P.host_total_splits, 0)) return;
      const int lo = P.window > 0 ? max(0, p - P.window + 1) : 0;
      const int first = lo / PAGE, np = p / PAGE - first + 1;
      SplitDesc d;
      d.t = t; d.b = b; d.p = p; d.lo = lo;
      if constexpr (decltype(OWN_)::value) {  // at most PLAN_OWN: the products fit 32 bits (np <= 2^27)
        d.pg0 = first + (int)((unsigned)(k * np) / (unsigned)n);
        d.pg1 = first + (int)((unsigned)((k + 1) * np) / (unsigned)n);
      } else {
        d.pg0 = first + (int)((int64_t)k * np / n);
        d.pg1 = first + (int)((int64_t)(k + 1) * np / n);
      }
      d.pad0 = d.pad1 = 0;
      P.split_desc[at] = d;
    };
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int n = max(ns[i], 0);
      if (__ballot(n > PLAN_OWN) == 0) {  // few splits each: a lane writes its own token's
        for (int k = 0; k < n; ++k) describe(std::true_type{}, start[i] + k, t0 + i, seq[i], pos[i], k, n);
        continue;
      }
      const int incl = wave_incl_scan(n);
      const int all = __shfl(incl, 63, 64);
      for (int j0 = 0; j0 < all; j0 += 64) {
        const int j = j0 + lane;
        int o = 0;  // the first lane with incl > j: the token of split j
#pragma unroll
        for (int step = 32; step; step >>= 1) o += __shfl(incl, o + step - 1, 64) <= j ? step : 0;
        const int src = min(o, 63);
        const int k = j - (__shfl(incl, src, 64) - __shfl(n, src, 64)), ns_o = __shfl(n, src, 64);
        const int at = __shfl(start[i], src, 64) + k, p = __shfl(pos[i], src, 64), sq = __shfl(seq[i], src, 64);
        if (j < all) describe(std::false_type{}, at, tile + V * (tid - lane + src) + i, sq, p, k, ns_o);
      }
    }
    base += total;
  }
  return base;
}

// Workgroups 1.. of the plan launch: the layer's first RMSNorm, y = x /
// sqrt(mean(x^2) + eps) * g, on four rows per workgroup (256 threads a row,
// float4 j of a thread at features 4 (t + 256 j)), so that the norm and the
// plan, both short and independent, share one launch.
template <typename T>
__device__ void plan_norm_rows(const RmsNorm& N) {
  __shared__ float part[16];
  constexpr int NVMAX = 8;  // hidden <= 8192
  const int tid = threadIdx.x, sub = tid & 255, grp = tid >> 8, H = N.hidden;
  const int row = (blockIdx.x - 1) * 4 + grp;
  const bool live = row < N.n_tokens;
  const float* x = N.x + (int64_t)(live ? row : 0) * H;
  float4 xv[NVMAX], gv[NVMAX];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < NVMAX; ++j) {
    const int i = (sub + 256 * j) * 4;
    if (i < H) {
      xv[j] = *reinterpret_cast<const float4*>(x + i);
      gv[j] = *reinterpret_cast<const float4*>(N.g + i);
      ss += xv[j].x * xv[j].x + xv[j].y * xv[j].y + xv[j].z * xv[j].z + xv[j].w * xv[j].w;
    }
  }
  ss = wave_sum(ss);
  if (lane_id() == 0) part[tid >> 6] = ss;
  __syncthreads();
  const float tot = part[4 * grp] + part[4 * grp + 1] + part[4 * grp + 2] + part[4 * grp + 3];
  const float inv = 1.0f / sqrtf(tot / (float)H + N.eps);
  if (!live) return;
  T* out = reinterpret_cast<T*>(N.out) + (int64_t)row * H;
#pragma unroll
  for (int j = 0; j < NVMAX; ++j) {
    const int i = (sub + 256 * j) * 4;
    if (i < H)
      store4(out + i, make_float4(xv[j].x * inv * gv[j].x, xv[j].y * inv * gv[j].y,
                                xv[j].z * inv * gv[j].z, xv[j].w * inv * gv[j].w));
  }
}

__global__ __launch_bounds__(1024) void attn_plan_kernel(AttnPlan P) {
  if (blockIdx.x > 0) {
    if (P.norm_dtype == 0) plan_norm_rows<float>(P.norm);
    else plan_norm_rows<bf16>(P.norm);
    return;
  }
  __shared__ int sums[160];
  __shared__ int cu_s[PLAN_SEQS + 1];
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int i = tid; i < P.n_zero; i += nt) P.zero[i] = 0;
  const int32_t* cu = P.cu_q;
  if (cu && P.batch <= PLAN_SEQS) {
    for (int i = tid; i <= P.batch; i += nt) cu_s[i] = cu[i];
    __syncthreads();
    cu = cu_s;
  }
  int total = 0;
  if (P.n_tokens <= PLAN_TILE * nt) total = plan_tokens<1>(P, cu, sums);
  else total = plan_tokens<4>(P, cu, sums);
  if (tid == 0) {
    P.split_start[P.n_tokens] = total;
    if (P.host_total_splits >= 0 && total != P.host_total_splits) set_error(P.err, 8);
  }
  if (!P.blk_start) return;
  // sequences: prefill blocks of prefill_qb tokens
  const int perb = (P.batch + nt - 1) / nt;
  const int b0 = min(P.batch, tid * perb), b1 = min(P.batch, b0 + perb);
  int local = 0;
  for (int b = b0; b < b1; ++b)
    if (is_prefill(P, b)) local += (P.cu_q[b + 1] - P.cu_q[b] + P.prefill_qb - 1) / P.prefill_qb;
  int run = block_exclusive_scan(local, sums, total);
  for (int b = b0; b < b1; ++b) {
    P.blk_start[b] = run;
    if (is_prefill(P, b)) run += (P.cu_q[b + 1] - P.cu_q[b] + P.prefill_qb - 1) / P.prefill_qb;
  }
  if (tid == 0) {
    P.blk_start[P.batch] = total;
    if (total != P.host_total_blocks) set_error(P.err, 8);
  }
}

hipError_t launch_attn_plan(const AttnPlan& p, hipStream_t s) {
  int blocks = 1;
  if (p.norm_dtype >= 0) {
    if (p.norm.hidden % 4 || p.norm.hidden > 8192) return hipErrorInvalidValue;
    blocks += (p.norm.n_tokens + 3) / 4;
  }
  hipLaunchKernelGGL(attn_plan_kernel, dim3(blocks), dim3(1024), 0, s, p);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// split: one wavefront per (split, KV head)
// ---------------------------------------------------------------------------

// One KV head's K and V of one page, loaded with the streaming policy: a page
// is read by one wavefront (C2 attention 218 -> 194 us).
template <typename T, int D>
struct PageFrags {
  Frag<T> k[D / 32];   // chunk c holds dims 32c + 8 * (lane / 16) .. +7 of key lane % 16
  Frag4<T> v[D / 16];  // block n holds V[4 * (lane / 16) + r][16n + lane % 16]
  __device__ __forceinline__ void load(const T* kp, const T* vp, int lane) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c) k[c].load_stream(kp + (64 * c + lane) * 8);
#pragma unroll
    for (int n = 0; n < D / 16; ++n) v[n].load_stream(vp + (64 * n + lane) * 4);
  }
};

// Online-softmax state of one wavefront: the running maximum (log2 units), the
// running sum and the value accumulator (lane (hl, grp) holds dims
// 16 n + 4 grp .. + 3 of query head hl).
template <int D>
struct SoftmaxAcc {
  float m = -INFINITY, l = 0.f;
  f32x4 acc[D / 16];
  __device__ __forceinline__ SoftmaxAcc() {
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // One page: S^T = K q^T on the matrix cores, mask keys outside [lo, p] (and
  // the whole page if `valid` is false), rescale, and O^T += V^T P^T.
  template <typename T>
  __device__ __forceinline__ void page(const PageFrags<T, D>& cur, const Frag<T> (&qf)[D / 32], bool valid,
                                       int key0, int lo, int p, float scale_log2) {
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 32; ++c) sc = mma32(cur.k[c], qf[c], sc);
    // sc[r] = score of key slot key0 + r for query head lane % 16
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int pos = key0 + r;
      x[r] = (valid && pos >= lo && pos <= p) ? sc[r] * scale_log2 : -INFINITY;
    }
    float mloc = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
    mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
    const float m_new = fmaxf(m, mloc);
    // m_new is -inf only while every key so far was masked (missing pages)
    const bool live = m_new != -INFINITY;
    const float alpha = live ? __builtin_amdgcn_exp2f(m - m_new) : 1.0f;
    float pr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pr[r] = live ? __builtin_amdgcn_exp2f(x[r] - m_new) : 0.f;
    l *= alpha;
#pragma unroll
    for (int n = 0; n < D / 16; ++n) {
      acc[n] *= alpha;
      acc[n] = mma16_p(cur.v[n], pr, acc[n], n == 0 ? &l : nullptr);
    }
    m = m_new;
  }
  // the sum over the wavefront's four key-row groups
  __device__ __forceinline__ float l_total() const {
    float t = l + __shfl_xor(l, 16, 64);
    return t + __shfl_xor(t, 32, 64);
  }
};

// The token, position and page range of split s (shared by both kernels).
struct SplitRange {
  int t, b, p, lo, pg0, pg1;
};
// (the plan kernel wrote it as one 32-byte record: a single load, where a
// search over split_start would chain several dependent ones)
__device__ __forceinline__ SplitRange split_range(const AttnSplit& P, int s) {
  const SplitDesc d = P.split_desc[s];
  SplitRange r;
  r.t = uniform(d.t);
  r.b = uniform(d.b);
  r.p = uniform(d.p);
  r.lo = uniform(d.lo);
  r.pg0 = uniform(d.pg0);
  r.pg1 = uniform(d.pg1);
  // a record the plan did not write (device arrays disagree with the host's
  // plan) may be stale: every field is checked before it addresses memory
  if (r.t < 0 || r.t >= P.n_tokens || r.b < 0 || r.b >= P.batch || r.p < 0 || r.p / PAGE >= P.max_pages ||
      r.pg0 < 0 || r.pg0 >= r.pg1 || r.pg1 > P.max_pages) {
    if (lane_id() == 0) set_error(P.err, 1);
    r.t = 0;
    r.b = 0;
    r.pg0 = r.pg1 = 0;
  }
  return r;
}

template <typename T, int D>
__device__ __forceinline__ void load_q(Frag<T> (&qf)[D / 32], const AttnSplit& P, int t, int g) {
  const int lane = lane_id(), G = P.hq / P.hkv, hl = lane & 15, grp = lane >> 4;
  const T* qb = reinterpret_cast<const T*>(P.q) + ((int64_t)t * P.hq + g * G + hl) * D + 8 * grp;
#pragma unroll
  for (int c = 0; c < D / 32; ++c) {
    if (hl < G) qf[c].load(qb + 32 * c); else qf[c].zero();
  }
}

template <typename T, int D, int WAVES, int PF>
__global__ __launch_bounds__(64 * WAVES) void attn_split_kernel(AttnSplit P) {
  const int lane = lane_id();
  const int item = blockIdx.x * WAVES + uniform(threadIdx.x >> 6);
  const int s = item / P.hkv, g = item - (item / P.hkv) * P.hkv;
  if (s >= P.n_splits) return;
  const SplitRange R = split_range(P, s);
  const int pg0 = R.pg0, pg1 = R.pg1;
  const int G = P.hq / P.hkv;
  const int hl = lane & 15, grp = lane >> 4;
  Frag<T> qf[D / 32];
  load_q<T, D>(qf, P, R.t, g);

  const T* kpool = reinterpret_cast<const T*>(P.k_pool);
  const T* vpool = reinterpret_cast<const T*>(P.v_pool);
  const int32_t* ptab = P.page_table + (int64_t)R.b * P.max_pages;
  const int64_t head_off = (int64_t)g * PAGE * D, page_elems = (int64_t)P.hkv * PAGE * D;
  SoftmaxAcc<D> st;

  // PF-deep ring of pages: while page i is consumed, pages i+1 .. i+PF-1 are
  // in flight and page i+PF is issued into its slot. Loads are branch-free: a
  // slot past the split re-reads the last page, a missing page reads page 0,
  // and both are masked out of the softmax instead of skipped. (The wait for
  // each page-table entry also waits for the pages in flight; reading 64
  // entries with one vector load up front avoids that but costs 17 VGPRs,
  // five wavefronts per SIMD down to four, and was 4% slower at 64
  // sequences: this kernel hides its latency with occupancy.)
  const int npg = pg1 - pg0;
  PageFrags<T, D> ring[PF];
  bool ok[PF];
  auto fetch = [&](int slot, int i) {
    const int pg = pg0 + min(i, npg - 1);
    int id = uniform(ptab[pg]);
    const bool good = id >= 0 && id < P.n_pages;
    if (!good && lane == 0 && i < npg) set_error(P.err, 1);
    id = good ? id : 0;
    ok[slot] = good && i < npg;
    ring[slot].load(kpool + id * page_elems + head_off, vpool + id * page_elems + head_off, lane);
  };
  auto consume = [&](int slot, int i) {
    st.page(ring[slot], qf, ok[slot], (pg0 + i) * PAGE + 4 * grp, R.lo, R.p, P.scale_log2);
  };
  if (npg > 0) {
#pragma unroll
    for (int u = 0; u < PF; ++u) fetch(u, u);
    int i = 0;
    for (; i + PF <= npg; i += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        consume(u, i + u);
        fetch(u, i + u + PF);
      }
    }
#pragma unroll
    for (int u = 0; u < PF; ++u)
      if (i + u < npg) consume(u, i + u);
  }

  const float l_tot = st.l_total();
  if (hl < G) {
    const int64_t row = (int64_t)s * P.hq + g * G + hl;
    if (grp == 0) {
      P.part_ml[row * 2 + 0] = st.m;
      P.part_ml[row * 2 + 1] = l_tot;
    }
    float* pa = P.part_acc + row * D + 4 * grp;
#pragma unroll
    for (int n = 0; n < D / 16; ++n)
      *reinterpret_cast<float4*>(pa + 16 * n) = make_float4(st.acc[n][0], st.acc[n][1], st.acc[n][2], st.acc[n][3]);
  }
}

// Sliding-window layers: every decode token's window spans at most MAXP pages
// and is one split. One wavefront per (token, KV head) reads the window's page
// ids with one vector load (lane j: page j), issues every page's K and V loads
// at once, and finishes the token itself: the sink joins the normaliser and o
// is written in the layer dtype, so no partials and no combine pass are
// needed. (The split-K kernel, whose pages follow a page-table load each and
// keep two in flight, left short windows waiting on memory latency.)
//
// The KV heads of a token go to one workgroup of WW wavefronts (wavefront w:
// head w), the workgroups in eight contiguous ranges, one per XCD (workgroups
// are dealt to the XCDs round robin): a token's pages, which hold all its KV
// heads side by side, are then read by one compute unit.
template <typename T, int D, int MAXP, int WW>
__global__ __launch_bounds__(64 * WW) void attn_window_kernel(AttnSplit P) {
  const int lane = lane_id();
  const int items = P.n_splits * P.hkv;
  const int nblk = (items + WW - 1) / WW, chunk = (nblk + 7) >> 3;
  const int blk = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= chunk || blk >= nblk) return;
  const int item = blk * WW + uniform(threadIdx.x >> 6);
  if (item >= items) return;  // no barriers below: a wavefront may leave alone
  const int s = item / P.hkv, g = item - (item / P.hkv) * P.hkv;
  const SplitRange R = split_range(P, s);
  if (R.pg0 == R.pg1) return;  // an invalid record (error bit set): no token to finish
  const int npg = min(R.pg1 - R.pg0, MAXP);
  if (lane == 0 && R.pg1 - R.pg0 > MAXP) set_error(P.err, 8);  // the launch does not fit this plan
  const int G = P.hq / P.hkv;
  const int hl = lane & 15, grp = lane >> 4;
  const int my_id = lane < npg ? P.page_table[(int64_t)R.b * P.max_pages + R.pg0 + lane] : 0;
  Frag<T> qf[D / 32];
  load_q<T, D>(qf, P, R.t, g);
  const T* kpool = reinterpret_cast<const T*>(P.k_pool);
  const T* vpool = reinterpret_cast<const T*>(P.v_pool);
  const int64_t head_off = (int64_t)g * PAGE * D, page_elems = (int64_t)P.hkv * PAGE * D;
  // Every page is requested before the first is used, unconditionally (slots
  // past the window re-read its last page, a missing page reads page 0; both
  // masked), and the error bit is set after the loads: a conditional load or
  // atomic among them leaves the compiler unable to count the loads in
  // flight, and it then waits for each page before requesting the next.
  PageFrags<T, D> pages[MAXP];
  bool ok[MAXP];
  bool bad = false;
#pragma unroll
  for (int u = 0; u < MAXP; ++u) {
    int id = __shfl(my_id, min(u, npg - 1), 64);
    const bool good = id >= 0 && id < P.n_pages;
    bad = bad || (!good && u < npg);
    ok[u] = good && u < npg;
    id = good ? id : 0;
    pages[u].load(kpool + id * page_elems + head_off, vpool + id * page_elems + head_off, lane);
  }
  if (bad && lane == 0) set_error(P.err, 1);
  SoftmaxAcc<D> st;
#pragma unroll
  for (int u = 0; u < MAXP; ++u)
    if (u < npg) st.page(pages[u], qf, ok[u], (R.pg0 + u) * PAGE + 4 * grp, R.lo, R.p, P.scale_log2);
  const float l_tot = st.l_total();
  if (hl < G) {
    // o_h = 2^{m - M} acc / (2^{sink log2e - M} + 2^{m - M} l), M = max(sink log2e, m)
    const int h = g * G + hl;
    float M = P.sinks ? P.sinks[h] * LOG2E : -INFINITY;
    float L = P.sinks ? 1.0f : 0.0f;
    float f = 0.f;
    if (st.m != -INFINITY) {
      if (st.m > M) {
        L *= __builtin_amdgcn_exp2f(M - st.m);
        M = st.m;
      }
      f = __builtin_amdgcn_exp2f(st.m - M);
      L += f * l_tot;
    }
    T* o = reinterpret_cast<T*>(P.o) + ((int64_t)R.t * P.hq + h) * D + 4 * grp;
#pragma unroll
    for (int n = 0; n < D / 16; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) Elem<T>::store(o, 16 * n + r, L > 0.f ? f * st.acc[n][r] / L : 0.f);
  }
}

#ifndef MCPU_WINDOW_WAVES
#define MCPU_WINDOW_WAVES 8
#endif
constexpr int WINDOW_WAVES = MCPU_WINDOW_WAVES;  // wavefronts per window workgroup

template <typename T, int D, int WAVES = 1, int PF = 2>
hipError_t split_impl(const AttnSplit& p, hipStream_t s) {
  int64_t items = (int64_t)p.n_splits * p.hkv;
  int blocks = (int)((items + WAVES - 1) / WAVES);
  if (blocks == 0) return hipSuccess;
  if (p.o) {
    constexpr int WW = WINDOW_WAVES;
    const int64_t nblk = (items + WW - 1) / WW, grid = (nblk + 7) / 8 * 8;
    hipLaunchKernelGGL((attn_window_kernel<T, D, WINDOW_MAX_PAGES, WW>), dim3((unsigned)grid), dim3(64 * WW), 0, s, p);
  } else {
    hipLaunchKernelGGL((attn_split_kernel<T, D, WAVES, PF>), dim3(blocks), dim3(64 * WAVES), 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_attn_split(int dtype, int head_dim, const AttnSplit& p, hipStream_t s) {
  if (dtype == 0) return head_dim == 32 ? split_impl<float, 32>(p, s) : split_impl<float, 64>(p, s);
  return head_dim == 32 ? split_impl<bf16, 32>(p, s) : split_impl<bf16, 64>(p, s);
}

// ---------------------------------------------------------------------------
// combine: o_h = sum_s 2^{m_s - M} acc_s / (2^{sink_h log2e - M} + sum_s 2^{m_s - M} l_s)
// ---------------------------------------------------------------------------

// A wavefront merges the splits of one query head of K tokens, n_waves / hq
// apart (1 up to COMBINE_WAVES wavefronts): in a step that also prefills most
// tokens have no splits, and one look at K tokens' split ranges skips them all
// (31 K tokens with 48 decoding: 133 -> 10.7 us against a wavefront per token and
// head; bound by their launches). K stays below the tokens per decoding one.
//
// WIDE: per 64 splits, lane j holds split j's maximum and sum; the partial rows are
// read four dims per lane, 256 / D rows per load and eight loads at a time, so
// that one token with many splits waits for few round trips (16 K keys: 25 ->
// 5.3 us). Otherwise the splits are merged in order, lane i owning dim i, four
// rows at a time: about 0.33 us per split of the longest list, but no cross-lane
// steps and a fifth of the registers, where WIDE takes about 0.44 us per
// thousand wavefronts. The shorter of the two is taken (wide -> in order: 512
// tokens of one to 15 splits 18.4 -> 10.0 us, 9000 of one 204 -> 116); lists of
// up to four are one round of loads either way and go in order.
constexpr int COMBINE_WAVES = 65536;
constexpr int COMBINE_WAVES_PER_SPLIT = 750;  // 0.33 us of a split in order, in wavefronts of the wide form

template <typename T, int D, bool WIDE>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnCombine P, int stride, int K) {
  constexpr int LR = D / 4, RW = 64 / LR, U = 8;  // lanes per row, rows per load, loads in flight
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = lane_id(), sub = lane / LR, dim = 4 * (lane % LR);
  if (item >= stride * P.hq) return;
  const int tb = uniform(item / P.hq), h = uniform(item - (item / P.hq) * P.hq);
  int b0 = 0, b1 = 0;  // lane k: the split range of token tb + k * stride
  if (lane < K && tb + lane * stride < P.n_tokens) {
    b0 = min(P.split_start[tb + lane * stride], P.n_splits);
    b1 = min(P.split_start[tb + lane * stride + 1], P.n_splits);
  }
  // tokens without splits are prefill tokens: their rows come from the prefill kernel
  for (uint64_t todo = __ballot(b0 < b1); todo; todo &= todo - 1) {
    const int k = __builtin_ctzll(todo);
    const int s0 = __builtin_amdgcn_readlane(b0, k), s1 = __builtin_amdgcn_readlane(b1, k);
    float M = P.sinks ? P.sinks[h] * LOG2E : -INFINITY;
    if constexpr (!WIDE) {
      float L = P.sinks ? 1.0f : 0.0f, a = 0.f;  // the sink's own term, 2^(sink - M)
      for (int s = s0; s < s1; s += 4) {
        float m[4], l[4], v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          m[u] = -INFINITY;
          l[u] = v[u] = 0.f;
          if (s + u < s1) {  // uniform
            const int64_t row = (int64_t)(s + u) * P.hq + h;
            m[u] = P.part_ml[row * 2];
            l[u] = P.part_ml[row * 2 + 1];
            if (lane < D) v[u] = P.part_acc[row * D + lane];
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (m[u] == -INFINITY) continue;  // a split whose pages were all missing
          if (m[u] > M) {
            const float r = __builtin_amdgcn_exp2f(M - m[u]);
            L *= r;
            a *= r;
            M = m[u];
          }
          const float f = __builtin_amdgcn_exp2f(m[u] - M);
          L += f * l[u];
          a += f * v[u];
        }
      }
      T* o = reinterpret_cast<T*>(P.o) + ((int64_t)(tb + k * stride) * P.hq + h) * D;
      if (lane < D) Elem<T>::store(o, lane, L > 0.f ? a / L : 0.f);
      continue;
    }
    float L = P.sinks && lane == 0 ? 1.0f : 0.0f;  // summed over lanes at the end
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int base = s0; base < s1; base += 64) {
      const int n = min(64, s1 - base);
      float m = -INFINITY, l = 0.f;
      if (lane < n) {
        const float2 ml = *reinterpret_cast<const float2*>(P.part_ml + ((int64_t)(base + lane) * P.hq + h) * 2);
        m = ml.x;
        l = ml.y;
      }
      const float Mn = fmaxf(M, wave_max(m));
      const bool missing = m == -INFINITY;  // a split whose pages were all missing: its row is not read
      float f = 0.f;
      if (Mn != -INFINITY) {
        const float r = __builtin_amdgcn_exp2f(M - Mn);
        L *= r;
        a.x *= r; a.y *= r; a.z *= r; a.w *= r;
        M = Mn;
        f = __builtin_amdgcn_exp2f(m - Mn);
        if (!missing) L += f * l;
      }
      const float fx = missing ? -1.0f : f;
      for (int j = 0; j < n; j += U * RW) {
        float4 v[U];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int row = j + u * RW + sub;
          w[u] = __shfl(fx, row & 63, 64);
          const bool use = row < n && w[u] != -1.0f;
          w[u] = use ? w[u] : 0.f;
          v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (use) v[u] = *reinterpret_cast<const float4*>(P.part_acc + ((int64_t)(base + row) * P.hq + h) * D + dim);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          a.x += w[u] * v[u].x; a.y += w[u] * v[u].y; a.z += w[u] * v[u].z; a.w += w[u] * v[u].w;
        }
      }
    }
    L = wave_sum(L);
#pragma unroll
    for (int o = LR; o < 64; o <<= 1) {
      a.x += __shfl_xor(a.x, o, 64);
      a.y += __shfl_xor(a.y, o, 64);
      a.z += __shfl_xor(a.z, o, 64);
      a.w += __shfl_xor(a.w, o, 64);
    }
    if (sub == 0) {
      T* o = reinterpret_cast<T*>(P.o) + ((int64_t)(tb + k * stride) * P.hq + h) * D + dim;
      const float r[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) Elem<T>::store(o, i, L > 0.f ? r[i] / L : 0.f);
    }
  }
}

hipError_t launch_attn_combine(int dtype, int head_dim, const AttnCombine& p, hipStream_t s) {
  if (p.n_tokens == 0) return hipSuccess;
  const int64_t waves = (int64_t)p.n_tokens * p.hq;
  const int64_t per_dec = std::max(1, p.n_tokens / std::max(p.n_dec, 1));
  const int K = (int)std::min<int64_t>({64, (waves + COMBINE_WAVES - 1) / COMBINE_WAVES, per_dec});
  const int stride = (p.n_tokens + K - 1) / K;
  const bool wide = p.max_splits > 4 && (int64_t)p.max_splits * COMBINE_WAVES_PER_SPLIT > (int64_t)p.n_dec * p.hq;
  dim3 grid((unsigned)(((int64_t)stride * p.hq + 3) / 4)), block(256);
#define COMBINE(T, D)                                                                                        \
  do {                                                                                                       \
    if (wide) hipLaunchKernelGGL((attn_combine_kernel<T, D, true>), grid, block, 0, s, p, stride, K);       \
    else hipLaunchKernelGGL((attn_combine_kernel<T, D, false>), grid, block, 0, s, p, stride, K);           \
  } while (0)
  if (dtype == 0) {
    if (head_dim == 32) COMBINE(float, 32);
    else COMBINE(float, 64);
  } else {
    if (head_dim == 32) COMBINE(bf16, 32);
    else COMBINE(bf16, 64);
  }
#undef COMBINE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// prefill: a chunk of new tokens attending causally to its sequence's pages
// ---------------------------------------------------------------------------

// A workgroup of four wavefronts owns QB consecutive new tokens of one
// sequence and one KV head. The matrix-core columns are (token, query head)
// pairs, 64 per wavefront: 64 / G tokens times the G query heads that share
// the KV head. The workgroup walks the pages from the first key any of its
// tokens sees to its last token's page, two pages (32 keys) per step, staged
// through LDS (double buffered) for all four wavefronts. Per step a wavefront
// forms S^T = K Q^T for both pages and its four 16-column tiles, masks keys
// outside each column's causal (and window) range, updates the running
// maximum and normaliser per column, and accumulates O^T += V^T P^T with one
// 16x16x32 product per tile that consumes both pages' scores as they sit in
// the lanes. The sink enters the normaliser at the end.
template <int G>
struct PrefillShape {
  static constexpr int TPW = 64 / G;    // tokens per wavefront
  static constexpr int QB = 4 * TPW;    // tokens per workgroup
};

// Only the groupings with a kernel instance (prefill_impl) report a block
// size; for the others the planner sends every chunk to split-K attention.
int prefill_block_tokens(int group) {
  switch (group) {
    case 4: return PrefillShape<4>::QB;
    case 8: return PrefillShape<8>::QB;
    default: return 0;
  }
}

template <typename T, int D, int G>
__global__ __launch_bounds__(256) void attn_prefill_kernel(AttnPrefill P) {
  using SH = PrefillShape<G>;
  constexpr int PE = PAGE * D;                          // elements of one page of one KV head
  constexpr int CH = 16 / sizeof(T);                    // elements per 16-byte chunk
  constexpr int NCH = 4 * PE / CH;                      // chunks per step (K and V of two pages)
  constexpr int PT = NCH / 256;                         // chunks per thread
  static_assert(NCH % 256 == 0, "a step's pages must split evenly over the workgroup");
  __shared__ __align__(16) T kv[2][4][PE];              // [buffer][K page a, K page b, V pages a and b interleaved]
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = blockIdx.x % P.hkv;
  const int blk = P.n_blocks - 1 - (int)(blockIdx.x / P.hkv);  // latest (heaviest) blocks first
  int lo_b = 0, hi_b = P.batch - 1;                            // sequence: last b with blk_start[b] <= blk
  while (lo_b < hi_b) {
    const int mid = (lo_b + hi_b + 1) >> 1;
    if (P.blk_start[mid] <= blk) lo_b = mid; else hi_b = mid - 1;
  }
  const int b = uniform(lo_b);
  const int q0 = P.cu_q[b], q1 = P.cu_q[b + 1];
  const int t0 = uniform(q0 + (blk - P.blk_start[b]) * SH::QB);
  const int ntok = min(SH::QB, q1 - t0);
  const int p_first = uniform(P.seq_lens[b] + (t0 - q0)), p_last = p_first + ntok - 1;
  const int lo = P.window > 0 ? max(0, p_first - P.window + 1) : 0;
  const int pg_lo = lo / PAGE;
  int n_steps = (p_last / PAGE - pg_lo + 2) / 2;
  if (ntok <= 0 || p_first < 0 || p_last / PAGE >= P.max_pages) {
    if (tid == 0) set_error(P.err, 1);
    n_steps = 0;
  }
  const int32_t* ptab = P.page_table + (int64_t)b * P.max_pages;
  const int64_t page_elems = (int64_t)P.hkv * PE;

  // this lane's column in each of the wavefront's four 16-column tiles
  const int fr = lane & 15, grp = lane >> 4;
  int pos[4], head[4];
  bool valid[4];
  Frag<T> qf[4][D / 32];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = 16 * j + fr;
    const int ti = wave * SH::TPW + c / G;
    valid[j] = ti < ntok;
    pos[j] = p_first + ti;
    head[j] = g * G + c % G;
    const int trow = min(max(t0 + ti, 0), P.n_tokens - 1);  // in range even if the tables disagree
    const T* qp = reinterpret_cast<const T*>(P.q) + ((int64_t)trow * P.hq + head[j]) * D + 8 * grp;
#pragma unroll
    for (int cc = 0; cc < D / 32; ++cc) {
      qf[j][cc].load(qp + 32 * cc);
      qf[j][cc].keep_if(valid[j]);
    }
  }

  // staging: chunk i of a step is piece i / (PE / CH) (K a, K b, V a, V b) at
  // element offset (i % (PE / CH)) * CH; pages past the range repeat the last
  // one and missing pages read page 0 (both masked below)
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  struct Regs {
    u32x4 v[PT];
  };
  // page ids are wave-uniform: read them with scalar loads, whose wait counter
  // is separate from the vector loads kept in flight below
  auto page_id = [&](int step, int which, bool& ok) __attribute__((always_inline)) {
    const int pg = uniform(min(pg_lo + 2 * step + which, p_last / PAGE));
    const int id = load_uniform(ptab, pg);
    ok = id >= 0 && id < P.n_pages;
    return ok ? id : 0;
  };
  auto fetch = [&](Regs& st, int step) __attribute__((always_inline)) {
    step = min(step, max(n_steps - 1, 0));
    bool oka, okb;
    const int ida = page_id(step, 0, oka), idb = page_id(step, 1, okb);
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const int i = tid + 256 * u, piece = i / (PE / CH), off = (i % (PE / CH)) * CH;
      const T* pool = reinterpret_cast<const T*>(piece < 2 ? P.k_pool : P.v_pool);
      const int id = (piece & 1) ? idb : ida;
      st.v[u] = *reinterpret_cast<const u32x4*>(pool + id * page_elems + (int64_t)g * PE + off);
    }
  };
  // K pages keep the page format; the V pages of a step are interleaved in
  // blocks of 256 elements (the 64 lanes' 4-value fragments of one 16-dim
  // tile): [tile n][page a, page b], so the two halves of a PV operand are
  // 512 bytes apart and load as one register quadruple
  auto stage = [&](const Regs& st, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const int i = tid + 256 * u, piece = i / (PE / CH), off = (i % (PE / CH)) * CH;
      T* dst = piece < 2 ? &kv[buf][piece][off] : &kv[buf][2][((off >> 8) * 2 + piece - 2) * 256 + (off & 255)];
      *reinterpret_cast<u32x4*>(dst) = st.v[u];
    }
  };

  // Per column: running maximum m (log2 units) and the accumulators of
  // O^T = V^T P^T, plus a tile against ones that sums the (rounded) weights.
  // The maximum is raised lazily: a step rescales only when some column's
  // scores exceed its m by more than RESCALE (weights then stay below
  // 2^RESCALE); every weight uses the same m as its normaliser, so the result
  // is the same quotient.
  constexpr float RESCALE = 8.0f;
  const float inv_scale = 1.0f / P.scale_log2;
  float m_run[4], m_sub[4], thr[4];
  f32x4 acc[D / 16][4], accl[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    m_run[j] = -INFINITY;
    m_sub[j] = 0.f;
    thr[j] = -INFINITY;
    accl[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  Frag4<T> one;
  ones(one);
  // keys a step may need to mask: past the wave's first token (causal), before
  // its last token's window, or on a missing or out-of-range page
  const int pos_lo_w = p_first + wave * SH::TPW;
  const int pos_hi_w = min(pos_lo_w + SH::TPW - 1, p_last);
  const int pg_last = p_last / PAGE;

  auto compute = [&](int step, int buf) __attribute__((always_inline)) {
    bool ok[2];
    page_id(step, 0, ok[0]);
    page_id(step, 1, ok[1]);
    const int pg0 = pg_lo + 2 * step, k0 = pg0 * PAGE;
    const bool edge = k0 + 2 * PAGE - 1 > pos_lo_w || (P.window > 0 && k0 < pos_hi_w - P.window + 1) ||
                      !ok[0] || !ok[1] || pg0 + 1 > pg_last;
    // scores: sc[pg][j][r] = q(column j) . k(key 4 grp + r of page pg)
    f32x4 sc[2][4];
#pragma unroll
    for (int pg = 0; pg < 2; ++pg) {
      Frag<T> kf[D / 32];
#pragma unroll
      for (int cc = 0; cc < D / 32; ++cc) kf[cc].load(&kv[buf][pg][(64 * cc + lane) * 8]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sc[pg][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < D / 32; ++cc) sc[pg][j] = mma32(kf[cc], qf[j][cc], sc[pg][j]);
      }
    }
    // wave-uniform: mask keys outside each column's range. The empty asm
    // keeps this a branch: if-converted, its compares and selects would run
    // on every step.
    if (__builtin_expect(edge, 0)) {
      asm volatile("");
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int hi = pos[j], lo_c = P.window > 0 ? pos[j] - P.window + 1 : 0;
#pragma unroll
        for (int pg = 0; pg < 2; ++pg)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int kp = k0 + pg * PAGE + 4 * grp + r;
            const bool in = ok[pg] && pg0 + pg <= pg_last && kp >= lo_c && kp <= hi;
            sc[pg][j][r] = in ? sc[pg][j][r] : -INFINITY;
          }
      }
    }
    // Each lane takes the largest of its 8 raw scores per column; the step
    // rescales only when one of them exceeds the column's threshold
    // (m + RESCALE in raw score units), and only then forms the column
    // maximum across the four row groups.
    float mloc[4];
    bool raise = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      mloc[j] = vmax(vmax(vmax(sc[0][j][0], sc[0][j][1]), vmax(sc[0][j][2], sc[0][j][3])),
                     vmax(vmax(sc[1][j][0], sc[1][j][1]), vmax(sc[1][j][2], sc[1][j][3])));
      raise = raise || mloc[j] > thr[j];
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {  // wave-uniform rescale (kept a branch)
      asm volatile("");
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float mstep = max_over_rows(mloc[j]) * P.scale_log2;
        const float m_new = fmaxf(m_run[j], mstep);
        const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run[j] - m_new);
        accl[j] *= alpha;
#pragma unroll
        for (int n = 0; n < D / 16; ++n) acc[n][j] *= alpha;
        m_run[j] = m_new;
        m_sub[j] = m_new == -INFINITY ? 0.f : m_new;  // masked scores give 2^-inf = 0
        thr[j] = (m_new + RESCALE) * inv_scale;
      }
    }
    PVFrag<T> vf[D / 16];
#pragma unroll
    for (int n = 0; n < D / 16; ++n) vf[n].load(&kv[buf][2][2 * n * 256 + lane * 4], &kv[buf][2][(2 * n + 1) * 256 + lane * 4]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float msub = m_sub[j];
      float pa[4], pb[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pa[r] = __builtin_amdgcn_exp2f(fmaf(sc[0][j][r], P.scale_log2, -msub));
        pb[r] = __builtin_amdgcn_exp2f(fmaf(sc[1][j][r], P.scale_log2, -msub));
      }
      accl[j] = mma32_pv(one, one, pa, pb, accl[j]);
#pragma unroll
      for (int n = 0; n < D / 16; ++n) acc[n][j] = mma32_pv(vf[n], pa, pb, acc[n][j]);
    }
  };

  // Step j's pages are loaded into register set j % R and staged into LDS
  // buffer j & 1: while step s is computed, steps s + 1 .. s + R are in flight
  // (L2 latency exceeds one step's products). The loop is unrolled R times so
  // set indices are constants; only the products are conditional (loads past
  // the last step are clamped and their staged copies never read).
  constexpr int R = 4;
  if (n_steps > 0) {
    Regs rs[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      fetch(rs[u], u);
      __builtin_amdgcn_sched_barrier(0);
    }
    stage(rs[0], 0);
    fetch(rs[0], R);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    for (int step = 0; step < n_steps; step += R) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        if (step + u < n_steps) compute(step + u, u & 1);
        __builtin_amdgcn_sched_barrier(0);
        stage(rs[(u + 1) % R], (u + 1) & 1);
        fetch(rs[(u + 1) % R], step + u + 1 + R);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      }
    }
  }

  // normalise with the sink and store this lane's 4 dims of each column
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float l_tot = accl[j][0];  // every row of the ones tile holds the column's sum
    float M = m_run[j], scale = 1.0f;
    if (P.sinks) {
      const float sk = P.sinks[head[j]] * LOG2E;
      const float Mt = fmaxf(M, sk);
      const float f = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mt);
      l_tot = l_tot * f + __builtin_amdgcn_exp2f(sk - Mt);
      scale = f;
    }
    const float inv = l_tot > 0.f ? scale / l_tot : 0.f;
    if (valid[j]) {
      T* o = reinterpret_cast<T*>(P.o) + ((int64_t)(t0 + wave * SH::TPW + (16 * j + fr) / G) * P.hq + head[j]) * D +
             4 * grp;
#pragma unroll
      for (int n = 0; n < D / 16; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) Elem<T>::store(o, 16 * n + r, acc[n][j][r] * inv);
    }
  }
}

// bf16, head dim 64: the same split of the work, on 32 x 32 x 16 products. Per
// step (two pages, 32 keys) a wavefront forms S^T = K Q^T as one 32 x 32 tile
// per 32 columns and O^T += V^T P^T from it. A product of this size keeps the
// matrix cores busy for 32 cycles and the vector pipe for one issue slot, so
// the softmax of one wavefront runs beside the products of the other on its
// SIMD (and beside its own: the scores of step s + 1 are formed ahead of the
// softmax of step s); the 16 x 16 tiles of the kernel above block the pipe
// twice as often and need four cross-lane maxima where this needs two.
//
// Lane l of a score tile holds column l % 32 and, with h = l / 32, the keys
// 8 q + 4 h + r (q, r < 4; element 4 q + r). The value product of page p takes
// its eight k-slots 4 (q % 2) + r straight from elements q / 2 == p, and its
// other operand, the value rows 8 (q % 2) + 4 h + r of one dim, is two 8-byte
// pieces of the page format 256 bytes apart: one two-address LDS read. Row
// sums are dot products of the packed weights with ones.
//
// Pages go straight to LDS (wavefront 0: K of the first page, 1: of the second,
// 2 and 3: their V) through PRS stages; the 16-byte pieces of V are permuted
// on the way (128-byte block b of a 512-byte dim tile to b ^ (tile & 1)) so
// that the lanes of a half tile read all banks.
//
// The maximum of a column is raised only when a lane's share of a step's
// weights would pass 2^8 (WEIGHT_LIMIT, the bound of a single weight in the
// kernel above): the accumulators keep fp32's headroom for values up to 2^108
// and more, and the largest weights are near one, where they are 1 exactly
// whenever the maximum was just raised. A limit of 2^40 was no faster, lost
// values beyond 2^75 to infinity and doubled the squared error of columns whose
// first visible keys score low.
//
// Bound: the vector pipe, about 126 instructions per wavefront and step (the 64
// x 32 exponentials cost two slots each; counted 6.9 per product, the matrix cores
// 47% busy). Measured against the 16 x 16 tiles,
// 64 query heads on 8 KV heads: twelve chunks (32 K tokens) behind up
// to 24 K keys 10.36 -> 8.27 ms, six chunks (1.8 K tokens) behind up to 16 K
// 383 -> 273 us.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* lds_void_t;
constexpr int PRS = 6;  // LDS stages of two pages' K and V (8 KB)

template <int G>
__global__ __launch_bounds__(256) void attn_prefill_wide_kernel(AttnPrefill P) {
  using SH = PrefillShape<G>;
  constexpr int D = 64, PE = PAGE * D, PB = 2 * PE;  // page elements and bytes of one KV head
  __shared__ __align__(1024) uint8_t s0[4 * PB];
  __shared__ __align__(1024) uint8_t s1[4 * PB];
  __shared__ __align__(1024) uint8_t s2[4 * PB];
  __shared__ __align__(1024) uint8_t s3[4 * PB];
  __shared__ __align__(1024) uint8_t s4[4 * PB];
  __shared__ __align__(1024) uint8_t s5[4 * PB];
  auto stage_of = [&](int s) __attribute__((always_inline)) {
    return s == 0 ? s0 : s == 1 ? s1 : s == 2 ? s2 : s == 3 ? s3 : s == 4 ? s4 : s5;
  };
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = blockIdx.x % P.hkv;
  const int blk = P.n_blocks - 1 - (int)(blockIdx.x / P.hkv);  // latest (heaviest) blocks first
  int lo_b = 0, hi_b = P.batch - 1;                            // sequence: last b with blk_start[b] <= blk
  while (lo_b < hi_b) {
    const int mid = (lo_b + hi_b + 1) >> 1;
    if (P.blk_start[mid] <= blk) lo_b = mid; else hi_b = mid - 1;
  }
  const int b = uniform(lo_b);
  const int q0 = P.cu_q[b], q1 = P.cu_q[b + 1];
  const int t0 = uniform(q0 + (blk - P.blk_start[b]) * SH::QB);
  const int ntok = min(SH::QB, q1 - t0);
  const int p_first = uniform(P.seq_lens[b] + (t0 - q0)), p_last = p_first + ntok - 1;
  const int lo = P.window > 0 ? max(0, p_first - P.window + 1) : 0;
  const int pg_lo = lo / PAGE, pg_last = p_last / PAGE;
  int n_steps = uniform((pg_last - pg_lo + 2) / 2);
  if (ntok <= 0 || p_first < 0 || pg_last >= P.max_pages) {
    if (tid == 0) set_error(P.err, 1);
    n_steps = 0;
  }
  const int32_t* ptab = P.page_table + (int64_t)b * P.max_pages;

  // this lane's column in each of the wavefront's two 32-column tiles
  const int fc = lane & 31, h = lane >> 5;
  int pos[2], head[2];
  bool valid[2];
  Frag<bf16> qf[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = 32 * j + fc, ti = wave * SH::TPW + c / G;
    valid[j] = ti < ntok;
    pos[j] = p_first + ti;
    head[j] = g * G + c % G;
    const int trow = min(max(t0 + ti, 0), P.n_tokens - 1);  // in range even if the tables disagree
    const bf16* qp = reinterpret_cast<const bf16*>(P.q) + ((int64_t)trow * P.hq + head[j]) * D + 8 * h;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      qf[j][cc].load(qp + 16 * cc);
      qf[j][cc].keep_if(valid[j]);
    }
  }

  // page ids of steps base .. base + 31, lane i: page pg_lo + 2 base + i (the
  // last page past the range). A block of IDB steps and the requests ahead of it
  // find their ids in one register; the next block's are loaded a block ahead.
  constexpr int IDB = 4 * PRS;
  static_assert(IDB + PRS - 1 <= 32, "a block's ids and those requested ahead of it");
  auto ids_of = [&](int base) __attribute__((always_inline)) {
    return n_steps > 0 ? ptab[min(pg_lo + 2 * base + lane, pg_last)] : 0;
  };
  int ids = ids_of(0), base = 0;
  const int step_bytes = P.hkv * PB;  // bytes of a page in one pool (below 2^31: hkv * 2 KB)
  const uint8_t* pool = reinterpret_cast<const uint8_t*>(wave < 2 ? P.k_pool : P.v_pool) + (int64_t)g * PB;
  // the wavefront's piece of a step: 2 KB, lane l of load u at byte 1024 u + 16 l
  uint32_t vo[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t at = 1024u * u + 16u * lane;
    vo[u] = wave < 2 ? at : at ^ (((at >> 9) & 1u) << 7);
  }
  // a page's id, or 0 with good = false where the table has none
  auto page_of = [&](int step, int which, bool& good) __attribute__((always_inline)) {
    const int id = __builtin_amdgcn_readlane(ids, 2 * (step - base) + which);
    good = id >= 0 && id < P.n_pages;
    return good ? id : 0;
  };
  // request a step's pages (past the end: the last page again, not used)
  auto request = [&](uint8_t* stg, int step) __attribute__((always_inline)) {
    bool good;
    const int id = page_of(step, wave & 1, good);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(pool) + (int64_t)id * step_bytes, 0, PB, 0x00020000);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t)(stg + wave * PB + 1024 * u), 16, vo[u], 0, 0, 0);
  };

  constexpr float WEIGHT_LIMIT = 0x1p8f;  // of a lane's 16 weights in a step
  float m_run[2], m_sub[2], limit[2], l[2];  // limit: -inf until a key is visible
  f32x16 acc[2][2];  // [dim tile][column tile]
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    m_run[j] = -INFINITY;
    m_sub[j] = 0.f;
    limit[j] = -INFINITY;
    l[j] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[dt][j][e] = 0.f;
  }
  const int pos_lo_w = p_first + wave * SH::TPW;
  const int pos_hi_w = min(pos_lo_w + SH::TPW - 1, p_last);
  // fragment addresses: key fc of the step (page fc / 16), dims 8 h .. of a
  // 16-dim chunk; dim fc of a tile of 32, value rows 4 h .. and 8 + 4 h ..
  const uint32_t ko = (fc >> 4) * PB + ((h * 16 + (fc & 15)) * 16);
  const uint32_t vbase = (fc >> 4) * 512 + (fc & 15) * 8 + (((uint32_t)h ^ ((fc >> 4) & 1)) << 7);

  struct Scores {
    f32x16 t[2];
  };
  auto load_keys = [&](u32x4_t (&kf)[4], const uint8_t* stg) __attribute__((always_inline)) {
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) kf[cc] = *reinterpret_cast<const u32x4_t*>(stg + ko + 512 * cc);
  };
  auto scores = [&](Scores& sc, const u32x4_t (&kf)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) sc.t[j][e] = 0.f;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        sc.t[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf[cc]),
                                                          __builtin_bit_cast(bf16x8_t, qf[j][cc].v), sc.t[j], 0, 0, 0);
  };
  // step's softmax and value products from its scores, and the scores of the next step
  auto attend = [&](Scores& sc, Scores& sn, const uint8_t* stg, const uint8_t* nxt, int step) __attribute__((always_inline)) {
    u32x4_t kf[4];
    load_keys(kf, nxt);
    bool ok[2];
    page_of(step, 0, ok[0]);
    page_of(step, 1, ok[1]);
    const int pg0 = pg_lo + 2 * step, k0 = pg0 * PAGE;
    const bool edge = k0 + 2 * PAGE - 1 > pos_lo_w || (P.window > 0 && k0 < pos_hi_w - P.window + 1) ||
                      !ok[0] || !ok[1] || pg0 + 1 > pg_last;
    if (__builtin_expect(edge, 0)) {  // wave-uniform; the empty asm keeps it a branch
      asm volatile("");
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int hi = pos[j], lo_c = P.window > 0 ? pos[j] - P.window + 1 : 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int kp = k0 + 8 * (e >> 2) + 4 * h + (e & 3), pg = e >> 3;
          const bool in = ok[pg] && pg0 + pg <= pg_last && kp >= lo_c && kp <= hi;
          sc.t[j][e] = in ? sc.t[j][e] : -INFINITY;
        }
      }
    }
    u32x4_t pw[2][2];  // [column tile][page]: the weights, packed
    float sum[2];
    auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sum[j] = 0.f;
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sc.t[j][e], P.scale_log2, -m_sub[j]));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sc.t[j][e + 1], P.scale_log2, -m_sub[j]));
          const uint32_t w = pack_bf16(p0, p1);
          pw[j][e >> 3][(e & 7) >> 1] = w;
          sum[j] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w), __builtin_bit_cast(bf16x2_t, 0x3F803F80u), sum[j], false);
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    scores(sn, kf);
    weights();
    // the next scores' eight products among the 96 vector instructions of the weights
#define PF_MIX                                        \
  __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  \
  __builtin_amdgcn_sched_group_barrier(0x402, 12, 0);
    PF_MIX PF_MIX PF_MIX PF_MIX PF_MIX PF_MIX PF_MIX PF_MIX
#undef PF_MIX
    // The maximum only has to keep the weights in range (bf16 and fp32 are
    // relative), so it is raised when a step's sum says that they are not, and
    // until a column has seen a key; the weights are then formed again.
    const bool raise = sum[0] > limit[0] || sum[1] > limit[1];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {  // wave-uniform (kept a branch)
      asm volatile("");
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float mloc = sc.t[j][0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mloc = vmax(mloc, sc.t[j][e]);
        const uint32_t u = __float_as_uint(mloc);
        auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        const float mstep = vmax(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * P.scale_log2;
        const float m_new = fmaxf(m_run[j], mstep);
        const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run[j] - m_new);
        l[j] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) acc[dt][j] *= alpha;
        m_run[j] = m_new;
        m_sub[j] = m_new == -INFINITY ? 0.f : m_new;  // masked scores give 2^-inf = 0
        limit[j] = m_new == -INFINITY ? -INFINITY : WEIGHT_LIMIT;
      }
      weights();
    }
    u32x4_t vf[2][2];  // [page][dim tile]
#pragma unroll
    for (int pg = 0; pg < 2; ++pg)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const uint8_t* v = stg + (2 + pg) * PB + 1024 * dt + vbase;
        const u32x2_t a = *reinterpret_cast<const u32x2_t*>(v), c = *reinterpret_cast<const u32x2_t*>(v + 256);
        vf[pg][dt] = __builtin_shufflevector(a, c, 0, 1, 2, 3);
      }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      l[j] += sum[j];
#pragma unroll
      for (int pg = 0; pg < 2; ++pg)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          acc[dt][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vf[pg][dt]),
                                                               __builtin_bit_cast(bf16x8_t, pw[j][pg]), acc[dt][j], 0, 0, 0);
    }
  };

  // Step s sits in stage s % PRS. In step s its scores are there already; step
  // s + PRS - 1 is requested into the stage step s - 1 left, the scores of step
  // s + 1 are formed, and before the barrier a wavefront waits for its loads of
  // step s + 2.
  if (n_steps > 0) {
    auto publish = [&]() __attribute__((always_inline)) {
      constexpr int N = 2 * (PRS - 3);
      // the barrier hands the stages over: this wavefront's reads of the step's
      // stage have returned (lgkmcnt), its loads of step s + 2 have landed, and
      // the empty asm keeps LDS accesses on their side of it (to the compiler
      // the barrier itself touches no memory)
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(N | (7 << 4));  // vmcnt(N) expcnt(7) lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int s = 0; s < PRS - 1; ++s) {
      request(stage_of(s), s);
      __builtin_amdgcn_sched_barrier(0);
    }
    publish();
    Scores sc[2];
    {
      u32x4_t kf[4];
      load_keys(kf, s0);
      scores(sc[0], kf);
    }
    auto one = [&](auto U_, int step) __attribute__((always_inline)) {
      constexpr int U = decltype(U_)::value;
      if (step < n_steps) {  // uniform
        request(stage_of((U + PRS - 1) % PRS), step + PRS - 1);
        attend(sc[U % 2], sc[(U + 1) % 2], stage_of(U), stage_of((U + 1) % PRS), step);
      }
      publish();
    };
    while (true) {
      const int ids_next = ids_of(base + IDB), stop = min(n_steps, base + IDB);
      for (int step = base; step < stop; step += PRS) {
        one(std::integral_constant<int, 0>{}, step);
        one(std::integral_constant<int, 1>{}, step + 1);
        one(std::integral_constant<int, 2>{}, step + 2);
        one(std::integral_constant<int, 3>{}, step + 3);
        one(std::integral_constant<int, 4>{}, step + 4);
        one(std::integral_constant<int, 5>{}, step + 5);
      }
      if (stop == n_steps) break;
      base = stop;
      ids = ids_next;
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // no load into LDS may outlive the workgroup

  // normalise with the sink and store this lane's dims 32 dt + 8 q + 4 h .. + 3 of each column
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t u = __float_as_uint(l[j]);
    auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    float l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    float M = m_run[j], scale = 1.0f;
    if (P.sinks) {
      const float sk = P.sinks[head[j]] * LOG2E;
      const float Mt = fmaxf(M, sk);
      const float f = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mt);
      l_tot = l_tot * f + __builtin_amdgcn_exp2f(sk - Mt);
      scale = f;
    }
    const float inv = l_tot > 0.f ? scale / l_tot : 0.f;
    if (valid[j]) {
      bf16* o = reinterpret_cast<bf16*>(P.o) + ((int64_t)(t0 + wave * SH::TPW + (32 * j + fc) / G) * P.hq + head[j]) * D + 4 * h;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          store4(o + 32 * dt + 8 * q, make_float4(acc[dt][j][4 * q] * inv, acc[dt][j][4 * q + 1] * inv,
                                                  acc[dt][j][4 * q + 2] * inv, acc[dt][j][4 * q + 3] * inv));
    }
  }
}

template <typename T, int D>
static hipError_t prefill_impl(int group, const AttnPrefill& p, hipStream_t s) {
  dim3 grid((unsigned)(p.n_blocks * p.hkv)), block(256);
  // bf16 with head dim 64 takes the wide products (figures at the kernel);
  // float has no such tile, and only the smallest configuration has head dim 32.
  // Its pages go to LDS by 16-byte direct loads, which are used on 16-byte
  // aligned pools only.
  if constexpr (sizeof(T) == 2 && D == 64) {
    if ((uintptr_t)p.k_pool % 16 == 0 && (uintptr_t)p.v_pool % 16 == 0) {
      switch (group) {
        case 4: hipLaunchKernelGGL(attn_prefill_wide_kernel<4>, grid, block, 0, s, p); break;
        case 8: hipLaunchKernelGGL(attn_prefill_wide_kernel<8>, grid, block, 0, s, p); break;
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
  }
  switch (group) {
    case 4: hipLaunchKernelGGL((attn_prefill_kernel<T, D, 4>), grid, block, 0, s, p); break;
    case 8: hipLaunchKernelGGL((attn_prefill_kernel<T, D, 8>), grid, block, 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_attn_prefill(int dtype, int head_dim, int group, const AttnPrefill& p, hipStream_t s) {
  if (p.n_blocks == 0) return hipSuccess;
  if (dtype == 0) return head_dim == 32 ? prefill_impl<float, 32>(group, p, s) : prefill_impl<float, 64>(group, p, s);
  return head_dim == 32 ? prefill_impl<bf16, 32>(group, p, s) : prefill_impl<bf16, 64>(group, p, s);
}

// ---------------------------------------------------------------------------
// KV append: copy new keys / values into their pages, bit for bit
// ---------------------------------------------------------------------------

template <typename T, int D>
__global__ __launch_bounds__(256) void kv_append_kernel(KvAppend P) {
  const int t = blockIdx.x;
  const int b = P.cu_q ? seq_of_token(P.cu_q, P.batch, t) : t;
  const int pos = P.seq_lens[b] + (P.cu_q ? t - P.cu_q[b] : 0);
  const int lp = pos >= 0 ? pos / PAGE : -1;
  int page = (lp >= 0 && lp < P.max_pages) ? P.page_table[(int64_t)b * P.max_pages + lp] : -1;
  if (page < 0 || page >= P.n_pages) {
    if (threadIdx.x == 0) set_error(P.err, 1);
    return;
  }
  const int slot = pos % PAGE;
  const T* kn = reinterpret_cast<const T*>(P.k_new) + (int64_t)t * P.hkv * D;
  const T* vn = reinterpret_cast<const T*>(P.v_new) + (int64_t)t * P.hkv * D;
  T* kp = reinterpret_cast<T*>(P.k_pool) + (int64_t)page * P.hkv * PAGE * D;
  T* vp = reinterpret_cast<T*>(P.v_pool) + (int64_t)page * P.hkv * PAGE * D;
  for (int e = threadIdx.x; e < P.hkv * D; e += blockDim.x) {
    const int g = e / D, i = e - g * D;
    kp[(int64_t)g * PAGE * D + k_off(slot, i)] = kn[e];
    vp[(int64_t)g * PAGE * D + v_off(slot, i)] = vn[e];
  }
}

hipError_t launch_kv_append(int dtype, int head_dim, const KvAppend& p, hipStream_t s) {
  if (p.n_tokens == 0) return hipSuccess;
  dim3 grid(p.n_tokens), block(256);
  if (dtype == 0) {
    if (head_dim == 32) hipLaunchKernelGGL((kv_append_kernel<float, 32>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((kv_append_kernel<float, 64>), grid, block, 0, s, p);
  } else {
    if (head_dim == 32) hipLaunchKernelGGL((kv_append_kernel<bf16, 32>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((kv_append_kernel<bf16, 64>), grid, block, 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace mcpu
