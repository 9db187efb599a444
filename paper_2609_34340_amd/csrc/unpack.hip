// Receive side of the Sec. 5 buffer layout, and the combine direction.
//
// A receive buffer holds the slices addressed to one rank in step order, one
// token row per slot whose stride is the row rounded up to 128 bytes (Sec. 5
// low-latency protocol: every row starts 128-byte aligned).  The dispatch
// receive is unpacked into the expert-major output: local expert m's rows from
// source 0, then source 1, ..., each source's rows in token order, which is
// the order of the stream from that source (Sec. 5: the receive kernel writes
// the output layout directly).  The combine returns every row to its source
// rank with a schedule planned on the transposed demand (the return AlltoAllv
// of expert parallelism); its pack reads the expert-major rows in stream
// order and its unpack puts every returned row at (token, routing slot).
//
// Kernels
//   map    one workgroup per step.  It takes the lane that moves rows to (or
//          from) this rank at its step, sums the volumes of this rank's
//          earlier steps (where the slice sits in the receive or send buffer)
//          and of its earlier steps with the same peer (where it sits in that
//          stream), and writes, for every row of the slice, the row index on
//          the other side: an expert-major output row, or token * k + slot.
//          The workgroup of the last step also checks that every peer's
//          stream is covered exactly.
//   copy   one workgroup per buffer row, each XCD a contiguous eighth of
//          the rows: 16-byte loads issued a pass at a time ahead of the
//          non-temporal stores.
//   transpose  D^T for the combine's plan, in 32 x 32 LDS tiles.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "divide.h"
#include "internal.h"

namespace vp {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

__device__ inline void report(int32_t* status, int code) { atomicCAS(status, 0, code); }

constexpr int kMapThreads = 512;
constexpr int kMapWaves = kMapThreads / 64;
constexpr int kMapRows = 4;   // rows of a slice that a thread has in flight

struct MapArgs {
  int mode, self, N, k_max, eloc, E, k;
  int64_t rb, T;
  int64_t rows_cap;   // rows the buffer side holds (receive slots, or send rows)
  int64_t map_cap;    // rows the other side holds (expert-major output, or T * k)
  const int32_t *Kp, *dst, *recv_src;
  const int64_t* bytes;
  const int32_t* counts;        // [N][E] dispatch assignments per (source rank, expert)
  const int32_t* sorted_tok;
  const uint8_t* sorted_slot;
  const int64_t* dest_off;
  int64_t* step_off;            // pack combine: [k_max + 1]
  int32_t* map;                 // [rows_cap]
  int64_t* total;               // rows in the buffer
  int32_t* status;
};

// Sums of two values over the block; every thread gets them.
__device__ void block_sum2(int64_t& u, int64_t& v, int64_t (*red)[2]) {
  for (int o = 32; o > 0; o >>= 1) {
    u += __shfl_xor(u, o);
    v += __shfl_xor(v, o);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = u;
    red[threadIdx.x >> 6][1] = v;
  }
  __syncthreads();
  u = v = 0;
  for (int i = 0; i < kMapWaves; ++i) {
    u += red[i][0];
    v += red[i][1];
  }
}

// Exclusive scan of v[0, n) in LDS by the whole block; returns the total.
__device__ int64_t block_excl_scan(int64_t* v, int n, int64_t* red) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int per = (n + kMapThreads - 1) / kMapThreads;
  const int b = min(tid * per, n), e = min(b + per, n);
  int64_t s = 0;
  for (int i = b; i < e; ++i) s += v[i];
  int64_t incl = s;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  __syncthreads();
  if (lane == 63) red[w] = incl;
  __syncthreads();
  int64_t run = incl - s, total = 0;
  for (int i = 0; i < kMapWaves; ++i) {
    if (i < w) run += red[i];
    total += red[i];
  }
  for (int i = b; i < e; ++i) {
    const int64_t t = v[i];
    v[i] = run;
    run += t;
  }
  __syncthreads();
  return total;
}

// Bound by latency, a chain of dependent loads: the lanes of this rank in this
// and the earlier steps, then their volumes, then the rows.  The first round
// of every load is issued before anything is waited for (the schedule arrays
// have k_max rows, so also before K is known; indexes taken from them are
// clamped and the results masked), volumes are divided in floating point, and
// the experts of one rank are scanned by one wavefront.  16 ranks, 49 steps,
// up to 117,000 rows: 16.0 us with one load waited for at a time, 9.7 us now.
__global__ void __launch_bounds__(kMapThreads) map_kernel(MapArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int64_t red2[kMapWaves][2], red[kMapWaves];
  __shared__ int32_t sK, sst;
  const int k = blockIdx.x, tid = threadIdx.x, N = a.N, self = a.self, eloc = a.eloc;
  const bool recv = a.mode != kModeCombinePack, experts = a.mode != kModeCombineUnpack;
  if (tid == 0) {   // one read, so that every early exit below is taken by the whole block
    sK = *a.Kp;
    sst = *a.status;
  }
  int64_t* tot = (int64_t*)smem;   // [N] rows per peer (last step only)
  // expert-major output: expert m's rows start at base[m] = rows of experts
  // before m from every source + rows of m from sources before the peer; the
  // peer's stream holds its rows for expert m from cum[m] on
  int64_t* base = tot + N;         // [eloc]
  int64_t* part = base + eloc;     // [eloc]
  int64_t* cum = part + eloc;      // [eloc + 1]
  // this step's lane and the one of step tid: the rank whose lane lands here,
  // or this rank's destination
  const int32_t* lanes = recv ? a.recv_src : a.dst;
  const int kt = min(tid, a.k_max - 1);
  const int lane_raw = lanes[(size_t)k * N + self], lane_t = lanes[(size_t)kt * N + self];
  const int n_cnt = experts ? N * eloc : 0;
  int32_t cnt0 = 0;   // the first round of the counts of this rank's experts
  if (tid < n_cnt) cnt0 = a.counts[(size_t)(tid / eloc) * a.E + (size_t)self * eloc + tid % eloc];
  for (int j = tid; j < N; j += kMapThreads) tot[j] = 0;
  if (experts)
    for (int m = tid; m < eloc; m += kMapThreads) base[m] = part[m] = 0;
  // 1. this step: the lane carrying rows to or from this rank, and its peer
  bool ok = lane_raw >= 0 && lane_raw < N;
  const int peer = ok ? lane_raw : 0, src = recv ? peer : self;
  const int64_t x = a.bytes[(size_t)k * N + src];
  const int back = a.dst[(size_t)k * N + src];
  const int peer_t = lane_t >= 0 && lane_t < N ? lane_t : 0, src_t = recv ? peer_t : self;
  const int64_t x_t = a.bytes[(size_t)kt * N + src_t];
  const int back_t = a.dst[(size_t)kt * N + src_t];
  __syncthreads();
  const int K = sK;
  if (K < 0 || K > a.k_max) {
    if (k == 0 && tid == 0) report(a.status, VP_ERR_INVALID_ARGUMENT);
    return;
  }
  if (sst != 0) return;
  if (k >= K) {
    if (k == 0 && tid == 0) {   // an empty schedule moves nothing
      *a.total = 0;
      if (a.step_off) a.step_off[0] = 0;
    }
    return;
  }
  ok = ok && (!recv || back == self) && x >= 0 && (x == 0 || peer != self);
  const int64_t nu = ok ? exact_div(x, a.rb) : 0;
  if (!ok || nu * a.rb != x) {
    if (tid == 0) report(a.status, VP_ERR_INVALID_ARGUMENT);
    return;
  }

  // 2. rows of this rank's earlier steps, in total and with the same peer;
  //    the last step's workgroup also counts every peer's rows.  A lane that
  //    does not match the schedule, or not whole rows, is reported by its
  //    step's own workgroup and left out here.
  const bool last = k == K - 1;
  int64_t g0 = 0, q0 = 0;
  const int kend = last ? K : k;
  auto earlier = [&](int kk, int lane_kk, int p, int64_t xx, int bk) {
    if (lane_kk < 0 || lane_kk >= N || (recv && bk != self)) return;
    const int64_t rows = exact_div(xx, a.rb);
    if (kk < k) {
      g0 += rows;
      if (p == peer) q0 += rows;
    }
    if (last && xx > 0) atomicAdd((unsigned long long*)&tot[p], (unsigned long long)rows);
  };
  if (tid < kend) earlier(tid, lane_t, peer_t, x_t, back_t);
  for (int kk = tid + kMapThreads; kk < kend; kk += kMapThreads) {
    const int l = lanes[(size_t)kk * N + self], p = l >= 0 && l < N ? l : 0, s = recv ? p : self;
    earlier(kk, l, p, a.bytes[(size_t)kk * N + s], a.dst[(size_t)kk * N + s]);
  }
  // 3. last step: every peer's stream must be delivered whole -- the rows of
  //    the peer's assignments to this rank's experts (dispatch receive, and the
  //    same rows sent back by the combine), or this rank's rows for that peer
  //    (combine receive).  And the expert totals.
  for (int idx = tid; idx < n_cnt; idx += kMapThreads) {
    const int i = idx / eloc, m = idx - i * eloc;
    const int64_t c = idx == tid ? cnt0 : a.counts[(size_t)i * a.E + (size_t)self * eloc + m];
    if (last && i != self) atomicAdd((unsigned long long*)&tot[i], (unsigned long long)-c);
    atomicAdd((unsigned long long*)&base[m], (unsigned long long)c);
    if (i < peer) atomicAdd((unsigned long long*)&part[m], (unsigned long long)c);
    if (i == peer) cum[m] = c;
  }
  if (last && !experts)
    for (int p = tid; p < N; p += kMapThreads)
      if (p != self)
        atomicAdd((unsigned long long*)&tot[p], (unsigned long long)-(a.dest_off[p + 1] - a.dest_off[p]));
  int64_t b0 = 0, len = 0;   // combine receive: the peer's rows in the sorted lists
  if (!experts) {
    b0 = a.dest_off[peer];
    len = a.dest_off[peer + 1] - b0;
  }
  block_sum2(g0, q0, red2);
  if (tid == 0) {
    if (a.step_off) a.step_off[k] = g0 * a.rb;
    if (last) {
      *a.total = g0 + nu;
      if (a.step_off) a.step_off[K] = g0 * a.rb + x;
    }
  }
  if (last)
    for (int p = tid; p < N; p += kMapThreads)
      if (tot[p] != 0) report(a.status, VP_ERR_INVALID_ARGUMENT);
  if (g0 < 0 || q0 < 0 || g0 > a.rows_cap || nu > a.rows_cap - g0) {
    if (tid == 0) report(a.status, g0 < 0 || q0 < 0 ? VP_ERR_INVALID_ARGUMENT : VP_ERR_CAPACITY);
    return;
  }
  if (nu == 0) return;

  // 4. the row on the other side of every row of this slice
  if (!experts) {
    if (b0 < 0 || len < 0 || b0 > a.map_cap || len > a.map_cap - b0 || q0 > len || nu > len - q0) {
      if (tid == 0) report(a.status, VP_ERR_INVALID_ARGUMENT);   // sorted lists hold T * k entries
      return;
    }
    const int32_t* tok = a.sorted_tok + b0 + q0;
    const uint8_t* slot = a.sorted_slot + b0 + q0;
    for (int64_t u0 = tid; u0 < nu; u0 += kMapRows * kMapThreads) {
      int32_t t[kMapRows];
      int c[kMapRows];
#pragma unroll
      for (int m = 0; m < kMapRows; ++m) {
        const int64_t u = min(u0 + m * kMapThreads, nu - 1);
        t[m] = tok[u];
        c[m] = slot[u];
      }
#pragma unroll
      for (int m = 0; m < kMapRows; ++m) {
        const int64_t u = u0 + m * kMapThreads;
        if (u >= nu) break;
        if (t[m] < 0 || t[m] >= a.T || c[m] >= a.k) report(a.status, VP_ERR_INVALID_ARGUMENT);
        else a.map[g0 + u] = (int32_t)((int64_t)t[m] * a.k + c[m]);
      }
    }
    return;
  }
  int64_t out_rows, stream_rows;
  if (eloc <= 64) {   // both scans in every wavefront; the first one leaves them in LDS
    const int lane = tid & 63;
    const int64_t bv = lane < eloc ? base[lane] : 0, cv = lane < eloc ? cum[lane] : 0;
    int64_t bi = bv, ci = cv;
    for (int o = 1; o < eloc; o <<= 1) {
      const int64_t by = __shfl_up(bi, o), cy = __shfl_up(ci, o);
      if (lane >= o) {
        bi += by;
        ci += cy;
      }
    }
    out_rows = __shfl(bi, eloc - 1);
    stream_rows = __shfl(ci, eloc - 1);
    __syncthreads();
    if (tid < eloc) {
      base[tid] = bi - bv;
      cum[tid] = ci - cv;
    }
    __syncthreads();
  } else {
    out_rows = block_excl_scan(base, eloc, red);
    stream_rows = block_excl_scan(cum, eloc, red);
  }
  if (q0 > stream_rows || nu > stream_rows - q0 || out_rows > a.map_cap) {
    if (tid == 0)
      report(a.status, out_rows > a.map_cap && !(q0 > stream_rows || nu > stream_rows - q0) ? VP_ERR_CAPACITY
                                                                                            : VP_ERR_INVALID_ARGUMENT);
    return;
  }
  for (int64_t u = tid; u < nu; u += kMapThreads) {
    const int64_t q = q0 + u;
    int lo = 0, hi = eloc - 1;   // the last expert whose rows start at or before q
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cum[mid] <= q) lo = mid;
      else hi = mid - 1;
    }
    const int64_t row = base[lo] + part[lo] + (q - cum[lo]);
    if (row < 0 || row >= a.map_cap) {
      report(a.status, VP_ERR_INVALID_ARGUMENT);
      continue;
    }
    a.map[g0 + u] = (int32_t)row;
  }
}

// Buffer row g <-> mapped row map[g]: read from the mapped side (map_src) or
// write to it.  Rows are whole 16-byte vectors.  One workgroup per row; TH
// threads move it in passes of V vectors per thread, every load of a pass
// issued before its stores (about 2 KiB in flight per wavefront, as for the
// dispatch scatter).
template <int TH, int V>
__global__ void __launch_bounds__(TH) copy_rows_kernel(const unsigned char* __restrict__ src, int64_t src_stride,
                                                       unsigned char* __restrict__ dst, int64_t dst_stride,
                                                       int64_t vpr, const int32_t* __restrict__ map, int map_src,
                                                       const int64_t* total, int64_t rows_cap,
                                                       const int32_t* status) {
  if (*status != 0) return;
  int64_t U = *total;
  U = U < rows_cap ? U : rows_cap;
  // XCD x (block % 8) copies the x-th eighth of the buffer's rows, in order
  // (measured 4-6 % faster than rows dealt to the XCDs in turn); the grid
  // covers rows_cap rounded up to eight, and blocks past the rows exit
  const int64_t per = (U + 7) / 8;
  const int64_t j = blockIdx.x >> 3;
  if (j >= per) return;
  const int64_t g = (int64_t)(blockIdx.x & 7) * per + j;
  if (g >= U) return;
  const int64_t m = map[g];
  const int64_t sr = map_src ? m : g, dr = map_src ? g : m;
  const u32x4* s = (const u32x4*)(src + sr * src_stride);
  u32x4* d = (u32x4*)(dst + dr * dst_stride);
  for (int64_t e0 = threadIdx.x; e0 < vpr; e0 += (int64_t)V * TH) {
    u32x4 r[V];
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (e0 + i * TH < vpr) r[i] = s[e0 + i * TH];
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (e0 + i * TH < vpr) __builtin_nontemporal_store(r[i], d + e0 + i * TH);
  }
}

constexpr int kTile = 32;

__global__ void __launch_bounds__(kTile * 8) transpose_kernel(const int64_t* __restrict__ D, int N,
                                                              int64_t* __restrict__ DT) {
  __shared__ int64_t tile[kTile][kTile + 1];
  const int bx = blockIdx.x * kTile, by = blockIdx.y * kTile;
  const int tx = threadIdx.x & (kTile - 1), ty = threadIdx.x / kTile;
  for (int r = ty; r < kTile; r += 8) {
    const int i = by + r, j = bx + tx;
    if (i < N && j < N) tile[r][tx] = D[(size_t)i * N + j];
  }
  __syncthreads();
  for (int r = ty; r < kTile; r += 8) {
    const int j = bx + r, i = by + tx;
    if (i < N && j < N) DT[(size_t)j * N + i] = tile[tx][r];
  }
}

constexpr size_t kHeader = 256;   // [0]: rows in the buffer (int64)

}  // namespace

int64_t slot_bytes(int64_t row_bytes) { return (row_bytes + 127) / 128 * 128; }

size_t unpack_workspace(int64_t rows) { return kHeader + align_up((size_t)rows * 4, 256); }

size_t unpack_lds_bytes(int mode, int32_t N, int32_t eloc) {
  return (size_t)N * 8 + (mode == kModeCombineUnpack ? 0 : (size_t)(3 * eloc + 1) * 8);
}

vp_status launch_unpack(const UnpackLaunch& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int eloc = a.E / a.N;
  const size_t lds = unpack_lds_bytes(a.mode, a.N, eloc);
  if (lds > 64 * 1024) return set_error(VP_ERR_UNSUPPORTED, "too many ranks or local experts for the row map");
  char* ws = (char*)a.ws;
  int64_t* total = (int64_t*)ws;
  int32_t* map = (int32_t*)(ws + kHeader);
  MapArgs m{a.mode, a.self_rank, a.N, a.k_max, eloc, a.E, a.k, a.row_bytes, a.T, a.rows_cap, a.map_cap,
            a.K, a.dst, a.recv_src, a.bytes, a.counts, a.sorted_tok, a.sorted_slot, a.dest_off, a.step_off,
            map, total, a.status};
  hipLaunchKernelGGL(map_kernel, dim3(a.k_max), dim3(kMapThreads), lds, s, m);
  if (a.rows_cap > 0) {
    if (a.rows_cap >= ((int64_t)1 << 31) - 8) return set_error(VP_ERR_UNSUPPORTED, "too many buffer rows");
    const int64_t vpr = a.row_bytes / 16;
    const dim3 grid((unsigned)((a.rows_cap + 7) / 8 * 8));   // rows past the buffer's count exit at once
    const unsigned char* sp = (const unsigned char*)a.src;
    unsigned char* dp = (unsigned char*)a.dst_buf;
    const int ms = a.mode == kModeCombinePack ? 1 : 0;
    // about 2 KiB per wavefront: rows up to 2, 4 and 8 KiB take 1, 2 and 4
    // wavefronts of two vectors per thread, longer rows 8 wavefronts of one
    if (vpr <= 128)
      hipLaunchKernelGGL((copy_rows_kernel<64, 2>), grid, dim3(64), 0, s, sp, a.src_stride, dp, a.dst_stride, vpr,
                         map, ms, total, a.rows_cap, a.status);
    else if (vpr <= 256)
      hipLaunchKernelGGL((copy_rows_kernel<128, 2>), grid, dim3(128), 0, s, sp, a.src_stride, dp, a.dst_stride, vpr,
                         map, ms, total, a.rows_cap, a.status);
    else if (vpr <= 512)
      hipLaunchKernelGGL((copy_rows_kernel<256, 2>), grid, dim3(256), 0, s, sp, a.src_stride, dp, a.dst_stride, vpr,
                         map, ms, total, a.rows_cap, a.status);
    else
      hipLaunchKernelGGL((copy_rows_kernel<512, 1>), grid, dim3(512), 0, s, sp, a.src_stride, dp, a.dst_stride, vpr,
                         map, ms, total, a.rows_cap, a.status);
  }
  if (hipGetLastError() != hipSuccess) return set_error(VP_ERR_HIP, "unpack launch failed");
  return VP_OK;
}

vp_status launch_transpose(const int64_t* D, int32_t N, int64_t* DT, void* stream) {
  const unsigned b = (unsigned)((N + kTile - 1) / kTile);
  hipLaunchKernelGGL(transpose_kernel, dim3(b, b), dim3(kTile * 8), 0, (hipStream_t)stream, D, N, DT);
  if (hipGetLastError() != hipSuccess) return set_error(VP_ERR_HIP, "transpose launch failed");
  return VP_OK;
}

}  // namespace vp
