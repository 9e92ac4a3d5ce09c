// Few long rows: every row divided among several workgroups.
//
// A call with fewer rows than half the compute units leaves the others idle for as long as one row takes (V = 151936: 23 us of
// mostly vector arithmetic, whatever the neighbours do).  Here a row is cut into segments of 32 KiB, one workgroup each:
//   dppo_split_stat_kernel  the statistics of a segment, one record per (row, segment), and the row's logits at its sampled and
//                           top-K ids (p.gath), so that nothing reads another segment once gradients are being written
//   dppo_split_grad_kernel  the records of the row combined and its epilogue evaluated by every workgroup of the row for
//                           itself (by one wave, while the segment's loads travel), then the segment's gradient; the row's first
//                           workgroup writes the per-token outputs.  The second read of a segment comes from the caches: fewer
//                           rows than 128 are 39 MB at V = 151936, and workgroup ids, so dies, are those of the first kernel.
//   dppo_split_rows_kernel  forward only: one wave per row
// The row whose loss term is the last to be left adds them all up, beside the other workgroups' gradients.
// Bound by launches and latencies (two kernels, 2 us each when empty) up to some 30 rows, then by the memory traffic of the two passes.
// V = 151936, Top-20 TV, calls in a graph, us, one workgroup per row / divided, a third kernel for the loss / as it is.  Inputs the same from call to call, in the caches: 8
// tokens 23.4 / 11.7 / 10.2, 64 23.7 / 14.9 / 13.4, 128 25.8 / 20.7 / 19.8, forward only 15.7 / 9.8 / 8.9, 16.0 / 11.3 / 10.5, 16.5 / 15.4 / 14.3; inputs that
// change, from memory: 25.6 / 13.3 / 11.5, 26.3 / 17.4 / 15.8, 27.5 / 23.9 / 23.0, forward only 15.7 / 11.5 / 10.2, 16.2 / 14.2 / 12.9, 16.8 / 17.2 / 15.9.
// Segments of 16 or 64 KiB, and 128 or 512 threads: the same to 30 % slower.  Code that few workgroups need (edges of a row, the
// sampled token) stands behind branches of the whole workgroup: a kernel this short runs each instruction once and waits
// for its fetch (100 tokens: 21.6 -> 20.1 us).
// A kernel boundary instead of a handshake between workgroups: nothing waits for another workgroup, and the scratch needs no
// particular contents (the first kernel clears the count of rows).
//
// Any V, pitch and 2-byte alignment (logits and gradient sharing their misalignment): rows are handled in their
// frame, the aligned 16-byte blocks from the start of the 128-byte line that holds the row's first entry to the block that
// holds its last (see the register-resident kernel); what the frame holds besides the row becomes -inf.
#include "dppo_common.hpp"
#include "dppo_launch.hpp"
#include "dppo_resident_parts.hpp"

namespace dppo {
namespace {

constexpr int kThreads = 256;
constexpr int kChunks = 8;                                   // 16-byte chunks per thread: all loads of a segment in flight at once
constexpr int kWaves = kThreads / kWave;
static_assert(kThreads * kChunks == kSplitVecs, "a segment is one workgroup's chunks");

// A row's segment as a thread sees it: chunk i is block v0 + i * kThreads of the row's frame.
struct Segment {
  int h;              // entries of the frame in front of the row
  int nvec;           // blocks of the frame
  int v0;             // this thread's first block
  bool last, ragged;  // uniform: blocks past the frame in this segment; an incomplete block of the row in it
};
__device__ __forceinline__ Segment segment_of(const KParams& p, int row, int seg) {
  Segment s;
  s.h = static_cast<int>(((reinterpret_cast<uintptr_t>(p.logits) + static_cast<uint64_t>(row) * static_cast<uint64_t>(p.ld) * 2u) >> 1) & 63u);
  s.nvec = (s.h + p.V + 7) >> 3;
  s.v0 = seg * kSplitVecs + static_cast<int>(threadIdx.x);
  s.last = (seg + 1) * kSplitVecs >= s.nvec;
  s.ragged = (seg == 0 && s.h != 0) || (s.last && ((s.h + p.V) & 7) != 0);
  return s;
}
// All loads of the segment (blocks past the frame read as zeros).
__device__ __forceinline__ void load_segment(const KParams& p, int row, const Segment& s, u32x4 (&buf)[kChunks]) {
  const row_rsrc_t r = make_row_rsrc(reinterpret_cast<const char*>(p.logits) + static_cast<int64_t>(row) * p.ld * 2 - 2 * s.h,
                                     (static_cast<uint32_t>(s.h + p.V) * 2u + 3u) & ~3u);
#pragma unroll
  for (int i = 0; i < kChunks; ++i) buf[i] = row_load16(r, static_cast<uint32_t>(s.v0) * 16u, i * kThreads * 16u);
}
// The chunk of this thread that holds the sampled token a of the row, -1 if none does.
__device__ __forceinline__ int chunk_of(const Segment& s, int a) {
  const int d = ((a + s.h) >> 3) - s.v0;
  return (d >= 0 && d < kSplitVecs && d % kThreads == 0) ? d / kThreads : -1;
}
__device__ __forceinline__ bool holds(int seg, const Segment& s, int a) { return ((a + s.h) >> 3) / kSplitVecs == seg; }
// Blocks past the frame, entries outside the row and the sampled token become -inf.  Only the first and last segments and
// the one with the sampled token have any: three branches of the whole workgroup, so that the others run (and fetch)
// nothing of this code.
__device__ __forceinline__ void mask_segment(const KParams& p, int seg, const Segment& s, int a, u32x4 (&buf)[kChunks]) {
  const u32x4 neg_inf = {kNegInfPair, kNegInfPair, kNegInfPair, kNegInfPair};
  if (s.last) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) if (s.v0 + i * kThreads >= s.nvec) buf[i] = neg_inf;
  }
  if (s.ragged) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int v = s.v0 + i * kThreads, e0 = 8 * v - s.h;           // entries e0 .. e0 + 7 of the row
      if (v < s.nvec && (e0 < 0 || e0 + 8 > p.V)) buf[i] = keep16(buf[i], max(-e0, 0), min(p.V - e0, 8));
    }
  }
  if (holds(seg, s, a)) {
    const int ia = chunk_of(s, a);
#pragma unroll
    for (int i = 0; i < kChunks; ++i) if (i == ia) buf[i] = patch16(buf[i], (a + s.h) & 7, 0xFF80u);
  }
}

template <bool DIAG>
__global__ __launch_bounds__(kThreads) void dppo_split_stat_kernel(const KParams p, SplitRecord* __restrict__ rec, float* __restrict__ gath, int segs) {
  __shared__ float sh_b[kWaves];
  __shared__ double sh_s[kWaves], sh_t[kWaves];
  const int row = static_cast<int>(blockIdx.x) / segs, seg = static_cast<int>(blockIdx.x) - row * segs;
  const int lane = threadIdx.x & (kWave - 1), wid = uniform_i(threadIdx.x / kWave);
  const int a = uniform_i(p.sampled[row]);
  const Segment s = segment_of(p, row, seg);
  u32x4 buf[kChunks];
  load_segment(p, row, s, buf);
  if (!(a >= 0 && a < p.V)) {                                      // an ignored row has no statistics
    if (blockIdx.x == 0 && threadIdx.x == 0) rec[0].rows = 0;
    return;
  }
  if (seg == 0) {
    const uint16_t* zrow = p.logits + static_cast<int64_t>(row) * p.ld;
    for (int k = threadIdx.x; k <= p.K; k += kThreads) {
      const int id = (k == 0) ? a : p.tk_ids[static_cast<int64_t>(row) * p.K + k - 1];
      if (id >= 0 && id < p.V) gath[static_cast<int64_t>(row) * (p.K + 1) + k] = bf16_bits_to_float(zrow[id]);
    }
  }
  mask_segment(p, seg, s, a, buf);
  PackedRowStat<DIAG> ps;
#pragma unroll
  for (int i = 0; i < kChunks; i += 2) ps.add2(buf[i], buf[i + 1]);
  const float bw = -wave_max(-ps.b);
  const double dw = static_cast<double>(bw - ps.b), scw = static_cast<double>(fast_exp2(bw - ps.b));      // exact powers of two
  const double sw = wave_sum(ps.sd * scw);
  const double tw = DIAG ? wave_sum(scw * (static_cast<double>(ps.tsum()) + dw * ps.sd)) : 0.0;
  if (lane == 0) { sh_b[wid] = bw; sh_s[wid] = sw; sh_t[wid] = tw; }
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = sh_b[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) b = fminf(b, sh_b[w]);
    double S = 0.0, T = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const double dd = static_cast<double>(b - sh_b[w]), sc = static_cast<double>(fast_exp2(b - sh_b[w]));
      S += sh_s[w] * sc;
      if (DIAG) T += sc * (sh_t[w] + dd * sh_s[w]);
    }
    rec[blockIdx.x] = SplitRecord{S, T, b, 0u};
  }
}

// The inputs of a row's epilogue, by one full wave: all requested at once (one memory latency).
struct RowInputs {
  SplitRecord r;      // lane l < segs: segment l's record
  float scalars, za;  // see load_row_scalars; the logit of the sampled token
  TopkLane tk;        // entry as it stands in memory, not yet looked at
};
__device__ __forceinline__ RowInputs load_row(const KParams& p, int row, const SplitRecord* rec, int segs, int lane) {
  RowInputs in;
  in.r = SplitRecord{0.0, 0.0, 3.0e38f, 0u};
  if (lane < segs) {
    const SplitRecord* r = rec + static_cast<int64_t>(row) * segs + lane;
    in.r.s = r->s; in.r.t = r->t; in.r.b = r->b;
  }
  in.scalars = load_row_scalars(p, row, lane);
  const float* gath = p.gath + static_cast<int64_t>(row) * (p.K + 1);
  in.za = gath[0];
  in.tk.id = -1; in.tk.lp = 0.f; in.tk.z = 0.f;
  if (lane < p.K) {
    in.tk.id = p.tk_ids[static_cast<int64_t>(row) * p.K + lane];
    in.tk.lp = p.tk_lp[static_cast<int64_t>(row) * p.K + lane];
    in.tk.z = gath[1 + lane];
  }
  return in;
}
// The row's epilogue from its segments' records; `o` is what row_store writes.
__device__ __forceinline__ RowResult split_row(const KParams& p, const EpiParams& ep, int row, int a, RowInputs in, int segs, int lane, RowOut& o) {
  RowScalars rs;
  rs.a = a;
  rs.za = in.za;
  unpack_row_scalars(in.scalars, rs);
  if (!(in.tk.id >= 0 && in.tk.id < p.V && in.tk.id != a)) in.tk.id = -1;
  const RowPre q = row_pre(rs, in.tk, p.K > 0, p.relax_log_alpha);
  // the common offset must also cover z[a_t], whose own term the epilogue adds
  const SplitRecord r = in.r;
  const float b = fminf(-wave_max(-r.b), -ceilf(fmaxf(rs.za, kNegBig) * kLog2e));
  const double d = static_cast<double>(b - r.b), sc = static_cast<double>(fast_exp2(b - r.b));
  const double S = wave_sum(r.s * sc), T = p.diag ? wave_sum(lane < segs ? sc * (r.t + d * r.s) : 0.0) : 0.0;
  return row_post(ep, row, q, a, nullptr, b, S, T, lane, 0.0, o);
}

// Leaves a row's loss term, by one lane: written past the die's L2 and waited for before the row is counted, so that whoever finds the count
// complete finds the terms (read past the L2 again).
__device__ __forceinline__ void leave_loss_term(double term, int row, double* row_loss) {
  __hip_atomic_store(row_loss + row, term, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// Counts rows: true for those that are the last.
__device__ __forceinline__ bool count_rows(int rows, const KParams& p, SplitRecord* rec) {
  return __hip_atomic_fetch_add(&rec[0].rows, static_cast<uint32_t>(rows), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + static_cast<uint32_t>(rows) == static_cast<uint32_t>(p.T);
}
// The scalar loss from the terms of all rows, by one wave: lane l those numbered l, l + 64, ..., then a tree (the order of the general sum
// for up to 128 rows).
__device__ __forceinline__ void sum_loss(const KParams& p, const double* row_loss, float* loss, int lane) {
  double v = 0.0;
  for (int r = lane; r < p.T; r += kWave) v += __hip_atomic_load(row_loss + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if (lane == 0) *loss = static_cast<float>(static_cast<double>(p.loss_scale) * v);
}

__device__ __forceinline__ void ignored_row(const KParams& p, int row) {
  p.divergence[row] = 0.f;
  p.mask[row] = 0;
  if (p.loss_tok) p.loss_tok[row] = 0.f;
  if (p.diag) {
    for (int k = 0; k < 8; ++k) p.diag[static_cast<int64_t>(row) * 8 + k] = 0.f;
  }
}

__global__ __launch_bounds__(kThreads) void dppo_split_rows_kernel(const KParams p, SplitRecord* rec, int segs, double* row_loss, float* loss) {
  const int lane = threadIdx.x & (kWave - 1), wid = uniform_i(threadIdx.x / kWave);
  const int row0 = static_cast<int>(blockIdx.x) * kWaves, row = row0 + wid;
  if (row < p.T) {
    const RowInputs in = load_row(p, row, rec, segs, lane);
    const int a = uniform_i(p.sampled[row]);
    double term = 0.0;
    if (a >= 0 && a < p.V) {
      const EpiParams ep = epi_params(p);
      RowOut o;
      term = split_row(p, ep, row, a, in, segs, lane, o).loss_term;
      row_store(ep, row, o, lane);
    } else if (lane == 0) {
      ignored_row(p, row);
    }
    if (lane == 0) leave_loss_term(term, row, row_loss);
  }
  __syncthreads();
  if (wid != 0) return;
  bool last = false;
  if (lane == 0) last = count_rows(min(kWaves, p.T - row0), p, rec);
  if (__any(last)) sum_loss(p, row_loss, loss, lane);
}

__global__ __launch_bounds__(kThreads) void dppo_split_grad_kernel(const KParams p, SplitRecord* rec, int segs, double* row_loss, float* loss) {
  __shared__ RowCoef sh_rc;
  // The segments in the opposite order, on the same dies: what the first kernel read last is what their L2 still holds.
  const int idx = static_cast<int>((gridDim.x - 8u - (blockIdx.x & ~7u)) | (blockIdx.x & 7u));
  if (idx >= p.T * segs) return;
  const int row = idx / segs, seg = idx - row * segs;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = uniform_i(tid / kWave);
  RowInputs in;
  if (wid == 0) in = load_row(p, row, rec, segs, lane);            // in front of the segment: loads return in order
  const Segment s = segment_of(p, row, seg);
  u32x4 buf[kChunks];
  load_segment(p, row, s, buf);
  const int a = uniform_i(p.sampled[row]);
  const bool live = (a >= 0 && a < p.V);
  RowCoef rc;
  rc.coef = 0.f; rc.kexp = 0.f; rc.g_a = 0.f;
  bool last = false;                       // (first lane of the row's first workgroup)
  if (live) {
    RowOut o;
    RowResult res;
    if (wid == 0) {
      res = split_row(p, epi_params(p), row, a, in, segs, lane, o);
      if (lane == 0) sh_rc = res.rc;
    }
    __syncthreads();
    if (wid == 0 && seg == 0) {
      row_store(epi_params(p), row, o, lane);
      if (lane == 0) {
        leave_loss_term(res.loss_term, row, row_loss);
        last = count_rows(1, p, rec);
      }
    }
    rc.coef = uniform_f(sh_rc.coef);
    rc.kexp = uniform_f(sh_rc.kexp);
    rc.g_a = uniform_f(sh_rc.g_a);
  } else if (seg == 0 && tid == 0) {
    ignored_row(p, row);
    leave_loss_term(0.0, row, row_loss);
    last = count_rows(1, p, rec);
  }
  // Of the frame only complete blocks of the row's own entries leave as 16-byte stores, an incomplete first or last block entry by
  // entry.  A masked, zero-advantage or ignored row's gradient is exactly zero whatever the logits hold.
  uint16_t* grow = p.grad + static_cast<int64_t>(row) * p.ld;
  const uint32_t sgn = (rc.coef < 0.f) ? 0x80008000u : 0u;
  const bool zero = rc.coef == 0.f;
  if (!zero) mask_segment(p, seg, s, a, buf);
  u32x4 (&o)[kChunks] = buf;
#pragma unroll
  for (int i = 0; i < kChunks; ++i) o[i] = zero ? u32x4{0u, 0u, 0u, 0u} : grad8(buf[i], rc.kexp, sgn);
  if (!zero && holds(seg, s, a)) {
    const int ia = chunk_of(s, a);
#pragma unroll
    for (int i = 0; i < kChunks; ++i) if (i == ia) o[i] = patch16(o[i], (a + s.h) & 7, float_to_bf16_bits(rc.g_a));
  }
  if (!s.ragged) {        // (past the frame: dropped by the range check)
    const row_rsrc_t r = make_row_rsrc(grow - s.h, static_cast<uint32_t>(s.h + p.V) * 2u);
#pragma unroll
    for (int i = 0; i < kChunks; ++i) __builtin_amdgcn_raw_buffer_store_b128(o[i], r, static_cast<uint32_t>(s.v0) * 16u, i * kThreads * 16u, 2);
  } else {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int v = s.v0 + i * kThreads, e0 = 8 * v - s.h;
      if (e0 >= 0 && e0 + 8 <= p.V) {
        __builtin_nontemporal_store(o[i], reinterpret_cast<u32x4*>(grow + e0));
      } else if (v < s.nvec) {
        const uint32_t w[4] = {o[i].x, o[i].y, o[i].z, o[i].w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e0 + e >= 0 && e0 + e < p.V) grow[e0 + e] = static_cast<uint16_t>((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu));
      }
    }
  }
  if (wid == 0 && seg == 0 && __any(last)) sum_loss(p, row_loss, loss, lane);
}

}  // namespace

int split_segments(int64_t V) { return static_cast<int>(((V + 70) / 8 + kSplitVecs - 1) / kSplitVecs); }

size_t split_scratch_bytes(int64_t T, int64_t V, int32_t K) {
  return static_cast<size_t>(T) * (sizeof(double) + static_cast<size_t>(split_segments(V)) * sizeof(SplitRecord) + static_cast<size_t>(K + 1) * sizeof(float));
}

hipError_t launch_split(KParams p, bool grad, void* scratch, float* loss, hipStream_t s) {
  const int segs = split_segments(p.V);
  if (segs > kWave || p.T <= 0) return hipErrorInvalidValue;
  // [loss terms | records | gathered logits]
  double* row_loss = static_cast<double*>(scratch);
  SplitRecord* rec = reinterpret_cast<SplitRecord*>(row_loss + p.T);
  float* gath = reinterpret_cast<float*>(rec + static_cast<int64_t>(p.T) * segs);
  p.gath = gath;
  const dim3 grid(static_cast<unsigned>(p.T) * static_cast<unsigned>(segs)), wg(kThreads);
  if (p.diag) hipLaunchKernelGGL(dppo_split_stat_kernel<true>, grid, wg, 0, s, p, rec, gath, segs);
  else        hipLaunchKernelGGL(dppo_split_stat_kernel<false>, grid, wg, 0, s, p, rec, gath, segs);
  if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  if (grad) hipLaunchKernelGGL(dppo_split_grad_kernel, dim3((grid.x + 7u) & ~7u), wg, 0, s, p, rec, segs, row_loss, loss);
  else      hipLaunchKernelGGL(dppo_split_rows_kernel, dim3((p.T + kWaves - 1) / kWaves), wg, 0, s, p, rec, segs, row_loss, loss);
  return hipGetLastError();
}

}  // namespace dppo
