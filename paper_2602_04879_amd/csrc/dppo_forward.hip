// Forward-only kernel: the per-token outputs of the loss, no gradient.
//
// Nothing needs a row after its statistics, so nothing is kept: a workgroup streams its row through a
// window of kWindow 16-byte chunks per thread (each pair of chunks is requested again, kWindow chunks
// further on, as soon as it has been consumed) into the online statistics, one LDS exchange and
// barrier, and wave 0 evaluates the per-token epilogue while the other waves are already in the next row.
//
// Bound by HBM reads, with the vector ALUs close behind (one exponential and about five other
// instructions per entry, seven with the entropy diagnostic).  Measured against the register-resident kernel's
// forward-only form, which kept the row for nothing at one workgroup per compute unit and spilled (V = 151936):
// 32768 tokens 1.74 -> 1.52 ms (6.5 TB/s), with diagnostics 2.18 -> 1.65; 8192 tokens 448 -> 406 and 570 -> 428 us;
// V = 50257, 16384 tokens 429 -> 338 us; against the two-pass kernel's forward form, V = 256000, 4096 tokens: 423 -> 354 us.
//
// Thread t of the workgroup takes vectors t, t + 512, ... of the row, two at a time, as the
// register-resident kernel's 512-thread shapes do: the per-token outputs of a forward-only call are those
// of a forward + backward one bit for bit.
//
// Any V, pitch and 2-byte alignment: RAGGED rows are handled in their frame, the aligned 16-byte
// blocks from the start of the 128-byte line that holds the row's first entry to the block that holds
// its last (see the register-resident kernel); what the frame holds besides the row becomes -inf.
#include "dppo_common.hpp"
#include "dppo_launch.hpp"
#include "dppo_resident_parts.hpp"

namespace dppo {
namespace {

constexpr int kThreads = 512;
constexpr int kWindow = 8;        // chunks in flight per thread (12: 1 % slower, 16: spills)

// PackedRowStat for a kernel with registers to spare: the entries are unpacked once, for the maximum
// (two entries per v_max3) and for the exponentials, where the packed form takes a packed maximum and
// minimum and unpacks for the exponentials; and two pairs of chunks go through side by side.  The same
// offset after every pair and the same order of the sums, so the same bits.  (V = 151936, 32768 tokens, with the
// packed form 1.61 ms, with diagnostics 1.79.)
template <bool DIAG>
struct UnpackedRowStat {
  float zmax = kNegBig, b = 3.0e38f;
  double sd = 0.0;
  float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
  __device__ __forceinline__ void add4(const u32x4 (&v)[4]) {
    float z[4][8], bn[2], sc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int i = 2 * q; i < 2 * q + 2; ++i) {
        unpack8(v[i], z[i]);
#pragma unroll
        for (int e = 0; e < 8; e += 2) zmax = fmaxf(fmaxf(zmax, z[i][e]), z[i][e + 1]);
      }
      bn[q] = -ceilf(zmax * kLog2e);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float d = bn[q] - b;
      sc[q] = fast_exp2(d);
      if (DIAG) { t0 = sc[q] * fmaf(d, static_cast<float>(sd), t0); t1 *= sc[q]; t2 *= sc[q]; t3 *= sc[q]; }
      b = bn[q];
      float gs = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float (&y)[8] = z[2 * q + i];
        float c;
        if (DIAG) {
          c = (term2(y[0], y[1], t0) + term2(y[2], y[3], t1)) + (term2(y[4], y[5], t2) + term2(y[6], y[7], t3));
        } else {
          c = ((ex(y[0]) + ex(y[1])) + (ex(y[2]) + ex(y[3]))) + ((ex(y[4]) + ex(y[5])) + (ex(y[6]) + ex(y[7])));
        }
        gs = (i == 0) ? c : gs + c;
      }
      sd = fma(sd, static_cast<double>(sc[q]), static_cast<double>(gs));
    }
  }
  __device__ __forceinline__ float ex(float z) const { return fast_exp2(fmaf(z, kLog2e, b)); }
  __device__ __forceinline__ float term2(float z0, float z1, float& t) const {
    const float x0 = fmaf(z0, kLog2e, b), x1 = fmaf(z1, kLog2e, b);
    const float e0 = fast_exp2(x0), e1 = fast_exp2(x1);
    t = fma_ex(e0, x0, fma_ex(e1, x1, t));
    return e0 + e1;
  }
  __device__ __forceinline__ float tsum() const { return (t0 + t1) + (t2 + t3); }
};

// Two workgroups per compute unit (four waves per SIMD: 128 registers).
template <bool DIAG, bool RAGGED>
__global__ __launch_bounds__(kThreads, 4) void dppo_forward_kernel(const KParams p) {
  constexpr int NW = kThreads / kWave;
  constexpr uint32_t kStride = kThreads * 16u;          // bytes between a thread's consecutive chunks
  // two sets, used by alternate rows: wave 0 may still read one row's while the others publish the next one's
  __shared__ float sh_b[2][NW];
  __shared__ double sh_s[2][NW], sh_t[2][NW];
  int par = 0;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = uniform_i(tid / kWave);
  const uint32_t voff = static_cast<uint32_t>(tid) * 16u;
  const u32x4 neg_inf = {kNegInfPair, kNegInfPair, kNegInfPair, kNegInfPair};
  const int64_t pitch = p.ld * 2;
  const char* logits = reinterpret_cast<const char*>(p.logits);
  const EpiParams ep = epi_params(p);
  double loss_acc = 0.0;                               // meaningful in wave 0 only

  auto head_of = [&](int r) -> int {
    return RAGGED ? static_cast<int>(((reinterpret_cast<uintptr_t>(logits) + static_cast<uint64_t>(r * pitch)) >> 1) & 63u) : 0;
  };
  // view of a row (RAGGED: of its frame, up to the 4-byte word holding its last entry); has = false: of zero bytes
  auto load_view = [&](int r, bool has) -> row_rsrc_t {
    const int h = head_of(r);
    return make_row_rsrc(logits + r * pitch - 2 * h, has ? ((static_cast<uint32_t>(h + p.V) * 2u + 3u) & ~3u) : 0u);
  };
  u32x4 buf[kWindow];
  int row = static_cast<int>(blockIdx.x);
  // Fetched one row ahead: the sampled id and (wave 0, lane k < K) the id and log-prob of top-K entry k,
  // so that the logits they point at can be requested at the top of the row.
  int a_next = p.sampled[row];
  int tkid_next = -1;
  float tklp_next = 0.f;
  if (wid == 0 && lane < p.K) {
    tkid_next = p.tk_ids[static_cast<int64_t>(row) * p.K + lane];
    tklp_next = p.tk_lp[static_cast<int64_t>(row) * p.K + lane];
  }
  __builtin_amdgcn_sched_barrier(0);
  {
    const row_rsrc_t zr = load_view(row, true);
#pragma unroll
    for (int i = 0; i < kWindow; ++i) buf[i] = row_load16<true>(zr, voff, i * kStride);
  }
  for (; row < p.T;) {
    const int a = uniform_i(a_next);
    const int next = row + static_cast<int>(gridDim.x);
    const bool more = next < p.T;
    if (more) a_next = p.sampled[next];
    const int tkid = tkid_next;
    const float tklp = tklp_next;
    if (more && wid == 0 && lane < p.K) {
      tkid_next = p.tk_ids[static_cast<int64_t>(next) * p.K + lane];
      tklp_next = p.tk_lp[static_cast<int64_t>(next) * p.K + lane];
    }
    const bool live = (a >= 0 && a < p.V);
    const uint16_t* zrow = p.logits + static_cast<int64_t>(row) * p.ld;
    TopkLane tk;
    tk.id = -1; tk.lp = 0.f; tk.z = 0.f;
    uint32_t za_bits = 0, tkz_bits = 0;      // raw until the statistics are through: a use up here would be a wait
    float packed_scalars = 0.f;
    if (live && wid == 0) {
      za_bits = zrow[a];
      packed_scalars = load_row_scalars(p, row, lane);
      if (tkid >= 0 && tkid < p.V && tkid != a) {
        tk.id = tkid;
        tk.lp = tklp;
        tkz_bits = zrow[tkid];
      }
    }
    const int h = head_of(row);
    const int nvec = (h + p.V + 7) >> 3;
    const int vl = nvec - 1, il = vl / kThreads, tl = vl - il * kThreads, t = h + p.V - 8 * vl;      // last block: chunk il of thread tl, t entries
    const int nchunk = live ? (nvec + kThreads - 1) / kThreads : 0;
    const int avec = (a + h) >> 3, ia = avec / kThreads, sub = (a + h) & 7;
    const bool owner = avec - ia * kThreads == tid;
    const row_rsrc_t zr = load_view(row, true);
    UnpackedRowStat<DIAG> ps;
    // What is not the row's own, and the sampled token's own term, becomes -inf (uniform tests first).
    if (RAGGED && tid < 8 && h > 8 * tid) buf[0] = keep16(buf[0], min(h - 8 * tid, 8), 8);
#pragma unroll 1
    for (int c0 = 0; c0 < nchunk; c0 += kWindow) {
      if (c0 <= ia && ia < c0 + kWindow) {
#pragma unroll
        for (int i = 0; i < kWindow; ++i)
          if (c0 + i == ia && owner) buf[i] = patch16(buf[i], sub, 0xFF80u);
      }
      if (c0 + kWindow > il) {
#pragma unroll
        for (int i = 0; i < kWindow; ++i) {
          if (c0 + i == il && tid == tl && t < 8) buf[i] = keep16(buf[i], 0, t);
          if (c0 + i >= il && (c0 + i) * kThreads + tid >= nvec) buf[i] = neg_inf;         // lanes past the row loaded 0
        }
      }
#pragma unroll
      for (int g = 0; g < kWindow; g += 4) {
        if (c0 + g >= nchunk) break;
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i] = buf[g + i];
          buf[g + i] = row_load16<true>(zr, voff, static_cast<uint32_t>(c0 + g + i + kWindow) * kStride);
        }
        ps.add4(v);
      }
    }
    {   // the next row's first chunks travel during this row's epilogue
      const row_rsrc_t zn = load_view(more ? next : row, more);
#pragma unroll
      for (int i = 0; i < kWindow; ++i) buf[i] = row_load16<true>(zn, voff, i * kStride);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (live) {
      const float bw = -wave_max(-ps.b);
      const double dw = static_cast<double>(bw - ps.b), scw = static_cast<double>(fast_exp2(bw - ps.b));
      const double sw = wave_sum(ps.sd * scw);
      const double tw = DIAG ? wave_sum(scw * (static_cast<double>(ps.tsum()) + dw * ps.sd)) : 0.0;
      if (lane == 0) { sh_b[par][wid] = bw; sh_s[par][wid] = sw; sh_t[par][wid] = tw; }
      __syncthreads();
      if (wid == 0) {
        asm volatile("" : "+v"(za_bits), "+v"(packed_scalars), "+v"(tkz_bits), "+v"(tk.lp), "+v"(tk.id));
        RowScalars rs;
        rs.a = a;
        rs.za = __uint_as_float(za_bits << 16);
        unpack_row_scalars(packed_scalars, rs);
        tk.z = __uint_as_float(tkz_bits << 16);
        float bb = -ceilf(fmaxf(rs.za, kNegBig) * kLog2e);       // the offset must also cover z[a_t]
#pragma unroll
        for (int w = 0; w < NW; ++w) bb = fminf(bb, sh_b[par][w]);
        double S_rest = 0.0, T_rest = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const double dd = static_cast<double>(bb - sh_b[par][w]), sc = static_cast<double>(fast_exp2(bb - sh_b[par][w]));   // exact power of two
          S_rest += sh_s[par][w] * sc;
          if (DIAG) T_rest += sc * (sh_t[par][w] + dd * sh_s[par][w]);
        }
        // (with diagnostics the inlined form spills fifty registers: 2-5 % slower from 1000 tokens on; without, 1000 tokens of
        // V = 57000, 151936 and 256000: 36.9 / 24.7, 70.5 / 52.4, 106 / 83 us as a call / inlined)
        const RowResult rr = DIAG ? row_epilogue_call(ep, row, rs, tk, zrow, bb, S_rest, T_rest, lane)
                                  : row_epilogue(ep, row, rs, tk, zrow, bb, S_rest, T_rest, lane);
        loss_acc += rr.loss_term;
      }
      par ^= 1;
    } else if (tid == 0) {
      p.divergence[row] = 0.f;
      p.mask[row] = 0;
      if (p.loss_tok) p.loss_tok[row] = 0.f;
      if (p.diag) {
        for (int k = 0; k < 8; ++k) p.diag[static_cast<int64_t>(row) * 8 + k] = 0.f;
      }
    }
    row = next;
  }
  if (tid == 0) p.partial[blockIdx.x] = loss_acc;
}

}  // namespace

hipError_t launch_forward(const KParams& p, bool ragged, int grid, hipStream_t s) {
  const dim3 g(grid), b(kThreads);
  if (p.diag) {
    if (ragged) hipLaunchKernelGGL((dppo_forward_kernel<true, true>), g, b, 0, s, p);
    else        hipLaunchKernelGGL((dppo_forward_kernel<true, false>), g, b, 0, s, p);
  } else {
    if (ragged) hipLaunchKernelGGL((dppo_forward_kernel<false, true>), g, b, 0, s, p);
    else        hipLaunchKernelGGL((dppo_forward_kernel<false, false>), g, b, 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace dppo
