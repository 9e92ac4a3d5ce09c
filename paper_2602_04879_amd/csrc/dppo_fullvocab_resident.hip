// Trust region on the EXACT full-vocabulary divergence (App. B), register-resident form (the
// backward of both variants, and the forward-only TV form): total variation 1/2 sum_j |mu_j - pi_j| or KL(mu || pi) = sum_j mu_j ln(mu_j / pi_j)
// between the rollout policy's and the trainer's next-token distributions, both given as rows of
// bf16 logits, and the gradient of the masked surrogate over the trainer's row.
//
// A persistent workgroup of 512 threads, one per compute unit (two for rows of up to 49152 entries), owns
// one row at a time.  The trainer
// row z stays packed in its vector registers (as in the register-resident loss kernel: V = 151936
// is 297 KiB of a compute unit's 512 KiB register file), the rollout row y streams past it a few
// 16-byte chunks per thread at a time and is never kept in registers:
//   pass 1   statistics of z (sampled token left out) and of y, and for the KL form the cross term
//            sum_j 2^(y_j..) (y_j - z_j); KL = E_mu[y - z] - lse(y) + lse(z) needs nothing else.
//   pass 2   (TV only) sum_j min(pi_j, mu_j) with z from the registers and y read again; the first
//            chunks of y each thread consumed in pass 1 wait for it in LDS, the later ones (read a
//            few microseconds earlier, partly still in the L2) are requested again.
//   epilogue on one wave: mask, loss term, gradient coefficient.
//   gradient every resident entry, the whole row in one run of 16-byte stores; then the next row of
//            z and the first chunks of the next row of y are requested in one run of loads.
// z is read once, y once (KL) or about one and a half times (TV), the gradient written once: 6
// (7) bytes per vocabulary entry where the general kernel moves 8 (10).
// All row traffic goes through range-checked buffer views (loads past the row return 0 and are
// turned into -inf, stores past it are dropped), so the passes are straight-line code.
// Preconditions (checked by the host): V % 8 == 0, V / 8 <= 512 * NCHUNK, the three matrices
// 16-byte aligned with pitches that are multiples of 8 entries.
#include "dppo_common.hpp"
#include "dppo_launch.hpp"
#include "dppo_resident_parts.hpp"

namespace dppo {
namespace {

constexpr int kThreads = 512;
// Shapes (chunks of z per thread).  Up to 12 chunks two workgroups share a compute unit (128 registers,
// 72 KiB of LDS for y each), from 14 on one owns it.
constexpr bool two_per_cu(int nchunk) { return nchunk <= 12; }
constexpr bool kl_shape(int nchunk) { return nchunk != 12; }      // shapes of the KL form (see fullvocab_resident_chunks)
constexpr int window_of(int nchunk) { return nchunk <= 8 ? nchunk : 4; }   // chunks of y in flight per thread (32 and 38 chunks: 4, 8 and 12 measure the same)
// chunks every row of a shape fills (shorter rows take the next smaller one): only later ones can have lanes past the row
constexpr int full_chunks(int nchunk) { return nchunk <= 16 ? nchunk - 2 : nchunk <= 24 ? nchunk - 4 : nchunk == 32 ? 24 : 32; }
constexpr int keep_of(int nchunk) { return two_per_cu(nchunk) ? 9 : 18; }   // TV form: chunks of y kept in LDS between the passes (8 KiB each, 144 of the 160 KiB)

// Running sum of 2^(x*log2e + b) over one row with an integer offset b <= -max*log2e that only
// ever decreases (lowering it rescales the sums by an exact power of two).  T: also sum 2^x * x,
// which feeds the entropy diagnostic.  U: also sum 2^x * (x_j - other_j) in natural units, the
// cross term of the KL form (a vanished term adds nothing even where the other row is -inf too).
template <bool T, bool U>
struct RowStat {
  float b = 3.0e38f, t = 0.f, u = 0.f;
  double s = 0.0;      // float64, fed with fp32 sums of eight entries (see sum8)
  __device__ __forceinline__ void cover(float vmax) {
    const float bn = fminf(b, -ceilf(fmaxf(vmax, kNegBig) * kLog2e));
    const float d = bn - b, sc = fast_exp2(d);
    if (T) t = sc * fmaf(d, static_cast<float>(s), t);
    if (U) u *= sc;
    s *= static_cast<double>(sc);
    b = bn;
  }
  __device__ __forceinline__ float term(float v, float other) {
    const float x = fmaf(v, kLog2e, b), e = fast_exp2(x);
    if (T) t = fma_ex(e, x, t);
    if (U) u = fmaf(e, fminf(fmaxf(v - other, -3.0e38f), 3.0e38f), u);     // NaN (-inf - -inf) -> -3e38, times e = 0
    return e;
  }
  __device__ __forceinline__ void add8(const float (&v)[8], const float (&other)[8]) {
    cover(fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7]))));
    add8_covered(v, other);
  }
  // Entries that the offset covers already.
  __device__ __forceinline__ void add8_covered(const float (&v)[8], const float (&other)[8]) {
    // the eight exponentials summed pairwise as they are formed (few of them alive at a time)
    const float q0 = (term(v[0], other[0]) + term(v[1], other[1])) + (term(v[2], other[2]) + term(v[3], other[3]));
    const float q1 = (term(v[4], other[4]) + term(v[5], other[5])) + (term(v[6], other[6]) + term(v[7], other[7]));
    s += static_cast<double>(q0 + q1);
  }
};

// The largest entry of a row's chunks, on the packed bf16 patterns as signed 16-bit integers: non-negative patterns order like the
// floats and every negative one stays below them; where every entry of a lane is negative the float maximum is the integer minimum.
template <int N>
__device__ __forceinline__ float packed_max(const u32x4 (&v)[N]) {
  s16x2 m = as_s16x2(0x80008000u);
#pragma unroll
  for (int i = 0; i < N; ++i)
    m = __builtin_elementwise_max(m, __builtin_elementwise_max(__builtin_elementwise_max(as_s16x2(v[i].x), as_s16x2(v[i].y)), __builtin_elementwise_max(as_s16x2(v[i].z), as_s16x2(v[i].w))));
  int top = max(static_cast<int>(m.x), static_cast<int>(m.y));
  if (__any(top < 0)) {
    s16x2 n = as_s16x2(0x7FFF7FFFu);
#pragma unroll
    for (int i = 0; i < N; ++i)
      n = __builtin_elementwise_min(n, __builtin_elementwise_min(__builtin_elementwise_min(as_s16x2(v[i].x), as_s16x2(v[i].y)), __builtin_elementwise_min(as_s16x2(v[i].z), as_s16x2(v[i].w))));
    top = top < 0 ? min(static_cast<int>(n.x), static_cast<int>(n.y)) : top;
  }
  return __uint_as_float(static_cast<uint32_t>(top) << 16);
}

// DYN: rows handed out at run time from a counter (as in the register-resident kernel of the Binary
// / Top-K variants: the dies do not run at one speed, and with rows fixed by the workgroup index the
// slowest compute unit ends the kernel), the loss terms to one slot per row.
template <int NCHUNK, bool TV, bool DIAG, bool GRAD, bool DYN>
__global__ __launch_bounds__(kThreads, two_per_cu(NCHUNK) ? 4 : 2) void dppo_fullvocab_resident_kernel(const KParams p) {
  static_assert(GRAD || TV, "forward only, the KL form reads each row once anyway: the general kernel serves it");
  static_assert(GRAD || !DYN, "rows at run time: the gradient forms only");
  static_assert(NCHUNK >= 32 || GRAD, "shorter rows: the gradient forms only");
  constexpr int kWindow = window_of(NCHUNK);
  constexpr int THREADS = kThreads, NW = THREADS / kWave;
  constexpr uint32_t kStride = THREADS * 16u;      // bytes between a thread's consecutive chunks
  constexpr int KEEP = TV ? (keep_of(NCHUNK) < NCHUNK ? keep_of(NCHUNK) : NCHUNK) : 0;
  constexpr int REREAD = NCHUNK - KEEP;            // TV form: chunks of y that pass 2 reads from memory again
  constexpr int FULLCHUNKS = full_chunks(NCHUNK);  // only later chunks can have lanes past the row
  __shared__ float sh_bz[NW], sh_by[NW];
  __shared__ double sh_sz[NW], sh_tz[NW], sh_sy[NW], sh_uy[NW], sh_acc[NW];
  __shared__ RowCoef sh_rc;
  __shared__ float sh_norm[3];
  __shared__ double sh_frac;
  __shared__ int sh_row[2];
  // chunks wave 0 parks around its float64 arithmetic (the TV form's kept chunks of y leave room for
  // 8), and chunks whose refill waits for the epilogue (forward only)
  constexpr int kPark = NCHUNK < 32 ? 0 : TV ? 8 : 16;
  constexpr int kLate = GRAD ? 0 : 8;
  __shared__ u32x4 sh_park[kPark > 0 ? kPark * kWave : 1];
  // every thread parks its own 16 bytes per kept chunk and takes them back itself: no synchronisation
  __shared__ u32x4 sh_y[KEEP > 0 ? KEEP * THREADS : 1];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = uniform_i(tid / kWave);
  const int nvec = p.V >> 3;
  const uint32_t row_bytes = static_cast<uint32_t>(p.V) * 2u;
  const uint32_t voff = static_cast<uint32_t>(tid) * 16u;
  const u32x4 neg_inf = {kNegInfPair, kNegInfPair, kNegInfPair, kNegInfPair};
  const int64_t pitch = p.ld * 2, pitch_y = p.mu_ld * 2;
  const char* zbase = reinterpret_cast<const char*>(p.logits);
  const char* ybase = reinterpret_cast<const char*>(p.mu_logits);
  char* gbase = reinterpret_cast<char*>(p.grad);
  const EpiParams ep = epi_params(p);
  double loss_acc = 0.0;   // meaningful in wave 0 only

  u32x4 buf[NCHUNK];       // the resident row of z; chunk i of thread tid is vector i*THREADS + tid
  u32x4 yb[kWindow];       // the window on y
  // In pass 1 the rollout row is marked non-temporal where it is not read again (KL form); in the
  // TV form the first read is plain, so that the second finds what it can in the caches.
  constexpr bool kY1Nt = !TV;
  // Short rows: both rows are in registers at once, so a thread's offsets are known before its first exponential, and no chunk
  // pays for a maximum of its own and the rescaling (bound by vector arithmetic: 2-3 % of a call; with pass 2's saved subtraction
  // V = 32000, 8192 tokens, TV 351 -> 339 us, KL 318 -> 313; 8200 entries 202 -> 198).
  constexpr bool kWhole = kWindow == NCHUNK;
  // Rows fixed by the workgroup index: neighbouring rows to the workgroups of one die, then every gridDim.x-th.
  // With two workgroups per compute unit the rows left over when all workgroups have had the same number
  // go round the dies instead, one compute unit after the other: as neighbours they were two to a compute
  // unit behind the memory of a die or two (V = 32000, 600 tokens: TV 52.3 us, now 40.3).  And so do the rows
  // of a call of one round, where a die's first rows can all lie on the same memory channel (V = 16384, 512 tokens,
  // KL: 25.3 us, now 21.5).  (One workgroup per compute unit: 2-6 % slower that way at V = 65536 and 131072.)
  constexpr bool kSpread = two_per_cu(NCHUNK);
  const int grid = static_cast<int>(gridDim.x), whole = kSpread ? p.T - p.T % grid : p.T;
  auto row_after = [&](int r) -> int { return !kSpread || r + grid < whole ? r + grid : r < whole ? whole + static_cast<int>(blockIdx.x) : p.T; };
  int row = kSpread && grid == p.T ? static_cast<int>(blockIdx.x) : first_row_of_workgroup();
  int next = row_after(row);
  constexpr int kNoRow = 0x7fffffff;
  if (DYN) {
    if (tid == 0) {
      sh_row[0] = atomicAdd(p.row_counters, 1);
      sh_row[1] = atomicAdd(p.row_counters, 1);
    }
    __syncthreads();
    row = uniform_i(sh_row[0]);
    next = uniform_i(sh_row[1]);
    __syncthreads();
    if (row >= p.T) return;            // every row already handed out: nothing to do, and no address to form
  }
  // (in front of the rows: the compiler's one wait at the head of the loop covers both ways into it)
  int a_next = p.sampled[row];
  __builtin_amdgcn_sched_barrier(0);
  {
    const row_rsrc_t zr = make_row_rsrc(zbase + row * pitch, row_bytes);
    const row_rsrc_t yr = make_row_rsrc(ybase + row * pitch_y, row_bytes);
#pragma unroll
    for (int i = 0; i < NCHUNK; ++i) buf[i] = row_load16<false>(zr, voff, i * kStride);
#pragma unroll
    for (int i = 0; i < kWindow; ++i) yb[i] = row_load16<kY1Nt>(yr, voff, i * kStride);
  }

  for (; row < p.T;) {
    const int a = uniform_i(a_next);
    const bool more = next < p.T;
    if (more) a_next = p.sampled[next];
    // DYN: request the row after next now (thread 0); the answer is published at this row's first barrier
    int drawn = 0, next2 = kNoRow;
    if (DYN && more && tid == 0) drawn = atomicAdd(p.row_counters, 1);
    const bool live = (a >= 0 && a < p.V);
    const uint16_t* zrow = p.logits + static_cast<int64_t>(row) * p.ld;
    const row_rsrc_t yr = make_row_rsrc(ybase + row * pitch_y, row_bytes);
    // The workgroup's next rows; without one the refills go through views of zero bytes: their
    // loads touch no memory.
    const row_rsrc_t zn = make_row_rsrc(zbase + (more ? next : row) * pitch, more ? row_bytes : 0u);
    const row_rsrc_t yn = make_row_rsrc(ybase + (more ? next : row) * pitch_y, more ? row_bytes : 0u);
    const int avec = a >> 3;
    const int ia = live ? avec / THREADS : -1;               // chunk holding a_t (uniform)
    const bool owner = live && (avec - ia * THREADS == tid);
    const int sub = a & 7;

    RowCoef rc;
    rc.coef = 0.f; rc.kexp = 0.f; rc.g_a = 0.f;
    if (live) {
      // Requested now, looked at behind pass 1 (raw bits until then): a use up here would be a wait for
      // everything requested in front of it, i.e. the whole row.
      uint32_t za_bits = zrow[a];
      float packed_scalars = (wid == 0) ? load_row_scalars(p, row, lane) : 0.f;
      // ---- pass 1 ------------------------------------------------------------------------------
      RowStat<DIAG, false> st;       // z, without a_t
      RowStat<false, !TV> cs;        // y, and for the KL form y - z
      if (kWhole) {
#pragma unroll
        for (int i = FULLCHUNKS; i < NCHUNK; ++i)
          if (i * THREADS + tid >= nvec) { buf[i] = neg_inf; yb[i % kWindow] = neg_inf; }
        cs.b = -ceilf(fmaxf(packed_max(yb), kNegBig) * kLog2e);
        st.b = -ceilf(fmaxf(packed_max(buf), kNegBig) * kLog2e);
      }
#pragma unroll
      for (int i = 0; i < NCHUNK; ++i) {
        u32x4 zq = buf[i], yq = yb[i % kWindow];
        if (i + kWindow < NCHUNK) yb[i % kWindow] = row_load16<kY1Nt>(yr, voff, (i + kWindow) * kStride);
        // lanes past the row loaded 0: make them -inf in both rows (they then add nothing)
        if (!kWhole && i >= FULLCHUNKS && i * THREADS + tid >= nvec) { zq = neg_inf; yq = neg_inf; }
        if (TV && i < KEEP) sh_y[i * THREADS + tid] = yq;
        float z[8], y[8];
        unpack8(zq, z);
        unpack8(yq, y);
        if (kWhole) cs.add8_covered(y, z); else cs.add8(y, z);
        // the sampled token's own term is left out of the sum over z (its chunk index is uniform:
        // a scalar test per chunk, the selects run once per row)
        if (i == ia) {
#pragma unroll
          for (int e = 0; e < 8; ++e) z[e] = (owner && e == sub) ? -INFINITY : z[e];
        }
        if (kWhole) st.add8_covered(z, z); else st.add8(z, z);
        // One chunk at a time: the running sums pass through an empty assembly statement, so this
        // chunk's arithmetic is done before the next one's starts.  (Without it the compiler
        // gathers the arithmetic of all chunks behind the last load, with every unpacked value
        // alive at once: over a thousand spilled registers.)
        asm volatile("" : "+v"(st.s), "+v"(st.t), "+v"(st.b), "+v"(cs.s), "+v"(cs.u), "+v"(cs.b));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (TV) {
        // the second pass over y starts to travel while the statistics are combined
#pragma unroll
        for (int i = 0; i < kWindow; ++i)
          if (i < REREAD) yb[i] = row_load16<true>(yr, voff, (KEEP + i) * kStride);
      }
      asm volatile("" : "+v"(za_bits), "+v"(packed_scalars));
      const float z_a = __uint_as_float(za_bits << 16);
      // workgroup-wide offsets = the smallest ones; rescaling to them is exact
      const float wbz = -wave_max(-st.b), wby = -wave_max(-cs.b);
      if (lane == 0) { sh_bz[wid] = wbz; sh_by[wid] = wby; }
      if (DYN && tid == 0) sh_row[0] = more ? drawn : kNoRow;
      __syncthreads();
      if (DYN) next2 = uniform_i(sh_row[0]);
      float bz = -ceilf(fmaxf(z_a, kNegBig) * kLog2e), by = sh_by[0];      // the offset must also cover z[a_t]
#pragma unroll
      for (int w = 0; w < NW; ++w) { bz = fminf(bz, sh_bz[w]); by = fminf(by, sh_by[w]); }
      {
        const double dd = static_cast<double>(bz - st.b), sc = static_cast<double>(fast_exp2(bz - st.b));
        const double scy = static_cast<double>(fast_exp2(by - cs.b));
        const double sd = wave_sum(st.s * sc);
        const double td = DIAG ? wave_sum(sc * (static_cast<double>(st.t) + dd * st.s)) : 0.0;
        const double sy = wave_sum(cs.s * scy);
        const double uy = TV ? 0.0 : wave_sum(static_cast<double>(cs.u) * scy);
        if (lane == 0) { sh_sz[wid] = sd; sh_tz[wid] = td; sh_sy[wid] = sy; sh_uy[wid] = uy; }
      }
      __syncthreads();
      // Wave 0 forms the two normalisers and their logarithms (float64, with its last chunks parked
      // in shared memory meanwhile: beside the resident row there are no registers for that) and,
      // for the TV form, hands what pass 2 needs to the other waves through shared memory.
      double S_rest = 0.0, T_rest = 0.0, Sy = 0.0, Uy = 0.0, l2z = 0.0, l2y = 0.0;
      auto park = [&]() {
        if (kPark > 0) {
#pragma unroll
          for (int i = 0; i < kPark; ++i) sh_park[i * kWave + lane] = buf[NCHUNK - 1 - i];
        }
      };
      auto unpark = [&]() {
        if (kPark > 0) {
#pragma unroll
          for (int i = 0; i < kPark; ++i) buf[NCHUNK - 1 - i] = sh_park[i * kWave + lane];
        }
      };
      if (wid == 0) {
        park();
#pragma unroll
        for (int w = 0; w < NW; ++w) { S_rest += sh_sz[w]; T_rest += sh_tz[w]; Sy += sh_sy[w]; Uy += sh_uy[w]; }
        const double xa = static_cast<double>(z_a) * static_cast<double>(kLog2e) + static_cast<double>(bz);
        const double S = S_rest + exp2_d(xa);
        l2z = log2_d(S);
        l2y = log2_d(Sy);
        if (TV) {
          // The integer part of log2 S goes into the (integer) offset, which stays exact, and only
          // the fractions in [0, 1) remain: y's is left out of pass 2 and applied to its sum in float64, so z's
          // exponents take the difference of the two, in fp32; a probability keeps a relative
          // error of about 1e-7 however large the offset is.
          const double nz = floor(l2z), ny = floor(l2y);
          if (lane == 0) {
            sh_norm[0] = bz - static_cast<float>(nz); sh_norm[1] = by - static_cast<float>(ny);
            sh_norm[2] = static_cast<float>((l2y - ny) - (l2z - nz));
            sh_frac = l2y - ny;
          }
          unpark();
        }
      }
      double D = 0.0;               // meaningful in wave 0
      if (TV) {
        // ---- pass 2: TV = 1/2 sum |pi_j - mu_j| = 1 - sum_j min(pi_j, mu_j) -----------------------
        // One exponential per entry: the minimum is taken on the base-2 log-probabilities
        // z_j*log2e + b - log2 S, both raised by the fraction of y's log2 S
        // (offsets and fractions from wave 0, see above).
        __syncthreads();
        const float bz2 = sh_norm[0], by2 = sh_norm[1], dzy = sh_norm[2];
        double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
        for (int j = 0; j < NCHUNK; ++j) {
          // first the chunks of y that are read again (the LAST ones pass 1 read, a few microseconds
          // ago: part of them is still in the L2), then the ones kept in LDS
          const int i = (j < REREAD) ? KEEP + j : j - REREAD;
          asm volatile("" : "+v"(buf[i]));     // unpack again here: nothing unpacked in pass 1 is kept alive
          u32x4 zq = buf[i], yq;
          if (j < REREAD) {
            yq = yb[j % kWindow];              // last use of the row: non-temporal loads
            if (j + kWindow < REREAD) yb[j % kWindow] = row_load16<true>(yr, voff, (KEEP + j + kWindow) * kStride);
            if (i >= FULLCHUNKS && i * THREADS + tid >= nvec) yq = neg_inf;
          } else {
            yq = sh_y[i * THREADS + tid];      // kept with its lanes past the row already -inf
          }
          if (i >= FULLCHUNKS && i * THREADS + tid >= nvec) zq = neg_inf;
          float z[8], y[8];
          unpack8(zq, z);
          unpack8(yq, y);
          double& acc = (j & 1) ? acc1 : acc0;
          auto mn = [&](int e) { return fast_exp2(fminf(fmaf(z[e], kLog2e, bz2) + dzy, fmaf(y[e], kLog2e, by2))); };
          // eight entries among themselves (pairwise, as they are formed), then into float64
          const float q0 = (mn(0) + mn(1)) + (mn(2) + mn(3)), q1 = (mn(4) + mn(5)) + (mn(6) + mn(7));
          acc += static_cast<double>(q0 + q1);
          asm volatile("" : "+v"(acc0), "+v"(acc1));
          __builtin_amdgcn_sched_barrier(0);
        }
        if (!GRAD) {
          // forward only: nothing needs the rows any more, the next ones start to travel now -- but
          // for the last kLate chunks, whose registers the float64 epilogue of wave 0 works in; they
          // are requested behind it (they are consumed last, and the delay is the epilogue's length)
#pragma unroll
          for (int i = 0; i < NCHUNK - kLate; ++i) buf[i] = row_load16<false>(zn, voff, i * kStride);
#pragma unroll
          for (int i = 0; i < kWindow; ++i) yb[i] = row_load16<kY1Nt>(yn, voff, i * kStride);
          __builtin_amdgcn_sched_barrier(0);
        }
        const double wa = wave_sum(acc0 + acc1);
        if (lane == 0) sh_acc[wid] = wa;
        __syncthreads();
        double tot = 0.0;
        if (wid == 0) {
#pragma unroll
          for (int w = 0; w < NW; ++w) tot += sh_acc[w];
          tot *= exp2_d(-sh_frac);
        }
        D = fmax(1.0 - tot, 0.0);
        if (tot != tot) D = tot;                  // NaN logits propagate
        if (GRAD && wid == 0) park();             // (forward only, the chunks refilled late are free anyway)
      } else if (wid == 0) {
        // KL = E_mu[y - z] - lse(y) + lse(z), the log-sum-exps in base 2 against their offsets
        const double lse2_z = l2z - static_cast<double>(bz), lse2_y = l2y - static_cast<double>(by);
        D = Uy / Sy + kLn2 * (lse2_z - lse2_y);
        D = (D > 0.0 || D != D) ? D : 0.0;       // rounding can leave -1e-8 for identical rows
      }
      // ---- epilogue on wave 0 (inlined but in two shapes, see below) ------------------------------
      // With the gradient the resident row is still needed afterwards, and the epilogue's float64
      // arithmetic finds no registers beside a long one: from 32 chunks on wave 0 parks its last chunks in shared memory around
      // it (its own 16 bytes per lane and chunk, no synchronisation) instead of spilling to scratch
      // memory, whose round trips would sit on the path the other seven waves wait for.
      if (wid == 0) {
        RowScalars rs;
        rs.a = a;
        rs.za = z_a;
        unpack_row_scalars(packed_scalars, rs);
        TopkLane tk;
        tk.id = -1; tk.lp = 0.f; tk.z = 0.f;
        // through an empty asm statement, so that the addresses of the per-token outputs are formed
        // here and not held in registers across the passes
        int row_e = row;
        asm volatile("" : "+s"(row_e));
        // (inlined, in the two shapes that spill most that way a call; us as a call / inlined, 1024 and 8192 tokens: TV V = 16384 36 / 31, 218 / 190,
        // 32000 51 / 47, 336 / 320; KL 16384 35 / 31, 186 / 171; TV 49152 73 / 75, 499 / 524, KL 32000 46 / 47, 306 / 309)
        const RowResult res = NCHUNK == 12 || (!TV && NCHUNK == 8) ? row_epilogue_call(ep, row_e, rs, tk, zrow, bz, S_rest, T_rest, lane, D)
                                          : row_epilogue(ep, row_e, rs, tk, zrow, bz, S_rest, T_rest, lane, D);
        rc = res.rc;
        if (DYN) { if (lane == 0) p.row_loss[row] = res.loss_term; }
        else loss_acc += res.loss_term;
        if (GRAD && lane == 0) sh_rc = rc;
        if (GRAD) unpark();
      }
      // (forward only, this barrier also keeps the next row's statistics from overwriting the
      // shared sums while a slower wave still reads them)
      __syncthreads();
      if (!GRAD) {
#pragma unroll
        for (int i = NCHUNK - kLate; i < NCHUNK; ++i) buf[i] = row_load16<false>(zn, voff, i * kStride);
      }
      if (GRAD) {
        rc.coef = uniform_f(sh_rc.coef);
        rc.kexp = uniform_f(sh_rc.kexp);
        rc.g_a = uniform_f(sh_rc.g_a);
      }
    } else {
      if (tid == 0) {
        p.divergence[row] = 0.f;
        p.mask[row] = 0;
        if (p.loss_tok) p.loss_tok[row] = 0.f;
        if (p.diag) {
          for (int k = 0; k < 8; ++k) p.diag[static_cast<int64_t>(row) * 8 + k] = 0.f;
        }
        if (DYN) p.row_loss[row] = 0.0;
      }
      if (DYN) {
        if (tid == 0) sh_row[0] = more ? drawn : kNoRow;
        __syncthreads();
        next2 = uniform_i(sh_row[0]);
        __syncthreads();
      }
    }

    // ---- gradient out, next rows in -----------------------------------------------------------
    if (!GRAD) {
      if (!live) {       // an ignored row skipped the passes and with them the refill
#pragma unroll
        for (int i = 0; i < NCHUNK; ++i) buf[i] = row_load16<false>(zn, voff, i * kStride);
#pragma unroll
        for (int i = 0; i < kWindow; ++i) yb[i] = row_load16<kY1Nt>(yn, voff, i * kStride);
      }
    } else {
      char* gr = gbase + row * pitch;
      const row_desc_t gout = make_row_desc(gr, row_bytes);
      const uint32_t sgn = (rc.coef < 0.f) ? 0x80008000u : 0u;
      if (rc.coef == 0.f) {
        // Masked, zero-advantage or ignored row: its gradient is exactly zero whatever the logits
        // hold.  Overwrite the resident copy with -inf so that the loop below writes 2^-inf = 0.
#pragma unroll
        for (int i = 0; i < NCHUNK; ++i) buf[i] = neg_inf;
      }
#pragma unroll
      for (int i = 0; i < NCHUNK; ++i) {
        asm volatile("" : "+v"(buf[i]));       // unpack again here: nothing unpacked in an earlier pass is kept alive
        float z[8];
        unpack8(buf[i], z);
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = fast_exp2(fmaf(z[e], kLog2e, rc.kexp));
        const u32x4 o = {pack_bf16x2(z[0], z[1]) ^ sgn, pack_bf16x2(z[2], z[3]) ^ sgn, pack_bf16x2(z[4], z[5]) ^ sgn, pack_bf16x2(z[6], z[7]) ^ sgn};
        row_store16_untracked(gout, voff, i * kStride, o);
      }
      // Keep the instruction scheduler from hoisting the refills above the stores: a refill can
      // only reuse its chunk's registers once the store has been given them.
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NCHUNK; ++i) buf[i] = row_load16<false>(zn, voff, i * kStride);
#pragma unroll
      for (int i = 0; i < kWindow; ++i) yb[i] = row_load16<kY1Nt>(yn, voff, i * kStride);
      __builtin_amdgcn_sched_barrier(0);
      if (rc.coef != 0.f && owner) {
        // The vector store above wrote the softmax term at a_t.  Once it has completed, the owning
        // thread writes the sampled token's own entry over it.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        reinterpret_cast<uint16_t*>(gr)[a] = float_to_bf16_bits(rc.g_a);
      }
    }
    row = next;
    next = DYN ? next2 : row_after(row);
  }
  if (!DYN && tid == 0) p.partial[blockIdx.x] = loss_acc;
}

template <int NCHUNK>
hipError_t launch_chunks(const KParams& p, bool tv, bool grad, int grid, hipStream_t s) {
  const bool diag = p.diag != nullptr, dyn = p.row_counters != nullptr;
  if (dyn && !grad) return hipErrorInvalidValue;       // rows at run time: the gradient forms only
  const dim3 g(grid), b(kThreads);
  constexpr bool kDyn = !two_per_cu(NCHUNK);        // rows at run time: one workgroup per compute unit
  if (dyn && !kDyn) return hipErrorInvalidValue;
#define DPPO_FORM(TVF, D, G, Y) hipLaunchKernelGGL((dppo_fullvocab_resident_kernel<NCHUNK, TVF, D, G, Y>), g, b, 0, s, p)
  if (!grad) {
    if constexpr (NCHUNK >= 32) {
      if (diag) DPPO_FORM(true, true, false, false); else DPPO_FORM(true, false, false, false);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (tv) {
    if (diag) { if (dyn) DPPO_FORM(true, true, true, kDyn); else DPPO_FORM(true, true, true, false); }
    else      { if (dyn) DPPO_FORM(true, false, true, kDyn); else DPPO_FORM(true, false, true, false); }
  } else {
    if constexpr (kl_shape(NCHUNK)) {
      if (diag) { if (dyn) DPPO_FORM(false, true, true, kDyn); else DPPO_FORM(false, true, true, false); }
      else      { if (dyn) DPPO_FORM(false, false, true, kDyn); else DPPO_FORM(false, false, true, false); }
    } else {
      return hipErrorInvalidValue;
    }
  }
#undef DPPO_FORM
  return hipGetLastError();
}

}  // namespace

// Chunks of 512 x 16 bytes that cover a row in this form, 0 where it does not apply.  It applies to
// the backward of both variants and to the forward-only TV form (which reads both rows twice; the
// forward-only KL form reads each row once in the general kernel too), on rows of 98312 .. 155648
// entries, a multiple of 8, every matrix 16-byte aligned with a pitch that is a multiple of 8; to the
// backward from 8200 entries on if there is a row for every compute unit.  Measured against the general
// kernel, which reads what it needs again (us, general / this; TV and KL): V = 98304, 8192 tokens 1285 / 963 and
// 1207 / 842; 65536: 919 / 666 and 930 / 601; 49152, 8192 tokens 595 / 500 (TV); 32000, 8192 tokens 424 / 322
// and 348 / 309; 16384, 8192 tokens 254 / 191 and 202 / 176; 32000, 520 tokens 39 / 32 and 36 / 33.
//
// The KL form's general kernel reads only z again, so idle lanes and waves count: this form needs a row that fills its
// shape, and below 65536 entries (from there on the general kernel runs one workgroup per compute unit, a third
// slower) one that leaves room for a second workgroup.  The lines were drawn when the general kernel made its epilogue as
// a call; inlined, it takes back what few rows gained, and they have not moved.  General = 1, at 256 to 1024 and at 2048 to 8192 tokens: four chunks,
// 10240 entries 0.99-1.02 and 0.98-1.00, 12288 (75 %) 0.95-0.96 and 0.90-0.94, 16384 0.84-0.99 and 0.87-0.94; six, 18432 (75 %) 1.00-1.05 and 0.95-0.99, 20480
// 0.95-0.97 and 0.88-0.94; eight, 24584 (75 %) 1.07-1.16 and 0.98-1.02, 25600 (78 %) 1.08-1.13 and 0.95-1.04, 28672 1.04-1.08 and 0.92-0.97, 32000 0.96-1.01
// and 0.87-0.90; ten, 34816 (85 %) 1.06-1.13 and 0.99-1.02, 35840 (87 %) 1.02-1.08 and 0.96-0.99, 40960 0.98-1.03 and 0.95-0.98; twelve: never (kl_shape).
// With one workgroup per compute unit (14 and 16 chunks) it gains up to four rows per compute
// unit and where many are handed out at run time: 57344 entries 0.83-1.00 and 0.96-1.01, 65528 0.82-0.98 and 0.91-0.96; 51200 (89 %) 0.88-1.09 and 1.01-1.07.
#define DPPO_FULL_SHAPES(X) X(4) X(6) X(8) X(10) X(12) X(14) X(16) X(20) X(24) X(32) X(38)
int fullvocab_resident_chunks(const KParams& p, bool tv, bool grad, int cus) {
  if (!(grad || tv) || !p.mu_logits || p.V % 8 != 0 || p.ld % 8 != 0 || p.mu_ld % 8 != 0) return 0;
  if ((reinterpret_cast<uintptr_t>(p.logits) | reinterpret_cast<uintptr_t>(p.mu_logits) | (grad ? reinterpret_cast<uintptr_t>(p.grad) : 0)) & 15u) return 0;
  const int64_t nvec = p.V / 8;
  if (nvec <= kThreads * 24 && (!grad || p.T < cus || nvec <= kThreads * 2)) return 0;
  auto kl_gains = [&](int c) {
    if (p.V >= 65536) return true;
    const int full = static_cast<int>(32 * nvec / (static_cast<int64_t>(kThreads) * c));       // 32nds of the shape that the row fills
    if (!two_per_cu(c)) return full >= 30 && (p.T <= 4 * cus || p.T >= 16 * cus);
    return kl_shape(c) && full >= (c == 4 ? 24 : c <= 8 ? 25 : 28);
  };
#define DPPO_FULL_TRY(C) if (nvec <= kThreads * C) return (tv || kl_gains(C)) ? C : 0;
  DPPO_FULL_SHAPES(DPPO_FULL_TRY)
#undef DPPO_FULL_TRY
  return 0;
}

int fullvocab_resident_per_cu(int chunks) { return two_per_cu(chunks) ? 2 : 1; }

hipError_t launch_fullvocab_resident(const KParams& p, bool tv, bool grad, int chunks, int grid, hipStream_t s) {
#define DPPO_FULL_LAUNCH(C) if (chunks == C) return launch_chunks<C>(p, tv, grad, grid, s);
  DPPO_FULL_SHAPES(DPPO_FULL_LAUNCH)
#undef DPPO_FULL_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace dppo
