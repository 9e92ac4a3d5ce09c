// bf16 matrix product on the matrix cores, C[M, N] = A[M, K] * B[N, K]^T with fp32 accumulation:
// both operands row-major with the contraction index contiguous (what an nn.Linear forward is:
// activations [T, d] times weight [V, d] transposed), C row-major: bf16 rounded to nearest even,
// or fp32, optionally added to what C holds.
//
// Workgroups of 256 threads (4 waves, one per SIMD), one per compute unit, form 256 x 256 tiles of C, each wave a
// 128 x 128 quadrant as 8 x 8 products of v_mfma_f32_16x16x32_bf16 (256 fp32 accumulators per
// lane, the whole accumulation register file).  That shape is chosen for power: with every
// compute unit busy the clock is set by the power limit, and a loop of nothing but 16x16x32
// products sustains about 13 % more than one of 32x32x16 products (measured, 2.2-2.3 against
// 1.9-2.0 PFLOP/s).  The contraction runs in steps of 64: the A and B panels of a step (256 x 64
// each, 32 KiB) are loaded from global memory straight into LDS, 16 bytes per
// lane, in a layout swizzled so that the fragment reads (one 16-byte read per lane: 8 consecutive
// k of one row) spread over all banks.
// What bounds it besides the power limit is the latency of those loads: a step is 2048 cycles of products, loads from beyond the L2 take as long, and a panel's
// place is free only from the middle of its own step on.  So all 160 KiB of LDS are panels, five of them: two of the near operand (activations,
// which the Infinity Cache holds), loaded a step and a half ahead, three of the far one (the weight; the logits' gradient for the weight's), loaded
// two and a half ahead.  And a workgroup forms several tiles one behind the other: the next tile's first panels are loaded during the last steps of a
// tile, whose stores travel behind the next one's products.  Measured, us, V = 151936, one tile per workgroup and two panels each / as it is:
// A B^T 300 x 2048 267 / 233, 1000 x 2048 519 / 491, 2048 x 1024 591 / 538, 2048 x 2048 1007 / 940, 8192 x 1024 2162 / 2028, 8192 x 4096 6841 / 6717; A B 1000 x 2048 3110 / 2750,
// 8192 x 4096 6902 / 6677; bf16 A^T B 1000 x 2048 608 / 544, 2048 x 2048 1045 / 947, 4096 x 4096 3790 / 3420, 8192 x 4096 7407 / 7213 (fp32, added to C, 8174 / 7930).  One round of tiles whose
// operands the L2 holds is up to 2.5 % slower (A B^T 4096 x 4096, K = 8192: 175 / 179).
// (With operands of zeros, which draw no power, 2048 x 2048 931 / 760, of 520 for the products alone: 130 of the rest are the stores, whose 32 MiB leave at
// once and fill the dies' way to memory for five microseconds; held back in registers and spread over the next tile's first six steps they cost the
// same but for 1 %, written in whole lines through shared memory too.)
// A 16x16x32 product occupies the matrix pipe for 16 cycles and a wave issues at most one
// instruction every 4, so whatever else the wave issues has to sit in the shadow of a product:
// the matrix-core instructions are written as assembly statements in a fixed order (that also
// keeps each accumulator in place in its own registers, which the register allocator does not
// manage by itself at this pressure), with one fragment read or one panel load pinned behind
// every second to fourth of them.
// Panel rows past M or N are zeros (their products are never stored): all
// loads go through range-checked buffer resources over exactly the rows a tile owns.  K must be
// a multiple of 64, rows 16-byte aligned (checked by the host).
//
// A second form of the same kernel takes both operands with the contraction index as the ROW
// index, C[M, N] = A[K, M]^T * B[K, N] (what the gradient of a weight is: logit gradients [T, V]
// transposed times activations [T, d]), with no transposed copies: the panels of a step are 64
// rows of 512 bytes, and the LDS transpose read (ds_read_b64_tr_b16) hands every lane the
// consecutive k of one column.  There K is arbitrary: rows past it read as zeros.
#include <algorithm>
#include <type_traits>
#include <utility>
#include "dppo_common.hpp"
#include "dppo_launch.hpp"

namespace dppo {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// f(std::integral_constant<int, 0>{}), ..., f(N - 1): a loop whose index is a constant
template <typename F, int... I>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled(std::make_integer_sequence<int, N>{}, f);
}

// The accumulators of a 256 x 256 tile are the whole accumulation register file, named in the statements that use it: block (i, j) of 16 x 16 is
// a[4 (8 i + j)] .. + 3.  As values of the compiler's they were moved, some between a tile's products and some in front of its stores, wherever
// a workgroup forms one tile behind another, and it does not keep the distances that such moves need from products in assembly statements.
// The compiler itself uses this file for nothing unless it runs out of the other 256 registers: the build compiles this source with spills to it switched
// off and refuses assembly that mentions one of its registers outside the statements below, whatever the compiler's version.
template <int M, bool FIRST>
__device__ __forceinline__ void product(bf16x8 x, bf16x8 y) {      // block M += x y, or = x y
  if constexpr (FIRST) asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, 0" ::"v"(x), "v"(y), "n"(4 * M), "n"(4 * M + 3));
  else                 asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(x), "v"(y), "n"(4 * M), "n"(4 * M + 3));
}
template <int R>
__device__ __forceinline__ float accumulator() {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(R));
  return v;
}
// row block I: eight blocks of four columns each per lane
template <int I>
__device__ __forceinline__ void accumulators(f32x4 (&row)[8]) {
  unrolled<8>([&](auto j) __attribute__((always_inline)) {
    constexpr int R = 4 * (8 * I + decltype(j)::value);
    row[decltype(j)::value] = f32x4{accumulator<R>(), accumulator<R + 1>(), accumulator<R + 2>(), accumulator<R + 3>()};
  });
}
// the whole file is in use (what the register count of a kernel is taken from)
#define DPPO_ALL_ACCUMULATORS() asm volatile("" ::: "a0","a1","a2","a3","a4","a5","a6","a7","a8","a9","a10","a11","a12","a13","a14","a15","a16","a17","a18","a19","a20","a21","a22","a23","a24","a25","a26","a27","a28","a29","a30","a31", \
  "a32","a33","a34","a35","a36","a37","a38","a39","a40","a41","a42","a43","a44","a45","a46","a47","a48","a49","a50","a51","a52","a53","a54","a55","a56","a57","a58","a59","a60","a61","a62","a63", \
  "a64","a65","a66","a67","a68","a69","a70","a71","a72","a73","a74","a75","a76","a77","a78","a79","a80","a81","a82","a83","a84","a85","a86","a87","a88","a89","a90","a91","a92","a93","a94","a95", \
  "a96","a97","a98","a99","a100","a101","a102","a103","a104","a105","a106","a107","a108","a109","a110","a111","a112","a113","a114","a115","a116","a117","a118","a119","a120","a121","a122","a123","a124","a125","a126","a127", \
  "a128","a129","a130","a131","a132","a133","a134","a135","a136","a137","a138","a139","a140","a141","a142","a143","a144","a145","a146","a147","a148","a149","a150","a151","a152","a153","a154","a155","a156","a157","a158","a159", \
  "a160","a161","a162","a163","a164","a165","a166","a167","a168","a169","a170","a171","a172","a173","a174","a175","a176","a177","a178","a179","a180","a181","a182","a183","a184","a185","a186","a187","a188","a189","a190","a191", \
  "a192","a193","a194","a195","a196","a197","a198","a199","a200","a201","a202","a203","a204","a205","a206","a207","a208","a209","a210","a211","a212","a213","a214","a215","a216","a217","a218","a219","a220","a221","a222","a223", \
  "a224","a225","a226","a227","a228","a229","a230","a231","a232","a233","a234","a235","a236","a237","a238","a239","a240","a241","a242","a243","a244","a245","a246","a247","a248","a249","a250","a251","a252","a253","a254","a255")

constexpr int kBM = 256, kBN = 256, kBK = 64;
constexpr int kRowBytes = kBK * 2;                    // one panel row in LDS: 128 bytes = 8 vectors
constexpr int kPanelBytes = kBM * kRowBytes;          // 32 KiB (kBM == kBN)

// LDS byte offset of the 16-byte vector `kvec` (0..7) of panel row `row`: the vector index is
// XOR-ed with bits 1..3 of the row, so 16 consecutive rows at one kvec cover all 64 banks once.
__device__ __forceinline__ uint32_t lds_off(int row, int kvec) {
  return static_cast<uint32_t>(row) * kRowBytes + static_cast<uint32_t>((kvec ^ ((row >> 1) & 7)) << 4);
}

// 16 rows x 128 columns of a tile (eight accumulators of four columns each) leave as bf16: row `row` of this lane, from column col0
// on.  Two neighbouring blocks exchange halves between lane rows (one v_permlane16_swap per register pair), after
// which a lane owns 8 consecutive columns: one 16-byte store, 64 contiguous bytes per row and instruction.
template <bool FULL>
__device__ __forceinline__ void store_row_block_bf16(uint16_t* __restrict__ C, int64_t ldc, int M, int N, int row, int col0, int fk, const f32x4 (&acc)[8]) {
  const bool quad_aligned = ((reinterpret_cast<uintptr_t>(C) & 15u) == 0) && (ldc % 8 == 0);
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const uint32_t lo0 = pack_bf16x2(acc[j][0], acc[j][1]), hi0 = pack_bf16x2(acc[j][2], acc[j][3]);
    const uint32_t lo1 = pack_bf16x2(acc[j + 1][0], acc[j + 1][1]), hi1 = pack_bf16x2(acc[j + 1][2], acc[j + 1][3]);
    if (quad_aligned) {
      const auto l = __builtin_amdgcn_permlane16_swap(lo0, lo1, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap(hi0, hi1, false, false);
      const u32x4 v = {l[0], h[0], l[1], h[1]};
      const int col = col0 + (j + (fk & 1)) * 16 + (fk >> 1) * 8;
      uint16_t* dst = C + static_cast<int64_t>(row) * ldc + col;
      // (a tile with rows or columns past the matrix: the same 16-byte stores, but for a vector across the
      // matrix's edge.  Two bytes at a time for the whole tile, one of four: 1000 x 151936 x 2048 0.75 ms, now 0.53.)
      if (FULL || (row < M && col + 8 <= N)) {
        *reinterpret_cast<u32x4*>(dst) = v;
      } else if (row < M) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (col + e < N) dst[e] = static_cast<uint16_t>((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu));
      }
    } else if (row < M) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = col0 + (j + h) * 16 + fk * 4;
        const uint32_t lo = h ? lo1 : lo0, hi = h ? hi1 : hi0;
        uint16_t* dst = C + static_cast<int64_t>(row) * ldc + col;
        if (col < N) dst[0] = static_cast<uint16_t>(lo & 0xffffu);
        if (col + 1 < N) dst[1] = static_cast<uint16_t>(lo >> 16);
        if (col + 2 < N) dst[2] = static_cast<uint16_t>(hi & 0xffffu);
        if (col + 3 < N) dst[3] = static_cast<uint16_t>(hi >> 16);
      }
    }
  }
}

// The same 16 rows x 128 columns, all in the matrix and on lines of 128 bytes, in whole lines: through `room` (this wave's own, kLineRoom bytes), where a row is
// 16 vectors of 16 bytes, vector v in place v ^ row, so that neither side meets its own banks; a store is four rows of 256 bytes then.
// Past the caches: a result is written once, and what many tiles store at the same time would take the L2 from the operands.  (In 64-byte pieces the
// same mark costs a third of the rate.)
constexpr int kLineRoom = 16 * 256;
__host__ __device__ __forceinline__ bool result_on_lines(const void* C, int64_t ldc) { return (reinterpret_cast<uintptr_t>(C) & 127u) == 0 && ldc % 64 == 0; }
__device__ __forceinline__ void store_row_block_lines(uint16_t* __restrict__ C, int64_t ldc, int lane, const f32x4 (&acc)[8], unsigned char* room) {
  const int frow = lane & 15, fk = lane >> 4;
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const auto l = __builtin_amdgcn_permlane16_swap(pack_bf16x2(acc[j][0], acc[j][1]), pack_bf16x2(acc[j + 1][0], acc[j + 1][1]), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(pack_bf16x2(acc[j][2], acc[j][3]), pack_bf16x2(acc[j + 1][2], acc[j + 1][3]), false, false);
    *reinterpret_cast<u32x4*>(room + frow * 256 + ((((j + (fk & 1)) * 2 + (fk >> 1)) ^ frow) << 4)) = u32x4{l[0], h[0], l[1], h[1]};
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = q * 4 + (lane >> 4), v = lane & 15;
    __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(room + r * 256 + ((v ^ r) << 4)), reinterpret_cast<u32x4*>(C + static_cast<int64_t>(r) * ldc + v * 8));
  }
}

// OUT selects what leaves a tile: bf16 (rounded to nearest even), fp32, or fp32 added to what C holds.
// kOutStats: nothing of C is stored.  The tile's logits, rounded to bf16 as a stored tile would be,
// leave as softmax statistics per row (GemmStats below): the forward of the hidden-state path then
// never writes a logit to memory.
// kOutSplit: the contraction is cut into ranges of steps, and the tile of a range leaves as fp32 for a second
// kernel to add up (see gemm_nn_splits).
enum : int { kOutBf16 = 0, kOutF32 = 1, kOutF32Add = 2, kOutStats = 3, kOutSplit = 4 };

// What leaves a tile of kOutStats.  Per row of the tile, over its 256 columns (those below N), of the logits ROUNDED to bf16:
// the integer offset b = -ceil(max * log2e), s = sum 2^(z*log2e + b) and t = sum 2^x * x (for
// the entropy), the row's sampled token left out as in the loss kernels.  A lane holds 32
// columns of each of its 8 rows; the four lanes of a row (lane, lane+16, +32, +48) combine by
// register swaps, the two waves of a row through shared memory.  The logit of the row's sampled token leaves from the registers (one tile in V / 256 holds it).
// With top-K ids the rounded tile itself goes to shared memory, into the panels of the products (64 rows of 512 bytes each, 32-byte blocks
// XOR-ed with the row so that a 16-lane write spreads over the banks), from where the logits at the ids that fall into this tile are picked.
// A value of each of the four rows of 16 lanes, combined over the rows in every lane (register swaps between lane rows: a shuffle through shared memory is 120 cycles
// that a wave alone on its SIMD waits for).
template <typename F>
__device__ __forceinline__ float across_rows(float v, F&& f) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
struct StatRoom {
  float part[2][kBM][3];
};
// quarter: room for 64 rows of the tile each.  Columns that do not exist come in whole blocks of 16 (the host sees to that), rows that do not
// exist are zeros and leave nothing.
__device__ __forceinline__ void tile_statistics(const int (&samp)[8], int M, int N, int m0, int n0, const GemmStats& gs, StatRoom& sh,
                                                unsigned char* const (&quarter)[4], int wid, int lane) {
  const int tid = wid * 64 + lane, wm = wid >> 1, wn = wid & 1, frow = lane & 15, fk = lane >> 4;
  const int K1 = gs.Ktop + 1;
  const int col0 = n0 + wn * 128;        // first column of this wave's quadrant
  unrolled<8>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    f32x4 acc[8];
    accumulators<i>(acc);
    const int rl = wm * 128 + i * 16 + frow;            // row inside the tile
    const int row = m0 + rl;
    const int a_loc = (row < M && samp[i] >= 0 && samp[i] < N) ? samp[i] - col0 : -1;
    float z[8][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t lo = pack_bf16x2(acc[j][0], acc[j][1]), hi = pack_bf16x2(acc[j][2], acc[j][3]);
      z[j][0] = __uint_as_float(lo << 16); z[j][1] = __uint_as_float(lo & 0xffff0000u);
      z[j][2] = __uint_as_float(hi << 16); z[j][3] = __uint_as_float(hi & 0xffff0000u);
    }
    if (gs.Ktop > 0) {
      unsigned char* rows = (wm ? quarter[2 + i / 4] : quarter[i / 4]) + ((i & 3) * 16 + frow) * 512;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2*>(rows + (((wn * 8 + j) ^ frow) << 5) + fk * 8) =
            u32x2{(__float_as_uint(z[j][0]) >> 16) | __float_as_uint(z[j][1]), (__float_as_uint(z[j][2]) >> 16) | __float_as_uint(z[j][3])};
      }
    }
    if (N - col0 < 128) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (col0 + j * 16 >= N) z[j][0] = z[j][1] = z[j][2] = z[j][3] = -INFINITY;
    }
    // The sampled token (rarely: one tile in V / 256 holds a row's), picked by selection and stored once: a store per column, each behind a branch of its own, was 256
    // branches a tile, 8 us where every column was looked at.
    if (__any(a_loc >= 0 && a_loc < 128)) {
      const int e_loc = a_loc - fk * 4;
      float za = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool here = e_loc == j * 16 + e;
          za = here ? z[j][e] : za;
          z[j][e] = here ? -INFINITY : z[j][e];
        }
      if (a_loc >= 0 && a_loc < 128 && ((a_loc >> 2) & 3) == fk) gs.gath[static_cast<int64_t>(row) * K1] = za;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 8; ++j) mx = fmaxf(fmaxf(fmaxf(mx, z[j][0]), z[j][1]), fmaxf(z[j][2], z[j][3]));
    mx = across_rows(mx, [](float x, float y) { return fmaxf(x, y); });
    const float b = -ceilf(fmaxf(mx, kNegBig) * kLog2e);
    float s = 0.f, t = 0.f;
    if (gs.want_t) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float e4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = fmaf(z[j][e], kLog2e, b);
          e4[e] = fast_exp2(x);
          t = fma_ex(e4[e], x, t);
        }
        s += (e4[0] + e4[1]) + (e4[2] + e4[3]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        s += (fast_exp2(fmaf(z[j][0], kLog2e, b)) + fast_exp2(fmaf(z[j][1], kLog2e, b))) +
             (fast_exp2(fmaf(z[j][2], kLog2e, b)) + fast_exp2(fmaf(z[j][3], kLog2e, b)));
    }
    s = across_rows(s, [](float x, float y) { return x + y; });
    if (gs.want_t) t = across_rows(t, [](float x, float y) { return x + y; });
    if (fk == 0) { sh.part[wn][rl][0] = b; sh.part[wn][rl][1] = s; sh.part[wn][rl][2] = t; }
  });
  __syncthreads();
  {
    const int row = m0 + tid;
    const float b0 = sh.part[0][tid][0], b1 = sh.part[1][tid][0], b = fminf(b0, b1);
    const float d0 = b - b0, d1 = b - b1, c0 = fast_exp2(d0), c1 = fast_exp2(d1);       // exact powers of two
    const float s = sh.part[0][tid][1] * c0 + sh.part[1][tid][1] * c1;
    const float t = c0 * fmaf(d0, sh.part[0][tid][1], sh.part[0][tid][2]) + c1 * fmaf(d1, sh.part[1][tid][1], sh.part[1][tid][2]);
    if (row < M) gs.part[static_cast<int64_t>(row) * gs.tiles_n + n0 / kBN] = f32x4{b, s, t, 0.f};
  }
  // ids fetched 22 at a time, one memory latency: 20 ids a row in one go, 64 in three.  Us, 16 at a time / 22: 300 x 4096 x 768 with 20 ids 35.6 / 34.6,
  // 5000 x 50304 x 768 435 / 424, with 64 497 / 494, with 8 407 / 414.
  const int n_ids = min(kBM, M - m0) * gs.Ktop;
  const int32_t* ids = gs.tk_ids + static_cast<int64_t>(m0) * gs.Ktop;
  constexpr int kAhead = 22;
  for (int i0 = tid; i0 < n_ids; i0 += kAhead * kBM) {
    int id[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) id[u] = (i0 + u * kBM < n_ids) ? ids[i0 + u * kBM] : -1;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int c = id[u] - n0;
      if (id[u] >= 0 && c >= 0 && c < kBN && id[u] < N) {
        const int idx = i0 + u * kBM, r = idx / gs.Ktop, k = idx - r * gs.Ktop, q = r >> 6;
        const unsigned char* rows = q == 0 ? quarter[0] : q == 1 ? quarter[1] : q == 2 ? quarter[2] : quarter[3];
        gs.gath[static_cast<int64_t>(m0 + r) * K1 + 1 + k] =
            bf16_bits_to_float(*reinterpret_cast<const uint16_t*>(rows + (r & 63) * 512 + (((c >> 4) ^ (r & 15)) << 5) + (c & 15) * 2));
      }
    }
  }
}

// Workgroup ids go round-robin over the 8 accelerator dies, each with its own L2.  Tiles are
// numbered block by block, a block being group_m x group_n tiles, at most 32, the number of workgroups
// that run together on a die, and each die gets a contiguous range of numbers: with 8 x 4 the workgroups sharing
// an L2 at any time share 8 A panels and 4 B panels (12 panel streams for 32 tiles).  Blocks at the
// edge are cut to the matrix: a number outside it would wait for a compute unit with free shared memory like
// any other workgroup (with whole blocks of 8 x 4 over one tile of rows seven of eight were: 64 tokens x 1024
// wide, logits + loss + hidden gradient 0.57 ms, now 0.23).  Blocks are 8 high where 8 divides the matrix's height or it is
// tall, the matrix's height below 8, else 4 high and 8 wide (18 x 127 tiles: 0.91 of the time with blocks of 6 x 5, 14 x 391: 0.94).
//
// Edge blocks are left whole, so that the rounds of 32 workgroups stay in step with the blocks, where that is
// less than 3 % of the numbers (the weight gradient at V = 151936, 594 tiles high: 7.8 ms, cut 8.4), and in blocks of 8 x 4,
// whole ones to each die, where cutting them saves no round (`even`), of whole 8 x 4 blocks / cut:
//  * tall matrices with as many rounds on the fullest die: 154 x 16 tiles 374 / 407 us, 171 x 15 1074 / 1196; and, where a
//    tile has at most 24 steps and is bound by its store, up to 15 % more: 594 x 7 tiles of 5 and 10 steps 372 / 396 and 480 / 522,
//    259 x 15 of 3 278 / 289 (of 64 steps, 594 x 7: 2079 / 1910; with a quarter more rounds, 143 x 7 of 17 steps: 199 / 171);
//  * contractions of 256 steps and more over two rounds or more (20 x 16 tiles, 2374 steps: 6687 / 6870, 32 x 14: 1496 / 1562): the
//    same rounds on fewer compute units at a higher clock.
struct TileMap {
  int tiles_m, tiles_n, group_m, group_n;
  int tiles;               // tiles_m * tiles_n
  int numbers, per_die;    // the same with whole edge blocks where the shares of the dies count those; a die's share (of all ranges)
  int split_steps;         // kOutSplit: steps of a range of the contraction
  int slots, run;          // workgroups of a die that run side by side; tiles each forms, one behind the other
  int start[9];            // die d: the tiles (of all ranges of the contraction) numbered start[d] .. start[d + 1] - 1
};
// A run is eight tiles at most, so that a workgroup that starts late, another kernel being on its compute unit, holds up no more than that, and 512 steps at
// most; tiles of 128 steps and more are worth no run: they gain a per cent by it, and workgroups that drift apart lose the panels they
// share.  Runs of 1 / 2 / 4 / 8 / 32 tiles, us, V = 151936: A B^T 2048 x 2048 975 / 954 / 943 / 938 / 933, 8192 x 4096 6838 / 6770 / 6738 / 6735 / 6712; A^T B
// 2048 x 2048 983 / 958 / 950 / 945 / 944, 8192 x 4096 (128 steps) 7150 / 7283 / 7377 / 7464 / 7570.
// No runs: a divided contraction (kOutSplit), which has 128 steps and more in all, and the statistics (kOutStats), which store next to nothing, want all of the panels for
// the tile with top-K ids, and with a next tile on its way keep more addresses than there are scalar registers.  Forward only, us, in runs (but for top-K ids,
// where the code for them stood unused) / without: 2048 x 50304 x 768 162 / 158, with 20 ids 210 / 189, of one workgroup per tile and two panels each 171 and 201; 64 x 32768 x 768 32.1 / 30.3, 38.5 / 35.0, 32.8 and 37.0;
// 2048 x 151936 x 2048 973 / 970, 1057 / 1021, 1015 and 1072; 8192 x 151936 x 4096 6925 / 6904, 7287 / 7144, 6990 and 7237.
constexpr int kMaxRun = 8;
TileMap tile_map(int64_t M, int64_t N, int64_t K, int64_t ranges, int cus, int max_run = kMaxRun) {
  TileMap t;
  t.tiles_m = static_cast<int>((M + kBM - 1) / kBM);
  t.tiles_n = static_cast<int>((N + kBN - 1) / kBN);
  const int64_t tiles = static_cast<int64_t>(t.tiles_m) * t.tiles_n, steps = (K + kBK - 1) / kBK;
  const bool tall = t.tiles_m >= 4 * static_cast<int64_t>(t.tiles_n);
  // whole blocks of 8 x 4, as many on each die: the tiles of the first die, which has the most, and its rounds of 32; and the same cut
  const int64_t blocks_m = (t.tiles_m + 7) / 8, blocks = (blocks_m * ((t.tiles_n + 3) / 4) + 7) / 8;
  const int64_t first = (blocks / blocks_m * t.tiles_m + std::min<int64_t>(blocks % blocks_m * 8, t.tiles_m)) * std::min(t.tiles_n, 4);
  const int64_t whole_rounds = (first + 31) / 32, cut_rounds = ((tiles + 7) / 8 + 31) / 32;
  const bool even = ranges == 1 && ((tall && (whole_rounds == cut_rounds || (steps <= 24 && whole_rounds * 100 <= cut_rounds * 115))) ||
                                    (steps >= 256 && cut_rounds >= 2 && whole_rounds == cut_rounds));
  t.group_m = even || t.tiles_m % 8 == 0 || (tall && t.tiles_m > 8) ? 8 : t.tiles_m < 8 ? t.tiles_m : 4;
  t.group_n = 32 / t.group_m;
  const int64_t whole_m = (t.tiles_m + t.group_m - 1) / t.group_m * t.group_m, whole_n = (t.tiles_n + t.group_n - 1) / t.group_n * t.group_n;
  const bool whole = even || (t.group_m * t.group_n == 32 && whole_m * whole_n * 100 < tiles * 103);
  const int64_t rows = whole ? whole_m : t.tiles_m, cols = whole ? whole_n : t.tiles_n;
  const int64_t share = (rows * cols * ranges + 7) / 8;
  // from eight rounds of workgroups per die on, dies start with a whole block (the last round is partly empty either way)
  const int64_t per_die = even || share >= 256 ? (share + 31) / 32 * 32 : share;
  t.tiles = static_cast<int>(tiles);
  t.numbers = static_cast<int>(rows * cols);
  t.per_die = static_cast<int>(per_die);
  t.split_steps = 0;
  // tiles in front of number v, edge blocks counted as the dies' shares count them (whole or cut)
  auto before = [&](int64_t v) -> int64_t {
    const int64_t range = v / (rows * cols);
    if (range >= ranges) return ranges * tiles;
    v -= range * rows * cols;
    const int64_t bn = v / (t.group_n * rows);
    v -= bn * t.group_n * rows;
    const int64_t width = std::min<int64_t>(t.group_n, cols - bn * t.group_n), real_width = std::min<int64_t>(t.group_n, t.tiles_n - bn * t.group_n);
    const int64_t bm = v / (t.group_m * width);
    v -= bm * t.group_m * width;
    const int64_t height = std::min<int64_t>(t.group_m, rows - bm * t.group_m), real_height = std::min<int64_t>(t.group_m, t.tiles_m - bm * t.group_m);
    const int64_t q = v / height, r = v % height;
    return range * tiles + bn * t.group_n * t.tiles_m + bm * t.group_m * real_width + std::min(q, real_width) * real_height +
           (q < real_width ? std::min(r, real_height) : 0);
  };
  int64_t most = 0;
  for (int d = 0; d <= 8; ++d) {
    t.start[d] = static_cast<int>(d == 8 ? ranges * tiles : before(d * per_die));
    if (d > 0) most = std::max<int64_t>(most, t.start[d] - t.start[d - 1]);
  }
  t.slots = static_cast<int>(std::min<int64_t>(most, std::max(1, cus / 8)));
  const int64_t rounds = (most + t.slots - 1) / t.slots;
  t.run = static_cast<int>(std::min<int64_t>(rounds, steps >= 128 ? 1 : std::max<int64_t>(1, std::min<int64_t>(max_run, 512 / steps))));
  return t;
}
inline dim3 tile_grid(const TileMap& t) {
  int most = 0;
  for (int d = 0; d < 8; ++d) most = std::max(most, t.start[d + 1] - t.start[d]);
  const int per_run = t.slots * t.run;
  return dim3(8u * static_cast<unsigned>(t.slots) * static_cast<unsigned>((most + per_run - 1) / per_run));
}

// One tile as the kernel sees it: the operands from the tile's first row (by rows: column) and the range's first k on.
struct TileAt {
  const uint16_t *a, *b;
  void* c;
  uint32_t bytes_a, bytes_b;      // of the views below
  int m0, n0, K;
};

// TA: A is [K, M]; TB: B is [K, N] (the contraction index is the ROW index of that operand; with
// both, C = A^T B; with TB alone, C = A B).  The panel of such an operand
// is then 64 rows of 512 bytes per step, and its fragment reads use the LDS transpose read
// (ds_read_b64_tr_b16: out of a 16-lane group's sixteen 8-byte blocks, lane i gets element i%4 of
// the blocks i/4, i/4 + 4, i/4 + 8, i/4 + 12), which turns four k rows of four neighbouring m
// into the four consecutive k of one m that a matrix-core operand wants.
//
// A workgroup forms a run of tiles (TileMap::run), one behind the other: while it multiplies the last steps of a
// tile it already loads the first of the next, and its stores travel behind the next tile's products (kOutSplit and kOutStats: one tile, the host asks for runs of one).
template <int OUT, bool TA, bool TB>
__global__ __launch_bounds__(256) void dppo_gemm_nt_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                           const uint16_t* __restrict__ B, int64_t ldb,
                                                           void* __restrict__ C, int64_t ldc, int M, int N, int K,
                                                           const TileMap map, const GemmStats gs) {
  // Five panels, all of the compute unit's shared memory: three of the operand that comes from far (`far`: A if FAR_A), two of the other.
  __shared__ __attribute__((aligned(16))) unsigned char panel0[kPanelBytes];
  __shared__ __attribute__((aligned(16))) unsigned char panel1[kPanelBytes];
  __shared__ __attribute__((aligned(16))) unsigned char panel2[kPanelBytes];
  __shared__ __attribute__((aligned(16))) unsigned char panel3[kPanelBytes];
  __shared__ __attribute__((aligned(16))) unsigned char panel4[kPanelBytes];
  auto far_panel = [&](int step) { return step % 3 == 0 ? panel0 : step % 3 == 1 ? panel1 : panel2; };
  auto near_panel = [&](int step) { return step % 2 == 0 ? panel3 : panel4; };
  constexpr bool FAR_A = TA;
  constexpr bool RUNS = OUT != kOutSplit && OUT != kOutStats;
  const int tid = threadIdx.x, lane = tid & 63, wid = uniform_i(tid >> 6);
  const int wm = wid >> 1, wn = wid & 1;

  // This workgroup's run: `map.run` tiles of its die, `map.slots` apart.
  const int die = static_cast<int>(blockIdx.x) & 7, nth = static_cast<int>(blockIdx.x) >> 3;      // nth workgroup of its die
  const int group = nth / map.slots;
  const int first = map.start[die] + group * map.slots * map.run;
  const int end = min(first + map.slots * map.run, map.start[die + 1]);
  int number = first + (nth - group * map.slots);
  if (number >= end) return;

  // requested here: no store waits for it
  const float factor = (OUT == kOutBf16 && TA && TB) ? uniform_f(*gs.factor) : 1.f;
  const uint32_t pitch_a = static_cast<uint32_t>(lda) * 2u, pitch_b = static_cast<uint32_t>(ldb) * 2u;
  auto locate = [&](int v) -> TileAt {
    TileAt t;
    t.a = A; t.b = B; t.c = C; t.K = K;
    if (OUT == kOutSplit) {
      // the range of the contraction is the outermost index, so the workgroups of a die still share panels
      const int split = v / map.tiles, k0 = split * map.split_steps * kBK;
      v -= split * map.tiles;
      t.a += TA ? static_cast<int64_t>(k0) * lda : static_cast<int64_t>(k0);
      t.b += TB ? static_cast<int64_t>(k0) * ldb : static_cast<int64_t>(k0);
      t.c = static_cast<float*>(C) + static_cast<int64_t>(split) * M * ldc;
      t.K = min(K - k0, map.split_steps * kBK);
    }
    // blocks run down the matrix, then on to the next group_n columns of tiles
    const int bn = v / (map.group_n * map.tiles_m);
    v -= bn * (map.group_n * map.tiles_m);
    const int width = min(map.group_n, map.tiles_n - bn * map.group_n);
    const int bm = v / (map.group_m * width);
    v -= bm * (map.group_m * width);
    const int height = min(map.group_m, map.tiles_m - bm * map.group_m);
    const int q = v / height;
    t.m0 = (bm * map.group_m + v - q * height) * kBM;
    t.n0 = (bn * map.group_n + q) * kBN;
    t.a += TA ? static_cast<int64_t>(t.m0) : static_cast<int64_t>(t.m0) * lda;
    t.b += TB ? static_cast<int64_t>(t.n0) : static_cast<int64_t>(t.n0) * ldb;
    // by rows: bytes of a row from the tile's first column on, in whole 16-byte vectors (the range
    // check works per 4 bytes, and the pitch, a multiple of 8 entries, covers them); else: bytes of the tile's rows
    t.bytes_a = TA ? ((static_cast<uint32_t>(M - t.m0) * 2u + 15u) & ~15u) : static_cast<uint32_t>(min(kBM, M - t.m0) - 1) * pitch_a + static_cast<uint32_t>(t.K) * 2u;
    t.bytes_b = TB ? ((static_cast<uint32_t>(N - t.n0) * 2u + 15u) & ~15u) : static_cast<uint32_t>(min(kBN, N - t.n0) - 1) * pitch_b + static_cast<uint32_t>(t.K) * 2u;
    return t;
  };
  // both by rows: rows past K read as zeros (range check)
  auto steps_of = [&](const TileAt& t) { return uniform_i((TA && TB) ? (t.K + kBK - 1) / kBK : t.K / kBK); };
  // Range-checked view of what a step of a tile reads of one operand (nothing of it, live = false: every load returns zeros and
  // touches no memory).  By rows: the step's k rows (those that exist) from the tile's first column on: what lies past the last row's
  // end reads as zero, what lies past a row's M (N) columns belongs to C rows (columns) that are never stored.  Else: the tile's rows,
  // from the step's k on; rows past the matrix read as zeros.  The k offset of a step goes into the base (scalar arithmetic), so
  // the per-lane offsets are the same for every step of every tile.
  auto view_a = [&](const TileAt& t, int step, bool live) -> row_rsrc_t {
    if (TA) return make_row_rsrc(t.a + static_cast<int64_t>(step) * kBK * lda, live ? static_cast<uint32_t>(min(kBK, t.K - step * kBK) - 1) * pitch_a + t.bytes_a : 0u);
    return make_row_rsrc(t.a + step * kBK, live ? t.bytes_a - static_cast<uint32_t>(step) * (kBK * 2) : 0u);
  };
  auto view_b = [&](const TileAt& t, int step, bool live) -> row_rsrc_t {
    if (TB) return make_row_rsrc(t.b + static_cast<int64_t>(step) * kBK * ldb, live ? static_cast<uint32_t>(min(kBK, t.K - step * kBK) - 1) * pitch_b + t.bytes_b : 0u);
    return make_row_rsrc(t.b + step * kBK, live ? t.bytes_b - static_cast<uint32_t>(step) * (kBK * 2) : 0u);
  };

  // Loader role: thread t moves LDS vector slot (t % 8) of rows t/8 + 32 i, i = 0..7, of each panel;
  // the slot holds global k-vector slot ^ ((row >> 1) & 7), the same for all eight rows.
  // By rows: load i of a panel (one KiB: two LDS rows) moves k rows 8 i + 2 wave + lane / 32, LDS slot lane % 32: the same global slot for every other i.
  // What differs from load to load is a scalar offset, which the range check counts (see row_rsrc_t; offsets stay below 2^31 here): rows of a tile or a step that do not
  // exist, and everything of a view of no bytes, read as zeros without an access.
  auto loader = [&](bool by_rows, uint32_t pitch, int i) -> uint32_t {
    if (!by_rows) return static_cast<uint32_t>(tid >> 3) * pitch + static_cast<uint32_t>(((tid & 7) ^ ((tid >> 4) & 7)) << 4);
    const int k = 8 * i + 2 * wid + (lane >> 5);
    return static_cast<uint32_t>(k) * pitch + ((static_cast<uint32_t>(lane & 31) ^ static_cast<uint32_t>(2 * ((k & 3) | (((k >> 3) & 1) << 2)))) << 4);
  };
  const uint32_t vo_a[2] = {loader(TA, pitch_a, 0), loader(TA, pitch_a, 1)}, vo_b[2] = {loader(TB, pitch_b, 0), loader(TB, pitch_b, 1)};
  // Global memory -> LDS directly (buffer_load ... lds): lane l of a wave-level load deposits its
  // 16 bytes at (LDS base of the instruction) + 16 l, which is exactly the loader layout above for
  // the base panel + i * 4096 + wave * 1024.  No staging registers, no LDS store
  // instructions; completion is counted with the other vector-memory loads.
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  auto load_a = [&](unsigned char* panel, row_rsrc_t r, int i) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(panel + wid * 1024 + i * 4096), 16, vo_a[TA ? i & 1 : 0], (TA ? 16u * (i >> 1) : 32u * i) * pitch_a, 0, 0);
  };
  auto load_b = [&](unsigned char* panel, row_rsrc_t r, int i) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(panel + wid * 1024 + i * 4096), 16, vo_b[TB ? i & 1 : 0], (TB ? 16u * (i >> 1) : 32u * i) * pitch_b, 0, 0);
  };
  // load i of the eight of a panel of the far / near operand
  auto load_far = [&](unsigned char* panel, row_rsrc_t r, int i) { if (FAR_A) load_a(panel, r, i); else load_b(panel, r, i); };
  auto load_near = [&](unsigned char* panel, row_rsrc_t r, int i) { if (FAR_A) load_b(panel, r, i); else load_a(panel, r, i); };
  auto view_far = [&](const TileAt& t, int step, bool live) { return FAR_A ? view_a(t, step, live) : view_b(t, step, live); };
  auto view_near = [&](const TileAt& t, int step, bool live) { return FAR_A ? view_b(t, step, live) : view_a(t, step, live); };

  // Fragment role: lane holds 8 consecutive k (k quarter `fk` of a 32-wide sub-step) of row `frow`
  // of a 16-row block.  The swizzle depends on the row only through frow, so one offset per
  // k-vector serves every block of both panels.
  const int frow = lane & 15, fk = lane >> 4;
  uint32_t foff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) foff[ks] = lds_off(frow, ks * 4 + fk);
  const uint32_t fbase_a = static_cast<uint32_t>(wm * 128) * kRowBytes;
  const uint32_t fbase_b = static_cast<uint32_t>(wn * 128) * kRowBytes;
  // TN panels: LDS row k (512 bytes = 32 slots of 16 bytes) holds in slot s the 8 columns of
  // global slot s ^ (2 g(k)), g(k) = (k & 3) | ((k >> 3) & 1) << 2: the sixteen k rows one transpose
  // read touches (k = 8 kg + j, kg = lane / 16, j = (lane % 16) / 4) then spread their 32-byte pieces
  // over all banks.  Lane (kg, j, q = lane % 4) reads the 8 bytes of columns 4 q .. 4 q + 3 of block t
  // in row 8 kg + j (+ 4 for the second half of the fragment, + 32 for the second sub-step).
  uint32_t toff_a[8], toff_b[8];
  if (TA || TB) {
    const int kg = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
    const uint32_t g2 = static_cast<uint32_t>(2 * (j | ((kg & 1) << 2)));
    const uint32_t rowoff = static_cast<uint32_t>(8 * kg + j) * 512u + static_cast<uint32_t>(q & 1) * 8u;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      toff_a[t] = rowoff + ((static_cast<uint32_t>(wm * 16 + 2 * t + (q >> 1)) ^ g2) << 4);
      toff_b[t] = rowoff + ((static_cast<uint32_t>(wn * 16 + 2 * t + (q >> 1)) ^ g2) << 4);
    }
  }
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
  // fragment t of a sub-step: 0..7 the B blocks, 8..15 the A blocks
  auto read_frag = [&](const unsigned char* far, const unsigned char* near, int ks, int t) -> bf16x8 {
    const unsigned char* stage = (t >= 8) == FAR_A ? far : near;
    if (t < 8 ? TB : TA) {
      const unsigned char* p = stage + (t < 8 ? toff_b[t & 7] : toff_a[t & 7]) + ks * (32 * 512);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * 512));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
    return *reinterpret_cast<const bf16x8*>(stage + (t < 8 ? fbase_b : fbase_a) + (t & 7) * 16 * kRowBytes + foff[ks]);
  };
#define DPPO_MFMA16(ACC, X, Y) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(ACC) : "v"(X), "v"(Y))
#define DPPO_PIN __builtin_amdgcn_sched_barrier(0)
  // Of this wave's memory accesses at most the VM youngest are in flight (they complete in order), and its LDS reads are done; then
  // everyone's.  The waits are written out: a barrier by itself, or the wait that the compiler puts in front of its own fragment
  // reads, would wait for more (the stores of the tile before) or, where the compiler thinks none is pending, for nothing.
  constexpr int kAnyVm = 63;
  auto meet = [&](auto vm) __attribute__((always_inline)) {
    constexpr int VM = decltype(vm)::value;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70);      // vmcnt(VM) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    DPPO_PIN;
  };

  // fragment q of the read order: the first A block, the 8 B blocks, then the other A blocks
  constexpr int kOrder[16] = {8, 0, 1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15};

  DPPO_ALL_ACCUMULATORS();
  TileAt tile = locate(number);
  {
    const int nk = steps_of(tile);
    unrolled<3>([&](auto sc) __attribute__((always_inline)) {
      constexpr int s = decltype(sc)::value;
      // (steps that the contraction does not have: sixteen or eight loads of nothing each, half a microsecond of an 8 us product of one step; a workgroup of one tile counts on them)
      if (RUNS && s > 0 && s >= nk) return;
      const row_rsrc_t rn = view_near(tile, s < nk ? s : 0, s < nk), rf = view_far(tile, s < nk ? s : 0, s < nk);
      if (s < 2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) load_near(near_panel(s), rn, i);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) load_far(far_panel(s), rf, i);
    });
  }
  // Of the forty loads the first sixteen, the first step's, are read at once.  A workgroup of one tile waits for no others here and for the next sixteen in the
  // middle of that step; where tiles follow, whose first steps begin behind their predecessor's stores, everything is awaited.
  meet(std::integral_constant<int, RUNS ? 0 : 24>{});
  for (;;) {
    // The panels hold the tile's first step, or its first two (three), for everyone.
    bf16x8 f0[16], f1[16];      // [0..7] B blocks, [8..15] A blocks
#pragma unroll
    for (int t = 0; t < 16; ++t) f0[kOrder[t]] = read_frag(far_panel(0), near_panel(0), 0, kOrder[t]);
    DPPO_PIN;
    // Pipeline over the contraction: step kt is multiplied out of far panel kt % 3 and near panel kt % 2; once every wave
    // has read its last fragments of them (the barrier in the middle of the step) the near panel of step kt + 2 and the far panel of step kt + 3
    // are loaded there, or, behind the tile's last steps, those of the same place of the next tile.  The fragments of each
    // 32-wide sub-step are read from LDS one sub-step ahead of the matrix-core instructions that consume them.  One barrier per step.
    const int nk = steps_of(tile);
    const bool has_next = RUNS && number + map.slots < end;
    TileAt next = tile;
    int nk_next = 0;
    // One step of the contraction: two 32-wide sub-steps of 64 matrix-core
    // instructions each (A block i = m / 8 against B block j = m % 8).  Every other instruction sits
    // directly behind a matrix-core instruction, where it issues while that one executes.
    // First sub-step: the 16 fragment reads of the second, behind the first 32 instructions, so they
    // have landed when the barrier is reached.  Second sub-step: the 16 fragment reads of the next
    // step's first sub-step and the panel loads, eight of the near operand two steps on and eight of the far one three steps on.
    // P: kt % 6.
    auto step = [&](int kt, auto phase, auto steady, auto first) __attribute__((always_inline)) {
      constexpr int P = decltype(phase)::value;
      constexpr bool STEADY = decltype(steady)::value, FIRST = decltype(first)::value;
      unrolled<64>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        product<m, FIRST>(f0[m & 7], f0[8 + (m >> 3)]); DPPO_PIN;
        if constexpr (m < 32 && (m & 1) == 0) { f1[kOrder[m >> 1]] = read_frag(far_panel(P), near_panel(P), 1, kOrder[m >> 1]); DPPO_PIN; }
      });
      // The next step's panels are complete (the eight youngest loads are the far panel of the step after it; a tile's second step: complete
      // since the tile began where there are runs) and this step's fully read.
      meet(std::integral_constant<int, (FIRST && RUNS ? kAnyVm : 8)>{});
      const bool own_n = STEADY || kt + 2 < nk, own_f = STEADY || kt + 3 < nk;
      const int sn = own_n ? kt + 2 : P % 2, sf = own_f ? kt + 3 : P % 3;
      const row_rsrc_t rn = STEADY ? view_near(tile, sn, true) : view_near(own_n ? tile : next, sn, own_n || sn < nk_next);
      const row_rsrc_t rf = STEADY ? view_far(tile, sf, true) : view_far(own_f ? tile : next, sf, own_f || sf < nk_next);
      unrolled<64>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        product<m, false>(f1[m & 7], f1[8 + (m >> 3)]); DPPO_PIN;
        if constexpr ((m & 3) == 0) { f0[kOrder[m >> 2]] = read_frag(far_panel(P + 1), near_panel(P + 1), 0, kOrder[m >> 2]); DPPO_PIN; }      // (a tile's last step: not used)
        if constexpr ((m & 3) == 2 && m < 32)  { load_near(near_panel(P), rn, m >> 2); DPPO_PIN; }
        if constexpr ((m & 3) == 2 && m >= 32) { load_far(far_panel(P), rf, (m >> 2) - 8); DPPO_PIN; }
      });
    };
    auto look_ahead = [&]() {
      if (has_next) {
        next = locate(number + map.slots);
        nk_next = steps_of(next);
      }
    };
    using Yes = std::true_type;
    using No = std::false_type;
#define DPPO_PHASE(P) std::integral_constant<int, P>{}
    if (nk <= 3) look_ahead();
    step(0, DPPO_PHASE(0), No{}, Yes{});
    int kt = 1;
    for (; kt + 8 < nk; kt += 6) {
      step(kt, DPPO_PHASE(1), Yes{}, No{});
      step(kt + 1, DPPO_PHASE(2), Yes{}, No{});
      step(kt + 2, DPPO_PHASE(3), Yes{}, No{});
      step(kt + 3, DPPO_PHASE(4), Yes{}, No{});
      step(kt + 4, DPPO_PHASE(5), Yes{}, No{});
      step(kt + 5, DPPO_PHASE(0), Yes{}, No{});
    }
    if (nk > 3) look_ahead();
    // (statistics: the sampled ids of the lane's eight rows, in time for the end of the tile)
    int samp[8];
    if (OUT == kOutStats) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = tile.m0 + wm * 128 + i * 16 + frow;
        samp[i] = (row < M) ? gs.sampled[row] : -1;
      }
    }
    // At most eight steps more.  (Left by one exit each: with a path around the steps that are not left, the compiler waits for the loads of a step
    // that it thinks may be read next.)
    for (;;) {
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(1), No{}, No{});
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(2), No{}, No{});
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(3), No{}, No{});
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(4), No{}, No{});
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(5), No{}, No{});
      if (kt >= nk) break;
      step(kt++, DPPO_PHASE(0), No{}, No{});
    }
#undef DPPO_PHASE
    // the matrix-core results must have landed before other instructions read the accumulators
    // (the products are assembly statements, so the compiler does not keep that distance by itself)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    DPPO_PIN;
    // The products were formed with the operands swapped (B fragment first), so a lane's four
    // accumulators of a 16 x 16 block are four consecutive COLUMNS (lane/16)*4 + 0..3 of row lane%16.
    const int m0 = tile.m0, n0 = tile.n0;
    const bool full = M - m0 >= kBM && N - n0 >= kBN;
    // Through an empty statement, so that the stores' addresses are formed here: kept from tile to tile they would be spilled, and
    // their reloads wait for the stores in front of them.
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int frow = lane_e & 15, fk = lane_e >> 4;
    const int row0 = m0 + wm * 128 + frow, col0 = n0 + wn * 128;
    // This wave's loads of the next tile's first steps have landed: from here on only the tile's own stores are in flight, and
    // the next wait for memory is in the next tile's second step.
    auto loads_landed = [&]() {
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
      DPPO_PIN;
    };
    if constexpr (OUT == kOutStats) {
      // in the panels, once every wave's last loads into them, of nothing, have ended
      meet(std::integral_constant<int, 0>{});
      static_assert(sizeof(StatRoom) <= kPanelBytes);
      StatRoom& room = *reinterpret_cast<StatRoom*>(panel2);
      unsigned char* const quarter[4] = {panel0, panel1, panel3, panel4};
      tile_statistics(samp, M, N, m0, n0, gs, room, quarter, wid, lane_e);
    } else if constexpr (OUT == kOutBf16) {
      auto store = [&](auto whole) __attribute__((always_inline)) {
        unrolled<8>([&](auto i) __attribute__((always_inline)) {
          f32x4 acc[8];
          accumulators<decltype(i)::value>(acc);
          if (TA && TB) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] *= factor;
          }
          store_row_block_bf16<decltype(whole)::value>(static_cast<uint16_t*>(tile.c), ldc, M, N, row0 + i * 16, col0, fk, acc);
        });
      };
      if (full) {
        store(std::true_type{});
        __builtin_amdgcn_s_waitcnt(0x8F70);      // vmcnt(32): the youngest 32 of the tile's stores may be in flight, no load in front of them
      } else {
        loads_landed();
        store(std::false_type{});
      }
    } else {
      loads_landed();
      // fp32: 16 bytes per lane as they are (the host requires 16-byte aligned rows for these forms)
      auto cptr = [&](int i, int j) { return static_cast<float*>(tile.c) + static_cast<int64_t>(row0 + i * 16) * ldc + (col0 + j * 16 + fk * 4); };
      auto store = [&](auto whole) __attribute__((always_inline)) {
        // C += tile: what C holds is requested one block of 16 rows AHEAD of the block being added and
        // stored (eight 16-byte loads per lane in flight behind eight stores), so that a lane waits for
        // memory eight times per tile and not sixty-four times.  (Written as load - add - store per
        // vector, the compiler keeps that order, every load behind the store in front of it.)
        constexpr bool AHEAD = OUT == kOutF32Add && decltype(whole)::value;
        f32x4 held[2][8];
        if (AHEAD) {
#pragma unroll
          for (int j = 0; j < 8; ++j) held[0][j] = __builtin_nontemporal_load(reinterpret_cast<f32x4*>(cptr(0, j)));
        }
        unrolled<8>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value;
          f32x4 acc[8];
          accumulators<i>(acc);
          if (AHEAD && i + 1 < 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j) held[(i + 1) & 1][j] = __builtin_nontemporal_load(reinterpret_cast<f32x4*>(cptr(i + 1, j)));
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            float* dst = cptr(i, j);
            const int row = row0 + i * 16, col = col0 + j * 16 + fk * 4;
            f32x4 v = acc[j];
            if (AHEAD) v += held[i & 1][j];
            if (decltype(whole)::value || (row < M && col + 3 < N)) {
              if (OUT == kOutF32Add && !AHEAD) v += *reinterpret_cast<const f32x4*>(dst);
              *reinterpret_cast<f32x4*>(dst) = v;
            } else if (row < M) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (col + e < N) dst[e] = (OUT == kOutF32Add ? dst[e] : 0.f) + v[e];
            }
          }
        });
      };
      if (full) store(std::true_type{});
      else store(std::false_type{});
    }
    if (!has_next) return;
    meet(std::integral_constant<int, kAnyVm>{});
    tile = next;
    number += map.slots;
  }
}

// ---- short contractions: C = bf16(factor A^T B) in tiles of 128 x 256 and steps of 32 ---------------
// The weight gradient of few tokens is bound by what its tiles write: alone on its compute unit, a 256 x 256 tile's first
// loads (2 us) and its store (7-8 us: every compute unit stores at the same time) leave the matrix cores idle, as long as
// 8 of its steps (1000 tokens are 16).  Here a stage is 24 KiB, three of them 72, and a lane holds 128 accumulators, so
// TWO workgroups share a compute unit and one's loads and stores pass behind the other's products.  The price is 1.5 x the LDS
// reads per product (a wave's 64 x 128 quadrant needs 12 fragments for 32 products, a 128 x 128 one 16 for 64).
// What is left is the rate of the stores: in the order of the accumulators they are pieces of 64 bytes, 4.2 TB/s; in whole lines past the caches (store_row_block_lines),
// us, 151936 x 2048, 64 tokens 148 / 110, 100 189 / 136, 200 236 / 179, 300 284 / 222.  (What both kinds of tiles measure: gemm_tn_short.)
// Two loads ahead are in flight per workgroup; the order of the sums over k is the same as in the larger tiles.
constexpr int kShortM = 128, kShortK = 32, kShortA = kShortK * kShortM * 2, kShortStage = kShortA + kShortK * kBN * 2;

template <bool FULL>
__device__ __forceinline__ void short_tile(unsigned char* lds0, unsigned char* lds1, unsigned char* lds2, const uint16_t* __restrict__ A, int64_t lda,
                                           const uint16_t* __restrict__ B, int64_t ldb, uint16_t* __restrict__ C, int64_t ldc,
                                           int M, int N, int K, int m0, int n0, const float* factor_ptr) {
  const int tid = threadIdx.x, lane = tid & 63, wid = uniform_i(tid >> 6);
  const int wm = wid >> 1, wn = wid & 1;
  const uint32_t pitch_a = static_cast<uint32_t>(lda) * 2u, pitch_b = static_cast<uint32_t>(ldb) * 2u;
  const float factor = uniform_f(*factor_ptr);
  f32x4 acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // Panels by rows as in the larger tiles: LDS row k of the A panel 256 bytes = 16 slots of 16 bytes, of the B panel 512 bytes = 32 slots, slot s
  // holding the columns of global slot s ^ 2 g(k).
  uint32_t toff_a[4], toff_b[8], vo_a[2], vo_b[4];
  {
    const int kg = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
    const uint32_t g2 = static_cast<uint32_t>(2 * (j | ((kg & 1) << 2)));
    const uint32_t k = static_cast<uint32_t>(8 * kg + j), sub = static_cast<uint32_t>(q & 1) * 8u;
#pragma unroll
    for (int t = 0; t < 4; ++t) toff_a[t] = k * 256u + sub + ((static_cast<uint32_t>(wm * 8 + 2 * t + (q >> 1)) ^ g2) << 4);
#pragma unroll
    for (int t = 0; t < 8; ++t) toff_b[t] = kShortA + k * 512u + sub + ((static_cast<uint32_t>(wn * 16 + 2 * t + (q >> 1)) ^ g2) << 4);
  }
  auto swizzle = [](int k) { return static_cast<uint32_t>(2 * ((k & 3) | (((k >> 3) & 1) << 2))); };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = 16 * i + 4 * wid + (lane >> 4);
    vo_a[i] = static_cast<uint32_t>(k) * pitch_a + ((static_cast<uint32_t>(lane & 15) ^ swizzle(k)) << 4);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = 8 * i + 2 * wid + (lane >> 5);
    vo_b[i] = static_cast<uint32_t>(k) * pitch_b + ((static_cast<uint32_t>(lane & 31) ^ swizzle(k)) << 4);
  }
  const uint32_t bytes_a = (static_cast<uint32_t>(M - m0) * 2u + 15u) & ~15u, bytes_b = (static_cast<uint32_t>(N - n0) * 2u + 15u) & ~15u;
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
  // Load idx of the 6 of a step: 0, 1 A panel, 2..5 B panel.  Issued from inline assembly, so that the compiler puts no waits of its own in
  // front of the fragment reads (around the loop it loses track of which stage a load goes to and waits for all of
  // them); the waits are written out below.  Before the load the wait states of row_store16_untracked.
  auto dma_one = [&](unsigned char* stage, int step, int idx) {
    const uint32_t kr = static_cast<uint32_t>(min(kShortK, K - step * kShortK));
    const bool b_panel = idx >= 2;
    const int i = b_panel ? idx - 2 : idx;
    const uint64_t base = b_panel ? reinterpret_cast<uint64_t>(B + static_cast<int64_t>(step) * kShortK * ldb + n0)
                                  : reinterpret_cast<uint64_t>(A + static_cast<int64_t>(step) * kShortK * lda + m0);
    const row_desc_t r = {static_cast<int>(base), static_cast<int>((base >> 32) & 0xffffu),
                          static_cast<int>((kr - 1) * (b_panel ? pitch_b : pitch_a) + (b_panel ? bytes_b : bytes_a)), 0x00020000};
    const uint32_t dst = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)(stage + (b_panel ? kShortA : 0) + wid * 1024 + i * 4096)));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(b_panel ? vo_b[i] : vo_a[i]), "s"(r) : "memory", "m0");
  };
  auto read_frag = [&](const unsigned char* p, uint32_t pitch) -> bf16x8 {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * pitch));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  const int nk = (K + kShortK - 1) / kShortK;
#pragma unroll
  for (int q = 0; q < 6; ++q) dma_one(lds0, 0, q);
  if (nk > 1) {
#pragma unroll
    for (int q = 0; q < 6; ++q) dma_one(lds1, 1, q);
  }
  auto step = [&](unsigned char* cur, unsigned char* free_stage, int kt, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    // This wave's six loads of this step have landed (the next step's six may be in flight) and its reads of the step before
    // are done; then everyone's.  (A plain s_barrier: the fence of __syncthreads() waits for every load in flight.)
    asm volatile("" ::: "memory");
    if (STEADY || kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x76);      // vmcnt(6) lgkmcnt(0)
    else                       __builtin_amdgcn_s_waitcnt(0x70);      // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    DPPO_PIN;
    const bool more = STEADY || kt + 2 < nk;
    bf16x8 fa[4], fb[8];
    fa[0] = read_frag(cur + toff_a[0], 256); DPPO_PIN;
#pragma unroll
    for (int t = 0; t < 8; ++t) { fb[t] = read_frag(cur + toff_b[t], 512); DPPO_PIN; }
#pragma unroll
    for (int t = 1; t < 4; ++t) { fa[t] = read_frag(cur + toff_a[t], 256); DPPO_PIN; }
#pragma unroll
    for (int m = 0; m < 32; ++m) {
      DPPO_MFMA16(acc[m >> 3][m & 7], fb[m & 7], fa[m >> 3]); DPPO_PIN;
      if (m % 5 == 0 && m / 5 < 6) { if (more) dma_one(free_stage, kt + 2, m / 5); DPPO_PIN; }
    }
  };
  int kt = 0;
  for (; kt + 4 < nk; kt += 3) {
    step(lds0, lds2, kt, std::true_type{});
    step(lds1, lds0, kt + 1, std::true_type{});
    step(lds2, lds1, kt + 2, std::true_type{});
  }
  for (; kt < nk; kt += 3) {
    step(lds0, lds2, kt, std::false_type{});
    if (kt + 1 < nk) step(lds1, lds0, kt + 1, std::false_type{});
    if (kt + 2 < nk) step(lds2, lds1, kt + 2, std::false_type{});
  }
  // the products have landed before anything else reads the accumulators (as in the larger tiles)
#define DPPO_THROUGH(CODE, I) asm volatile(CODE : "+a"(acc[I][0]), "+a"(acc[I][1]), "+a"(acc[I][2]), "+a"(acc[I][3]), \
                                               "+a"(acc[I][4]), "+a"(acc[I][5]), "+a"(acc[I][6]), "+a"(acc[I][7]) :: "memory")
  DPPO_THROUGH("s_nop 15\n\ts_nop 15", 0);
#pragma unroll
  for (int i = 1; i < 4; ++i) DPPO_THROUGH("", i);
#undef DPPO_THROUGH
  DPPO_PIN;
  const int frow = lane & 15, fk = lane >> 4;
  if (FULL && result_on_lines(C, ldc)) {
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));         // (addresses formed here, not kept from in front of the loop)
    // every wave is done with the stages
    __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    DPPO_PIN;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] *= factor;
      store_row_block_lines(C + static_cast<int64_t>(m0 + wm * 64 + i * 16) * ldc + n0 + wn * 128, ldc, lane_e, acc[i], ((i & 1) ? lds1 : lds0) + wid * kLineRoom);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] *= factor;
    store_row_block_bf16<FULL>(C, ldc, M, N, m0 + wm * 64 + i * 16 + frow, n0 + wn * 128, fk, acc[i]);
  }
}

struct ShortMap {
  int tiles_m, tiles_n, group_m, group_n, tiles, per_die;
};

__global__ __launch_bounds__(256, 2) void dppo_gemm_tn_short_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B, int64_t ldb,
                                                                    uint16_t* __restrict__ C, int64_t ldc, int M, int N, int K, const ShortMap map,
                                                                    const float* factor) {
  __shared__ __attribute__((aligned(16))) unsigned char lds0[kShortStage];
  __shared__ __attribute__((aligned(16))) unsigned char lds1[kShortStage];
  __shared__ __attribute__((aligned(16))) unsigned char lds2[kShortStage];
  const int tile = (static_cast<int>(blockIdx.x) & 7) * map.per_die + (static_cast<int>(blockIdx.x) >> 3);
  if (tile >= map.tiles) return;
  const int bn = tile / (map.group_n * map.tiles_m);
  int t = tile - bn * (map.group_n * map.tiles_m);
  const int width = min(map.group_n, map.tiles_n - bn * map.group_n);
  const int bm = t / (map.group_m * width);
  t -= bm * (map.group_m * width);
  const int height = min(map.group_m, map.tiles_m - bm * map.group_m);
  const int m0 = (bm * map.group_m + t % height) * kShortM, n0 = (bn * map.group_n + t / height) * kBN;
  if (M - m0 >= kShortM && N - n0 >= kBN) short_tile<true>(lds0, lds1, lds2, A, lda, B, ldb, C, ldc, M, N, K, m0, n0, factor);
  else                                    short_tile<false>(lds0, lds1, lds2, A, lda, B, ldb, C, ldc, M, N, K, m0, n0, factor);
}

// Numbers run block by block over 64 tiles, the workgroups that run together on a die, each die a contiguous range.  Eight tiles wide:
// four 0-4 % slower, sixteen 3-29 % where the matrix is 12 or 16 tiles wide (but for 151936 x 3008: 3-10 % faster).
ShortMap short_map(int64_t M, int64_t N) {
  ShortMap t;
  t.tiles_m = static_cast<int>((M + kShortM - 1) / kShortM);
  t.tiles_n = static_cast<int>((N + kBN - 1) / kBN);
  t.group_n = std::min(t.tiles_n, 8);
  t.group_m = 64 / t.group_n;
  t.tiles = t.tiles_m * t.tiles_n;
  t.per_die = (t.tiles + 7) / 8;
  return t;
}

}  // namespace

hipError_t launch_gemm_nt(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, void* C, int64_t ldc,
                          int M, int N, int K, int out, int cus, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const TileMap map = tile_map(M, N, K, 1, cus);
  const dim3 grid = tile_grid(map), wg(256);
  if (out == 0)      hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutBf16, false, false>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  else if (out == 1) hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutF32, false, false>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  else               hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutF32Add, false, false>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  return hipGetLastError();
}

// The first product of the hidden-state path with nothing of C stored: per row and column tile the
// softmax statistics of the bf16-rounded logits, and the logits at the sampled and top-K ids.
hipError_t launch_gemm_stats(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, int M, int N, int K,
                             const GemmStats& gs, int cus, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const TileMap map = tile_map(M, N, K, 1, cus, 1);
  if (gs.tiles_n != map.tiles_n || N % 16 != 0) return hipErrorInvalidValue;
  const dim3 grid = tile_grid(map), wg(256);
  hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutStats, false, false>), grid, wg, 0, s, A, lda, B, ldb, static_cast<void*>(nullptr), int64_t(0), M, N, K,
                     map, gs);
  return hipGetLastError();
}

// Which contractions are short.  Ratio of the times, these tiles / 256 x 256 ones, over V = 16000 .. 151936 and 64 .. 4160 columns, results of more than the Infinity Cache in turn:
//  * a last column of tiles that is cut, which the large tiles store behind a check per vector: up to 640 tokens 0.48-0.95 (results off the lines up to 1.11), 768 .. 1024
//    0.69-1.04;
//  * whole columns of tiles, results on lines: up to 640 0.61-1.04, 768 .. 896 0.80-1.05, 930 .. 1024 0.84-1.09, but 0.71-0.98 where the large tiles are at most one per compute unit
//    (V = 8192 and 16000); V = 151936, 2048 columns: 64 tokens 0.62, 200 0.66, 400 0.74, 640 0.84, 768 0.90, 900 0.96, 1000 1.04 (64 110 / 191 us, 300 222 / 284, 800 442 /
//    483, 1000 565 / 546);
//  * whole columns, other results, which both kinds leave in pieces of 64 bytes: up to 300 0.89-1.19, 400 .. 640 0.94-1.15 where the large tiles fill nine tenths of their rounds, 0.92-1.03
//    where they do not; 768 .. 1024 0.92-1.14.
static bool gemm_tn_short(const void* C, int64_t ldc, int64_t M, int64_t N, int64_t K, int cus) {
  const int64_t tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN), rounds = (tiles + cus - 1) / cus;
  if (N % kBN != 0) return K <= 1024;
  if (result_on_lines(C, ldc)) return K <= (rounds == 1 ? 1024 : 896);
  return K <= (tiles * 10 >= rounds * cus * 9 ? 384 : 640);
}

// C[M, N] bf16 = *factor A^T B, rounded once.
//
// The gradient of the weight in its own type.  Left in fp32 for a pass of its own to scale and round, it cost 12 bytes
// per entry where 2 do, and short contractions are bound by them.  V = 151936: 1000 tokens x 2048, fp32 product and
// conversion 743 + 322 us, here 546; 8192 x 4096 7.85 + 0.62 ms, here 7.15.
hipError_t launch_gemm_tn_bf16(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, void* C, int64_t ldc,
                               int M, int N, int K, const float* factor, int cus, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (gemm_tn_short(C, ldc, M, N, K, cus)) {
    const ShortMap map = short_map(M, N);
    hipLaunchKernelGGL(dppo_gemm_tn_short_kernel, dim3(8u * static_cast<unsigned>(map.per_die)), dim3(256), 0, s, A, lda, B, ldb, static_cast<uint16_t*>(C), ldc,
                       M, N, K, map, factor);
    return hipGetLastError();
  }
  const TileMap map = tile_map(M, N, K, 1, cus);
  GemmStats gs;
  gs.factor = factor;
  hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutBf16, true, true>), tile_grid(map), dim3(256), 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, gs);
  return hipGetLastError();
}

// C[M, N] (fp32; out 1: written, 2: added to) = A^T B with A [K, M], B [K, N] (row-major, the contraction index the row index)
hipError_t launch_gemm_tn(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, void* C, int64_t ldc,
                          int M, int N, int K, int out, int cus, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const TileMap map = tile_map(M, N, K, 1, cus);
  const dim3 grid = tile_grid(map), wg(256);
  if (out == 1) hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutF32, true, true>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  else          hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutF32Add, true, true>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  return hipGetLastError();
}

// The gradient of the hidden states contracts over the whole vocabulary (2374 steps of 64 at 151936
// entries) into few tiles: 1000 tokens of a 2048-wide model are 32 tiles for 256 compute units, 5000 of
// a 4096-wide one 320, a full round and a quarter.  So the contraction can be cut into ranges: every
// (tile, range) is a workgroup, fp32 partial tiles go to scratch and dppo_gemm_sum_kernel adds them in
// a fixed order and rounds once.  The number of ranges is the one with the least estimated time, in
// steps of a compute unit (1.46 us, measured): rounds of workgroups on the busiest die times (steps of
// a range + 8 for filling the pipeline and storing a tile), plus the partial sums' way out and back
// (at 4 TB/s, 5.8 MB per step) and the second launch.  It has to beat the undivided product by 3 %.
// Contractions of fewer than 128 steps (vocabularies below 8192: at most 0.2 ms undivided) stay whole,
// a range has 16 steps or more (but for the last, which has what is left), twice what filling the pipeline and
// storing the tile cost, and there are at most 16 (tile, range) pairs per compute unit, so that the partial sums take 4 MiB per
// compute unit at most.  Measured at V = 151936, logits + loss + hidden gradient, undivided against divided: 64 tokens x 1024 wide
// (63 ranges) 2.92 / 0.22 ms, 512 x 2048 (16) 3.42 / 0.67, 1000 x 2048 (8) 3.69 / 1.19, 2048 x 4096 (2) 5.24 / 3.91,
// 5000 x 4096 (4) 11.74 / 9.74, 8192 x 1024 (2) 6.57 / 4.99; 8192 x 4096 and 8192 x 2048 fill whole rounds and stay undivided.
int gemm_nn_splits(int64_t M, int64_t N, int64_t K, int cus, size_t scratch_bytes) {
  const int64_t nk = K / kBK;
  const int per_die = cus >= 8 ? cus / 8 : 1;
  int best = 1;
  double best_cost = 0.0;
  for (int64_t s = 1; s <= 64; ++s) {
    const TileMap t = tile_map(M, N, K, s, cus);
    if (s > 1 && (nk < 128 || nk / s < 16 || t.numbers * s > 16 * static_cast<int64_t>(cus))) break;
    if (s > 1 && static_cast<uint64_t>(s) * static_cast<uint64_t>(M) * static_cast<uint64_t>(N) * 4u > scratch_bytes) break;
    const int64_t busiest = std::min<int64_t>(t.per_die, t.numbers * s);
    double cost = static_cast<double>((busiest + per_die - 1) / per_die) * static_cast<double>((nk + s - 1) / s + 8);
    if (s > 1) cost = (cost + static_cast<double>(s * M * N) * 8.0 / 5.8e6 + 4.0) / 0.97;
    if (s == 1 || cost < best_cost) {
      best = static_cast<int>(s);
      best_cost = cost;
    }
  }
  return best;
}

namespace {
// Adds the fp32 partial results of the ranges of the contraction, [splits][M][N], in their order and
// rounds the sum to bf16 once.  Four columns per thread (N a multiple of 4); bound by the latency of reading the
// partial sums, which the products have just written: few tokens are few threads and many ranges, so sixteen loads are in flight
// per thread, and workgroups are one wave (one load at a time, 64 tokens x 768, 63 ranges: 17 us, now 6).
constexpr int kSumThreads = 64, kSumAhead = 16;
__global__ __launch_bounds__(kSumThreads) void dppo_gemm_sum_kernel(const f32x4* __restrict__ part, int splits, int64_t quads, int quads_row,
                                                                    uint16_t* __restrict__ C, int64_t ldc) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * kSumThreads + threadIdx.x;
  if (q >= quads) return;
  f32x4 v = part[q];
  for (int s = 1; s < splits; s += kSumAhead) {
    f32x4 x[kSumAhead];
#pragma unroll
    for (int u = 0; u < kSumAhead; ++u)
      if (s + u < splits) x[u] = part[static_cast<int64_t>(s + u) * quads + q];
#pragma unroll
    for (int u = 0; u < kSumAhead; ++u)
      if (s + u < splits) v += x[u];
  }
  const int64_t row = q / quads_row;
  uint16_t* dst = C + row * ldc + (q - row * quads_row) * 4;
  const uint32_t lo = pack_bf16x2(v[0], v[1]), hi = pack_bf16x2(v[2], v[3]);
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if ((reinterpret_cast<uintptr_t>(dst) & 7u) == 0) {
    *reinterpret_cast<u32x2*>(dst) = u32x2{lo, hi};
  } else {
    dst[0] = static_cast<uint16_t>(lo & 0xffffu);
    dst[1] = static_cast<uint16_t>(lo >> 16);
    dst[2] = static_cast<uint16_t>(hi & 0xffffu);
    dst[3] = static_cast<uint16_t>(hi >> 16);
  }
}
}  // namespace

// C[M, N] bf16 = A B with A [M, K] (contraction index contiguous) and B [K, N] (contraction index the row index); K % 64 == 0
hipError_t launch_gemm_nn(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, void* C, int64_t ldc,
                          int M, int N, int K, int splits, float* scratch, int cus, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (splits > 1) {
    if (N % 4 != 0 || !scratch) return hipErrorInvalidValue;
    const int split_steps = (K / kBK + splits - 1) / splits;
    const int used = (K / kBK + split_steps - 1) / split_steps;       // ranges that hold a step
    TileMap map = tile_map(M, N, K, used, cus, 1);
    map.split_steps = split_steps;
    hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutSplit, false, true>), tile_grid(map), dim3(256), 0, s, A, lda, B, ldb,
                       static_cast<void*>(scratch), static_cast<int64_t>(N), M, N, K, map, GemmStats{});
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    const int64_t quads = static_cast<int64_t>(M) * N / 4;
    hipLaunchKernelGGL(dppo_gemm_sum_kernel, dim3(static_cast<unsigned>((quads + kSumThreads - 1) / kSumThreads)), dim3(kSumThreads), 0, s,
                       reinterpret_cast<const f32x4*>(scratch), used, quads, N / 4, static_cast<uint16_t*>(C), ldc);
    return hipGetLastError();
  }
  const TileMap map = tile_map(M, N, K, 1, cus);
  const dim3 grid = tile_grid(map), wg(256);
  hipLaunchKernelGGL((dppo_gemm_nt_kernel<kOutBf16, false, true>), grid, wg, 0, s, A, lda, B, ldb, C, ldc, M, N, K, map, GemmStats{});
  return hipGetLastError();
}

}  // namespace dppo
