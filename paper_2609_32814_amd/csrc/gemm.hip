// Grouped, row-typed GEMM on gfx950 MFMA for fp32 operands: the forward
// projection, its activation gradient and its weight gradient (Alg. 1 and
// the VJPs of the appendix) in one kernel template.  bf16 operands run in
// the pipelined kernel of gemm_async.hip.
//
// Work decomposition.  C is cut into tiles of 64 rows x 64 columns.  A
// workgroup of 4 wavefronts (2 x 2) computes a tile, each wave one 32 x 32
// block with v_mfma_f32_32x32x2f32.
//
//  * FWD: a tile is (row type i, row tile of I_i, output group j, column
//    tile).  Its K range is the concatenation of the input groups in
//    B(i,j): {j, i} for the star law (one group when j = i), all of K for
//    the dense law.  Rows are gathered through the type plan's permutation,
//    so each tile multiplies only rows that share one support: the skipped
//    blocks are never read and never multiplied.
//  * BWD_DATA: a tile is (row type i, row tile, input group g, column tile of
//    g).  Its contraction runs over the output groups j with g in B(i,j): all
//    of N when g = i (eq. vjp-xi), only group g otherwise (eq. vjp-xj).  W is
//    read in place as W^T (its rows are K-contiguous for this product).
//  * BWD_WEIGHT: a tile is (input group g, output group j, row tile of g,
//    column tile of j, split).  Its contraction runs over the rows whose
//    support reaches block (g, j): all rows when g = j (eqs. vjp-wii,
//    vjp-wjj), the type-g rows otherwise (eq. vjp-wij).  Long contractions
//    are split into a fixed number of row ranges whose fp32 partials a
//    second kernel sums in a fixed order.  The bias gradient is summed from
//    the dY tiles that the diagonal tiles already stage.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s nominal; a 4096^3
// library product reaches 138).  An fp32 MFMA of 32 x 32 x 2 holds its SIMD
// for 64 cycles and takes one float per lane and operand, so LDS reads are
// far from a limit (32 bytes a clock of 128) and neither operand needs a
// transposed copy: a 4-byte read per lane and K index serves an operand that
// is contiguous along the tile rows.  What matters is that every SIMD has a
// tile: small tiles, three workgroups per CU, and operands copied ahead.
// Against 256 x 128 tiles staged through registers by one workgroup per CU
// (1111 rows of three types, 768 <-> 2304: 40 to 100 workgroups on the
// chip): forward 162 and 386 -> 37 and 47 us, activation gradients 192 and
// 460 -> 34 and 55 us, weight gradients 416 -> 44 us each.  128 x 128 tiles
// of the same kernel: 10 % faster on 4096 x 1024 x 4096 (311 against 351 us),
// three times slower where the long contractions are few (172 against 52 us),
// so they are not built; dense forwards that filled the chip with 256 x 128
// tiles exactly are the one loss (2048 x 4096 x 4096, 597 -> 612 us).
//
// Operands go from global memory straight into LDS (16 bytes per lane, 1 KB
// per copy instruction) in steps of 32 K elements, two steps ahead of the
// one being multiplied, in a ring of three 16 KB stages.  A wait counts the
// copies still allowed in flight, so a step never drains the ring; a step's
// copies go between its MFMAs (issued in a burst ahead of them: 4096 x 1024
// x 4096 weight gradient 390 -> 335 us).
//
// LDS layout of a stage.  K-contiguous operand (X and dY rows, W^T): 128
// bytes a row, 16-byte chunk c of row r at c ^ ((r >> 1) & 7).  Operand
// contiguous along the tile rows (W in the forward, X and dY in the weight
// gradient): one K index a row, its 16-byte chunks rotated by 8 for every
// other group of 4 K indexes, so the two lane halves of a 4-byte read sit
// in different halves of the 64 banks.
//
// Scheduling.  Each pass's tiles (pass 0: the longer contractions) are cut
// into 8 contiguous chunks, one per XCD (workgroups are dispatched
// round-robin over the 8 XCDs); consecutive tiles of a chunk share rows and
// weight panels in that XCD's L2.
//
// Epilogue.  The MFMA is issued with the operands swapped (it computes
// C^T blocks), so each lane ends with 4 consecutive columns of one row of
// C and writes them as one 16-byte store.  The activation and its
// derivative are the shared ones of common.hpp.
#include <algorithm>

#include "gemm_common.hpp"

namespace starq {

namespace {

using namespace gemm;

constexpr int kThreads = 256;        // 4 wavefronts, 2 x 2 over a tile
constexpr int TM = 64, TN = 64;      // tile of C
constexpr int BK = 32;               // K elements per step (128 bytes)
constexpr int kStages = 3;           // LDS ring
constexpr int kAhead = kStages - 1;  // steps copied ahead
constexpr int kABytes = TM * BK * 4;
constexpr int kStageBytes = kABytes + TN * BK * 4;  // 16 KB
constexpr int kPerCU = 3;                           // workgroups per CU
constexpr int CA = TM / 32, CB = TN / 32;           // copies per wave and step
constexpr int kChunks = 16;                         // 16-byte chunks per K index of a row-contiguous operand
static_assert(TM == 4 * kChunks && TN == 4 * kChunks && CA == CB, "one copy layout for both operands");

// 256 zero bytes: the source of every copy past a step's K range
__device__ __attribute__((aligned(256))) uint32_t g_f32_zero[64];

template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p)));
}

// Chunk of K-contiguous row r, and of K index k of a row-contiguous operand.
__device__ __forceinline__ int kc_chunk(int r, int c) { return c ^ ((r >> 1) & 7); }
__device__ __forceinline__ int rc_chunk(int k, int c) { return c ^ (8 * ((k >> 2) & 1)); }

// The four K values 4 (2 rs + lh) .. + 3 of tile row `row` (lane half lh
// supplies K element 4 kp + e of MFMA e; both operands use the same
// assignment, so the products pair up).
template <bool KC>
__device__ __forceinline__ void read_frag(const char* tile, int rs, int lh, int row, float (&f)[4]) {
  if constexpr (KC) {
    const float4 v = *reinterpret_cast<const float4*>(tile + row * 128 + kc_chunk(row, 2 * rs + lh) * 16);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 8 * rs + 4 * lh + e;
      f[e] = *reinterpret_cast<const float*>(tile + k * (16 * kChunks) + rc_chunk(k, row >> 2) * 16 + (row & 3) * 4);
    }
  }
}

template <int MODE, int LAW>
__global__ __launch_bounds__(kThreads, kPerCU) void star_gemm_f32_kernel(const GemmParams p) {
  constexpr bool kAKC = MODE != kModeBwdWeight;  // A K-contiguous
  constexpr bool kBKC = MODE == kModeBwdData;    // B K-contiguous
  // a step's copies of one wave: operands, and the weight gradient's perm
  // entries of a later step
  constexpr int kGroup = CA + CB + (MODE == kModeBwdWeight ? 1 : 0);
  __shared__ __attribute__((aligned(256))) char smem[kStages * kStageBytes];
  // weight gradient: rows (perm entries) of the positions of a step, for
  // each wave alone (copied 2 kAhead steps ahead, read kAhead steps ahead)
  constexpr int kRowSlots = 4;
  static_assert(kAhead + 1 <= kRowSlots, "perm ring");
  __shared__ __attribute__((aligned(16))) int32_t prow_s[MODE == kModeBwdWeight ? 4 : 1][kRowSlots][64];

  const float* __restrict__ Ag = static_cast<const float*>(p.A);
  const float* __restrict__ Bg = static_cast<const float*>(p.B);
  const void* zero = g_f32_zero;
  const int q = p.q;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int lr = lane & 31, lh = lane >> 5;
  const uint32_t lds0 = lds_addr(smem);

  // ---- tiles per class and pass: lane i holds class i (q <= 64) ----
  int32_t units = 0, cnt[2] = {0, 0}, pfx[2];
  if (lane < q) {
    if constexpr (MODE == kModeBwdWeight) units = (p.MTp[lane + 1] - p.MTp[lane]) * p.nsplit;
    else units = (p.offsets[lane + 1] - p.offsets[lane] + TM - 1) / TM;
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) cnt[ps] = units * ncols_sel(p, sel_for(MODE, LAW, ps), lane);
  }
  int32_t chunk[2], total[2];
#pragma unroll
  for (int ps = 0; ps < 2; ++ps) {
    int32_t v = cnt[ps];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    pfx[ps] = v;  // inclusive
    total[ps] = __builtin_amdgcn_readlane(v, 63);
    chunk[ps] = (total[ps] + 7) >> 3;
  }
  const int xcd = blockIdx.x & 7;

  for (int32_t slot = blockIdx.x >> 3; slot < chunk[0] + chunk[1]; slot += gridDim.x >> 3) {
    const int ps = slot < chunk[0] ? 0 : 1;
    const int32_t logical = xcd * chunk[ps] + (ps == 0 ? slot : slot - chunk[0]);
    if (logical >= total[ps]) continue;
    const int32_t mypfx = ps == 0 ? pfx[0] : pfx[1];
    const int cls = __popcll(__ballot(mypfx <= logical));
    const int32_t before = __builtin_amdgcn_readlane(mypfx - (ps == 0 ? cnt[0] : cnt[1]), cls);
    const Tile t = make_tile<MODE, LAW, TN, BK>(p, sel_for(MODE, LAW, ps), cls, logical - before,
                                                __builtin_amdgcn_readlane(units, cls), p.offsets, TM);

    // ---- copy sources of this tile ----
    // K-contiguous A: the lane's row of copy j (rows past the tile's end read
    // its first row; their products are not stored)
    int32_t arow[CA], brow[CB];
    const int kslot = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);  // chunk of every K-contiguous copy
    if constexpr (kAKC) {
#pragma unroll
      for (int j = 0; j < CA; ++j) {
        const int row = 8 * (wave + 4 * j) + (lane >> 3);
        arow[j] = p.perm[t.pos0 + (row < t.nrows ? row : 0)];
      }
    }
    if constexpr (kBKC) {
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        const int row = 8 * (wave + 4 * j) + (lane >> 3);
        brow[j] = t.cstart + (t.cstart + row < t.cend ? row : 0);
      }
    }
    // row of C this lane writes, -1 for none
    int32_t erow = -1;
    {
      const int row = 32 * wm + lr;
      if constexpr (MODE != kModeBwdWeight) erow = row < t.nrows ? p.perm[t.pos0 + row] : -1;
      else erow = t.rstart + row < t.rend ? t.rstart + row : -1;
    }

    // weight gradient: the rows at the positions of step s, into this wave's
    // perm slot (zeros past the step's range)
    auto copy_perm = [&](int32_t s) {
      if constexpr (MODE == kModeBwdWeight) {
        int32_t k0 = 0, kend = 0;
        if (s < t.nsteps) step_range<MODE, LAW, BK>(p, t, p.offsets, s, k0, kend);
        dma4(k0 + lane < kend ? static_cast<const void*>(p.perm + k0 + lane) : zero,
             lds_addr(&prow_s[wave][s & (kRowSlots - 1)][0]));
      }
    };
    // The operands of a step, in CA + CB copies: copy_begin picks the step
    // (past the last one: zeros) and reads the rows of its positions (weight
    // gradient), copy_a(j) and copy_b(j) issue one copy each.  Without a
    // branch, so that a step's copies can sit between its MFMAs.
    int32_t ck0 = 0, cklen = 0, prow[CA];
    uint32_t cla = lds0;
    auto copy_begin = [&](int32_t s) {
      int32_t kend = 0;
      ck0 = 0;
      if (s < t.nsteps) step_range<MODE, LAW, BK>(p, t, p.offsets, s, ck0, kend);
      cklen = kend - ck0;
      cla = lds0 + (s % kStages) * kStageBytes;
      if constexpr (MODE == kModeBwdWeight) {
#pragma unroll
        for (int j = 0; j < CA; ++j)
          prow[j] = prow_s[wave][s & (kRowSlots - 1)][(wave + 4 * j) * (64 / kChunks) + lane / kChunks];
      }
    };
    auto copy_a = [&](int j) {
      const int ci = wave + 4 * j;
      const float* g;
      bool ok;
      if constexpr (kAKC) {
        ok = 4 * kslot < cklen;
        g = Ag + arow[j] * static_cast<int64_t>(MODE == kModeFwd ? p.K : p.N) + ck0 + 4 * kslot;
      } else {
        const int k = ci * (64 / kChunks) + lane / kChunks;
        const int32_t col = t.rstart + 4 * rc_chunk(k, lane % kChunks);
        ok = k < cklen;
        g = Ag + static_cast<int64_t>(prow[j]) * p.K + (col < t.rend ? col : t.rstart);
      }
      dma16(ok ? static_cast<const void*>(g) : zero, cla + ci * 1024);
    };
    auto copy_b = [&](int j) {
      const int ci = wave + 4 * j;
      const float* g;
      bool ok;
      if constexpr (kBKC) {
        ok = 4 * kslot < cklen;
        g = Bg + static_cast<int64_t>(brow[j]) * p.N + ck0 + 4 * kslot;
      } else {
        const int k = ci * (64 / kChunks) + lane / kChunks;
        const int32_t col = t.cstart + 4 * rc_chunk(k, lane % kChunks);
        ok = k < cklen;
        g = Bg + static_cast<int64_t>(MODE == kModeFwd ? ck0 + k : prow[j]) * p.N + (col < t.cend ? col : t.cstart);
      }
      dma16(ok ? static_cast<const void*>(g) : zero, cla + kABytes + ci * 1024);
    };
    auto copy_step = [&](int32_t s) {
      copy_begin(s);
#pragma unroll
      for (int j = 0; j < CA; ++j) copy_a(j);
#pragma unroll
      for (int j = 0; j < CB; ++j) copy_b(j);
    };

    block_barrier();  // every wave is done with the previous tile's stages
    if constexpr (MODE == kModeBwdWeight) {
#pragma unroll
      for (int s = 0; s < kAhead; ++s) copy_perm(s);
      wait_vm<0>();
    }
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      copy_perm(s + kAhead);
      copy_step(s);
    }

    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    float colsum = 0.f;

    for (int32_t s = 0; s < t.nsteps; ++s) {
      wait_vm<(kAhead - 1) * kGroup>();  // this wave's copies of step s have landed
      block_barrier();                  // and everyone's; the stage of step s - 1 is free
      const char* As = smem + (s % kStages) * kStageBytes;
      const char* Bs = As + kABytes;
      // every fragment of the step is read ahead of its MFMAs: a CU with one
      // tile has no other wave to fill the LDS latency of each slice
      float fa[4][4], fb[4][4];
#pragma unroll
      for (int rs = 0; rs < 4; ++rs) {
        read_frag<kAKC>(As, rs, lh, 32 * wm + lr, fa[rs]);
        read_frag<kBKC>(Bs, rs, lh, 32 * wn + lr, fb[rs]);
      }
      copy_begin(s + kAhead);
      copy_perm(s + 2 * kAhead);
#pragma unroll
      for (int rs = 0; rs < 4; ++rs) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[rs][e], fa[rs][e], acc, 0, 0, 0);
        // the copies of step s + kAhead, spread over the slices
        __builtin_amdgcn_sched_barrier(0);
        if (rs < CA) copy_a(rs);
        else copy_b(rs - CA);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (MODE == kModeBwdWeight) {
        if (t.do_dbias) {
          // one column per thread, its share of the step's K indexes
          constexpr int kPart = BK * TN / kThreads;
          const int c = threadIdx.x % TN, k0 = (threadIdx.x / TN) * kPart;
#pragma unroll
          for (int k = k0; k < k0 + kPart; ++k)
            colsum += *reinterpret_cast<const float*>(Bs + k * (16 * kChunks) + rc_chunk(k, c >> 2) * 16 + (c & 3) * 4);
        }
      }
    }
    wait_vm<0>();  // the copies past the last step, before the stages are reused

    // ---- epilogue ----
    // lane holds C[row m][columns n .. n+3] with m = 32 wm + lr and
    // n = 32 wn + 8 a + 4 lh, values acc[4a .. 4a+3]
    const int64_t crow = erow * static_cast<int64_t>(MODE == kModeBwdData ? p.K : p.N);
    auto each = [&](auto fn) {  // fn(element index of C, column, the 4 values)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int32_t col = t.cstart + 32 * wn + 4 * lh + 8 * a;
        if (erow >= 0 && col < t.cend) {
          float v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = acc[4 * a + j];
          fn(crow + col, col, v);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[4 * a + j] = v[j];
        }
      }
    };
    if constexpr (MODE == kModeBwdWeight) {
      float* dw = p.nsplit > 1 ? p.partial + static_cast<int64_t>(t.split) * p.K * p.N : p.dW;
      each([&](int64_t idx, int32_t, float (&v)[4]) { store4(dw, 0, idx, v); });
    } else {
      if constexpr (MODE == kModeFwd) {
        if (p.bias)
          each([&](int64_t, int32_t col, float (&v)[4]) {
            const float4 bv = *reinterpret_cast<const float4*>(p.bias + col);
            v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
          });
        if (p.Z) each([&](int64_t idx, int32_t, float (&v)[4]) { store4(p.Z, p.ydtype, idx, v); });
        if (p.act != kActNone)
          each([&](int64_t, int32_t, float (&v)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = act_apply(p.act, v[j]);
          });
      } else if (p.Zprev) {
        each([&](int64_t idx, int32_t, float (&v)[4]) {
          float z[4];
          load4(p.Zprev, 0, idx, z);
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] *= act_deriv(p.act, z[j]);
        });
      }
      each([&](int64_t idx, int32_t, float (&v)[4]) { store4(p.Y, p.ydtype, idx, v); });
    }
    if constexpr (MODE == kModeBwdWeight) {
      if (t.do_dbias) {
        // the threads of a column, added in a fixed order
        float* red = reinterpret_cast<float*>(smem);
        block_barrier();  // every wave is done with the stages
        red[threadIdx.x] = colsum;
        __syncthreads();
        if (threadIdx.x < TN && t.cstart + static_cast<int32_t>(threadIdx.x) < t.cend) {
          float sum = 0.f;
#pragma unroll
          for (int g = 0; g < kThreads / TN; ++g) sum += red[g * TN + threadIdx.x];
          const int32_t col = t.cstart + threadIdx.x;
          if (p.nsplit > 1) p.dbias_part[static_cast<int64_t>(t.split) * p.N + col] = sum;
          else p.dbias[col] = sum;
        }
        __syncthreads();
      }
    }
  }
}

// out = sum over s of part[s], in split order (so the result does not depend
// on timing).  The partials of up to 8 splits are loaded together before
// any is added: one dependent load after another left each thread waiting
// out nsplit memory round trips.
__global__ void split_reduce_kernel(const float* __restrict__ part, int nsplit, int64_t n,
                                    float* __restrict__ out) {
  const int64_t n4 = n >> 2;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
      float4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = s0 + k < nsplit ? reinterpret_cast<const float4*>(part + static_cast<int64_t>(s0 + k) * n)[i]
                               : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (s0 + k < nsplit) {
          acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w;
        }
      }
    }
    reinterpret_cast<float4*>(out)[i] = acc;
  }
  // tail (n not a multiple of 4)
  const int64_t t = (n4 << 2) + blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (blockIdx.x == 0 && t < n) {
    float a = part[t];
    for (int s = 1; s < nsplit; ++s) a += part[static_cast<int64_t>(s) * n + t];
    out[t] = a;
  }
}

// The same for partials whose blocks have a pass's number of splits each:
// a workgroup takes 1024 consecutive columns of one row of dW (its input
// group is uniform), a thread four of them (one output group: widths are
// multiples of 8).  The first row of workgroups adds the chunk sums of the
// bias gradient, if any, in chunk order (a launch of its own for them took
// 4.6 us behind the column sums; here they run beside the rows of dW).
template <int LAW>
__global__ __launch_bounds__(256) void block_reduce_kernel(const GemmParams p, const float* chunks, int nchunks) {
  const int32_t n = (blockIdx.x * 256 + threadIdx.x) * 4;
  const int32_t k = static_cast<int32_t>(blockIdx.y + blockIdx.z * gridDim.y) - 1;
  if (k >= p.K || n >= p.N) return;
  if (k < 0) {
    if (!chunks) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c0 = 0; c0 < nchunks; c0 += 16) {
      float4 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        v[u] = c0 + u < nchunks ? *reinterpret_cast<const float4*>(chunks + static_cast<int64_t>(c0 + u) * p.N + n)
                                : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (c0 + u < nchunks) {
          acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w;
        }
      }
    }
    // (dbias need only be 4-byte aligned)
    p.dbias[n] = acc.x; p.dbias[n + 1] = acc.y; p.dbias[n + 2] = acc.z; p.dbias[n + 3] = acc.w;
    return;
  }
  int i = 0, j = 0;
  while (k >= p.S[i + 1]) ++i;
  for (int lo = 0, hi = p.q - 1; lo < hi;) {  // the last group that starts at or before n
    const int mid = (lo + hi + 1) >> 1;
    if (n >= p.R[mid]) lo = mid;
    else hi = mid - 1;
    j = lo;
  }
  bool first;  // pass 0
  if constexpr (LAW == 2) first = tensor_in_pass(p, sel_for(kModeBwdWeight, LAW, 0), i, j);
  else if constexpr (LAW == 3) first = graph_in_pass(p, sel_for(kModeBwdWeight, LAW, 0), i, j);
  else first = LAW == 1 || i == j;
  const int ns = first ? p.nsplit : p.nsplit1;
  const int64_t at = static_cast<int64_t>(k) * p.N + n, kn = static_cast<int64_t>(p.K) * p.N;
  // the further splits of pass 0
  const float* more = p.partial + p.nsplit1 * kn + static_cast<int64_t>(k) * p.rmax + n - p.R[j];
  auto part = [&](int s) {
    return s < p.nsplit1 ? p.partial + s * kn + at : more + static_cast<int64_t>(s - p.nsplit1) * p.K * p.rmax;
  };
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < ns; s0 += 8) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = s0 + u < ns ? *reinterpret_cast<const float4*>(part(s0 + u)) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (s0 + u < ns) {
        acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w;
      }
    }
  }
  *reinterpret_cast<float4*>(p.dW + at) = acc;
}

__global__ void fill_zero_kernel(float* __restrict__ dst, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = 0.f;
}

// One workgroup per tile (at most kMaxGrid; a workgroup then takes every
// gridDim-th of its XCD's tiles).
constexpr int64_t kMaxGrid = int64_t{1} << 20;

template <int MODE, int LAW>
hipError_t launch_law(const GemmParams& p0, hipStream_t stream) {
  GemmParams p = p0;
  const int32_t* G = MODE == kModeBwdData ? p.S : p.R;  // column groups of C
  p.NTp[0] = p.MTp[0] = 0;
  for (int g = 0; g < p.q; ++g) {
    p.NTp[g + 1] = p.NTp[g] + (G[g + 1] - G[g] + TN - 1) / TN;
    p.MTp[g + 1] = p.MTp[g] + (p.S[g + 1] - p.S[g] + TM - 1) / TM;
  }
  const int64_t units = MODE == kModeBwdWeight ? static_cast<int64_t>(p.MTp[p.q]) * p.nsplit
                                               : static_cast<int64_t>(p.M) / TM + p.q;
  // (each XCD's share of a pass rounds up)
  const int64_t per_xcd = (units * p.NTp[p.q] + 7) / 8 + 2;
  const int64_t grid = 8 * std::min(per_xcd, kMaxGrid / 8);
  hipLaunchKernelGGL((star_gemm_f32_kernel<MODE, LAW>), dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, stream,
                     p);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const GemmParams& p, hipStream_t stream) {
  switch (p.law) {
    case 1: return launch_law<MODE, 1>(p, stream);
    case 2: return launch_law<MODE, 2>(p, stream);
    case 3: return launch_law<MODE, 3>(p, stream);
    default: return launch_law<MODE, 0>(p, stream);
  }
}

}  // namespace

hipError_t launch_gemm(int mode, const GemmParams& p, hipStream_t stream) {
  if (p.elem != 0) return hipErrorInvalidValue;  // bf16 operands run in the pipelined kernel
  if (mode == kModeFwd) return launch_mode<kModeFwd>(p, stream);
  if (mode == kModeBwdWeight) return launch_mode<kModeBwdWeight>(p, stream);
  return launch_mode<kModeBwdData>(p, stream);
}

hipError_t launch_fill_zero(float* dst, int64_t n, hipStream_t stream) {
  const int blocks = static_cast<int>(std::min<int64_t>(1024, (n + 255) / 256 + 1));
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream, dst, n);
  return hipGetLastError();
}

hipError_t launch_block_reduce(const GemmParams& p, const float* chunks, int nchunks, hipStream_t stream) {
  const unsigned rows = static_cast<unsigned>(p.K) + 1, gy = std::min(rows, 32768u);
  const dim3 grid((p.N + 1023) / 1024, gy, (rows + gy - 1) / gy);
  switch (p.law) {
    case 1: hipLaunchKernelGGL(block_reduce_kernel<1>, grid, dim3(256), 0, stream, p, chunks, nchunks); break;
    case 2: hipLaunchKernelGGL(block_reduce_kernel<2>, grid, dim3(256), 0, stream, p, chunks, nchunks); break;
    case 3: hipLaunchKernelGGL(block_reduce_kernel<3>, grid, dim3(256), 0, stream, p, chunks, nchunks); break;
    default: hipLaunchKernelGGL(block_reduce_kernel<0>, grid, dim3(256), 0, stream, p, chunks, nchunks); break;
  }
  return hipGetLastError();
}

hipError_t launch_split_reduce(const GemmParams& p, hipStream_t stream) {
  const int64_t nKN = static_cast<int64_t>(p.K) * p.N;
  int blocks = static_cast<int>(std::min<int64_t>(2048, (nKN / 4 + 255) / 256 + 1));
  hipLaunchKernelGGL(split_reduce_kernel, dim3(blocks), dim3(256), 0, stream, p.partial,
                     p.nsplit, nKN, p.dW);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.dbias == nullptr) return e;
  return launch_sum_chunks(p.dbias_part, p.nsplit, p.N, p.dbias, stream);
}

}  // namespace starq
