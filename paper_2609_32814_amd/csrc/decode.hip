// Decode-step projection for few rows (one new token per sequence, M <= 64).
//
// Single-token FFN decode is a matrix-vector problem bound by weight
// bandwidth (Sec. 4.2 notes that decode needs its own implementation;
// Sec. 5.3).  The batched kernel's per-type gathering would read a shared
// diagonal block once per row type present; here every weight block that
// some row's support reaches is streamed exactly once per step, and rows
// whose support skips the block multiply zeros.
//
// A workgroup owns 64 output columns (inside one output group j) and one of
// `splits` equal shares of the K slices they need: K is cut into 32-row
// slices, and a slice is needed when some row's support reaches one of its
// input groups (k in B(t_b, j)).  What bounds it is the weight stream, and
// below about 20 MB the chain of round trips around it: types, slices,
// weights, hand-over.  64 columns make every row piece of a slice a whole
// 128-byte line, and splitting K fills the chip: each projection of 8 rows,
// 2560 <-> 9728, q = 4 (46 MB of weights), 81 -> 16 to 20 us against
// 16-column tiles over all of K (32-byte pieces, up to 128 slices copied and
// then waited for at once).  Each wavefront streams every fourth slice of
// the share straight from global memory into a ring of its own in LDS (four
// copies of 1 KB for the weights, one per 16 rows for their input pieces;
// two or three slices, so that two workgroups fit a CU), waits only for the
// oldest slice, reads it back with the LDS transpose read (two reads give
// every lane 8 consecutive K values of one column) and multiplies with
// v_mfma_f32_16x16x32_bf16.  No barrier in the stream.  The four
// wavefronts' sums are added in LDS in a fixed order.
//
// With more than one split, a workgroup stores its sums (agent-coherent
// stores, acknowledged before its arrival is counted) and the last of a
// tile's workgroups to arrive adds all of them in split order, so results do
// not depend on timing.  It also sets the tile's counter back to zero for
// the next projection.  Nobody waits for anybody.
//
// A small projection of more than 16 rows takes tiles of 16 columns without
// splits: with few slices the time is the workgroup's own end (the waves'
// sums through LDS, bias, activation, stores), which then spreads over four
// times as many workgroups.  See decode_phase_cols.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace starq {

namespace {

constexpr int kThreads = 256;
constexpr int SLICE = kDecodeSliceK;  // 32 K rows
constexpr int kWide = kDecodePhaseN / 16, kNarrow = kDecodeNarrowN / 16;  // 16-column blocks of a tile

typedef short v4i16_t __attribute__((ext_vector_type(4)));
#define STARQ_LDS __attribute__((address_space(3)))

// k in B(i, j): law 0 {i, j}; law 1 every group; law 2 (tensor power of
// the two-group law) every bit of k equal to that bit of i or of j; law 3
// (graph algebra, bit j of adj[i] for the edge i -> j) {i} for j = i, {i, j}
// for an edge, nothing otherwise
__device__ __forceinline__ bool in_support(int law, const uint64_t* adj, int i, int j, int k) {
  if (law == 2) return ((k ^ i) & (k ^ j)) == 0;
  if (law == 3) {
    // graph algebra: B(i,i) = {i}, B(i,j) = {i, j} for an edge i -> j, empty otherwise
    if (j == i) return k == i;
    return ((adj[i] >> j) & 1ull) && (k == i || k == j);
  }
  return law == 1 || k == i || k == j;
}

// the input group of index x: the last g with starts[g] <= x, by binary
// search over the starts (held in LDS: searched from the kernel's argument
// block, every step was a dependent scalar load)
__device__ __forceinline__ int group_of(const int32_t* starts, int q, int32_t x) {
  int lo = 0, hi = q - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (x >= starts[mid]) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Slices a wave holds in LDS: two workgroups per CU fit.
constexpr int wave_slots(int mb, int nb) { return nb == kNarrow ? 4 : (mb <= 2 ? 3 : 2); }

// 16-column block cb of slice row r sits at block cb ^ col_swz(r): the rows
// a transposing read takes together (0-3 and 8-11 of a 16-row half) then
// cover all banks.
__device__ __forceinline__ int col_swz(int r) { return ((r >> 1) & 1) | (((r >> 3) & 1) << 1); }

__device__ __forceinline__ void st_agent64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_agent64(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 64 zero bytes: the source of an input piece that no support reaches
__device__ __attribute__((aligned(64))) uint32_t g_decode_zero[16];

template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// MB: 16-row blocks of the step (M <= 16 MB); NB: 16-column blocks of a tile
template <int MB, int NB>
__global__ __launch_bounds__(kThreads, 2) void decode_phase_kernel(const DecodePhase p) {
  constexpr int TN = 16 * NB;
  constexpr int kSliceBytes = SLICE * TN * 2;
  constexpr int kSlots = wave_slots(MB, NB);
  // 16 x 16 blocks of the tile that a thread finishes (the waves' sums are
  // shared out by block): block wave + 4 it, column block of it and row block
  constexpr int kItems = (NB * MB + 3) / 4;
  constexpr int kSlot = kSliceBytes + MB * 1024;  // a slice's weights and input pieces
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ unsigned long long rowmask_s[kMaxQGroups];
  __shared__ int32_t S_s[kMaxQGroups + 1];
  __shared__ int16_t slices_s[kDecodeMaxK / SLICE];
  __shared__ int32_t wave_cnt_s[4];
  __shared__ int32_t last_s;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;

  // the status line reads zero: these kernels do not wait
  if (p.status && blockIdx.x == 0 && tid < kCounterStride) p.status[tid] = 0;

  const int nt = p.NTp[p.q];
  const int ct = blockIdx.x % nt, split = blockIdx.x / nt;
  const int j = __popcll(__ballot(lane < p.q && ct >= p.NTp[lane + 1]));
  const int32_t n0 = p.R[j] + (ct - p.NTp[j]) * TN;
  const int32_t nend = p.R[j + 1];

  // the input group starts, searched from LDS below
  for (int i = tid; i <= p.q; i += kThreads) S_s[i] = p.S[i];
  // which rows need block (g, j), per input group g: one row per lane, one
  // ballot per group
  {
    // a row whose type lies outside [0, q) has an empty support
    const int t = lane < p.M ? p.types[lane] : -1;
    const bool valid = t >= 0 && t < p.q;
    for (int g = wave; g < p.q; g += 4) {
      const unsigned long long m = __ballot(valid && in_support(p.law, p.adj, t, j, g));
      if (lane == 0) rowmask_s[g] = m;
    }
  }
  __syncthreads();
  // needed slices, in K order: one slice per thread a round (256 slices a
  // round), compacted with ballots
  const int nsl = (p.K + SLICE - 1) / SLICE;  // <= kDecodeMaxK / SLICE
  int32_t found = 0;                          // needed slices before this round
  for (int base = 0; base < nsl; base += kThreads) {
    const int sl = base + tid;
    bool need = false;
    if (sl < nsl) {
      for (int piece = 0; piece < SLICE / 8; ++piece) {
        const int32_t k = sl * SLICE + piece * 8;
        if (k < p.K && rowmask_s[group_of(S_s, p.q, k)]) need = true;
      }
    }
    const unsigned long long bal = __ballot(need);
    if (lane == 0) wave_cnt_s[wave] = __popcll(bal);
    __syncthreads();
    if (need) {
      int before = found + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
      for (int w = 0; w < wave; ++w) before += wave_cnt_s[w];
      slices_s[before] = static_cast<int16_t>(sl);
    }
    found += wave_cnt_s[0] + wave_cnt_s[1] + wave_cnt_s[2] + wave_cnt_s[3];
    __syncthreads();  // every thread has read the counts before the next round writes them
  }
  // this split's share of them
  const int lo = found * split / p.splits, hi = found * (split + 1) / p.splits;

  // compute: lane group G = lane/16 holds K rows 8G..8G+7 of a slice for
  // column lane%16 of each 16-column block (transpose reads), and the input
  // pieces of rows 16 mb + lane%16
  const int G = lane >> 4;
  const int pl = lane & 15;
  f32x4_t acc[NB][MB];
#pragma unroll
  for (int cb = 0; cb < NB; ++cb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[cb][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // this wave's slices: lo + wave + 4 t, t < n
  const int n = max(0, (hi - lo - wave + 3) >> 2);
  char* mine = lds + wave * (kSlots * kSlot);
  const uint32_t mine_lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(mine)));
  // Slice t into its slot: weights, 8 rows a copy (lane l: row l/8, 16 bytes
  // of it; a 16-column tile's 32 rows in one copy), then the rows' input pieces, one copy a row block (zeros where
  // the support skips them).  Rows past K repeat row K-1 and columns past
  // the group repeat its first ones (finite values; their products are
  // either multiplied by zero inputs or never stored).
  auto copy = [&](int t) {
    const int32_t k0 = slices_s[lo + wave + 4 * t] * SLICE;
    const uint32_t dst = mine_lds + (t % kSlots) * kSlot;
#pragma unroll
    for (int d = 0; d < NB; ++d) {
      const int r = SLICE / NB * d + lane / (2 * NB), c = lane % (2 * NB);
      int32_t col = n0 + 16 * (NB == kWide ? (c >> 1) ^ col_swz(r) : 0) + 8 * (c & 1);
      col = col < nend ? col : n0;
      dma16(p.W + static_cast<int64_t>(min(k0 + r, p.K - 1)) * p.N + col, dst + d * 1024);
    }
    const int32_t kk = k0 + 8 * G;
    const unsigned long long gm = kk < p.K ? rowmask_s[group_of(S_s, p.q, kk)] : 0ull;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = 16 * mb + pl;
      const bool ok = m < p.M && ((gm >> m) & 1ull);
      dma16(ok ? static_cast<const void*>(p.A + static_cast<int64_t>(m) * p.K + kk) : g_decode_zero,
            dst + kSliceBytes + mb * 1024);
    }
  };
  constexpr int kCopies = NB + MB;  // of a slice
  for (int t = 0; t < min(n, kSlots); ++t) copy(t);
  for (int t = 0; t < n; ++t) {
    // slice t has landed (the copies of the kSlots - 1 slices after it may
    // still be in flight)
    if (t + kSlots - 1 < n) wait_vm<(kSlots - 1) * kCopies>();
    else wait_vm<0>();
    const char* slot = mine + (t % kSlots) * kSlot;
    uint4 wf[NB], x[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) x[mb] = *reinterpret_cast<const uint4*>(slot + kSliceBytes + mb * 1024 + lane * 16);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      const int r = 8 * G + (pl >> 2);
      const char* a0 = slot + r * (2 * TN) + (NB == kWide ? cb ^ col_swz(r) : 0) * 32 + (pl & 3) * 8;
      const char* a1 = slot + (r + 4) * (2 * TN) + (NB == kWide ? cb ^ col_swz(r + 4) : 0) * 32 + (pl & 3) * 8;
      const v4i16_t w0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((STARQ_LDS v4i16_t*)(a0));
      const v4i16_t w1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((STARQ_LDS v4i16_t*)(a1));
      wf[cb].x = static_cast<uint16_t>(w0[0]) | (static_cast<uint32_t>(static_cast<uint16_t>(w0[1])) << 16);
      wf[cb].y = static_cast<uint16_t>(w0[2]) | (static_cast<uint32_t>(static_cast<uint16_t>(w0[3])) << 16);
      wf[cb].z = static_cast<uint16_t>(w1[0]) | (static_cast<uint32_t>(static_cast<uint16_t>(w1[1])) << 16);
      wf[cb].w = static_cast<uint16_t>(w1[2]) | (static_cast<uint32_t>(static_cast<uint16_t>(w1[3])) << 16);
    }
    // the slot is free once its reads are done
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    if (t + kSlots < n) copy(t + kSlots);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        // D[n][m] += W^T x^T: lane ends with 4 consecutive columns of row m
        acc[cb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8_t, wf[cb]), __builtin_bit_cast(bf16x8_t, x[mb]), acc[cb][mb], 0, 0, 0);
  }

  // add the four waves' sums in a fixed order: thread tid then holds, of row
  // block mb and column block cb of item wave + 4 it, columns n0 + 16 cb + 4
  // (lane / 16) .. + 3 of row 16 mb + lane % 16
  __syncthreads();  // every wave is done with its slots
  f32x4_t* red = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
  for (int cb = 0; cb < NB; ++cb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) red[((wave * NB + cb) * MB + mb) * 64 + lane] = acc[cb][mb];
  __syncthreads();
  f32x4_t z[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int item = min(wave + 4 * it, NB * MB - 1), cb = item % NB, mb = item / NB;
    z[it] = red[(cb * MB + mb) * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) z[it] += red[((w * NB + cb) * MB + mb) * 64 + lane];
  }

  if (NB == kWide && p.splits > 1) {
    // (item wave + 4 mb: column block wave of row block mb)
    // sums as two 8-byte words, one 16 MB x 64 block of them per (tile,
    // split); rows past M are not stored
    const int64_t block = static_cast<int64_t>(MB) * kThreads * 2;
    uint64_t* tile = p.part + static_cast<int64_t>(ct) * p.splits * block;
    uint64_t* dst = tile + split * block + 2 * tid;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if (16 * mb + pl < p.M) {
        const uint2 a = make_uint2(__float_as_uint(z[mb][0]), __float_as_uint(z[mb][1]));
        const uint2 b = make_uint2(__float_as_uint(z[mb][2]), __float_as_uint(z[mb][3]));
        st_agent64(dst + mb * 2 * kThreads, __builtin_bit_cast(uint64_t, a));
        st_agent64(dst + mb * 2 * kThreads + 1, __builtin_bit_cast(uint64_t, b));
      }
    }
    __builtin_amdgcn_s_waitcnt(0);  // the stores are acknowledged ...
    __syncthreads();                // ... every thread's
    if (tid == 0) {
      const int32_t n = __hip_atomic_fetch_add(p.cnt + ct, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_s = n == p.splits - 1;
    }
    __syncthreads();
    if (!last_s) return;
    if (tid == 0) __hip_atomic_store(p.cnt + ct, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      z[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (16 * mb + pl >= p.M) continue;
      const uint64_t* src = tile + 2 * tid + mb * 2 * kThreads;
      for (int s0 = 0; s0 < p.splits; s0 += 8) {
        uint64_t a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int s = min(s0 + u, p.splits - 1);
          a[u] = ld_agent64(src + s * block);
          b[u] = ld_agent64(src + s * block + 1);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (s0 + u < p.splits) {
            const uint2 av = __builtin_bit_cast(uint2, a[u]), bv = __builtin_bit_cast(uint2, b[u]);
            z[mb][0] += __uint_as_float(av.x); z[mb][1] += __uint_as_float(av.y);
            z[mb][2] += __uint_as_float(bv.x); z[mb][3] += __uint_as_float(bv.y);
          }
        }
      }
    }
  }

#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int item = wave + 4 * it;
    const int m = 16 * (item / NB) + pl;
    const int32_t n = n0 + 16 * (item % NB) + 4 * G;
    if (item >= NB * MB || m >= p.M || n >= nend) continue;
    f32x4_t v = z[it];
    if (p.bias) {
      const float4 bv = *reinterpret_cast<const float4*>(p.bias + n);
      v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
    }
    const int64_t o = static_cast<int64_t>(m) * p.N + n;
    if (p.mode == 0) {
      uint2 w;
      w.x = f32_to_bf16(act_apply(p.act, v[0])) | (static_cast<uint32_t>(f32_to_bf16(act_apply(p.act, v[1]))) << 16);
      w.y = f32_to_bf16(act_apply(p.act, v[2])) | (static_cast<uint32_t>(f32_to_bf16(act_apply(p.act, v[3]))) << 16);
      *reinterpret_cast<uint2*>(p.out_bf16 + o) = w;
      continue;
    }
    float hv[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.residual) {
      if (p.h_init) {
        const uint2 hi4 = *reinterpret_cast<const uint2*>(p.h_init + o);
        hv[0] = bf16_to_f32(hi4.x & 0xffffu); hv[1] = bf16_to_f32(hi4.x >> 16);
        hv[2] = bf16_to_f32(hi4.y & 0xffffu); hv[3] = bf16_to_f32(hi4.y >> 16);
      } else {
        const float4 hp = *reinterpret_cast<const float4*>(p.h_in + o);
        hv[0] = hp.x; hv[1] = hp.y; hv[2] = hp.z; hv[3] = hp.w;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) hv[e] += v[e];
    if (p.h_out) *reinterpret_cast<float4*>(p.h_out + o) = make_float4(hv[0], hv[1], hv[2], hv[3]);
    if (p.out_bf16) {
      uint2 w;
      w.x = f32_to_bf16(hv[0]) | (static_cast<uint32_t>(f32_to_bf16(hv[1])) << 16);
      w.y = f32_to_bf16(hv[2]) | (static_cast<uint32_t>(f32_to_bf16(hv[3])) << 16);
      *reinterpret_cast<uint2*>(p.out_bf16 + o) = w;
    }
    if (p.Y) {
#pragma unroll
      for (int e = 0; e < 4; ++e) store_out(p.Y, p.ydtype, o + e, hv[e]);
    }
  }
}

template <int MB, int NB>
hipError_t launch_nb(const DecodePhase& p, hipStream_t stream) {
  // the slots, reused for the waves' sums
  constexpr size_t smem = std::max<size_t>(4 * wave_slots(MB, NB) * (SLICE * NB * 32 + MB * 1024),
                                           static_cast<size_t>(4 * NB * MB) * 1024);
  static std::atomic<unsigned long long> lds_set{0};
  const hipError_t attr =
      ensure_lds_limit(reinterpret_cast<const void*>(decode_phase_kernel<MB, NB>), lds_set, static_cast<int>(smem));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((decode_phase_kernel<MB, NB>), dim3(static_cast<unsigned>(p.NTp[p.q] * p.splits)), dim3(kThreads),
                     smem, stream, p);
  return hipGetLastError();
}
template <int MB>
hipError_t launch_mb(const DecodePhase& p, hipStream_t stream) {
  if (p.cols == kDecodePhaseN) return launch_nb<MB, kWide>(p, stream);
  if (p.cols == kDecodeNarrowN && p.splits == 1) return launch_nb<MB, kNarrow>(p, stream);
  return hipErrorInvalidValue;
}

// Most slices a column tile can need: the support of output group j over the
// rows' types reaches at most min(q, M + 1) groups under the star and graph
// laws (B(t, j) within {t, j}), every group under the others; a group of s
// inputs spans at most ceil(s / 32) + 1 slices.
template <typename I>
int64_t most_slices(int law, int q, const I* S, int64_t M) {
  const int64_t reach = (law == 0 || law == 3) ? std::min<int64_t>(q, M + 1) : q;
  int64_t widest = 0;
  for (int g = 0; g < q; ++g) widest = std::max<int64_t>(widest, (S[g + 1] - S[g] + SLICE - 1) / SLICE + 1);
  return std::max<int64_t>(1, std::min<int64_t>((S[q] + SLICE - 1) / SLICE, reach * widest));
}

}  // namespace

// 16 columns where a tile has at most 32 slices (eight a wave) and the tiles
// are no more than the chip's CUs.  Measured with 40 layers, star law, q = 4,
// 16 against 64 columns, us a projection: 128 <-> 256, 64 rows, 8.8 and 10.8;
// 256 <-> 512, 17 rows 9.0 and 10.4, 64 rows 9.5 and 12.1; 768 <-> 3072, 64
// rows, 14.8 and 16.1; 1024 <-> 4096 (the limit of both), 64 rows, 16.3 and
// 17.9.  Up to 16 rows a thread of the wide tiles finishes one block as well,
// and 64 columns are level or faster.
int decode_phase_cols(int law, int q, const int64_t* S, const int64_t* R, int64_t M) {
  int64_t tiles = 0;
  for (int g = 0; g < q; ++g) tiles += (R[g + 1] - R[g] + kDecodeNarrowN - 1) / kDecodeNarrowN;
  return M > 16 && most_slices(law, q, S, M) <= 32 && tiles <= 256 ? kDecodeNarrowN : kDecodePhaseN;
}

// At most one workgroup per CU (256 / tiles, rounded down: with 129 to 255
// column tiles every tile has one split and the other CUs none, as the up
// projection of 2560 -> 9728 with its 152), of at least 16 slices (four a
// wave; 1024 <-> 4096 up to 16 rows stops at 128 workgroups by this).  Measured
// on 2560 <-> 9728, 8 rows of 4 types: 256 workgroups 15.5 to 19.8 us a
// projection, 512 (two per CU) 20.1, 768 23.0; 64 rows: 28.3, 34.2, 41.4 (a
// workgroup's start, its hand-over of partial sums and its arrival cost
// about 8 us whatever its share).  Shares of 8 slices where there is less
// work: 768 <-> 3072, 64 rows, 15.4 against 13.8 us.
int decode_phase_splits(int law, int q, const int64_t* S, int32_t tiles, int64_t M) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(256 / tiles, most_slices(law, q, S, M) / 16)));
}

size_t decode_phase_part_bytes(int32_t tiles, int splits, int64_t M) {
  return splits > 1 ? static_cast<size_t>(tiles) * splits * ((M + 15) / 16) * kThreads * 16 : 0;
}

hipError_t launch_decode_phase(const DecodePhase& p, hipStream_t stream) {
  switch ((p.M + 15) / 16) {
    case 1: return launch_mb<1>(p, stream);
    case 2: return launch_mb<2>(p, stream);
    case 3: return launch_mb<3>(p, stream);
    default: return launch_mb<4>(p, stream);
  }
}

}  // namespace starq
