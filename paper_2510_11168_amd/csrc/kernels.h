// HIP kernels of the ELMO head step for gfx950 (Algorithm 1 of the paper, one label chunk at a
// time): logits + sigmoid-BCE gradient epilogue, input-gradient product, fused weight-gradient +
// SGD + Kahan + stochastic-rounding update, and the small per-step helpers around them.
#pragma once
#include "numerics.h"
#include "tiles.h"

namespace elmo {

// ---------------------------------------------------------------------------------------------
// Small helpers
// ---------------------------------------------------------------------------------------------
__device__ inline uint32_t pack2_bf16(float a, float b) {   // hardware round-to-nearest-even
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}
// sigmoid on the transcendental unit: v_exp_f32 and v_rcp_f32 (about 1 ulp each), five instructions.
// The result is rounded to BF16 right away, so the last FP32 bits only matter next to a BF16 tie.
__device__ inline float sigmoidf_fast(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * z));
}
__device__ inline float softplusf_fast(float z) { return fmaxf(z, 0.0f) + __logf(1.0f + __expf(-fabsf(z))); }

template <int NW> __device__ inline float block_sum(float v, float* red /*>= NW floats of LDS*/) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < NW; ++i) s += red[i];
  return s;
}

__global__ void __launch_bounds__(kThreads) k_fill_u32(uint32_t* __restrict__ p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) p[i] = v;
}

// ---------------------------------------------------------------------------------------------
// Per-batch label index: the positives (CSR by sample) regrouped by 128-label tile, so that the
// logits epilogue of a tile finds its few positives with two loads (Algorithm 1 filters the
// COO pairs of each chunk; here the filter is a counting sort done once per step).
// ---------------------------------------------------------------------------------------------
// Eight lanes share a sample row (its positives are few, and one lane per row would walk them as a
// chain of dependent loads).  Label ids sorted by falling frequency put most positives of a batch
// into the first few bins; atomics on one address serialise in L2, so every workgroup first counts
// the bins below kHotBins in LDS and touches each of those global counters once.
constexpr int kRowLanes = 8;
constexpr int kHotBins = 2048;                                   // labels 0 .. 262143
__global__ void __launch_bounds__(kThreads) k_label_hist(const int* __restrict__ indptr, const int* __restrict__ indices,
                                                         int B, int64_t L, int64_t nnz, int* __restrict__ cnt,
                                                         int* __restrict__ bad) {
  __shared__ int hot[kHotBins];
  for (int i = threadIdx.x; i < kHotBins; i += kThreads) hot[i] = 0;
  __syncthreads();
  const int t = blockIdx.x * kThreads + threadIdx.x;
  const int b = t / kRowLanes, sub = t % kRowLanes;
  if (b < B) {
    const int p0 = indptr[b], p1 = indptr[b + 1];
    if (p0 < 0 || p1 < p0 || p1 > nnz) {
      if (bad && sub == 0) atomicOr(bad, 1);
    } else {
      for (int p = p0 + sub; p < p1; p += kRowLanes) {
        const int l = indices[p];
        const bool in_range = l >= 0 && l < L;
        if (bad && (!in_range || (p > p0 && l <= indices[p - 1]))) atomicOr(bad, 2);   // out of range, or not strictly ascending
        if (in_range) {
          const int bin = l >> 7;
          if (bin < kHotBins) atomicAdd(&hot[bin], 1);
          else atomicAdd(&cnt[bin], 1);
        }
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kHotBins; i += kThreads) {
    const int c = hot[i];
    if (c) atomicAdd(&cnt[i], c);
  }
}
// Exclusive scan of cnt[0..nb) into ptr[0..nb] (ptr[nb] = total) and cur[0..nb) = ptr.  One
// workgroup; the bins pass through LDS in segments so that global memory is read and written in
// whole lines (a thread's run of consecutive bins would otherwise touch 64 lines per load), every
// thread sums a run of a segment, the 1024 run totals are scanned in LDS.
constexpr int kScanRun = 15, kScanSeg = kScanRun * 1024;
__global__ void __launch_bounds__(1024) k_label_scan(const int* __restrict__ cnt, int nb, int* __restrict__ ptr, int* __restrict__ cur) {
  __shared__ int seg[kScanSeg];
  __shared__ int part[1024];
  const int tid = threadIdx.x;
  int carry = 0;
  for (int base = 0; base < nb; base += kScanSeg) {
    const int m = min(kScanSeg, nb - base);
    for (int i = tid; i < m; i += 1024) seg[i] = cnt[base + i];
    __syncthreads();
    const int i0 = min(tid * kScanRun, m), i1 = min(i0 + kScanRun, m);
    int sum = 0;
    for (int i = i0; i < i1; ++i) sum += seg[i];
    part[tid] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int t = tid >= o ? part[tid - o] : 0;
      __syncthreads();
      part[tid] += t;
      __syncthreads();
    }
    int run = carry + part[tid] - sum;               // exclusive prefix of this thread's run
    for (int i = i0; i < i1; ++i) {
      const int v = seg[i];
      seg[i] = run;
      run += v;
    }
    carry += part[1023];
    __syncthreads();
    for (int i = tid; i < m; i += 1024) {
      const int v = seg[i];
      ptr[base + i] = v;
      cur[base + i] = v;
    }
    __syncthreads();
  }
  if (tid == 0) ptr[nb] = carry;
}
// Positives into their bins.  For the bins below kHotBins a workgroup ranks its positives in LDS,
// reserves one range per bin with a single global atomic and then writes; a thread keeps up to
// four such positives in registers between the two phases, anything beyond goes the direct way.
__global__ void __launch_bounds__(kThreads) k_label_scatter(const int* __restrict__ indptr, const int* __restrict__ indices,
                                                            int B, int64_t L, int64_t nnz, int* __restrict__ cur,
                                                            int2* __restrict__ pos) {
  __shared__ int hot[kHotBins];
  for (int i = threadIdx.x; i < kHotBins; i += kThreads) hot[i] = 0;
  __syncthreads();
  const int t = blockIdx.x * kThreads + threadIdx.x;
  const int b = t / kRowLanes, sub = t % kRowLanes;
  int lab[4] = {-1, -1, -1, -1}, rank[4] = {0, 0, 0, 0};
  if (b < B) {
    const int p0 = indptr[b], p1 = indptr[b + 1];
    if (!(p0 < 0 || p1 < p0 || p1 > nnz)) {
      int kept = 0;
      for (int p = p0 + sub; p < p1; p += kRowLanes) {
        const int l = indices[p];
        if (l < 0 || l >= L) continue;
        const int bin = l >> 7;
        if (bin < kHotBins && kept < 4) {
          const int r = atomicAdd(&hot[bin], 1);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k == kept) { lab[k] = l; rank[k] = r; }
          ++kept;
        } else {
          const int slot = atomicAdd(&cur[bin], 1);
          if (slot < nnz) pos[slot] = make_int2(l, b);
        }
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kHotBins; i += kThreads) {
    const int c = hot[i];
    hot[i] = c ? atomicAdd(&cur[i], c) : 0;          // first slot of this workgroup's range in bin i
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (lab[k] >= 0) {
      const int slot = hot[lab[k] >> 7] + rank[k];
      if (slot < nnz) pos[slot] = make_int2(lab[k], b);
    }
}

// The same index by one workgroup of 1024 threads with all bins in LDS: counts, exclusive prefix, positives
// into their slots.  The three kernels above cost a launch each (4-5 us apart) and a single-workgroup scan of
// all bins in memory (16 us at 23438 bins); this one runs beside the workgroups that stage the inputs, in the
// same launch.  Its passes are chains of memory round trips, so the row pointers and first labels of
// eight rows per thread are fetched at once, and what a row has beyond kRowWalk positives is left to whole waves at the
// end of a pass: eight rows of 3000 positives 128 apart among 1024 rows, 3 M labels, whose chains all fell to the same
// eight threads, took 1277 us (the kernels above 333), now 80.  Same treatment of malformed rows as above (skipped; flagged
// when `flag` is given); positions never exceed nnz.
constexpr int kSetupThreads = 1024;
constexpr int kIndexMaxBins = 32768;                             // 128 KiB of LDS: labels 0 .. 4194303
constexpr int kIndexMaxNnz = 65536;
constexpr int kRowWalk = 64;
constexpr int kSetupMaxSmem = 159 * 1024;                        // beside the static part
// One CU places 64 positives in about the time of 64 scattered stores and takes a round of latencies per 1024 rows, the kernels
// above pay launches and their scan of the bins: where the lines cross (set-up of a step, one workgroup / kernels):
//   782 bins:    1024 rows of 7 13 / 18 us, of 16 20 / 18; 2048 rows of 4 20 / 20; 4096 rows of 1 32 / 22
//   23438 bins:  512 rows of 64 43 / 42; 2048 rows of 7 26 / 32, of 16 41 / 35; 3072 rows of 4 30 / 32, of 16 58 / 35
// With at most one row per group of lanes the walk is never longer than the kernels' (64 rows of 1000: 64 / 240 us).
inline bool index_in_one_workgroup(int64_t nb, int B, int64_t nnz) {
  if (nb > kIndexMaxBins || nnz > kIndexMaxNnz || (nb + B) * 4 > kSetupMaxSmem) return false;
  return B <= kSetupThreads / kRowLanes || nnz + 4 * (int64_t)B + 10 * std::max<int64_t>(B - 1024, 0) <= 17500 + nb * 3 / 4;
}
struct IndexArgs {
  const int* indptr; const int* indices;
  int64_t L, nnz;
  int nb;                                                        // bins; 0 = the index is built by the kernels above
  int* ptr; int2* pos; int* flag;
};
// f(label, row, place in `indices` of a positive that has one before it in its row, or 0) for the first kRowWalk positives of
// every row; the rows that have more are collected in long_rows if it is given.
template <class F>
__device__ __forceinline__ void for_each_positive(const IndexArgs& ia, int B, int tid, int* long_rows, int* n_long, F&& f) {
  constexpr int NR = 8, RPP = kSetupThreads / kRowLanes;         // rows in flight per thread, rows per pass
  const int sub = tid % kRowLanes;
  for (int r0 = tid / kRowLanes; r0 < B; r0 += NR * RPP) {
    int p0[NR], p1[NR], l[NR], most = 0;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int r = r0 + k * RPP;
      p0[k] = r < B ? ia.indptr[r] : 0;
      p1[k] = r < B ? ia.indptr[r + 1] : 0;
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      if (p0[k] < 0 || p1[k] < p0[k] || p1[k] > ia.nnz) { f(-1, -1, 0); p0[k] = p1[k] = 0; }
      l[k] = p0[k] + sub < p1[k] ? ia.indices[p0[k] + sub] : 0;
      most = max(most, p1[k] - p0[k]);
    }
    if (most > kRowWalk)
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (p1[k] - p0[k] > kRowWalk) {
          if (long_rows && sub == 0) long_rows[atomicAdd(n_long, 1)] = r0 + k * RPP;
          p1[k] = p0[k] + kRowWalk;
        }
#pragma unroll
    for (int k = 0; k < NR; ++k)
      for (int p = p0[k] + sub; p < p1[k]; p += kRowLanes) f(p == p0[k] + sub ? l[k] : ia.indices[p], r0 + k * RPP, p > p0[k] ? p : 0);
  }
}
// The rest of the collected rows, a wave each.
template <class F>
__device__ __forceinline__ void for_each_left_positive(const IndexArgs& ia, int tid, const int* long_rows, int n, F&& f) {
  const int lane = tid & 63;
  for (int i = tid >> 6; i < n; i += kSetupThreads / 64) {
    const int r = long_rows[i], end = ia.indptr[r + 1];
    for (int p = ia.indptr[r] + kRowWalk + lane; p < end; p += 64) f(ia.indices[p], r, p);
  }
}
__device__ inline void label_index(const IndexArgs& ia, int B, int* h) {
  __shared__ int wsum[kSetupThreads / 64];
  __shared__ int bad, n_long;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int* long_rows = h + ia.nb;                                    // [B]
  for (int i = tid; i < ia.nb; i += kSetupThreads) h[i] = 0;
  if (tid == 0) bad = n_long = 0;
  __syncthreads();
  const auto count = [&](int l, int b, int p) {
    if (b < 0) { if (ia.flag) atomicOr(&bad, 1); return; }
    const bool in_range = l >= 0 && l < ia.L;
    if (ia.flag && (!in_range || (p > 0 && l <= ia.indices[p - 1]))) atomicOr(&bad, 2);
    if (in_range) atomicAdd(&h[l >> 7], 1);
  };
  for_each_positive(ia, B, tid, long_rows, &n_long, count);
  __syncthreads();
  const int n = n_long;
  if (n) {
    for_each_left_positive(ia, tid, long_rows, n, count);
    __syncthreads();
  }
  const int run = ((ia.nb + kSetupThreads - 1) / kSetupThreads) | 1;      // odd: consecutive threads' runs start in different banks
  const int i0 = min(tid * run, ia.nb), i1 = min(i0 + run, ia.nb);
  int sum = 0;
  for (int i = i0; i < i1; ++i) sum += h[i];
  int scan = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(scan, o, 64);
    scan += lane >= o ? t : 0;
  }
  if (lane == 63) wsum[wave] = scan;
  __syncthreads();
  int at = scan - sum, total = 0;
#pragma unroll
  for (int w = 0; w < kSetupThreads / 64; ++w) {
    at += w < wave ? wsum[w] : 0;
    total += wsum[w];
  }
  for (int i = i0; i < i1; ++i) {
    const int v = h[i];
    h[i] = at;
    at += v;
  }
  __syncthreads();
  const int most = (int)ia.nnz;
  for (int i = tid; i < ia.nb; i += kSetupThreads) ia.ptr[i] = min(h[i], most);
  if (tid == 0) {
    ia.ptr[ia.nb] = min(total, most);
    if (ia.flag) *ia.flag = bad;
  }
  __syncthreads();
  const auto place = [&](int l, int b, int) {
    if (b < 0 || l < 0 || l >= ia.L) return;
    const int slot = atomicAdd(&h[l >> 7], 1);
    if (slot < most) ia.pos[slot] = make_int2(l, b);
  };
  for_each_positive(ia, B, tid, nullptr, nullptr, place);
  for_each_left_positive(ia, tid, long_rows, n, place);
}

// Step set-up.  Workgroup 0 builds the label index (or nothing); the others stage the inputs (Algorithm 1:
// "X.t().to(float8_e4m3fn)"), one tile of 64 samples x 128 columns each: the E4M3 cast Xq [Bp, d] used by the
// logits product and the transposed BF16 copy XT [d, Bp] used by the weight-gradient product, turned in LDS so
// that both sides are read and written 8 and 16 bytes at a time (2-byte stores at a stride of Bp took 46 us for
// 4096 x 768).  Rows B..Bp-1 are zero padding.  Either output may be absent.  cnt: bin counters to clear for
// the separate index kernels.
constexpr int kXtPitch = 64 * 2 + 16;                             // bytes per staged column of 64 samples
// X is the caller's and may begin at any of its elements (one 16-byte load all the same: global loads need no alignment)
typedef u32x4 u32x4_at2 __attribute__((aligned(2)));
template <int NT>
__device__ __forceinline__ void stage_inputs(const uint16_t* __restrict__ X, int B, int Bp, int d, uint8_t* __restrict__ Xq, uint16_t* __restrict__ XT,
                                             int tile, char* smem) {
  const int tiles_c = d >> 7, b0 = tile / tiles_c * 64, c0 = tile % tiles_c * 128, tid = threadIdx.x;
#pragma unroll
  for (int t = tid; t < 1024; t += NT) {
    const int r = t >> 4, c = (t & 15) * 8;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (b0 + r < B) v = *reinterpret_cast<const u32x4_at2*>(X + (size_t)(b0 + r) * d + c0 + c);
    if (Xq) {
      uint32_t q[2] = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e >> 2] |= e4m3_rne(bf16_decode((v[e >> 1] >> (16 * (e & 1))) & 0xFFFFu)) << (8 * (e & 3));
      *reinterpret_cast<uint2*>(Xq + (size_t)(b0 + r) * d + c0 + c) = make_uint2(q[0], q[1]);
    }
    if (XT)
#pragma unroll
      for (int e = 0; e < 8; ++e) *reinterpret_cast<uint16_t*>(smem + (c + e) * kXtPitch + r * 2) = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
  }
  if (!XT) return;
  __syncthreads();
#pragma unroll
  for (int t = tid; t < 1024; t += NT) {
    const int cb = t >> 8, o = (t >> 5) & 7, c = t & 31;
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(XT) + (size_t)((c0 >> 5) + cb) * blk_strip(Bp) + blk_off((b0 >> 3) + o, c)) =
        *reinterpret_cast<const u32x4*>(smem + (cb * 32 + c) * kXtPitch + o * 16);
  }
}
// LDS of a launch that indexes nb bins and B rows, or that only stages (nb = 0)
inline size_t setup_smem(int nb, int B) {
  const size_t index = nb ? (size_t)(nb + B) * 4 : 0;
  return index > 128 * kXtPitch ? index : 128 * kXtPitch;
}
__global__ void __launch_bounds__(kSetupThreads) k_step_setup(const uint16_t* __restrict__ X, int B, int Bp, int d,
                                                              uint8_t* __restrict__ Xq, uint16_t* __restrict__ XT, IndexArgs ia,
                                                              int* __restrict__ cnt, size_t n_cnt) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x;
  if (cnt) {
    const size_t t0 = (size_t)blockIdx.x * kSetupThreads + tid;
    for (size_t i = t0; i < n_cnt; i += (size_t)gridDim.x * kSetupThreads) cnt[i] = 0;
    if (ia.flag && t0 == 0) *ia.flag = 0;
  }
  if (blockIdx.x == 0) {
    if (ia.nb) label_index(ia, B, reinterpret_cast<int*>(smem));
    return;
  }
  stage_inputs<kSetupThreads>(X, B, Bp, d, Xq, XT, blockIdx.x - 1, smem);
}

// ---------------------------------------------------------------------------------------------
// The three matrix products share one shape: 512-thread workgroups (8 waves) computing a 256 x 256 output tile (logits also 128 x 128),
// operands streamed by asynchronous global->LDS loads through a ring of LDS stages (tiles.h: ring_pipeline_pp for
// the logits, ring_alternate for the other two).  One workgroup per CU.  On this part the matrix cores and the L2->LDS
// fill do not overlap for free: a tile of this size halves the fill traffic per flop of a 256 x 128 tile.
// ---------------------------------------------------------------------------------------------
constexpr int kGemmThreads = 512;
constexpr int kGemmWaves = 8;
constexpr int kWideRingBytes = 2 * (256 + 256) * 128;            // K-contiguous operands, 128-byte slabs, 2 stages

// Register fragments of one step of a product: FM x FN blocks of 32 x 32 outputs.
template <int FM, int FN> struct FragBF16 { bf16x8 a[FM], b[FN]; };

template <int FN> __device__ inline void zero_acc(f32x16 (&acc)[2][FN]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
}

// Classifier dropout on a weight slab that has landed in LDS (appendix "Low-Memory Dropout for
// Classifier": mask after the load, before the product).  The slab is ROWS weight rows of ROWB
// bytes of consecutive columns in the tile_off<ROWB> layout; blk0 is the mask block of its first
// 16 elements and blk_stride the mask blocks per weight row (d / 16).  Every thread draws whole
// mask blocks and zeroes the dropped elements in place.
template <int ROWS, int ROWB, bool FP8>
__device__ __forceinline__ void drop_slab(char* tile, uint64_t blk0, uint32_t blk_stride, uint64_t seed, uint64_t step,
                                          uint32_t thresh, int tid) {
  constexpr int UPR = ROWB / (FP8 ? 16 : 32);                  // mask blocks per slab row
  static_assert((ROWS * UPR) % kGemmThreads == 0, "slab size");
  const uint32_t tb = thresh * 0x01010101u;
#pragma unroll
  for (int u0 = 0; u0 < ROWS * UPR; u0 += kGemmThreads) {
    const int u = u0 + tid, r = u / UPR, k = u % UPR;
    const U4 rb = drop_block(blk0 + (uint64_t)r * blk_stride + k, seed, step);
    if (FP8) {
      u32x4* p = reinterpret_cast<u32x4*>(tile + tile_off<ROWB>(r, k));
      u32x4 w = *p;
      w[0] &= keep_bytes(rb.x, tb);
      w[1] &= keep_bytes(rb.y, tb);
      w[2] &= keep_bytes(rb.z, tb);
      w[3] &= keep_bytes(rb.w, tb);
      *p = w;
    } else {
      // byte mask -> one 16-bit mask per element (v_perm_b32 doubles each byte)
      u32x4* p0 = reinterpret_cast<u32x4*>(tile + tile_off<ROWB>(r, 2 * k));
      u32x4* p1 = reinterpret_cast<u32x4*>(tile + tile_off<ROWB>(r, 2 * k + 1));
      u32x4 a = *p0, b = *p1;
      uint32_t m = keep_bytes(rb.x, tb);
      a[0] &= __builtin_amdgcn_perm(m, m, 0x01010000u);
      a[1] &= __builtin_amdgcn_perm(m, m, 0x03030202u);
      m = keep_bytes(rb.y, tb);
      a[2] &= __builtin_amdgcn_perm(m, m, 0x01010000u);
      a[3] &= __builtin_amdgcn_perm(m, m, 0x03030202u);
      m = keep_bytes(rb.z, tb);
      b[0] &= __builtin_amdgcn_perm(m, m, 0x01010000u);
      b[1] &= __builtin_amdgcn_perm(m, m, 0x03030202u);
      m = keep_bytes(rb.w, tb);
      b[2] &= __builtin_amdgcn_perm(m, m, 0x01010000u);
      b[3] &= __builtin_amdgcn_perm(m, m, 0x03030202u);
      *p0 = a;
      *p1 = b;
    }
  }
}

// The same for the four rows of a 32-row slab of 256 columns that a wave has loaded itself (dma_tile<32, ROWB, 8>): a lane draws one mask
// block, of row 4 wave + lane / 16, columns 16 (lane % 16) .. +15.
template <int ROWB, bool FP8>
__device__ __forceinline__ void drop_own_rows(char* tile, int wave, int lane, uint64_t blk0, uint32_t blk_stride, uint64_t seed, uint64_t step,
                                              uint32_t thresh) {
  static_assert(ROWB == (FP8 ? 256 : 512), "256 columns");
  const int r = 4 * wave + (lane >> 4), k = lane & 15;
  const U4 rb = drop_block(blk0 + (uint64_t)r * blk_stride + k, seed, step);
  const uint32_t tb = thresh * 0x01010101u;
  const uint32_t m[4] = {keep_bytes(rb.x, tb), keep_bytes(rb.y, tb), keep_bytes(rb.z, tb), keep_bytes(rb.w, tb)};
  if (FP8) {
    u32x4* p = reinterpret_cast<u32x4*>(tile + tile_off<ROWB>(r, k));
    *p = *p & u32x4{m[0], m[1], m[2], m[3]};
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h) {                                // byte mask -> one 16-bit mask per element
      u32x4* p = reinterpret_cast<u32x4*>(tile + tile_off<ROWB>(r, 2 * k + h));
      *p = *p & u32x4{__builtin_amdgcn_perm(m[2 * h], m[2 * h], 0x01010000u), __builtin_amdgcn_perm(m[2 * h], m[2 * h], 0x03030202u),
                      __builtin_amdgcn_perm(m[2 * h + 1], m[2 * h + 1], 0x01010000u), __builtin_amdgcn_perm(m[2 * h + 1], m[2 * h + 1], 0x03030202u)};
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Logits + fused epilogue (Algorithm 1: matmul_fp8, sigmoid_, "-= 1" at the positives).
// One workgroup computes a 256 (samples) x 256 (labels) tile of Z = Xq W_c^T with FP32
// accumulation over the full embedding width, then G = sigmoid(Z) - Y, and stores G^T as
// BF16 in blocks of 32 labels (tiles.h, blk_off), the order in which the other two products take it.  Z never reaches memory.
// FP8: both operands E4M3, v_mfma_f32_32x32x64_f8f6f4.  BF16: v_mfma_f32_32x32x16_bf16.
// The positives of the tile's two 128-label bins are turned into a bit mask in LDS behind the loads of the first
// slab; after the K loop every wave finishes its accumulators in registers (sigmoid, minus the mask
// bit, BF16) and stores them a KiB at a time, without LDS and without a workgroup barrier.
// Rows of G^T between n and the next multiple of 128 are written as zeros (the input-gradient
// product reads whole 32-label blocks).
// ---------------------------------------------------------------------------------------------
// TB x TB output tiles: TB = 256, or 128 for padded batches of at most 128 rows, where half of a
// 256-row tile would be padding and the kernel is bound by the stream of W: 128 x 128 tiles need
// 66 KiB of LDS, so two workgroups share a CU and one's epilogue overlaps the other's loads.
template <int TB> constexpr int logits_mask_offset() { return 2 * (TB + TB) * 128; }   // positives mask: behind the ring
template <int TB> constexpr int logits_rows_offset() { return logits_mask_offset<TB>() + TB * (TB / 32) * 4 + 32; }
template <int TB> constexpr int logits_smem() { return logits_rows_offset<TB>() + (TB == 128 ? 132 * 4 : 0); }   // row pointers of a direct step

// One half (0 or 1) of the product of a 128-byte K slab of the logits tile: A = TB sample rows,
// B = TB label rows, K-contiguous in LDS.  Wave (wm, wn) owns samples 64 wm .. +63 and labels
// 32 FN wn .. +32 FN - 1; acc[i][j] is its 32 x 32 block (i, j).
template <bool FP8, int FN>
__device__ __forceinline__ void logits_slab_product(const char* sa, const char* sb, int half, int wm, int wn, int lane,
                                                    f32x16 (&acc)[2][FN]) {
  if (FP8) {
    i32x8 a[2], b[FN];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = frag_fp8(sa, wm * 64 + 32 * i, half, lane);
#pragma unroll
    for (int j = 0; j < FN; ++j) b[j] = frag_fp8(sb, wn * 32 * FN + 32 * j, half, lane);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[i], b[j], acc[i][j], 0, 0, 0, 0, 0, 0);
  } else {
#pragma unroll
    for (int kk = 2 * half; kk < 2 * half + 2; ++kk) {
      bf16x8 a[2], b[FN];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = frag_bf16(sa, wm * 64 + 32 * i, kk, lane);
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = frag_bf16(sb, wn * 32 * FN + 32 * j, kk, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
}

// Z tile = Xa[TB rows] . Wc[TB rows]^T over the full embedding width (rowb bytes per row), FP32
// accumulators.  Waves as (8 / WGN) x WGN with WGN = 2 (TB = 256, 64 x 128 per wave) or 4
// (TB = 128, 64 x 32 per wave).
template <bool FP8, int TB, int FN, class Prep = NoPrep, class Extra = NoPrep>
__device__ __forceinline__ void logits_tile_product(const char* __restrict__ Xa, int a_valid, const char* __restrict__ Wc, int w_valid,
                                                    size_t rowb, char* smem, int wave, int lane, f32x16 (&acc)[2][FN],
                                                    Prep&& prep = Prep{}, Extra&& extra = Extra{}) {
  constexpr int WGN = TB / 32 / FN;
  static_assert(WGN == (TB == 256 ? 2 : 4), "wave layout");
  const int wm = wave / WGN, wn = wave % WGN;
  zero_acc(acc);
  ring_pipeline_pp<TB, 128, TB, 128, 2, kGemmWaves, true>(
      Xa, rowb, a_valid, 0, 128, 8, Wc, rowb, w_valid, 0, 128, 8, (int)(rowb >> 7), smem, wave, lane,
      [&](const char* sa, const char* sb, int h) { logits_slab_product<FP8, FN>(sa, sb, h, wm, wn, lane, acc); },
      static_cast<Prep&&>(prep), static_cast<Extra&&>(extra));
}

// A small BF16 step needs neither an E4M3 cast of X nor, with this few positives, an index of them: every workgroup finds
// its tile's in the CSR lists themselves, and the transposed copy of X, which only the
// next kernel reads, is made by workgroups of the same launch behind the `tiles` that have logits to compute.  That takes the set-up launch out of the
// chain of a step that is all launches (8192 labels, d = 256, B = 64: 25.6 -> 21.0 us).
struct DirectArgs { const int* indptr; const int* indices; int nnz; int tiles; uint16_t* XT; };
// Positives that every tile looks at: four per thread, however they are spread over the rows.
constexpr int kDirectMaxNnz = 4 * kGemmThreads;
constexpr int kDirectWalk = 16;
// mark(row, label - lo) for the positives of a direct step among the `count` labels from lo on, by all threads of a workgroup (B <= 128; `ptr`: 129
// ints of LDS).  The first kDirectWalk of a row are read by four threads, four loads each in flight together, which is all there is where rows
// are short.  Where one is longer the whole list is read by place, four loads a thread, and a place that
// holds one of the tile's labels looks for its row.  (Long rows walked to their end by their four threads: 1 M labels, d = 256, B = 64,
// one row of 1800: 1421 us a step, now 540, 559 with an
// index; every list read by place only: 8192 labels, d = 256, B = 64 18.3 -> 18.6 us.)  Malformed rows are
// skipped; beside one the others may overlap, and are walked by their own threads.  Contains a barrier, which also orders what
// the caller wrote to LDS before it.
template <class F> __device__ __forceinline__ void mark_direct_positives(const DirectArgs& da, int B, int tid, int lo, int count, int* ptr, F&& mark) {
  constexpr int WALK = kDirectWalk / 4, PER = kDirectMaxNnz / kGemmThreads;
  const int r = tid >> 2, sub = tid & 3, lane = tid & 63;
  const int begin = r < B ? da.indptr[r] : INT32_MAX, end = r < B ? da.indptr[r + 1] : INT32_MAX;
  if (sub == 0) ptr[r + 1] = end;
  if (tid == 0) ptr[0] = begin;
  const bool sound = r < B && begin >= 0 && begin <= end && end <= da.nnz;    // (also keeps begin + 15 from wrapping to a place before the list)
  const auto mark_label = [&](int row, int label) {
    const uint32_t at = (uint32_t)label - (uint32_t)lo;
    if (label >= 0 && at < (uint32_t)count) mark(row, (int)at);
  };
  int l[WALK > PER ? WALK : PER];
#pragma unroll
  for (int i = 0; i < WALK; ++i) l[i] = sound && sub + 4 * i < end - begin ? da.indices[begin + sub + 4 * i] : -1;
  barrier_lds();
  const int p0 = ptr[2 * lane], p1 = ptr[2 * lane + 1], p2 = ptr[2 * lane + 2];
#pragma unroll
  for (int i = 0; i < WALK; ++i) mark_label(r, l[i]);
  if (__builtin_amdgcn_ballot_w64((2 * lane < B && p1 - p0 > kDirectWalk) || (2 * lane + 1 < B && p2 - p1 > kDirectWalk)) == 0ull) return;
  if (__builtin_amdgcn_ballot_w64(p0 > p1 || p1 > p2) != 0ull || ptr[0] < 0 || ptr[B] > da.nnz) {
    if (sound)
      for (int p = begin + kDirectWalk + sub; p < end; p += 4) mark_label(r, da.indices[p]);
    return;
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) l[i] = tid + i * kGemmThreads < da.nnz ? da.indices[tid + i * kGemmThreads] : -1;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int p = tid + i * kGemmThreads;
    if ((uint32_t)l[i] - (uint32_t)lo >= (uint32_t)count) continue;
    int row = 0;                                                         // the last row that begins at or before p
#pragma unroll
    for (int o = 64; o > 0; o >>= 1) row += ptr[row + o] <= p ? o : 0;
    if (row < B && ptr[row] <= p && p < ptr[row + 1]) mark_label(row, l[i]);   // (places before the first row or behind the last belong to none)
  }
}
// DROP: the W slabs are masked in LDS as they land (drop_slab) and Z is scaled by 1 / (1 - p);
// elem0 = flat index of the chunk's first weight element.
template <bool FP8, bool LOSS, int TB, bool DROP>
__global__ void __launch_bounds__(kGemmThreads, TB == 256 ? 1 : 2)
k_logits(const char* __restrict__ Xa, int a_rows, const char* __restrict__ Wc, int n, int d, int Bp, int B,
         uint16_t* __restrict__ Gt, const int* __restrict__ binptr, const int2* __restrict__ pos, int tile0,
         float* __restrict__ loss_slots, uint64_t seed, uint64_t step, uint64_t elem0, DropArgs dr, DirectArgs da) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int WGN = TB == 256 ? 2 : 4, FN = TB / 32 / WGN;   // waves along the labels, 32-label blocks per wave
  constexpr bool MAY_DIRECT = !FP8 && TB == 128;
  if (MAY_DIRECT && da.tiles && (int)blockIdx.x >= da.tiles) {           // X^T for the kernels after this one
    stage_inputs<kGemmThreads>(reinterpret_cast<const uint16_t*>(Xa), B, Bp, d, nullptr, da.XT, blockIdx.x - da.tiles, smem);
    return;
  }
  constexpr int MW = TB / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
  const int tiles_b = (Bp + TB - 1) / TB;
  const int wg = xcd_logical_id(blockIdx.x, MAY_DIRECT && da.tiles ? da.tiles : gridDim.x);
  const int lt = wg / tiles_b, bt = wg % tiles_b;
  const int b0 = bt * TB, l0 = lt * TB;
  const size_t rowb = (size_t)d * (FP8 ? 1 : 2);

  uint32_t* ym = reinterpret_cast<uint32_t*>(smem + logits_mask_offset<TB>());   // [TB labels][MW] bits over the samples
  float* red = reinterpret_cast<float*>(smem + logits_mask_offset<TB>() + TB * MW * 4);
  const int rows_out = min(TB, ((n - l0 + 127) >> 7) << 7);              // rows of G^T this tile writes
  const int gt0 = tile0 + lt * (TB / 128);                               // first of the tile's one or two bins

  // ---- positives of this tile's bins that fall into this batch tile -> bit mask.  The mask lives
  // behind the ring and is built behind the loads of the first slab, which its own two round trips overlap; the K
  // loop's first barrier publishes it.
  auto build_mask = [&]() {
    for (int i = tid; i < TB * MW; i += kGemmThreads) ym[i] = 0u;
    if (MAY_DIRECT && da.indptr) {                                       // (the batch is one tile)
      mark_direct_positives(da, B, tid, gt0 << 7, min(TB, n - l0), reinterpret_cast<int*>(smem + logits_rows_offset<TB>()),
                            [&](int r, int at) { atomicOr(&ym[at * MW + (r >> 5)], 1u << (r & 31)); });
      __builtin_amdgcn_s_waitcnt(0xC07F);
      return;
    }
    const int p0 = binptr[gt0], p1 = binptr[gt0 + (rows_out >> 7)];
    barrier_lds();
    for (int p = p0 + tid; p < p1; p += kGemmThreads) {
      const int2 e = pos[p];
      const int lr_ = e.x - (gt0 << 7), br = e.y - b0;
      if (br >= 0 && br < TB && lr_ >= 0 && lr_ < TB) atomicOr(&ym[lr_ * MW + (br >> 5)], 1u << (br & 31));
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                                  // in LDS ahead of that barrier
  };

  f32x16 acc[2][FN];
  const char* xa = Xa + (size_t)b0 * rowb;
  const char* wc = Wc + (size_t)l0 * rowb;
  if constexpr (DROP) {
    const uint64_t blk_tile = (elem0 + (uint64_t)l0 * d) >> 4;     // mask block of the tile's first element
    logits_tile_product<FP8, TB, FN>(
        xa, a_rows - b0, wc, n - l0, rowb, smem, wave, lane, acc,
        [&](char* sb, int ks) {
          drop_slab<TB, 128, FP8>(sb, blk_tile + (uint64_t)ks * (FP8 ? 8 : 4), (uint32_t)d >> 4, seed, step, dr.thresh, tid);
        },
        build_mask);
  } else {
    logits_tile_product<FP8, TB, FN>(xa, a_rows - b0, wc, n - l0, rowb, smem, wave, lane, acc, NoPrep{}, build_mask);
  }

  // ---- G = sigmoid(Z) - Y in registers, BF16, stored as two octets of a label block (1 KiB) per instruction.
  // Each wave finishes its own 64-sample x (32 FN)-label block on its own: one wave's stores overlap another's
  // arithmetic, and this phase is bound by the vector ALU (two transcendental instructions per value).
  // Turned through LDS into 128-byte segments of label rows the launch took 147 us per 131072 E4M3 labels (d = 768,
  // 1024 samples), now 133.
  // Positives are a handful per sample among millions of labels: a 32 x 32 block whose mask words
  // are all zero, in a tile without ragged rows, takes the short form (sigmoid only); the wave
  // votes, so the choice is uniform.
  constexpr int WROWS = 32 * FN;
  float loss = 0.0f;
  const bool tile_full = n - l0 >= TB, in_batch = b0 + wm * 64 < Bp;
  const size_t strip = blk_strip(Bp);
  char* gt = reinterpret_cast<char*>(Gt) + (size_t)((l0 + wn * WROWS) >> 5) * strip + (size_t)((b0 >> 3) + wm * 8) * 512;
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int l = wn * WROWS + 32 * j + (lane & 31);
      const bool row_ok = l0 + l < n;
      const uint32_t ybits = (ym[l * MW + 2 * wm + i] >> (4 * (lane >> 5))) & 0x0F0F0F0Fu;
      const bool plain = !LOSS && tile_full && __builtin_amdgcn_ballot_w64(ybits != 0u) == 0ull;
#pragma unroll
      for (int qp = 0; qp < 2; ++qp) {                               // 16 samples: two octets
        uint32_t o[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int q = 2 * qp + h, b = wm * 64 + 32 * i + 8 * q + 4 * (lane >> 5);
          float g[4];
          if (plain) {
#pragma unroll
            for (int e = 0; e < 4; ++e) g[e] = sigmoidf_fast(DROP ? acc[i][j][4 * q + e] * dr.scale : acc[i][j][4 * q + e]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float z = DROP ? acc[i][j][4 * q + e] * dr.scale : acc[i][j][4 * q + e];
              const float y = (float)((ybits >> (8 * q + e)) & 1u);
              g[e] = row_ok ? sigmoidf_fast(z) - y : 0.0f;
              if (LOSS) loss += (row_ok && b0 + b + e < B) ? softplusf_fast(z) - y * z : 0.0f;
            }
          }
          o[h][0] = pack2_bf16(g[0], g[1]);
          o[h][1] = pack2_bf16(g[2], g[3]);
        }
        // a lane holds half of each octet, the lane 32 further the other half: after the exchange the lower lanes hold the first
        // octet and the upper ones the second
        const auto s0 = __builtin_amdgcn_permlane32_swap(o[0][0], o[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(o[0][1], o[1][1], false, false);
        // streaming store: the gradients are written once here and read by other kernels later (measured 157 -> 150 us
        // per chunk against a plain store; the same hint on the weight stores of the update kernels and on
        // the asynchronous loads changed nothing or made them slower)
        if (in_batch && wn * WROWS + 32 * j < rows_out)
          __builtin_nontemporal_store(u32x4{s0[0], s1[0], s0[1], s1[1]},
                                      reinterpret_cast<u32x4*>(gt + j * strip + blk_off(4 * i + 2 * qp + (lane >> 5), lane & 31)));
      }
    }
  if (LOSS) {
    const float s = block_sum<kGemmWaves>(loss, red);
    if (tid == 0) {
      loss_slots[(size_t)gt0 * tiles_b + bt] = s;                        // both bins' loss in the first bin's slot
      if (rows_out > 128) loss_slots[(size_t)(gt0 + 1) * tiles_b + bt] = 0.0f;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Input gradient (Algorithm 1: X_gradient += large_k_matmul(logits, W_i)), dX += G W_c with the
// weights as they are before this step's update.  The contraction runs over the labels; both
// operands are stored label-major, so fragments come from transposing LDS reads and E4M3
// weights are widened to BF16 in registers (no up-cast copy of W in memory).
// Workgroup = 256 samples x 256 embedding columns x one slice s of the chunk's labels; the FP32
// partial goes to dXacc[s] (owned by exactly this workgroup, so plain read-modify-write).
// Label rows beyond n inside the last 32-label slab are harmless: G^T holds zeros there and the
// weight rows are re-reads of row n-1.  Columns beyond d in the last column tile re-read the
// row's last 16 bytes and are not stored.
// ---------------------------------------------------------------------------------------------
// The FP32 partials live in the layout of the accumulators, not as matrix rows: a plane of R x d values
// is a row-major array of 32 x 32 blocks, a block is four groups of 64 lanes x 16 bytes (group q, lane:
// elements 4q .. 4q+3 of the lane's accumulator), so a wave moves 1 KiB per instruction.  What bounds this
// read-modify-write is the number of memory instructions and their round trips (as rows of 4-byte accesses
// it took 30 k of the input-gradient kernel's 364 k clocks); k_finalize turns the layout back.
__device__ inline f32x4* dx_block(float* plane, int d, int row0, int col0) {
  return reinterpret_cast<f32x4*>(plane + ((size_t)(row0 >> 5) * (d >> 5) + (col0 >> 5)) * 1024);
}
// NB blocks of a wave at src + b * 256.
template <int NB> __device__ __forceinline__ void load_acc_blocks(const f32x4* __restrict__ src, int lane, f32x16 (&acc)[NB]) {
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = src[b * 256 + q * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[b][4 * q + e] = v[e];
    }
}
// NB blocks of a wave, at dst + b * 256: += acc[b], or = acc[b] in the step's first pass over the plane
// (which is why the planes need no clearing).  The loads of one block are in flight while the block
// before it is added and stored.
template <int NB> __device__ __forceinline__ void add_acc_blocks(f32x4* __restrict__ dst, int lane, const f32x16 (&acc)[NB], bool first) {
  auto quad = [&](int b, int q) { return f32x4{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]}; };
  if (first) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[b * 256 + q * 64 + lane] = quad(b, q);
    return;
  }
  f32x4 old[2][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) old[0][q] = dst[q * 64 + lane];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b + 1 < NB)
#pragma unroll
      for (int q = 0; q < 4; ++q) old[(b + 1) & 1][q] = dst[(b + 1) * 256 + q * 64 + lane];
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[b * 256 + q * 64 + lane] = old[b & 1][q] + quad(b, q);
  }
}

// Ring stage: [32 labels x 256 samples of the gradients (one block's octets, as in memory) | W slab 32 labels x 256 columns].
constexpr int kDxStages = 4;
template <bool FP8> constexpr int dx_stage_bytes() { return 32 * 512 + 32 * (FP8 ? 256 : 512); }
template <bool FP8> constexpr int dx_smem_bytes() { return kDxStages * dx_stage_bytes<FP8>(); }

// Fragments of one step of 16 labels: four blocks of 32 samples, two of 32 columns (E4M3: as stored).
template <bool FP8> struct FragDx { bf16x8 a[4]; typename std::conditional<FP8, i32x2, bf16x8>::type b[2]; };

// The waves stand 2 x 4, 128 samples x 64 columns each: a weight fragment then feeds four MFMAs and is widened in two waves (64 x 128
// each: two MFMAs, four waves), and it is widened between the MFMAs, where the vector ALU is free, not before them.
// Alone, 131072 E4M3 labels x 768, 1024 samples: 156 us, 164 us as 64 x 128, 167 us widened ahead of the product.
template <bool FP8, bool DROP>
__global__ void __launch_bounds__(kGemmThreads, 1)
k_dx(const char* __restrict__ Gt, const char* __restrict__ Wc, float* __restrict__ dXacc, int n, int d, int Bp,
     int Bp256, int S, bool first, uint64_t seed, uint64_t step, uint64_t elem0, DropArgs dr) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int ESZ = FP8 ? 1 : 2, WROWB = 256 * ESZ, GBYTES = 32 * 512;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 2, wn = wave & 3;
  const int tiles_b = Bp256 >> 8, tiles_j = (d + 255) >> 8;
  const int wg = xcd_logical_id(blockIdx.x, gridDim.x);
  const int jt = wg % tiles_j, bt = (wg / tiles_j) % tiles_b, s = wg / (tiles_j * tiles_b);
  const int b0 = bt << 8, j0 = jt << 8;
  const int ksteps = (n + 31) >> 5, per = (ksteps + S - 1) / S;
  const int ks0 = s * per, ks1 = min(ks0 + per, ksteps);
  if (ks0 >= ks1 && !first) return;
  const size_t strip = blk_strip(Bp), strideB = (size_t)d * ESZ;

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  float* out = dXacc + (size_t)s * Bp256 * d;
  auto store = [&]() {
    const int col = j0 + wn * 64;
    if (col < d)
#pragma unroll
      for (int i = 0; i < 4; ++i) add_acc_blocks<2>(dx_block(out, d, b0 + wm * 128 + 32 * i, col), lane, acc[i], first);
  };
  if (ks0 >= ks1) { store(); return; }                 // a slice without labels in the first chunk still owns its plane
  const char* ga = Gt + (size_t)ks0 * strip;
  const char* gb = Wc + (size_t)ks0 * 32 * strideB + (size_t)j0 * ESZ;
  const int kibs = Bp >> 4, kib0 = (b0 >> 4) + 2 * wave;   // KiB of a strip; this wave's two of every slab (beyond the batch: the last one again)
  const int chunks_b = min(256, d - j0) * ESZ / 16;
  auto issue = [&](int ks, int to) {
    const char* g = ga + (size_t)ks * strip;
    char* st = smem + to;
    dma_kib_of(g, kib0, kibs, st + 2 * wave * 1024, lane);
    dma_kib_of(g, kib0 + 1, kibs, st + (2 * wave + 1) * 1024, lane);
    dma_tile<32, WROWB, kGemmWaves>(gb + (size_t)ks * 32 * strideB, strideB, n - (ks0 + ks) * 32, st + GBYTES, wave, lane, chunks_b);
  };
  auto ld = [&](FragDx<FP8>& f, const char* st, int kk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f.a[i] = frag_tr_blk(st, 16 * kk, wm * 128 + 32 * i, lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (FP8) f.b[j] = frag_tr_raw8<WROWB>(st + GBYTES, 16 * kk, wn * 64 + 32 * j, lane);
      else f.b[j] = frag_tr_bf16<WROWB>(st + GBYTES, 16 * kk, wn * 64 + 32 * j, lane);
    }
  };
  auto mm = [&](const FragDx<FP8>& f) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 b;
      if constexpr (FP8) b = widen8(f.b[j]);
      else b = f.b[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], b, acc[i][j], 0, 0, 0);
    }
  };
  constexpr int LPS = 2 + dma_loads_per_wave<32, WROWB, kGemmWaves>();
  if constexpr (DROP) {
    // the same masked weights as in the logits product (appendix "Low-Memory Dropout for Classifier")
    const uint64_t blk_first = (elem0 + (uint64_t)ks0 * 32 * d + j0) >> 4;
    ring_alternate<kDxStages, dx_stage_bytes<FP8>(), LPS, FragDx<FP8>>(ks1 - ks0, smem, wave >= 4, issue, ld, mm, [&](char* st, int ks) {
      drop_own_rows<WROWB, FP8>(st + GBYTES, wave, lane, blk_first + (uint64_t)ks * 2 * d, (uint32_t)d >> 4, seed, step, dr.thresh);
    });
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] *= dr.scale;
  } else {
    ring_alternate<kDxStages, dx_stage_bytes<FP8>(), LPS, FragDx<FP8>>(ks1 - ks0, smem, wave >= 4, issue, ld, mm);
  }
  store();
}

// dX_out = BF16(sum over the S planes of FP32 partials); loss_out = sum of the tile losses.
// A workgroup turns one group of 64 lanes x 16 bytes (8 x 32 outputs) of the partials' layout into rows;
// its eight waves share the planes, so that the chain of dependent loads is S / 8 long: with one thread per
// output walking all S planes this kernel took 38 us at 64 outputs rows x 256 columns and 256 planes.
// The last workgroup of the grid sums the losses.
constexpr int kFinalWaves = 8;
__global__ void __launch_bounds__(64 * kFinalWaves) k_finalize(const float* __restrict__ dXacc, int S, int plane_rows, int B, int d, int groups,
                                                               float scale, uint16_t* __restrict__ dX_out, const float* __restrict__ loss_slots,
                                                               int nslots, float* __restrict__ loss_out) {
  __shared__ f32x4 part[kFinalWaves][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x == groups) {
    float s = 0.0f;
    for (int i = tid; i < nslots; i += 64 * kFinalWaves) s += loss_slots[i];
    const float t = block_sum<kFinalWaves>(s, reinterpret_cast<float*>(part));
    if (tid == 0) *loss_out = t;
    return;
  }
  const int u = blockIdx.x, blk = u >> 2, q = u & 3;
  const size_t plane = (size_t)plane_rows * d / 4;
  const f32x4* src = reinterpret_cast<const f32x4*>(dXacc) + (size_t)u * 64 + lane;
  f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int k = wave; k < S; k += kFinalWaves) s += src[k * plane];
  part[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 1; w < kFinalWaves; ++w) s += part[w][lane];
  const int row = (blk / (d >> 5)) * 32 + 8 * q + 4 * (lane >> 5), col = (blk % (d >> 5)) * 32 + (lane & 31);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (row + e < B) dX_out[(size_t)(row + e) * d + col] = (uint16_t)bf16_rne(s[e] * scale);
}

// ---------------------------------------------------------------------------------------------
// Fused weight gradient + SGD + (Kahan) + rounding, in place (Algorithm 1, fuse_update).
// One workgroup owns a 256 (labels) x 256 (columns) tile of W_c: grad = G^T X accumulated in FP32
// over the whole batch on the BF16 matrix cores, then per element the FP32 update of
// numerics.h, rounded stochastically (Eq. 1) or to nearest, written back in the storage format.
// The weight gradient only ever exists as MFMA accumulators and one LDS tile (staged in two
// halves of 128 columns).
// ---------------------------------------------------------------------------------------------
constexpr int kGPitch = 132;                                     // floats per staged gradient row of 128 columns
constexpr int kUpdateEpiBytes = kGemmWaves * 32 * kGPitch * 4;   // one 32 x 128 FP32 half-block per wave
constexpr int kUpdateStages = 4, kUpdateStageBytes = (256 + 256) * 64;    // [8 blocks of gradients | 8 blocks of inputs] x 32 samples
constexpr int kUpdateSmem = kUpdateEpiBytes > kUpdateStages * kUpdateStageBytes ? kUpdateEpiBytes : kUpdateStages * kUpdateStageBytes;

// N (8 or 16) consecutive elements of one weight row: storage bits in, storage bits out.
// E4M3: w[0 .. N/4-1] hold 4 codes each; BF16: w[0 .. N/2-1] hold 2 patterns each.  c[0 .. N/2-1]: BF16 compensation.
// WD = false ignores wd (the two extra operations of the decay are not even selected away).
template <int FMT, bool SR, bool KAHAN, bool WD, int N>
__device__ inline void update_wd(uint32_t (&w)[8], uint32_t (&c)[8], const float (&g)[N], float lr, float wd_, const U4 (&rb)[N / 8]) {
  const float wd = WD ? wd_ : 0.0f;
  uint32_t rw[N / 2];
#pragma unroll
  for (int i = 0; i < N / 8; ++i) {
    rw[4 * i] = rb[i].x; rw[4 * i + 1] = rb[i].y; rw[4 * i + 2] = rb[i].z; rw[4 * i + 3] = rb[i].w;
  }
  if (FMT == FMT_E4M3) {
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
      // four codes at a time: the packed conversion decodes two E4M3 bytes per instruction (exact)
      const f32x2 wlo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[q], 1.0f, false);
      const f32x2 whi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[q], 1.0f, true);
      const float wv[4] = {wlo[0], wlo[1], whi[0], whi[1]};
      uint32_t out = 0u;
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 4 * q + e;
        const float gi = wd != 0.0f ? __fadd_rn(g[i], __fmul_rn(wd, wv[e])) : g[i];   // L2 weight decay as a gradient term
        const float u = __fmul_rn(lr, gi);
        float t;
        y[e] = 0.0f;
        if (KAHAN) {
          const float cv = u2f((i & 1) ? (c[i >> 1] & 0xFFFF0000u) : (c[i >> 1] << 16));
          y[e] = __fsub_rn(-u, cv);
          t = __fadd_rn(wv[e], y[e]);
        } else {
          t = __fsub_rn(wv[e], u);
        }
        if (SR) {
          const uint32_t rnd = (i & 1) ? (rw[i >> 1] & 0xFFFF0000u) : (rw[i >> 1] << 16);
          out = e4m3_sr_pack(t, rnd, out, e);
        } else {
          out |= e4m3_rne(t) << (8 * e);
        }
      }
      w[q] = out;
      if (KAHAN) {
        const f32x2 nlo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(out, 1.0f, false);
        const f32x2 nhi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(out, 1.0f, true);
        c[2 * q] = pack2_bf16(__fsub_rn(__fsub_rn(nlo[0], wv[0]), y[0]), __fsub_rn(__fsub_rn(nlo[1], wv[1]), y[1]));   // hardware round-to-nearest-even
        c[2 * q + 1] = pack2_bf16(__fsub_rn(__fsub_rn(nhi[0], wv[2]), y[2]), __fsub_rn(__fsub_rn(nhi[1], wv[3]), y[3]));
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      uint32_t wb = (w[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu;
      uint32_t cb = KAHAN ? (c[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu : 0u;
      const uint32_t r16 = SR ? ((rw[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu) : 0u;
      update_element<FMT, SR, KAHAN>(wb, cb, g[i], lr, wd, r16);
      w[i >> 1] = (i & 1) ? (w[i >> 1] & 0x0000FFFFu) | (wb << 16) : (w[i >> 1] & 0xFFFF0000u) | wb;
      if (KAHAN) c[i >> 1] = (i & 1) ? (c[i >> 1] & 0x0000FFFFu) | (cb << 16) : (c[i >> 1] & 0xFFFF0000u) | cb;
    }
  }
}

// DROP: the weight gradient is that of the masked model: zero where the step's mask drops the
// element, scaled by 1 / (1 - p) elsewhere.
// WD: the update includes the weight-decay term (a template parameter because this phase is bound
// by the vector ALU: the common wd = 0 case should not compute the term and select it away).
template <int FMT, bool SR, bool KAHAN, bool DROP, bool WD>
__global__ void __launch_bounds__(kGemmThreads, 1)
k_update(const char* __restrict__ Gt, const char* __restrict__ XT, char* __restrict__ Wc, uint16_t* __restrict__ Cc,
         int n, int d, int Bp, float lr, float wd, uint64_t seed, uint64_t step, uint64_t elem0, DropArgs dr) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int ESZ = FMT == FMT_E4M3 ? 1 : 2;
  constexpr int WQ = FMT == FMT_E4M3 ? 1 : 2;       // 16-byte loads per 16 weights
  // (the epilogue's wave index is a vector value, the K loop's a scalar one; scalar in both measures the same within 1 %)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  const int tiles_j = (d + 255) >> 8;
  const int wg = xcd_logical_id(blockIdx.x, gridDim.x);
  const int lt = wg / tiles_j, jt = wg % tiles_j;
  const int l0 = lt << 8, j0 = jt << 8;
  // Every wave finishes its own 64 (labels) x 128 (columns) block of the tile on its own, in two
  // halves of 32 labels: per half the lane handles 4 passes x 16 consecutive columns of one row
  // (row = 8 pass + lane / 8; eight lanes cover the 128 columns of a row, i.e. whole 128-byte
  // lines of E4M3 weights -- halves of 64 columns measured 3.5 % slower for E4M3 with
  // compensation and 7 % faster for BF16).  The first half's weights (and compensation) are fetched behind the loads of
  // the first slabs (two passes) and right after the product (two), the second half's pass by pass while the first is being updated, so the
  // read-modify-write does not wait on memory.  A wave whose columns lie beyond d (the last
  // column tile of a d = 128 (mod 256) head) has nothing to update.
  const int wl0 = l0 + wm * 64, wj0 = j0 + wn * 128;
  const bool has_cols = wj0 < d;
  const int urow = lane >> 3, useg = lane & 7;
  u32x4 wreg[4][WQ];
  u32x4 creg[4][2];
  auto fetch = [&](int it, int half) {
    const int l = min(wl0 + 32 * half + it * 8 + urow, n - 1);
    const size_t eoff = (size_t)l * d + wj0 + useg * 16;
#pragma unroll
    for (int q = 0; q < WQ; ++q) wreg[it][q] = *reinterpret_cast<const u32x4*>(Wc + eoff * ESZ + 16 * q);
    if (KAHAN) {
      creg[it][0] = *reinterpret_cast<const u32x4*>(Cc + eoff);
      creg[it][1] = *reinterpret_cast<const u32x4*>(Cc + eoff + 8);
    }
  };

  f32x16 acc[2][4];
  zero_acc(acc);
  // K loop over the batch in slabs of 32 samples; a wave loads one 32-row block of each operand (beyond the last: that one again)
  const int uw = __builtin_amdgcn_readfirstlane(wave);
  const size_t strip = blk_strip(Bp);
  const char* ga = Gt + (size_t)((l0 >> 5) + min(uw, ((n - l0 + 31) >> 5) - 1)) * strip;
  const char* gb = XT + (size_t)((j0 >> 5) + min(uw, ((d - j0) >> 5) - 1)) * strip;
  ring_alternate<kUpdateStages, kUpdateStageBytes, 4, FragBF16<2, 4>>(
      Bp >> 5, smem, uw >= 4,
      [&](int ks, int to) {
        char* st = smem + to + uw * 2048;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          dma_kib(ga + (size_t)ks * 2048 + 1024 * i, st + 1024 * i, lane);
          dma_kib(gb + (size_t)ks * 2048 + 1024 * i, st + 16384 + 1024 * i, lane);
        }
      },
      [&](FragBF16<2, 4>& f, const char* st, int kk) {
#pragma unroll
        for (int i = 0; i < 2; ++i) f.a[i] = frag_blk(st + (wm * 2 + i) * 2048, kk, lane);
#pragma unroll
        for (int j = 0; j < 4; ++j) f.b[j] = frag_blk(st + 16384 + (wn * 4 + j) * 2048, kk, lane);
      },
      [&](const FragBF16<2, 4>& f) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
      },
      NoPrep{},
      [&]() {       // passes 0 and 1 of the first half before the product, passes 2 and 3 right after it
        if (has_cols) { fetch(0, 0); fetch(1, 0); }
      });
  if (!has_cols) return;                             // after the ring's last barrier: no barrier follows
#pragma unroll
  for (int it = 2; it < 4; ++it) fetch(it, 0);

  // This wave's LDS area: a 32 x 128 FP32 half-block, [label][column], turns the MFMA layout into
  // 16 consecutive columns per lane.  Nothing below synchronises the workgroup.
  float* gs = reinterpret_cast<float*>(smem) + wave * (32 * kGPitch);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) gs[acc_row(v, lane) * kGPitch + 32 * j + (lane & 31)] = acc[h][j][v];
    __builtin_amdgcn_s_waitcnt(0xC07F);              // the wave's own LDS writes (its lanes read each other's)
    asm volatile("" ::: "memory");

    // ---- per-element update
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = it * 8 + urow;
      const int l = wl0 + 32 * h + row;
      uint32_t w[8], c[8];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        w[q] = wreg[it][0][q];
        if (WQ == 2) w[4 + q] = wreg[it][WQ - 1][q];
        if (KAHAN) { c[q] = creg[it][0][q]; c[4 + q] = creg[it][1][q]; }
      }
      float g[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(gs + row * kGPitch + useg * 16 + 4 * q);
        g[4 * q] = t[0]; g[4 * q + 1] = t[1]; g[4 * q + 2] = t[2]; g[4 * q + 3] = t[3];
      }
      if (h == 0) fetch(it, 1);
      if (l >= n) continue;
      const size_t eoff = (size_t)l * d + wj0 + useg * 16;
      if (DROP) {
        const U4 mb = drop_block((elem0 + eoff) >> 4, seed, step);
        const uint32_t tb = dr.thresh * 0x01010101u;
        const uint32_t km[4] = {keep_bytes(mb.x, tb), keep_bytes(mb.y, tb), keep_bytes(mb.z, tb), keep_bytes(mb.w, tb)};
#pragma unroll
        for (int i = 0; i < 16; ++i) g[i] = ((km[i >> 2] >> (8 * (i & 3))) & 1u) ? g[i] * dr.scale : 0.0f;
      }
      U4 rb[2];
      if (SR) {
        const uint64_t blk = (elem0 + eoff) >> 3;
        rb[0] = sr_block(blk, seed, step);
        rb[1] = sr_block(blk + 1, seed, step);
      }
      update_wd<FMT, SR, KAHAN, WD, 16>(w, c, g, lr, wd, rb);
      char* wp = Wc + eoff * ESZ;
      *reinterpret_cast<u32x4*>(wp) = u32x4{w[0], w[1], w[2], w[3]};
      if (WQ == 2) *reinterpret_cast<u32x4*>(wp + 16) = u32x4{w[4], w[5], w[6], w[7]};
      if (KAHAN) {
        *reinterpret_cast<u32x4*>(Cc + eoff) = u32x4{c[0], c[1], c[2], c[3]};
        *reinterpret_cast<u32x4*>(Cc + eoff + 8) = u32x4{c[4], c[5], c[6], c[7]};
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Small batches (padded batch <= 128): input gradient and fused update in ONE pass over the
// weights.  At small batch the step is bound by memory traffic, and running the two products as
// separate kernels reads every weight twice; here a workgroup streams tiles of 32 labels x 256
// columns of W_c (and of the compensation) exactly once, and from each tile, while it sits in LDS,
// forms both  dX[:, cols] += G W_tile  (old weights, transposing reads)  and  grad = G^T X[:, cols]
// followed by the same per-element update as k_update.  Workgroup (g, c) owns column block c
// (256 columns) and the g-th contiguous range of label tiles of the chunk; its 128 x 256 slice of
// dX stays in registers over all its tiles and is added to dXacc[g] at the end (one owner).
// The X operand of the gradient product lives in registers for the whole kernel.
// Stage of the 3-deep ring: [W 32 x 256 el | G^T 32 x 256 B | comp 32 x 512 B].
// ---------------------------------------------------------------------------------------------
template <int FMT, bool KAHAN> constexpr int dxu_stage_bytes() {
  return 32 * 256 * (FMT == FMT_E4M3 ? 1 : 2) + 32 * 256 + (KAHAN ? 32 * 512 : 0);
}
constexpr int kDxuGsBytes = 32 * 260 * 4;
// With dropout one more W tile: the masked copy the input-gradient product reads (the update
// needs the stored weights, so the tile cannot be masked in place).
// Three stages, also where the LDS holds more: with six of 16 KiB 1 M E4M3 labels without compensation, B = 128, take 1177 us a step, with
// three 1052.
constexpr int kDxuStages = 3;
template <int FMT, bool KAHAN, bool DROP = false> constexpr int dxu_smem_bytes() {
  return kDxuStages * dxu_stage_bytes<FMT, KAHAN>() + kDxuGsBytes + (DROP ? 32 * 256 * (FMT == FMT_E4M3 ? 1 : 2) : 0);
}

// The body is a separate inlined function with restrict-qualified parameters on purpose: inlining
// it tags every LDS access inside with alias information, without which the compiler puts a full
// vmcnt(0) wait in front of the transposing LDS reads (it cannot tell them from the asynchronous
// loads still in flight for later stages) and the ring stops prefetching.  The waits that are
// needed are the explicit ones below.
template <int FMT, bool SR, bool KAHAN, bool DX, bool WD, bool DROP>
__device__ __forceinline__ void dx_update_body(const char* __restrict__ Gt, const char* __restrict__ XT, char* __restrict__ Wc,
                                               uint16_t* __restrict__ Cc, float* __restrict__ dXacc, int n, int d, int Bp,
                                               float lr, float wd, uint64_t seed, uint64_t step, uint64_t elem0, int tiles_per_group,
                                               bool first, DropArgs dr, char* smem) {
  constexpr int ESZ = FMT == FMT_E4M3 ? 1 : 2;
  constexpr int WROWB = 256 * ESZ;
  constexpr int WBYTES = 32 * WROWB, GBYTES = 32 * 256, SBYTES = dxu_stage_bytes<FMT, KAHAN>();
  constexpr int LPS = WROWB / 256 + 1 + (KAHAN ? 2 : 0);     // asynchronous loads per wave and tile
  constexpr int NST = kDxuStages;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = d >> 8;
  const int wg = xcd_logical_id(blockIdx.x, gridDim.x);
  const int g = wg / C, c = wg % C;
  const int ntiles = (n + 31) >> 5;
  const int t0 = g * tiles_per_group, t1 = min(t0 + tiles_per_group, ntiles);
  if (t0 >= t1 && !(DX && first)) return;                    // (in the first pass every group writes its dX plane)
  const int j0 = c << 8;
  const size_t strip = blk_strip(Bp);
  char* ring = smem;
  float* gs = reinterpret_cast<float*>(smem + NST * SBYTES);
  char* wmk = smem + NST * SBYTES + kDxuGsBytes;          // DROP: masked copy of the current W tile

  // X^T fragments of this wave's 32 columns (B operand of grad = G^T X), resident for the kernel
  bf16x8 xt[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    const int o = min(2 * ks + (lane >> 5), (Bp >> 3) - 1);
    xt[ks] = *reinterpret_cast<const bf16x8*>(XT + (size_t)((j0 >> 5) + wave) * strip + blk_off(o, lane & 31));
  }
  const int bt = wave & 3, jh = wave >> 2;                  // dX block of this wave: rows 32*bt.., columns 128*jh..
  f32x16 dxa[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) dxa[t][v] = 0.0f;

  auto issue = [&](int t) {
    char* st = ring + (t % NST) * SBYTES;
    const int l0 = t << 5, valid = n - l0;
    dma_tile<32, WROWB, kGemmWaves>(Wc + ((size_t)l0 * d + j0) * ESZ, (size_t)d * ESZ, valid, st, wave, lane);
    // rows of G^T past n exist and hold zeros (written by the logits kernel): no clamping, so they add nothing to dX
    dma_kib_of(Gt + (size_t)t * strip, wave, Bp >> 4, st + WBYTES + wave * 1024, lane);
    if (KAHAN)
      dma_tile<32, 512, kGemmWaves>(reinterpret_cast<const char*>(Cc) + ((size_t)l0 * d + j0) * 2, (size_t)d * 2, valid,
                                    st + WBYTES + GBYTES, wave, lane);
  };
  for (int s = 0; s < NST - 1; ++s)
    if (t0 + s < t1) issue(t0 + s);
  for (int t = t0; t < t1; ++t) {
    // Tile t has landed once only younger operations are outstanding: the loads of the tiles after it and, at least, the
    // stores of tile t-1's update (vector loads and stores retire in issue order on gfx9-family
    // parts and share vmcnt).  Every wave issues NSTORE stores per full tile; the only tile that
    // can be ragged is the last one of the chunk, after which nothing is waited for.
    constexpr int NSTORE = ESZ + (KAHAN ? 2 : 0);
    if (t == t0 || t + NST - 1 > t1) wait_slabs<LPS, NST - 2>(t1 - 1 - t);
    else wait_vmcnt<(NST - 2) * LPS + NSTORE>();
    barrier_nofence();
    if (t + NST - 1 < t1) issue(t + NST - 1);
    const char* ws = ring + (t % NST) * SBYTES;
    const char* gsl = ws + WBYTES;
    const char* cs = gsl + GBYTES;
    const int l0 = t << 5;
    const int l = tid >> 4, seg = tid & 15;                 // this thread's part of the tile: one label row, 16 consecutive columns
    const size_t eoff = (size_t)(l0 + l) * d + j0 + seg * 16;
    uint32_t w[8], km[4];
    auto load_w = [&]() {
      if (FMT == FMT_E4M3) {
        const u32x4 t4 = *reinterpret_cast<const u32x4*>(ws + tile_off<WROWB>(l, seg));
        w[0] = t4[0]; w[1] = t4[1]; w[2] = t4[2]; w[3] = t4[3];
      } else {
        const u32x4 ta = *reinterpret_cast<const u32x4*>(ws + tile_off<WROWB>(l, 2 * seg));
        const u32x4 tb = *reinterpret_cast<const u32x4*>(ws + tile_off<WROWB>(l, 2 * seg + 1));
        w[0] = ta[0]; w[1] = ta[1]; w[2] = ta[2]; w[3] = ta[3]; w[4] = tb[0]; w[5] = tb[1]; w[6] = tb[2]; w[7] = tb[3];
      }
    };
    if (DROP) {
      // the step's keep mask of these 16 elements (appendix "Low-Memory Dropout for Classifier"):
      // the input-gradient product reads a masked copy, the update below masks the gradient
      load_w();
      const U4 mb = drop_block((elem0 + eoff) >> 4, seed, step);
      const uint32_t tb = dr.thresh * 0x01010101u;
      km[0] = keep_bytes(mb.x, tb); km[1] = keep_bytes(mb.y, tb); km[2] = keep_bytes(mb.z, tb); km[3] = keep_bytes(mb.w, tb);
      if (DX) {
        if (FMT == FMT_E4M3) {
          *reinterpret_cast<u32x4*>(wmk + tile_off<WROWB>(l, seg)) = u32x4{w[0] & km[0], w[1] & km[1], w[2] & km[2], w[3] & km[3]};
        } else {
          u32x4 a, b;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            a[2 * q] = w[2 * q] & __builtin_amdgcn_perm(km[q], km[q], 0x01010000u);
            a[2 * q + 1] = w[2 * q + 1] & __builtin_amdgcn_perm(km[q], km[q], 0x03030202u);
            b[2 * q] = w[4 + 2 * q] & __builtin_amdgcn_perm(km[2 + q], km[2 + q], 0x01010000u);
            b[2 * q + 1] = w[5 + 2 * q] & __builtin_amdgcn_perm(km[2 + q], km[2 + q], 0x03030202u);
          }
          *reinterpret_cast<u32x4*>(wmk + tile_off<WROWB>(l, 2 * seg)) = a;
          *reinterpret_cast<u32x4*>(wmk + tile_off<WROWB>(l, 2 * seg + 1)) = b;
        }
        barrier_lds();
      }
    }
    const char* wdx = DROP ? wmk : ws;                      // what the input-gradient product reads

    // grad[32 labels x 32 columns of this wave] = G^T X, four reads in flight (behind a test each, every MFMA waited for its own)
    f32x16 wa;
#pragma unroll
    for (int v = 0; v < 16; ++v) wa[v] = 0.0f;
#pragma unroll
    for (int k0 = 0; k0 < 8; k0 += 4)
      if (16 * k0 < Bp) {
        bf16x8 fg[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) fg[i] = frag_blk(gsl, k0 + i, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) wa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fg[i], xt[k0 + i], wa, 0, 0, 0);
      }
    // dX[32 samples x 128 columns of this wave] += G W_tile (weights as stored before the update)
    if (DX) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 a = frag_tr_blk(gsl, 16 * kk, 32 * bt, lane);
        typename std::conditional<FMT == FMT_E4M3, i32x2, bf16x8>::type fb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (FMT == FMT_E4M3) fb[q] = frag_tr_raw8<WROWB>(wdx, 16 * kk, 128 * jh + 32 * q, lane);
          else fb[q] = frag_tr_bf16<WROWB>(wdx, 16 * kk, 128 * jh + 32 * q, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x8 b;
          if constexpr (FMT == FMT_E4M3) b = widen8(fb[q]);
          else b = fb[q];
          dxa[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, dxa[q], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) gs[acc_row(v, lane) * 260 + 32 * wave + (lane & 31)] = wa[v];
    barrier_lds();

    // per-element update
    if (l0 + l < n) {
      uint32_t cc[8];
      if (!DROP) load_w();
      if (KAHAN) {
        const u32x4 ta = *reinterpret_cast<const u32x4*>(cs + tile_off<512>(l, 2 * seg));
        const u32x4 tb = *reinterpret_cast<const u32x4*>(cs + tile_off<512>(l, 2 * seg + 1));
        cc[0] = ta[0]; cc[1] = ta[1]; cc[2] = ta[2]; cc[3] = ta[3]; cc[4] = tb[0]; cc[5] = tb[1]; cc[6] = tb[2]; cc[7] = tb[3];
      }
      float gr[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 t4 = *reinterpret_cast<const f32x4*>(gs + l * 260 + seg * 16 + 4 * q);
        gr[4 * q] = t4[0]; gr[4 * q + 1] = t4[1]; gr[4 * q + 2] = t4[2]; gr[4 * q + 3] = t4[3];
      }
      if (DROP) {
#pragma unroll
        for (int i = 0; i < 16; ++i) gr[i] = ((km[i >> 2] >> (8 * (i & 3))) & 1u) ? gr[i] * dr.scale : 0.0f;
      }
      U4 rb[2];
      if (SR) {
        const uint64_t blk = (elem0 + eoff) >> 3;
        rb[0] = sr_block(blk, seed, step);
        rb[1] = sr_block(blk + 1, seed, step);
      }
      update_wd<FMT, SR, KAHAN, WD, 16>(w, cc, gr, lr, wd, rb);
      char* wp = Wc + eoff * ESZ;
      *reinterpret_cast<u32x4*>(wp) = u32x4{w[0], w[1], w[2], w[3]};
      if (ESZ == 2) *reinterpret_cast<u32x4*>(wp + 16) = u32x4{w[4], w[5], w[6], w[7]};
      if (KAHAN) {
        *reinterpret_cast<u32x4*>(Cc + eoff) = u32x4{cc[0], cc[1], cc[2], cc[3]};
        *reinterpret_cast<u32x4*>(Cc + eoff + 8) = u32x4{cc[4], cc[5], cc[6], cc[7]};
      }
    }
  }
  if (DX) {
    if (DROP) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) dxa[q][v] *= dr.scale;
    }
    // rows beyond the padded batch are never read
    if (32 * bt < Bp) add_acc_blocks<4>(dx_block(dXacc + (size_t)g * 128 * d, d, 32 * bt, j0 + 128 * jh), lane, dxa, first);
  }
}

template <int FMT, bool SR, bool KAHAN, bool DX, bool WD, bool DROP>
__global__ void __launch_bounds__(kGemmThreads, 1)
k_dx_update(const char* __restrict__ Gt, const char* __restrict__ XT, char* __restrict__ Wc, uint16_t* __restrict__ Cc,
            float* __restrict__ dXacc, int n, int d, int Bp, float lr, float wd, uint64_t seed, uint64_t step, uint64_t elem0,
            int tiles_per_group, bool first, DropArgs dr) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  dx_update_body<FMT, SR, KAHAN, DX, WD, DROP>(Gt, XT, Wc, Cc, dXacc, n, d, Bp, lr, wd, seed, step, elem0, tiles_per_group, first, dr, smem);
}

// ---------------------------------------------------------------------------------------------
// The same in tiles of 32 labels x 128 columns, for padded batches of up to 256 rows (which of the two: plan.h).  With twice the samples the X operand of the
// gradient product (64 registers a lane) and the slice of dX (128) no longer fit into one wave, so the waves have a role each: waves
// 0-3 form the gradient of 32 columns over all samples, waves 4-7 the dX of 64 samples x 128 columns, 16 MFMAs a tile either way, and a
// SIMD holds one of each.  The update of a tile, by all eight, comes one tile late: while the upper waves update tile t - 1 the
// lower ones multiply tile t, then they change places, so the matrix cores work behind the vector ALU (a tile's update is some
// 1.5 k clocks of it on a SIMD, its products 1 k) and a tile costs one barrier.  The new weights are read
// from the tile into registers an iteration before they are updated, so that the ring gets their stage back.
// 131072 BF16 labels with compensation, B = 256, d = 768, per pass of 43520 labels: input gradient 36 us and update 71 us as separate
// kernels, 81 us here, and a launch and a third of the partial sums less; all waves in the same role, products and update in
// turn (two waves to a gradient sum, 128 samples each): 95 us; the sums of earlier passes added at the end, not loaded at the start: 88 us.
// ---------------------------------------------------------------------------------------------
template <int FMT, bool KAHAN> constexpr int dxw_stage_bytes() {
  return 32 * 128 * (FMT == FMT_E4M3 ? 1 : 2) + 32 * 512 + (KAHAN ? 32 * 256 : 0);
}
// Ring depth: what 160 KiB hold, from 3 to 6 (300000 E4M3 labels, d = 640, B = 128: 3 stages 315 us a step, 6 stages 283).
constexpr int one_pass_stages(int other, int stage) {
  const int fit = (160 * 1024 - other) / stage;
  return fit < 3 ? 3 : fit > 6 ? 6 : fit;
}
constexpr int kDxwGsBytes = 32 * 128 * 4;                        // a gradient tile; rows 4 .. 7 of eight have their column halves exchanged, for the banks
__device__ inline int dxw_gs(int row, int col) { return row * 128 + (col ^ ((row & 4) << 3)); }
// two gradient tiles, and with dropout the masked copy of the W tile that the input gradient reads and its keep bits
template <int FMT, bool DROP> constexpr int dxw_other_bytes() { return 2 * kDxwGsBytes + (DROP ? 32 * 128 * (FMT == FMT_E4M3 ? 1 : 2) + 512 : 0); }
template <int FMT, bool KAHAN, bool DROP> constexpr int dxw_stages() { return one_pass_stages(dxw_other_bytes<FMT, DROP>(), dxw_stage_bytes<FMT, KAHAN>()); }
template <int FMT, bool KAHAN, bool DROP> constexpr int dxw_smem_bytes() {
  return dxw_stages<FMT, KAHAN, DROP>() * dxw_stage_bytes<FMT, KAHAN>() + dxw_other_bytes<FMT, DROP>();
}
template <int FMT, bool SR, bool KAHAN, bool WD, bool DROP, bool LOWER>
__device__ __forceinline__ void dx_update_wide_role(const char* __restrict__ Gt, const char* __restrict__ XT, char* __restrict__ Wc,
                                                    uint16_t* __restrict__ Cc, float* __restrict__ plane, int n, int d, int Bp, float lr,
                                                    float wd, uint64_t seed, uint64_t step, uint64_t elem0, int t0, int t1, int j0, bool first,
                                                    DropArgs dr, char* __restrict__ smem) {
  constexpr int ESZ = FMT == FMT_E4M3 ? 1 : 2, WROWB = 128 * ESZ;
  constexpr int WBYTES = 32 * WROWB, GBYTES = 32 * 512, SBYTES = dxw_stage_bytes<FMT, KAHAN>();
  constexpr bool LOADS_W = ESZ == 2 || LOWER;                // 4 KiB of E4M3 weights: by the lower waves alone
  constexpr int LPS = (LOADS_W ? 1 : 0) + 2 + (KAHAN ? 1 : 0), NSTORE = 1 + (KAHAN ? 1 : 0);   // loads and stores per wave and tile
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rw = wave & 3;
  constexpr int NST = dxw_stages<FMT, KAHAN, DROP>();
  const size_t strip = blk_strip(Bp);
  char* gs0 = smem + NST * SBYTES;
  char* wmk = gs0 + 2 * kDxwGsBytes;
  uint16_t* keep = reinterpret_cast<uint16_t*>(wmk + WBYTES);

  const int xoct = (Bp >> 3) - 1, KS = Bp >> 4;              // last octet of the samples; k16 steps over them: 4, 8, 12 or 16
  bf16x8 xt[LOWER ? 16 : 1];                                 // lower: X^T fragments of columns 32 rw ..
  f32x16 dxa[LOWER ? 1 : 2][4];                              // upper: dX of samples 64 rw .., all columns
  if constexpr (LOWER) {
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      xt[ks] = *reinterpret_cast<const bf16x8*>(XT + (size_t)((j0 >> 5) + rw) * strip + blk_off(min(2 * ks + (lane >> 5), xoct), lane & 31));
  } else {
    // the sums of the passes before are where this one's begin: their loads are all in flight at once, beside the first tiles'
    zero_acc(dxa);
    if (!first)
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (64 * rw + 32 * s < Bp) load_acc_blocks<4>(dx_block(plane, d, 64 * rw + 32 * s, j0), lane, dxa[s]);
  }
  auto issue = [&](int t) {
    char* st = smem + (t % NST) * SBYTES;
    const int l0 = t << 5, valid = n - l0;
    if constexpr (LOADS_W) dma_tile<32, WROWB, ESZ == 2 ? 8 : 4>(Wc + ((size_t)l0 * d + j0) * ESZ, (size_t)d * ESZ, valid, st, wave, lane);
    // rows of G^T past n exist and hold zeros (written by the logits kernel): no clamping, so they add nothing to dX
#pragma unroll
    for (int i = 0; i < 2; ++i) dma_kib_of(Gt + (size_t)t * strip, 2 * wave + i, KS, st + WBYTES + (2 * wave + i) * 1024, lane);
    if constexpr (KAHAN)
      dma_tile<32, 256, kGemmWaves>(reinterpret_cast<const char*>(Cc) + ((size_t)l0 * d + j0) * 2, (size_t)d * 2, valid, st + WBYTES + GBYTES, wave, lane);
  };
  // this thread's part of a tile: one label row, eight consecutive columns; its weights and compensation, an iteration ahead of their update
  const int l = tid >> 4, seg = tid & 15;
  uint32_t w[8], cc[8];
  auto fetch = [&](const char* st) {
    if constexpr (ESZ == 1) {
      const uint2 v = *reinterpret_cast<const uint2*>(st + tile_off<WROWB>(l, seg >> 1) + (seg & 1) * 8);
      w[0] = v.x; w[1] = v.y;
    } else {
      const u32x4 v = *reinterpret_cast<const u32x4*>(st + tile_off<WROWB>(l, seg));
      w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
    }
    if constexpr (KAHAN) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(st + WBYTES + GBYTES + tile_off<256>(l, seg));
      cc[0] = v[0]; cc[1] = v[1]; cc[2] = v[2]; cc[3] = v[3];
    }
  };
  uint32_t kept = 0;                                         // DROP: keep bits of the eight weights
  // DROP, lower: this thread's part of the step's keep mask (appendix "Low-Memory Dropout for Classifier"), a row's 16 elements, drawn a
  // tile ahead; the input gradient reads a masked copy of the tile, the update masks the gradient
  const int mr = (tid & 255) >> 3, mb = tid & 7;
  uint32_t m[4];
  auto draw = [&](int t) {
    const U4 b = drop_block((elem0 + (size_t)((t << 5) + mr) * d + j0 + mb * 16) >> 4, seed, step);
    const uint32_t tb = dr.thresh * 0x01010101u;
    m[0] = keep_bytes(b.x, tb); m[1] = keep_bytes(b.y, tb); m[2] = keep_bytes(b.z, tb); m[3] = keep_bytes(b.w, tb);
  };
  if constexpr (DROP && LOWER) draw(t0);
  auto update = [&](int t, int rows) {                       // rows: n, or 0 where there is nothing to store
    const float* gs = reinterpret_cast<const float*>(gs0 + (t & 1) * kDxwGsBytes) + dxw_gs(l, seg * 8);
    const f32x4 ga = *reinterpret_cast<const f32x4*>(gs), gb = *reinterpret_cast<const f32x4*>(gs + 4);
    float g[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
    if (DROP) {
#pragma unroll
      for (int i = 0; i < 8; ++i) g[i] = ((kept >> i) & 1u) ? g[i] * dr.scale : 0.0f;
    }
    const int row = (t << 5) + l;
    const size_t eoff = (size_t)row * d + j0 + seg * 8;
    U4 rb[1];
    if (SR) rb[0] = sr_block((elem0 + eoff) >> 3, seed, step);
    update_wd<FMT, SR, KAHAN, WD, 8>(w, cc, g, lr, wd, rb);
    if ((uint32_t)row < (uint32_t)rows) {                    // (before the first tile the row may be negative)
      char* wp = Wc + eoff * ESZ;
      if constexpr (ESZ == 1) *reinterpret_cast<uint2*>(wp) = make_uint2(w[0], w[1]);
      else *reinterpret_cast<u32x4*>(wp) = u32x4{w[0], w[1], w[2], w[3]};
      if constexpr (KAHAN) *reinterpret_cast<u32x4*>(Cc + eoff) = u32x4{cc[0], cc[1], cc[2], cc[3]};
    }
  };
  for (int s = 0; s < NST - 1; ++s)
    if (t0 + s < t1) issue(t0 + s);
  for (int t = t0; t < t1; ++t) {
    // Younger than tile t's loads are those of the tiles after it and, from the third tile on, at least the stores of the last update
    // (loads and stores retire in issue order and share vmcnt).  Every wave issues its
    // stores in every tile but a ragged last one, after which nothing is waited for.
    if (t < t0 + 2 || t + NST - 1 > t1) wait_slabs<LPS, NST - 2>(t1 - 1 - t);
    else wait_vmcnt<(NST - 2) * LPS + NSTORE>();
    barrier_lds();                                           // tile t, and the gradient of tile t - 1
    if (t + NST - 1 < t1) issue(t + NST - 1);
    const char* st = smem + (t % NST) * SBYTES;
    const char* gsl = st + WBYTES;
    if constexpr (LOWER) {
      if constexpr (DROP) {
        uint32_t bits = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) bits |= (((m[i] & 0x01010101u) * 0x01020408u) >> 24 & 15u) << (4 * i);
        keep[mr * 8 + mb] = (uint16_t)bits;
        if constexpr (ESZ == 1) {
          const int o = tile_off<WROWB>(mr, mb);
          *reinterpret_cast<u32x4*>(wmk + o) = *reinterpret_cast<const u32x4*>(st + o) & u32x4{m[0], m[1], m[2], m[3]};
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int o = tile_off<WROWB>(mr, 2 * mb + h);
            *reinterpret_cast<u32x4*>(wmk + o) = *reinterpret_cast<const u32x4*>(st + o) &
                u32x4{__builtin_amdgcn_perm(m[2 * h], m[2 * h], 0x01010000u), __builtin_amdgcn_perm(m[2 * h], m[2 * h], 0x03030202u),
                      __builtin_amdgcn_perm(m[2 * h + 1], m[2 * h + 1], 0x01010000u), __builtin_amdgcn_perm(m[2 * h + 1], m[2 * h + 1], 0x03030202u)};
          }
        }
        barrier_lds();
      }
      f32x16 wa;                                             // grad[32 labels x 32 columns] = G^T X
#pragma unroll
      for (int v = 0; v < 16; ++v) wa[v] = 0.0f;
#pragma unroll
      for (int k0 = 0; k0 < 16; k0 += 4)                      // (four reads in flight; KS is a multiple of four)
        if (k0 < KS) {
          bf16x8 fg[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) fg[i] = frag_blk(gsl, k0 + i, lane);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 4; ++i) wa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fg[i], xt[k0 + i], wa, 0, 0, 0);
        }
      if constexpr (DROP) draw(t + 1);
      update(t - 1, t > t0 ? n : 0);
      float* gs = reinterpret_cast<float*>(gs0 + (t & 1) * kDxwGsBytes);
#pragma unroll
      for (int v = 0; v < 16; ++v) gs[dxw_gs(acc_row(v, lane), 32 * rw + (lane & 31))] = wa[v];
    } else {
      if constexpr (DROP) barrier_lds();
      update(t - 1, t > t0 ? n : 0);
      const char* wdx = DROP ? wmk : st;
      bf16x8 fa[2][2];                                       // dX += G W_tile (weights as stored before the update), all fragments read first
      typename std::conditional<ESZ == 1, i32x2, bf16x8>::type fb[2][4];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int s = 0; s < 2; ++s) fa[kk][s] = frag_tr_blk(gsl, 16 * kk, 64 * rw + 32 * s, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (ESZ == 1) fb[kk][q] = frag_tr_raw8<WROWB>(wdx, 16 * kk, 32 * q, lane);
          else fb[kk][q] = frag_tr_bf16<WROWB>(wdx, 16 * kk, 32 * q, lane);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x8 b;
          if constexpr (ESZ == 1) b = widen8(fb[kk][q]);
          else b = fb[kk][q];
#pragma unroll
          for (int s = 0; s < 2; ++s) dxa[s][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][s], b, dxa[s][q], 0, 0, 0);
        }
    }
    fetch(st);
    if constexpr (DROP) kept = keep[l * 8 + (seg >> 1)] >> (8 * (seg & 1));
  }
  if (t0 < t1) {
    barrier_lds();
    update(t1 - 1, n);
  }
  if constexpr (!LOWER) {
#pragma unroll
    for (int s = 0; s < 2; ++s)            // rows beyond the padded batch are never read; with dropout 1 / (1 - p) comes with the final sum
      if (64 * rw + 32 * s < Bp) add_acc_blocks<4>(dx_block(plane, d, 64 * rw + 32 * s, j0), lane, dxa[s], true);
  }
}

template <int FMT, bool SR, bool KAHAN, bool WD, bool DROP>
__global__ void __launch_bounds__(kGemmThreads, 1)
k_dx_update_wide(const char* __restrict__ Gt, const char* __restrict__ XT, char* __restrict__ Wc, uint16_t* __restrict__ Cc,
                 float* __restrict__ dXacc, int n, int d, int Bp, float lr, float wd, uint64_t seed, uint64_t step, uint64_t elem0,
                 int tiles_per_group, bool first, DropArgs dr) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int C = d >> 7, wg = xcd_logical_id(blockIdx.x, gridDim.x), g = wg / C, c = wg % C;
  const int t0 = g * tiles_per_group, t1 = min(t0 + tiles_per_group, (n + 31) >> 5);
  if (t0 >= t1 && !first) return;                            // (in the first pass every group writes its dX plane)
  float* plane = dXacc + (size_t)g * 256 * d;
  if (threadIdx.x < 256)
    dx_update_wide_role<FMT, SR, KAHAN, WD, DROP, true>(Gt, XT, Wc, Cc, plane, n, d, Bp, lr, wd, seed, step, elem0, t0, t1, c << 7, first, dr, smem);
  else
    dx_update_wide_role<FMT, SR, KAHAN, WD, DROP, false>(Gt, XT, Wc, Cc, plane, n, d, Bp, lr, wd, seed, step, elem0, t0, t1, c << 7, first, dr, smem);
}

// ---------------------------------------------------------------------------------------------
// Stand-alone quantiser (round to nearest even or stochastic rounding with the step's fields).
// Bound by memory (4 bytes read, 1 or 2 written per element), so a thread takes eight consecutive
// elements: two 16-byte loads, one 8- or 16-byte store, and with stochastic rounding the one Philox
// block (two where `first` is not a multiple of 8) that holds their fields.  One element per thread
// moved a byte per store and drew a whole block per element: 50 M elements to
// E4M3 took 69.7 us (3.6 TB/s), now 46.0 us (5.5 TB/s).
// WIDE: `groups` whole groups of eight are taken this way and the rest element by element.  Otherwise everything is, one
// element per thread: buffers that are not aligned to the wide accesses, and short stochastic calls, where the Philox rounds
// of one element are all there is to wait for and the two blocks and eight roundings of a group only lengthen the chain.
// ---------------------------------------------------------------------------------------------
// Elements from which a stochastic call takes the wide form; E4M3, one element / eight per thread: 0.1 M 2.4 / 3.1 us,
// 1.5 M 4.7 / 5.0, 2 M 5.5 / 5.5, 3 M 7.4 / 6.5.
constexpr int64_t kQuantWideSr = 2 << 20;
template <int FMT, bool SR, bool WIDE>
__global__ void __launch_bounds__(kThreads) k_quantize(const float* __restrict__ src, int64_t n, int64_t groups, uint64_t seed, uint64_t step,
                                                       uint64_t first, void* __restrict__ dst) {
  const int64_t t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x, nt = (int64_t)gridDim.x * kThreads;
  if constexpr (WIDE) {
    for (int64_t i = t0; i < groups; i += nt) {
      const f32x4 a = reinterpret_cast<const f32x4*>(src)[2 * i], b = reinterpret_cast<const f32x4*>(src)[2 * i + 1];
      uint32_t r[8];
      if (SR) {
        const uint64_t e = first + 8 * (uint64_t)i;
        const int o = (int)(e & 7);
        const U4 lo = sr_block(e >> 3, seed, step);
        U4 hi = lo;
        if (o) hi = sr_block((e >> 3) + 1, seed, step);
#pragma unroll
        for (int k = 0; k < 8; ++k) r[k] = sr_field(o + k < 8 ? lo : hi, (o + k) & 7);
      }
      uint32_t q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float t = k < 4 ? a[k & 3] : b[k & 3];
        q[k] = SR ? quant_sr<FMT>(t, r[k]) : quant_rne<FMT>(t);
      }
      if (FMT == FMT_E4M3) {
        reinterpret_cast<uint2*>(dst)[i] = make_uint2(q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24), q[4] | (q[5] << 8) | (q[6] << 16) | (q[7] << 24));
      } else {
        reinterpret_cast<u32x4*>(dst)[i] = u32x4{q[0] | (q[1] << 16), q[2] | (q[3] << 16), q[4] | (q[5] << 16), q[6] | (q[7] << 16)};
      }
    }
  }
  for (int64_t i = (WIDE ? 8 * groups : 0) + t0; i < n; i += nt) {
    const float t = src[i];
    uint32_t q;
    if (SR) {
      const uint64_t e = first + (uint64_t)i;
      const U4 rb = sr_block(e >> 3, seed, step);
      q = quant_sr<FMT>(t, sr_field(rb, (int)(e & 7)));
    } else {
      q = quant_rne<FMT>(t);
    }
    if (FMT == FMT_E4M3) reinterpret_cast<uint8_t*>(dst)[i] = (uint8_t)q;
    else reinterpret_cast<uint16_t*>(dst)[i] = (uint16_t)q;
  }
}

// Simulated (E, M) format: dst[i] = FP32 value of src[i] rounded to that format.
template <bool SR>
__global__ void __launch_bounds__(kThreads) k_quantize_em(const float* __restrict__ src, int64_t n, int E, int M, uint64_t seed,
                                                          uint64_t step, uint64_t first, float* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    int r16 = -1;
    if (SR) {
      const uint64_t e = first + (uint64_t)i;
      r16 = (int)sr_field(sr_block(e >> 3, seed, step), (int)(e & 7));
    }
    dst[i] = round_em(src[i], E, M, r16);
  }
}

// ---------------------------------------------------------------------------------------------
// AdamW with Kahan-compensated BF16 parameters (Section 4.1: Kahan summation for the encoder's
// parameters).  Elementwise, 8 elements per thread and pass; FP32 arithmetic, every operation
// rounded once; the moments are BF16 (stored round-to-nearest-even) or FP32.
//   m' = b1 m + o1 g;  v' = b2 v + (o2 g) g;  r = (m'/bc1) / (sqrt(v'/bc2) + eps) [+ wd p];  u = lr r
//   y = -u - c;  s = p + y;  p' = RNE_BF16(s);  c' = RNE_BF16((p' - p) - y)
// ---------------------------------------------------------------------------------------------
struct AdamArgs { float lr, b1, o1, b2, o2, bc1, bc2, eps, wd; };

__device__ inline void adamw_element(uint32_t& pb, uint32_t& cb, float& m, float& v, uint32_t gb, const AdamArgs& a) {
  const float p = bf16_decode(pb), c = bf16_decode(cb), g = bf16_decode(gb);
  m = __fadd_rn(__fmul_rn(a.b1, m), __fmul_rn(a.o1, g));
  v = __fadd_rn(__fmul_rn(a.b2, v), __fmul_rn(__fmul_rn(a.o2, g), g));
  const float mh = __fdiv_rn(m, a.bc1), vh = __fdiv_rn(v, a.bc2);
  float r = __fdiv_rn(mh, __fadd_rn(sqrtf(vh), a.eps));      // sqrtf and '/' are correctly rounded (the __fsqrt_rn intrinsic is not)
  if (a.wd != 0.0f) r = __fadd_rn(r, __fmul_rn(a.wd, p));
  const float u = __fmul_rn(a.lr, r);
  const float y = __fsub_rn(-u, c);
  const uint32_t q = bf16_rne(__fadd_rn(p, y));
  cb = bf16_rne(__fsub_rn(__fsub_rn(bf16_decode(q), p), y));
  pb = q;
}

template <bool STATE_BF16>
__global__ void __launch_bounds__(kThreads) k_kahan_adamw(uint16_t* __restrict__ P, uint16_t* __restrict__ C, void* __restrict__ Mv,
                                                          void* __restrict__ Vv, const uint16_t* __restrict__ G, int64_t n,
                                                          AdamArgs a) {
  const int64_t groups = n >> 3;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < groups; i += (int64_t)gridDim.x * kThreads) {
    u32x4 p4 = reinterpret_cast<const u32x4*>(P)[i], c4 = reinterpret_cast<const u32x4*>(C)[i];
    const u32x4 g4 = reinterpret_cast<const u32x4*>(G)[i];
    float m[8], v[8];
    if (STATE_BF16) {
      const u32x4 m4 = reinterpret_cast<const u32x4*>(Mv)[i], v4 = reinterpret_cast<const u32x4*>(Vv)[i];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        m[e] = bf16_decode((m4[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
        v[e] = bf16_decode((v4[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
      }
    } else {
      const f32x4 ma = reinterpret_cast<const f32x4*>(Mv)[2 * i], mb = reinterpret_cast<const f32x4*>(Mv)[2 * i + 1];
      const f32x4 va = reinterpret_cast<const f32x4*>(Vv)[2 * i], vb = reinterpret_cast<const f32x4*>(Vv)[2 * i + 1];
#pragma unroll
      for (int e = 0; e < 4; ++e) { m[e] = ma[e]; m[4 + e] = mb[e]; v[e] = va[e]; v[4 + e] = vb[e]; }
    }
    uint32_t pn[8], cn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pn[e] = (p4[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
      cn[e] = (c4[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
      adamw_element(pn[e], cn[e], m[e], v[e], (g4[e >> 1] >> (16 * (e & 1))) & 0xFFFFu, a);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      p4[q] = pn[2 * q] | (pn[2 * q + 1] << 16);
      c4[q] = cn[2 * q] | (cn[2 * q + 1] << 16);
    }
    reinterpret_cast<u32x4*>(P)[i] = p4;
    reinterpret_cast<u32x4*>(C)[i] = c4;
    if (STATE_BF16) {
      u32x4 m4, v4;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        m4[q] = bf16_rne(m[2 * q]) | (bf16_rne(m[2 * q + 1]) << 16);
        v4[q] = bf16_rne(v[2 * q]) | (bf16_rne(v[2 * q + 1]) << 16);
      }
      reinterpret_cast<u32x4*>(Mv)[i] = m4;
      reinterpret_cast<u32x4*>(Vv)[i] = v4;
    } else {
      reinterpret_cast<f32x4*>(Mv)[2 * i] = f32x4{m[0], m[1], m[2], m[3]};
      reinterpret_cast<f32x4*>(Mv)[2 * i + 1] = f32x4{m[4], m[5], m[6], m[7]};
      reinterpret_cast<f32x4*>(Vv)[2 * i] = f32x4{v[0], v[1], v[2], v[3]};
      reinterpret_cast<f32x4*>(Vv)[2 * i + 1] = f32x4{v[4], v[5], v[6], v[7]};
    }
  }
  // the last n % 8 elements, one thread each
  const int64_t tail = (groups << 3) + (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (tail < n) {
    uint32_t pb = P[tail], cb = C[tail];
    float m = STATE_BF16 ? bf16_decode(reinterpret_cast<uint16_t*>(Mv)[tail]) : reinterpret_cast<float*>(Mv)[tail];
    float v = STATE_BF16 ? bf16_decode(reinterpret_cast<uint16_t*>(Vv)[tail]) : reinterpret_cast<float*>(Vv)[tail];
    adamw_element(pb, cb, m, v, G[tail], a);
    P[tail] = (uint16_t)pb;
    C[tail] = (uint16_t)cb;
    if (STATE_BF16) {
      reinterpret_cast<uint16_t*>(Mv)[tail] = (uint16_t)bf16_rne(m);
      reinterpret_cast<uint16_t*>(Vv)[tail] = (uint16_t)bf16_rne(v);
    } else {
      reinterpret_cast<float*>(Mv)[tail] = m;
      reinterpret_cast<float*>(Vv)[tail] = v;
    }
  }
}

}  // namespace elmo
