// In-place perturbation pass theta <- rnd(theta + c Z), Z = a G + b U R (Eq. (10)),
// with G and R regenerated from the shared seed in registers / LDS and never
// stored (Sec. 3.1 step 5; Algorithm 1, client and edge-server blocks).  One
// pass reads and writes every parameter exactly once.
//
// Two persistent kernels per pass, each looping over a work list:
//   flat: tensors without a basis (embeddings, biases, LayerNorm, non-guided
//         rounds): one thread per Philox call, fully coalesced vector RMW;
//   tile: guided matrices: a block owns a [rows x 32P] column strip piece,
//         generates its slice of R once into LDS, stages U row blocks in LDS,
//         contracts U R in registers and fuses G, the mix and the axpy.
#include "internal.h"
#include "planes.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>

namespace zgr {

namespace {

struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }
__device__ __forceinline__ void from_f32(float x, float& o) { o = x; }
__device__ __forceinline__ void from_f32(float x, bf16_t& o) {     // round to nearest, ties to even (v_cvt_pk_bf16_f32)
  const __bf16 h = static_cast<__bf16>(x);
  o.bits = __builtin_bit_cast(uint16_t, h);
}

template <typename T, int P> struct alignas(sizeof(T) * P <= 16 ? sizeof(T) * P : 16) Vec { T v[P]; };

// P fp32 results into the storage type: fp32 as they are, bf16 rounded two at a time (one v_cvt_pk_bf16_f32 per pair,
// which leaves the pair in the dword it is stored from).
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
template <int P> __device__ __forceinline__ void round_into(Vec<float, P>& x, const float* f) {
#pragma unroll
  for (int j = 0; j < P; ++j) x.v[j] = f[j];
}
template <int P> __device__ __forceinline__ void round_into(Vec<bf16_t, P>& x, const float* f) {
#pragma unroll
  for (int j = 0; j < P; j += 2) {
    const bf16x2_t r = __builtin_convertvector(f32x2_t{f[j], f[j + 1]}, bf16x2_t);
    const uint32_t bits = __builtin_bit_cast(uint32_t, r);
    x.v[j].bits = (uint16_t)bits;
    x.v[j + 1].bits = (uint16_t)(bits >> 16);
  }
}

// theta pointers come out of descriptors in memory, so the compiler cannot know that they point to global
// memory and would emit FLAT accesses (which also tie up the LDS counter); say so explicitly.
template <typename V> __device__ __forceinline__ V load_global(const void* p) {
  typedef uint32_t R __attribute__((ext_vector_type(sizeof(V) / 4)));
  typedef const R __attribute__((address_space(1))) GR;
  const R r = *reinterpret_cast<GR*>(reinterpret_cast<uintptr_t>(p));
  V v;
  __builtin_memcpy(&v, &r, sizeof(V));
  return v;
}
template <> __device__ __forceinline__ float load_global<float>(const void* p) {
  typedef const float __attribute__((address_space(1))) GF;
  return *reinterpret_cast<GF*>(reinterpret_cast<uintptr_t>(p));
}
template <typename V> __device__ __forceinline__ void store_global(void* p, const V& v) {
  typedef uint32_t R __attribute__((ext_vector_type(sizeof(V) / 4)));
  typedef R __attribute__((address_space(1))) GR;
  R r;
  __builtin_memcpy(&r, &v, sizeof(V));
  *reinterpret_cast<GR*>(reinterpret_cast<uintptr_t>(p)) = r;
}

__device__ __forceinline__ float load_global_elem(const float* p) { return load_global<float>(p); }
__device__ __forceinline__ bf16_t load_global_elem(const bf16_t* p) {
  typedef const uint16_t __attribute__((address_space(1))) GH;
  bf16_t r; r.bits = *reinterpret_cast<GH*>(reinterpret_cast<uintptr_t>(p)); return r;
}
__device__ __forceinline__ void store_global_elem(float* p, float v) {
  typedef float __attribute__((address_space(1))) GF;
  *reinterpret_cast<GF*>(reinterpret_cast<uintptr_t>(p)) = v;
}
__device__ __forceinline__ void store_global_elem(bf16_t* p, bf16_t v) {
  typedef uint16_t __attribute__((address_space(1))) GH;
  *reinterpret_cast<GH*>(reinterpret_cast<uintptr_t>(p)) = v.bits;
}

// A descriptor or work-list entry read through the constant address space: these tables are never written by a
// kernel, and only a load the compiler knows to be invariant may use the scalar unit however many stores to theta
// surround it (as a vector load it would have to be waited for behind the stores issued just before it).
template <typename S> __device__ __forceinline__ S load_const(const S* p) {
  static_assert(sizeof(S) % 4 == 0, "whole words");
  typedef const uint32_t __attribute__((address_space(4))) CW;
  CW* w = reinterpret_cast<CW*>(reinterpret_cast<uintptr_t>(p));
  uint32_t buf[sizeof(S) / 4];
#pragma unroll
  for (size_t i = 0; i < sizeof(S) / 4; ++i) buf[i] = w[i];
  S s;
  __builtin_memcpy(&s, buf, sizeof(S));
  return s;
}

template <int P> __device__ __forceinline__ void gaussP(const u32x4 w, const RadiusEntry* tab, float* g);
template <> __device__ __forceinline__ void gaussP<4>(const u32x4 w, const RadiusEntry* tab, float* g) { gauss4(w, tab, g); }
template <> __device__ __forceinline__ void gaussP<8>(const u32x4 w, const RadiusEntry* tab, float* g) { gauss8(w, tab, g); }

// Element [row][l] of the basis: fp32 as stored, or restored from its 4-bit code as lambda (code - delta)
// (Sec. 3.4, first equation): the restore is fused into the operand load, the fp32 basis never exists in memory.
__device__ __forceinline__ float basis_at(const TensorDesc& d, int64_t row, int l) {
  if (d.Uq) {
    const uint32_t byte = d.Uq[row * d.ldu + (l >> 1)];
    const uint32_t code = (l & 1) ? (byte >> 4) : (byte & 15u);
    return d.qlambda * ((float)code - d.qdelta);
  }
  return load_global<float>(d.U + row * d.ldu + l);
}

// Layer pipeline (Sec. 3.3): a launch also fetches the basis data its successor will need, straight from pinned
// host memory into the staging slot the successor reads.  The last a.pull_blocks blocks of the grid do nothing
// else (a block that waited for the host link before computing would delay its share of the tiles by that long);
// the other blocks share the work list among themselves.  The kernel boundary makes the data visible.
__device__ __forceinline__ void pull_next_stage(const PerturbArgs& a, int part, int parts) {
  for (int t = 0; t < a.n_stage; ++t) {
    const StageCopy sc = a.stage[t];
    const uint64_t n16 = sc.bytes >> 4;
    const uint4* src = reinterpret_cast<const uint4*>(sc.src);
    uint4* dst = reinterpret_cast<uint4*>(sc.dst);
    for (uint64_t i = (uint64_t)part * blockDim.x + threadIdx.x; i < n16; i += (uint64_t)parts * blockDim.x) dst[i] = src[i];
    if (part == 0)
      for (uint64_t i = (n16 << 4) + threadIdx.x; i < sc.bytes; i += blockDim.x) sc.dst[i] = sc.src[i];
  }
}

__global__ void __launch_bounds__(256) stage_only_kernel(PerturbArgs a) { pull_next_stage(a, blockIdx.x, gridDim.x); }

// What a pass does with Z.
//   kOne:    theta <- rnd(theta + c Z), theta read from the second copy instead when a.from_copy is set
//   kBatch:  the same with a sum of perturbations in place of Z
//   kSpread: what three passes with c, -2c and c leave behind, from one generation of Z and one read of theta: copy 0 <- rnd(theta + c Z),
//            copy 1 <- rnd(copy 0 - 2c Z), theta <- rnd(copy 1 + c Z) (theta stays as it is when a.restore is 0)
// Vector instructions are what bounds kOne (the generator alone 425 cycles a call against 420 for the bytes, some 200 more for the rest); kSpread
// calls the generator once for four times a value's bytes and is bound by those.  Against three passes, when it was written: steps of 1.3B bf16
// parameters 29.0 -> 26.1 ms, of 350M 10.0 -> 9.1, of 125M 3.30 -> 3.21.
enum { kOne = 0, kBatch = 1, kSpread = 2 };

// The P Gaussians of Philox call q of one stream.  kBatch: instead the combination sum_i qcoef[i] * (those of step
// qstep[i]), accumulated in the order of the list; since Z is linear in (G, R), a batched pass is the single
// pass with this combination in place of G and of R and the coefficient 1.
template <int P, int MODE>
__device__ __forceinline__ void draw(uint32_t q_lo, uint32_t q_hi, uint32_t id_stream, const PerturbArgs& a, const RadiusEntry* tab, float* g) {
  if (MODE != kBatch) {
    gaussP<P>(philox4x32_10(q_lo, q_hi, id_stream, a.step, a.k0, a.k1), tab, g);
  } else {
#pragma unroll
    for (int j = 0; j < P; ++j) g[j] = 0.f;
    for (int i = 0; i < a.n_q; ++i) {
      float t[P];
      gaussP<P>(philox4x32_10(q_lo, q_hi, id_stream, a.qstep[i], a.k0, a.k1), tab, t);
      const float ci = a.qcoef[i];
#pragma unroll
      for (int j = 0; j < P; ++j) g[j] = __builtin_fmaf(ci, t[j], g[j]);
    }
  }
}
template <int P, int MODE>
__device__ __forceinline__ void draw(uint64_t q, uint32_t id_stream, const PerturbArgs& a, const RadiusEntry* tab, float* g) {
  draw<P, MODE>((uint32_t)q, (uint32_t)(q >> 32), id_stream, a, tab, g);
}

// Where the parameters of one tensor are read and written.
template <typename T> struct Places { const T* src; T* theta; T* copy0; T* copy1; };
template <typename T, int MODE> __device__ __forceinline__ Places<T> places_of(const TensorDesc& d, const PerturbArgs& a) {
  Places<T> w;
  w.theta = reinterpret_cast<T*>(d.theta);
  w.copy0 = MODE == kSpread ? reinterpret_cast<T*>(a.copy[0] + d.copy) : nullptr;
  w.copy1 = MODE == kSpread ? reinterpret_cast<T*>(a.copy[1] + d.copy) : nullptr;
  w.src = MODE == kOne && a.from_copy ? reinterpret_cast<const T*>(a.copy[1] + d.copy) : w.theta;
  return w;
}

// P parameters x (elements e0 .. e0 + P - 1) and their Z: every result rounded to the storage type before the next is taken from it.
template <typename T, int P, int MODE>
__device__ __forceinline__ void apply_z(const Places<T>& w, const PerturbArgs& a, int64_t e0, Vec<T, P> x, const float* z, float c) {
  auto add = [&](float coef) {
    float f[P];
#pragma unroll
    for (int j = 0; j < P; ++j) f[j] = __builtin_fmaf(coef, z[j], to_f32(x.v[j]));
    round_into<P>(x, f);
  };
  add(c);
  if (MODE != kSpread) { store_global(w.theta + e0, x); return; }
  store_global(w.copy0 + e0, x);
  add(-2.0f * c);
  store_global(w.copy1 + e0, x);
  if (a.restore) { add(c); store_global(w.theta + e0, x); }
}
template <typename T, int MODE>
__device__ __forceinline__ void apply_z_elem(const Places<T>& w, const PerturbArgs& a, int64_t e, float z, float c) {
  T x = load_global_elem(w.src + e);
  from_f32(__builtin_fmaf(c, z, to_f32(x)), x);
  if (MODE != kSpread) { store_global_elem(w.theta + e, x); return; }
  store_global_elem(w.copy0 + e, x);
  from_f32(__builtin_fmaf(-2.0f * c, z, to_f32(x)), x);
  store_global_elem(w.copy1 + e, x);
  if (a.restore) { from_f32(__builtin_fmaf(c, z, to_f32(x)), x); store_global_elem(w.theta + e, x); }
}

// The work list and the tensor descriptors are separate __restrict__ kernel parameters (besides being members
// of PerturbArgs): only then can the compiler tell that the stores to theta do not change them, and fetch them
// with scalar loads.  Fetched through the struct they become vector loads behind an s_waitcnt vmcnt(0), which
// drains every outstanding load and store of the wave once per work item.
// ------------------------------------------------------------------ flat
// Materialiser of Z for the isotropic tensors (test boundary only): one thread per Philox call.
template <typename T, int P>
__global__ void __launch_bounds__(256) fill_flat_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items,
                                                        const RadiusEntry* __restrict__ gtab, float* __restrict__ zout) {
  __shared__ RadiusEntry tab[kRadiusTabEntries];
  load_radius_table(tab, gtab);
  __syncthreads();
  for (int w = blockIdx.x; w < a.n_flat; w += gridDim.x) {
    const WorkItem it = items[w];
    const TensorDesc d = descs[it.tensor];
    const int64_t n = d.rows * d.cols;
    for (int g = threadIdx.x; g < it.count; g += 256) {
      const int64_t q = it.first + g;
      float G[P];
      draw<P, kOne>((uint64_t)q, d.id, a, tab, G);
      for (int j = 0; j < P; ++j) if (q * P + j < n) zout[q * P + j] = G[j];
    }
  }
}

// The registers of v as inputs of an empty statement: whatever they are waiting for (a load issued long ago) is
// waited for HERE.  The compiler places the wait for an outstanding load in front of the first use of its
// registers, and that wait also covers every store issued before it; anchoring it in front of a store, at a point
// where the load is a whole work item old, keeps the write it would otherwise have to sit out behind it.
template <typename V> __device__ __forceinline__ void wait_here_for(const V& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef uint32_t R __attribute__((ext_vector_type(sizeof(V) / 4 > 4 ? 4 : sizeof(V) / 4)));
  R r[sizeof(V) / sizeof(R)];
  __builtin_memcpy(r, &v, sizeof(V));
#pragma unroll
  for (size_t i = 0; i < sizeof(V) / sizeof(R); ++i) asm volatile("" ::"v"(r[i]));
#endif
}

// In-place pass over the isotropic tensors.  A work item is flat_groups_per_item Philox calls of one tensor; a
// thread owns the calls tid, tid + 256, ... of it (flat_slots of them, 64 bytes per lane).  The parameters of the NEXT item of the
// block are requested before the generator runs for the current one, so kFlatSlots vectors per lane are in
// flight under a whole item's arithmetic: the pass needs about 20 KB of reads in flight per compute unit to
// keep HBM busy, and one 8-byte request per lane at a time, waited for after one call, supplies less than that.
// The share of block `block` of `nblk`, 256 threads, the table in LDS.
template <typename T, int P, int MODE>
__device__ __forceinline__ void flat_share(const PerturbArgs& a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items, float c, const RadiusEntry* tab, int block, int nblk) {
  constexpr int kFlatSlots = flat_slots((int)sizeof(T), P);
  const int tid = threadIdx.x;
  // Requests the vectors of item w (the last item again once the list is exhausted).  A slot past the end of the
  // item or of the tensor re-reads the tensor's last whole vector, and a tensor shorter than one vector reads the
  // descriptor table instead: always in bounds, never used, and so the requests carry no condition at all (a
  // conditional request would make the compiler merge old and new registers behind it, with a wait).
  auto request = [&](int w, Vec<T, P>* buf) {
    const WorkItem it = load_const(items + (w < a.n_flat ? w : a.n_flat - 1));
    const TensorDesc d = load_const(descs + it.tensor);
    const int64_t n = d.rows * d.cols;
    const int64_t last = n >= P ? (n - P) / P * P : 0;
    const T* th = n >= P ? places_of<T, MODE>(d, a).src : reinterpret_cast<const T*>(descs);
#pragma unroll
    for (int j = 0; j < kFlatSlots; ++j) {
      int64_t e0 = (it.first + tid + 256 * j) * P;
      e0 = e0 < last ? e0 : last;
      buf[j] = load_global<Vec<T, P>>(th + e0);
    }
  };
  Vec<T, P> cur[kFlatSlots], nxt[kFlatSlots];
  request(block, cur);
#pragma unroll
  for (int j = 0; j < kFlatSlots; ++j) wait_here_for(cur[j]);      // nothing outstanding on entry to the loop
  for (int w = block; w < a.n_flat; w += nblk) {
    request(w + nblk, nxt);
    const WorkItem it = load_const(items + w);
    const TensorDesc d = load_const(descs + it.tensor);
    const int64_t n = d.rows * d.cols;
    const Places<T> at = places_of<T, MODE>(d, a);
    // an item starts at a multiple of its length, a power of two: its counters share their upper word
    const uint32_t q_lo = (uint32_t)it.first, q_hi = (uint32_t)((uint64_t)it.first >> 32);
    // the next item's vectors were requested a whole item ago and the youngest store is one call old: nothing to sit out
    auto arrived = [&]() {
#pragma unroll
      for (int i = 0; i < kFlatSlots; ++i) wait_here_for(nxt[i]);
    };
    if (it.count == 256 * kFlatSlots && (it.first + it.count) * P <= n) {
#pragma unroll
      for (int j = 0; j < kFlatSlots; ++j) {
        float G[P];
        draw<P, MODE>(q_lo + (uint32_t)(tid + 256 * j), q_hi, d.id, a, tab, G);
        if (j == kFlatSlots - 1) arrived();
        apply_z<T, P, MODE>(at, a, (it.first + tid + 256 * j) * P, cur[j], G, c);
      }
    } else {
#pragma unroll
      for (int j = 0; j < kFlatSlots; ++j) {
        const int g = tid + 256 * j;
        if (j == kFlatSlots - 1) arrived();
        if (g < it.count) {
          const int64_t e0 = (it.first + g) * P;
          float G[P];
          draw<P, MODE>(q_lo + (uint32_t)g, q_hi, d.id, a, tab, G);
          if (e0 + P <= n) {
            apply_z<T, P, MODE>(at, a, e0, cur[j], G, c);
          } else {
            // ragged end of a tensor: element by element
            for (int i = 0; i < P; ++i)
              if (e0 + i < n) apply_z_elem<T, MODE>(at, a, e0 + i, G[i], c);
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kFlatSlots; ++j) cur[j] = nxt[j];
  }
}
template <typename T, int P, int MODE>
__global__ void __launch_bounds__(256) perturb_flat_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items,
                                                           float c, const RadiusEntry* __restrict__ gtab) {
  __shared__ RadiusEntry tab[kRadiusTabEntries];
  const int nblk = (int)gridDim.x - a.pull_blocks;               // computing blocks
  if ((int)blockIdx.x >= nblk) { pull_next_stage(a, (int)blockIdx.x - nblk, a.pull_blocks); return; }
  load_radius_table(tab, gtab);
  __syncthreads();
  flat_share<T, P, MODE>(a, descs, items, c, tab, (int)blockIdx.x, nblk);
}

// ------------------------------------------------------------------ tile
typedef float f32x16 __attribute__((ext_vector_type(16)));

// One lane's P consecutive elements starting at flat index e0: G from the seed, Z = a G + (b U R), axpy.
template <typename T, int P, bool WRITE_Z, int MODE>
__device__ __forceinline__ void finish_row(const TensorDesc& d, const Places<T>& at, float* __restrict__ zout, int64_t e0, const float* ur,
                                           float c, const PerturbArgs& a, const RadiusEntry* tab) {
  float G[P];
  draw<P, MODE>((uint64_t)e0 / P, d.id, a, tab, G);
  if (WRITE_Z) {
#pragma unroll
    for (int j = 0; j < P; ++j) zout[e0 + j] = __builtin_fmaf(d.a, G[j], ur[j]);
  } else {
    const Vec<T, P> x = load_global<Vec<T, P>>(at.src + e0);
    float z[P];
#pragma unroll
    for (int j = 0; j < P; ++j) z[j] = __builtin_fmaf(d.a, G[j], ur[j]);
    apply_z<T, P, MODE>(at, a, e0, x, z, c);
  }
}

// Lane layout: column group cg = lane % 32 owns P consecutive columns, each half of a wave RPL consecutive rows (a lane makes one
// Philox call per row).  RPL = 16 is for passes that fill the chip; RPL = 1 spreads a small model's matrices over sixteen times the
// blocks (least-squares layer of 256 x 512: 17 us with 8 blocks of 128 rows, 5.3 with 128 blocks of 8).
// The share of block `block` of `nblk`; the table, at smem, is on its way into LDS.
template <typename T, int P, bool WRITE_Z, int MODE, int RPL>
__device__ __forceinline__ void tile_share(const PerturbArgs& a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items, float c, float* smem, float* __restrict__ zout, int kp,
                                           int block, int nblk) {
  const RadiusEntry* tab = reinterpret_cast<const RadiusEntry*>(smem);
  constexpr int TR = 8 * RPL;                        // rows a block covers at a time
  float* Us = smem + kRadiusTabEntries * 3;          // [TR][kp]
  float* Rs = Us + TR * kp;                          // [kp][TC]
  constexpr int TC = 32 * P;
  constexpr int RB = RPL < 8 ? RPL : (P == 4 ? 16 : 8);   // rows a lane holds at once
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cg = lane & 31, rh = lane >> 5;

  // A block takes a contiguous run of the list; the list orders the row tiles of one column strip one after the
  // other, so the slice of R in LDS is regenerated only when the strip (or the tensor) changes.
  const int per_block = (a.n_tiles + nblk - 1) / nblk;
  const int w_end = min(a.n_tiles, (block + 1) * per_block);
  int prev_tensor = -1;
  int64_t prev_col0 = -1;
  for (int w = block * per_block; w < w_end; ++w) {
    const WorkItem it = items[w];
    const TensorDesc d = descs[it.tensor];
    const int64_t row0 = it.first >> 32, col0 = it.first & 0xFFFFFFFFll;
    const int nrows = it.count, k = d.k, kpt = (k + 7) & ~7;
    const Places<T> at = places_of<T, MODE>(d, a);
    const bool same_strip = it.tensor == prev_tensor && col0 == prev_col0;
    prev_tensor = it.tensor; prev_col0 = col0;
    if (!same_strip) __syncthreads();                // table loaded / previous strip's readers of Rs done
    // this strip's slice of b*R: rows l < k, columns col0 .. col0+TC
    for (int idx = tid; idx < (same_strip ? 0 : kpt * 32); idx += 256) {
      const int l = idx >> 5, g = idx & 31;
      const int64_t col = col0 + (int64_t)g * P;
      float r[P];
#pragma unroll
      for (int j = 0; j < P; ++j) r[j] = 0.f;
      if (l < k && col < d.cols) {
        const uint64_t q = (uint64_t)((int64_t)l * d.cols + col) / P;
        draw<P, MODE>(q, d.id | 0x80000000u, a, tab, r);
#pragma unroll
        for (int j = 0; j < P; ++j) r[j] *= d.b;
      }
#pragma unroll
      for (int j = 0; j < P; ++j) Rs[l * TC + g * P + j] = r[j];
    }
    for (int r0 = 0; r0 < nrows; r0 += TR) {
      __syncthreads();                               // Rs written / previous row block's readers of Us done
      for (int idx = tid; idx < TR * kpt; idx += 256) {
        const int r = idx / kpt, l = idx - r * kpt;
        const int64_t row = row0 + r0 + r;
        Us[r * kp + l] = (l < k && r0 + r < nrows && row < d.rows) ? basis_at(d, row, l) : 0.f;
      }
      __syncthreads();
      const int64_t col = col0 + (int64_t)cg * P;
#pragma unroll 1
      for (int vb = 0; vb < RPL; vb += RB) {
        float acc[RB][P];
#pragma unroll
        for (int v = 0; v < RB; ++v)
#pragma unroll
          for (int j = 0; j < P; ++j) acc[v][j] = 0.f;
        for (int l0 = 0; l0 < kpt; l0 += 8) {
          float Rreg[8][P];
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < P; ++j) Rreg[i][j] = Rs[(l0 + i) * TC + cg * P + j];
#pragma unroll
          for (int v = 0; v < RB; ++v) {
            const int vv = vb + v;
            const int rloc = (2 * wave + rh) * RPL + vv;
            const float* u = Us + rloc * kp + l0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const float ui = u[i];
#pragma unroll
              for (int j = 0; j < P; ++j) acc[v][j] = __builtin_fmaf(ui, Rreg[i][j], acc[v][j]);
            }
          }
        }
        if (col < d.cols) {
#pragma unroll
          for (int v = 0; v < RB; ++v) {
            const int vv = vb + v;
            const int rloc = (2 * wave + rh) * RPL + vv;
            const int64_t row = row0 + r0 + rloc;
            if (r0 + rloc < nrows && row < d.rows) finish_row<T, P, WRITE_Z, MODE>(d, at, zout, row * d.cols + col, acc[v], c, a, tab);
          }
        }
      }
    }
  }
}
template <typename T, int P, bool WRITE_Z, int MODE, int RPL>
__global__ void __launch_bounds__(256) perturb_tile_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items,
                                                           float c, const RadiusEntry* __restrict__ gtab, float* __restrict__ zout, int kp) {
  extern __shared__ float smem[];
  const int nblk = (int)gridDim.x - a.pull_blocks;               // computing blocks
  if ((int)blockIdx.x >= nblk) { pull_next_stage(a, (int)blockIdx.x - nblk, a.pull_blocks); return; }
  load_radius_table(reinterpret_cast<RadiusEntry*>(smem), gtab);
  tile_share<T, P, WRITE_Z, MODE, RPL>(a, descs, items, c, smem, zout, kp, (int)blockIdx.x, nblk);
}

// ------------------------------------------------------------------ tile, U R on the matrix cores (k >= 16)
// v_mfma_f32_16x16x32_bf16 on the operands' planes (planes.h).  A wave covers 16 rows x 32P columns of a tile: lane (n = lane % 16,
// rg = lane / 16) ends up with rows 4 rg + v (v = 0..3) and, in each of the two column groups g, the P consecutive columns
// g*16P + P n + j -- one Philox call per (row, group) -- so Z never leaves registers.  Eight tiles of 16 columns are contracted at a time, both
// groups with P = 4, one after the other with P = 8: 32 accumulators.  The lane feeds row n of the wave's slab: eight consecutive entries of U,
// cut into planes once for the eight tiles.
// The strip's slice of b R waits in LDS as planes: [plane][l / 8][column], 16 bytes of eight l each, the columns of a tile next to each other.
// Instructions of a tile: six per 32 terms; 16 terms (or what is left of that many) take three, their six products side by side along
// the instruction's index (the half-waves rg < 2 and rg >= 2 hold different planes).
// Bound by the generator's vector instructions where one result is written (1.2e9 bf16 entries of rank 16 in 1.45 ms, 3.3 TB/s; four perturbations at
// once 4.54 ms), by writes where three are (2.2 ms, 4.4 TB/s).  On v_mfma_f32_16x16x4f32, whose 32 (rank 32: 64) cycles per four terms the vector
// instructions do not hide, with four waves to a radius table and theta requested one vector ahead, the same passes took 1.49, 4.6 and 2.3 ms, and
// 302e6 entries of rank 32 487 and 660 us, now 382 and 534.  Z is off from fp64 by 0.7e-7 of its norm at rank 16, 1.1e-7 at 64 (1.0 and 1.6e-7
// with the fp32 instruction).  Entries of U that planes don't hold (infinite, too large for bf16, or so small that their last plane is subnormal) send their wave
// to the fp32 instruction, and so do sums of perturbations with coefficients so far from 1 that planes don't hold R.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTilePasses = 3;      // runs of the tile list per block of the matrix-core kernel
constexpr int kTileWaves = 8;       // of 16 rows each, a tile's: one radius table and one slice of R serve them all
static_assert(16 * kTileWaves == kTileRowsPerIter, "a wave has one slab of a tile");

__device__ __forceinline__ f32x4 mfma_planes(planes_u32x4 x, planes_u32x4 y, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(planes_bf16x8, x), __builtin_bit_cast(planes_bf16x8, y), c, 0, 0, 0);
}
__device__ __forceinline__ void in_this_order() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// One entry of the tile list, and where a lane's row of U and its part of theta start (rows and columns past the end: the last ones).
struct Tile {
  TensorDesc d;
  int64_t row0, col0;
  int nrows, n8;            // n8: eights of the rank
  bool eights;              // the rank is a multiple of 8: rows of U are read eight entries at a time
};
__device__ __forceinline__ Tile tile_of(const TensorDesc* descs, const WorkItem* items, int w) {
  const WorkItem it = load_const(items + w);
  Tile t;
  t.d = load_const(descs + it.tensor);
  t.row0 = it.first >> 32; t.col0 = it.first & 0xFFFFFFFFll;
  t.nrows = it.count; t.n8 = (t.d.k + 7) >> 3; t.eights = (t.d.k & 7) == 0;
  return t;
}

// Eight entries of a lane's row of U as they lie: fp32 (16-byte loads aligned to 4) or 4-bit codes (one load of 4 bytes aligned to 1).
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_a1 __attribute__((aligned(1)));
struct RawEight { uint32_t w[8]; };
__device__ __forceinline__ void request_eight(const TensorDesc& d, int64_t row, int c8, RawEight& o) {
  if (d.Uq) {
    typedef const u32_a1 __attribute__((address_space(1))) GW;
    o.w[0] = *reinterpret_cast<GW*>(reinterpret_cast<uintptr_t>(d.Uq + row * d.ldu + 4 * c8));
  } else {
    typedef const u32x4_a4 __attribute__((address_space(1))) GV;
    GV* p = reinterpret_cast<GV*>(reinterpret_cast<uintptr_t>(d.U + row * d.ldu + 8 * c8));
    const planes_u32x4 lo = p[0], hi = p[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) { o.w[i] = lo[i]; o.w[4 + i] = hi[i]; }
  }
}
__device__ __forceinline__ void eight_of(const TensorDesc& d, const RawEight& r, float (&u)[8]) {
  if (d.Uq) {
    const uint32_t w = r.w[0];
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = d.qlambda * ((float)((w >> (4 * i)) & 15u) - d.qdelta);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = __uint_as_float(r.w[i]);
  }
}

// acc[t] = U R for the wave's 16 rows and the 16 columns of tile t, eight tiles from R's entries at Rs on; `first` holds the lane's first eight where t.eights.
// extreme: planes don't hold R.
template <int P>
__device__ __forceinline__ void contract(const Tile& tl, const RawEight& first, const planes_u32x4* Rs, bool extreme, int64_t urow, int n16, int rg, f32x4 (&acc)[8]) {
  constexpr int TC = 32 * P;
  const int n8 = tl.n8, plane = n8 * TC;                      // 16-byte entries of a plane of R
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bool held = true;
  auto cut_u = [&](int l8, int c8, bool in, PlanesOf<3>& o) {
    float u[8];
    if (tl.eights) {
      RawEight r = first;
      if (l8 > 0) request_eight(tl.d, urow, c8, r);
      eight_of(tl.d, r, u);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] = 8 * c8 + i < tl.d.k ? basis_at(tl.d, urow, 8 * c8 + i) : 0.f;
    }
    // Three planes hold a number that does not round up to infinity and whose last place is a normal number (2^-103 and above), and zero: twice its bits less those of
    // 2^-103 wrap round below that, zero least.
    constexpr uint32_t least = 24u << 24;
    float most = 0.f;
    uint32_t wrapped = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      u[2 * w] = in ? u[2 * w] : 0.f; u[2 * w + 1] = in ? u[2 * w + 1] : 0.f;         // past the end: zeros times R's last eight
      cut_pair_rounded(u[2 * w], u[2 * w + 1], w, o);
      most = fmaxf(fmaxf(most, __builtin_fabsf(u[2 * w])), __builtin_fabsf(u[2 * w + 1]));
      wrapped = max(wrapped, max((__float_as_uint(u[2 * w]) << 1) - least, (__float_as_uint(u[2 * w + 1]) << 1) - least));
    }
    held &= (most <= 0x1.fefffep127f) & (wrapped <= 0u - least);
  };
  PlanesOf<3> pu;
  int l8 = 0;
  for (; n8 - l8 > 2; l8 += 4) {                              // 32 terms
    const bool in = l8 + rg < n8;
    const int c8 = in ? l8 + rg : n8 - 1;
    cut_u(l8, c8, in, pu);
    const planes_u32x4* r = Rs + c8 * TC + n16;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const planes_u32x4 q[3] = {r[16 * t], r[plane + 16 * t], r[2 * plane + 16 * t]};
      for_terms<3, 3>([&](int x, int y) { acc[t] = mfma_planes(pu.p[x], q[y], acc[t]); });
      if (t & 1) in_this_order();                             // the operands of two tiles at a time: those of all would take 96 registers
    }
  }
  if (l8 < n8) {                                              // 16, or 8
    const bool low = rg < 2, in = l8 + (rg & 1) < n8;
    const int c8 = in ? l8 + (rg & 1) : n8 - 1;
    cut_u(l8, c8, in, pu);
#pragma unroll
    for (int w = 0; w < 4; ++w) pu.p[2][w] = low ? pu.p[2][w] : pu.p[0][w];
    const planes_u32x4* r = Rs + c8 * TC + n16;
    const planes_u32x4* ra = r + (low ? 0 : 2 * plane);       // U2 R0 and U0 R2
    const planes_u32x4* rb = r + (low ? plane : 0);           // U1 R1 and U1 R0, then U0 R1 and U0 R0
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const planes_u32x4 b = rb[16 * t];
      acc[t] = mfma_planes(pu.p[2], ra[16 * t], acc[t]);
      acc[t] = mfma_planes(pu.p[1], b, acc[t]);
      acc[t] = mfma_planes(pu.p[0], b, acc[t]);
      if (t & 1) in_this_order();
    }
  }
  if (__builtin_expect(extreme || __ballot(!held) != 0, 0)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t* r = reinterpret_cast<const uint16_t*>(Rs);
#pragma unroll 1
    for (int l = rg; l < 8 * n8; l += 4) {
      const float u = l < tl.d.k ? basis_at(tl.d, urow, l) : 0.f;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int e = ((l >> 3) * TC + 16 * t + n16) * 8 + (l & 7);
        const float x = low_float(r[e]) + (low_float(r[e + 8 * plane]) + low_float(r[e + 16 * plane]));
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(u, x, acc[t], 0, 0, 0);
        in_this_order();
      }
    }
  }
}

// What a lane requests is used one round of calls later: kAhead vectors of theta (and, with a tile's last ones, the next tile's U) are under way while
// those before them are worked on.  Requested one vector and one call ahead, the pass ran at the latency of the loads: a wait covers every load
// and store issued before it, and some 10 KB in flight per compute unit are half of what HBM needs at this rate.
template <typename T, int P> constexpr int vectors_ahead() { return 64 / (int)(sizeof(T) * P); }      // 16 registers

// The share of block `block` of `nblk`; the table, at smem, is on its way into LDS.  WHOLE: every tile has rows for every wave; looking after waves without costs 2 % of an in-place
// pass (1.2e9 bf16 entries of rank 16: 1.63 ms -> 1.66), in scalar registers that spill.
template <typename T, int P, bool WRITE_Z, int MODE, bool WHOLE>
__device__ __forceinline__ void tile_mfma_share(const PerturbArgs& a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items, float c, float* smem, float* __restrict__ zout,
                                                int block, int nblk) {
  const RadiusEntry* tab = reinterpret_cast<const RadiusEntry*>(smem);
  planes_u32x4* Rs = reinterpret_cast<planes_u32x4*>(smem + kRadiusTabEntries * 3);      // [3][kp / 8][TC]
  constexpr int TC = 32 * P, GC = 16 * P;            // tile columns, columns per group
  constexpr int kAhead = vectors_ahead<T, P>(), kRounds = 8 / kAhead, kGroups = 8 / P;      // kGroups: column groups contracted at a time
  // the row and the column group of a lane's vector number i
  auto row_of = [](int i) { return kGroups == 2 ? i >> 1 : i & 3; };
  auto group_of = [](int i) { return kGroups == 2 ? i & 1 : i >> 2; };
#if defined(__HIP_DEVICE_COMPILE__)
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#else
  const int wave = (int)threadIdx.x >> 6;
#endif
  const int tid = threadIdx.x, lane = tid & 63;
  const int n16 = lane & 15, rg = lane >> 4;
  // Every block takes kTilePasses contiguous runs of the list; the R slice is regenerated only when the column strip
  // changes (see above).  Consecutive block ids go round-robin to the 8 XCDs, so the list is cut into 8 chunks, one
  // per XCD, and in pass i the blocks q = 0, 1, ... of an XCD take the neighbouring runs i n + q of its chunk: at any
  // time the blocks of one XCD work on neighbouring column strips of the same few matrices, walk the same rows and
  // find each other's rows of U in their common L2, and a block's next run lies in other matrices.
  const bool by_xcd = (nblk & 7) == 0;
  // (a run shorter than a strip of a 2048-row matrix, 16 tiles, would only regenerate R slices more often: short
  // launches, e.g. one pipeline stage of streamed bases, take fewer runs per block)
  const int by_len = a.n_tiles / (nblk * 16);
  const int n_pass = !by_xcd || by_len < 1 ? 1 : (by_len < kTilePasses ? by_len : kTilePasses);
  const int per_xcd = nblk >> 3;
  const int64_t n_runs = (int64_t)nblk * n_pass;          // run r is tiles [r n / R, (r + 1) n / R): lengths differ by at most one
  int pass = -1, w = 0, w_end = 0;
  auto advance = [&]() {                             // the block's next tile; false behind the last one
    if (w + 1 < w_end) { ++w; return true; }
    while (++pass < n_pass) {
      const int run = by_xcd ? ((block & 7) * n_pass + pass) * per_xcd + (block >> 3) : block;
      if (n_runs == a.n_tiles) { w = run; w_end = run + 1; return true; }
      w = (int)((int64_t)run * a.n_tiles / n_runs);
      w_end = (int)(((int64_t)run + 1) * a.n_tiles / n_runs);
      if (w < w_end) return true;
    }
    return false;
  };
  // A wave without rows of a tile (a matrix's last tile, the tiles of a model of few) contracts nothing, and no lane reads theta that another wave may be
  // storing: a row or column past the tile is read as the wave's own last one, that of a wave without any, or behind the last tile, as the descriptor
  // table (in bounds, never used; a conditional request takes registers for old and new values behind it, which then spill).
  auto has_rows = [&](const Tile& t) { return 16 * wave < t.nrows; };
  auto u_row = [&](const Tile& t) { const int r = 16 * wave + n16; return t.row0 + (r < t.nrows ? r : t.nrows - 1); };
  auto request_u = [&](const Tile& t, RawEight& o) {
    if (!t.eights) return;
    const int c8 = t.n8 > 2 ? rg : rg & 1;
    request_eight(t.d, u_row(t), c8 < t.n8 ? c8 : t.n8 - 1, o);
  };
  auto request = [&](const Tile& t, int round, Vec<T, P>* buf, bool more) {
    if (WRITE_Z) return;
    const bool own = WHOLE || (more && has_rows(t));
    const T* src = own ? places_of<T, MODE>(t.d, a).src + (t.row0 * t.d.cols + t.col0) : reinterpret_cast<const T*>(descs);
    const int64_t cols_left = t.d.cols - t.col0;
    const uint32_t last_row = own ? (uint32_t)t.nrows - 1 : 0, last_col = !own ? 0 : cols_left < TC ? (uint32_t)cols_left - P : TC - P;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int v = row_of(round * kAhead + i), g = group_of(round * kAhead + i);
      uint32_t r = 16 * wave + 4 * rg + v, k = g * GC + P * n16;
      r = r < last_row ? r : last_row; k = k < last_col ? k : last_col;
      buf[i] = load_global<Vec<T, P>>(src + ((uint64_t)r * (uint32_t)t.d.cols + k));
    }
  };
  if (!advance()) return;                            // uniform over the block: no barrier follows
  Tile t = tile_of(descs, items, w);
  Vec<T, P> cur[kAhead], nxt[kAhead];
  RawEight u8{};
  request(t, 0, cur, true);
  request_u(t, u8);
  int prev_tensor = -1;
  int64_t prev_col0 = -1;
  for (bool more = true; more;) {
    const int tensor = load_const(items + w).tensor;
    const bool same_strip = tensor == prev_tensor && t.col0 == prev_col0;
    prev_tensor = tensor; prev_col0 = t.col0;
    if (!same_strip) {
      const int kpt = 8 * t.n8;
      __syncthreads();                               // table loaded / previous strip's readers of Rs done
      for (int idx = tid; idx < kpt * 32; idx += 64 * kTileWaves) {
        const int l = idx >> 5, g = idx & 31;
        const int64_t col = t.col0 + (int64_t)g * P;
        float r[P];
#pragma unroll
        for (int j = 0; j < P; ++j) r[j] = 0.f;
        if (l < t.d.k && col < t.d.cols) {
          draw<P, MODE>((uint64_t)((int64_t)l * t.d.cols + col) / P, t.d.id | 0x80000000u, a, tab, r);
#pragma unroll
          for (int j = 0; j < P; ++j) r[j] *= t.d.b;
        }
        // column g P + j is column n = g % 16 of tile j of its group: entry 16 tile + n
        uint16_t* o = reinterpret_cast<uint16_t*>(Rs + (l >> 3) * TC + (g >> 4) * 16 * P + (g & 15)) + (l & 7);
#pragma unroll
        for (int j = 0; j < P; j += 2) {
          PlanesOf<3> q;
          cut_pair_rounded(r[j], r[j + 1], 0, q);
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            o[x * t.n8 * TC * 8 + 128 * j] = (uint16_t)q.p[x][0];
            o[x * t.n8 * TC * 8 + 128 * (j + 1)] = (uint16_t)(q.p[x][0] >> 16);
          }
        }
      }
      __syncthreads();
    }
    f32x4 acc[8];
    const Places<T> at = places_of<T, MODE>(t.d, a);
    const int rbase = 16 * wave + 4 * rg;            // first of this lane's 4 rows (tile-relative)
    const int64_t origin = t.row0 * t.d.cols + t.col0, ebase = origin + (int64_t)rbase * t.d.cols + (int64_t)P * n16;
    // the calls' counters share their upper word in all but the tile that crosses 2^32 calls
    const uint32_t q_hi = (uint32_t)((uint64_t)origin / P >> 32);
    const bool full = 16 * wave + 16 <= t.nrows && t.row0 + t.nrows <= t.d.rows && t.col0 + TC <= t.d.cols &&
                      q_hi == (uint32_t)((uint64_t)(origin + (int64_t)(t.nrows - 1) * t.d.cols + TC - 1) / P >> 32);
    const bool any = WHOLE || 16 * wave < t.nrows;
    const int nrows = t.nrows;
    const TensorDesc d = t.d;
    const int64_t row0 = t.row0, col0 = t.col0;
    const uint32_t q0 = (uint32_t)((uint64_t)ebase / P), q_row = (uint32_t)((uint64_t)d.cols / P);
    auto z_of = [&](int v, int g, float* z) {
#pragma unroll
      for (int j = 0; j < P; ++j) z[j] = __builtin_fmaf(d.a, z[j], acc[(g % kGroups) * P + j][v]);
    };
#pragma unroll
    for (int round = 0; round < kRounds; ++round) {
      const bool last = round + 1 == kRounds;
      if (round * kAhead % (4 * kGroups) == 0 && any) contract<P>(t, u8, Rs + group_of(round * kAhead) * GC, MODE == kBatch && a.extreme, u_row(t), n16, rg, acc);
      if (last) {
        more = advance();
        if (more) t = tile_of(descs, items, w);
        request_u(t, u8);                            // behind the last tile it is requested again
      }
      request(t, last ? 0 : round + 1, nxt, !last || more);
      in_this_order();
      auto arrived = [&]() {                         // all that was requested, in front of the round's last store
        if (WRITE_Z) return;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) wait_here_for(nxt[i]);
        if (last) wait_here_for(u8);
      };
      if (full) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
          const int v = row_of(round * kAhead + i), g = group_of(round * kAhead + i);
          float z[P];
          draw<P, MODE>(q0 + (uint32_t)v * q_row + 16u * g, q_hi, d.id, a, tab, z);
          z_of(v, g, z);
          const int64_t e0 = ebase + (int64_t)v * d.cols + g * GC;
          if (i + 1 == kAhead) arrived();
          if (WRITE_Z) {
#pragma unroll
            for (int j = 0; j < P; ++j) zout[e0 + j] = z[j];
          } else {
            apply_z<T, P, MODE>(at, a, e0, cur[i], z, c);
          }
        }
      } else {
        arrived();
        if (any) {
#pragma unroll
          for (int i = 0; i < kAhead; ++i) {
            const int v = row_of(round * kAhead + i), g = group_of(round * kAhead + i);
            if (rbase + v >= nrows || row0 + rbase + v >= d.rows || col0 + g * GC + P * n16 >= d.cols) continue;
            const int64_t e0 = ebase + (int64_t)v * d.cols + g * GC;
            float z[P];
            draw<P, MODE>((uint64_t)e0 / P, d.id, a, tab, z);
            z_of(v, g, z);
            if (WRITE_Z) {
#pragma unroll
              for (int j = 0; j < P; ++j) zout[e0 + j] = z[j];
            } else {
              apply_z<T, P, MODE>(at, a, e0, cur[i], z, c);
            }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < kAhead; ++i) cur[i] = nxt[i];
    }
  }
}
template <typename T, int P, bool WRITE_Z, int MODE, bool WHOLE>
__global__ void __launch_bounds__(64 * kTileWaves) __attribute__((amdgpu_waves_per_eu(4, 8))) perturb_tile_mfma_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ items,
                                                                float c, const RadiusEntry* __restrict__ gtab, float* __restrict__ zout) {
  extern __shared__ float smem[];
  const int nblk = (int)gridDim.x - a.pull_blocks;               // computing blocks
  if ((int)blockIdx.x >= nblk) { pull_next_stage(a, (int)blockIdx.x - nblk, a.pull_blocks); return; }
  load_radius_table<64 * kTileWaves>(reinterpret_cast<RadiusEntry*>(smem), gtab);
  tile_mfma_share<T, P, WRITE_Z, MODE, WHOLE>(a, descs, items, c, smem, zout, (int)blockIdx.x, nblk);
}

// ------------------------------------------------------------------ a small model's two lists in one launch
// A block per entry, those of the flat list first (four waves of a block work on them): with so few the launches are latency.  One pass over a model of two blocks
// of 128 columns 10.3 us (fp32, rank 8) and 14.5 (bf16, rank 16) in two launches, 5.5 and 9.1 in one; four blocks of 256 columns, rank 16 19.9 and 13.3.
template <typename T, int P, int MODE>
__global__ void __launch_bounds__(256) perturb_small_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ flat, const WorkItem* __restrict__ tiles,
                                                            float c, const RadiusEntry* __restrict__ gtab, int kp) {
  extern __shared__ float smem[];
  load_radius_table(reinterpret_cast<RadiusEntry*>(smem), gtab);
  if ((int)blockIdx.x < a.n_flat) {
    __syncthreads();
    flat_share<T, P, MODE>(a, descs, flat, c, reinterpret_cast<const RadiusEntry*>(smem), (int)blockIdx.x, a.n_flat);
  } else {
    tile_share<T, P, false, MODE, kSmallTileRows / 8>(a, descs, tiles, c, smem, nullptr, kp, (int)blockIdx.x - a.n_flat, a.n_tiles);
  }
}
template <typename T, int P, int MODE>
__global__ void __launch_bounds__(64 * kTileWaves) __attribute__((amdgpu_waves_per_eu(4, 8))) perturb_small_mfma_kernel(PerturbArgs a, const TensorDesc* __restrict__ descs, const WorkItem* __restrict__ flat,
                                                                                                                        const WorkItem* __restrict__ tiles, float c, const RadiusEntry* __restrict__ gtab, int) {
  extern __shared__ float smem[];
  load_radius_table<64 * kTileWaves>(reinterpret_cast<RadiusEntry*>(smem), gtab);
  if ((int)blockIdx.x < a.n_flat) {
    __syncthreads();
    if (threadIdx.x < 256) flat_share<T, P, MODE>(a, descs, flat, c, reinterpret_cast<const RadiusEntry*>(smem), (int)blockIdx.x, a.n_flat);
  } else {
    tile_mfma_share<T, P, false, MODE, false>(a, descs, tiles, c, smem, nullptr, (int)blockIdx.x - a.n_flat, a.n_tiles);
  }
}

// ------------------------------------------------------------------ affine quantiser of a basis (cloud side of Sec. 3.4)
// min / max as order-preserving integers, so that integer atomics reduce them
__device__ __forceinline__ int32_t float_order(float x) { const int32_t b = __float_as_int(x); return b >= 0 ? b : (int32_t)(0x80000000u - (uint32_t)b); }
__device__ __forceinline__ float order_float(int32_t o) { return __int_as_float(o >= 0 ? o : (int32_t)(0x80000000u - (uint32_t)o)); }

__global__ void basis_minmax_init_kernel(int32_t* mm) { mm[0] = 0x7FFFFFFF; mm[1] = (int32_t)0x80000000; }
__global__ void __launch_bounds__(256) basis_minmax_kernel(const float* __restrict__ U, int64_t rows, int k, int ldu, int32_t* __restrict__ mm) {
  int32_t lo = 0x7FFFFFFF, hi = (int32_t)0x80000000;
  const int64_t n = rows * k;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int32_t o = float_order(U[(i / k) * ldu + (i % k)]);
    lo = o < lo ? o : lo; hi = o > hi ? o : hi;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const int32_t l2 = __shfl_xor(lo, off, 64), h2 = __shfl_xor(hi, off, 64);
    lo = l2 < lo ? l2 : lo; hi = h2 > hi ? h2 : hi;
  }
  if ((threadIdx.x & 63) == 0) { atomicMin(mm, lo); atomicMax(mm + 1, hi); }
}
__global__ void basis_minmax_finish_kernel(int32_t* mm) {
  float* f = reinterpret_cast<float*>(mm);
  const float lo = order_float(mm[0]), hi = order_float(mm[1]);
  f[0] = lo; f[1] = hi;
}
// one thread per output byte: codes of elements 2j and 2j + 1 of a row, round(x / lambda + delta) clipped to [0, 15]
__global__ void __launch_bounds__(256) basis_quantize_kernel(const float* __restrict__ U, int64_t rows, int k, int ldu, float lambda, float delta,
                                                             uint8_t* __restrict__ Uq, int ldq) {
#pragma clang fp contract(off)   // x / lambda is rounded before delta is added, as the definition has it
  const int kb = (k + 1) >> 1;
  const int64_t n = rows * kb;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / kb;
    const int j = (int)(i % kb);
    uint32_t byte = 0;
    for (int h = 0; h < 2; ++h) {
      const int l = 2 * j + h;
      if (l < k) {
        const float t = U[r * ldu + l] / lambda;
        float q = __builtin_rintf(t + delta);
        q = q < 0.f ? 0.f : (q > 15.f ? 15.f : q);
        byte |= (uint32_t)q << (4 * h);
      }
    }
    Uq[r * ldq + j] = (uint8_t)byte;
  }
}

// ------------------------------------------------------------------ debug kernels
__global__ void debug_philox_kernel(const uint32_t* __restrict__ ctr, uint32_t k0, uint32_t k1, uint32_t* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const u32x4 r = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
  out[4 * i] = r.x; out[4 * i + 1] = r.y; out[4 * i + 2] = r.z; out[4 * i + 3] = r.w;
}

template <int P>
__global__ void __launch_bounds__(256) debug_gauss_kernel(uint32_t k0, uint32_t k1, uint32_t step, uint32_t id_stream, int64_t first,
                                                          int64_t n, const RadiusEntry* __restrict__ gtab, float* __restrict__ out) {
  __shared__ RadiusEntry tab[kRadiusTabEntries];
  load_radius_table(tab, gtab);
  __syncthreads();
  const int64_t q0 = first / P, q1 = (first + n + P - 1) / P;
  for (int64_t q = q0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < q1; q += (int64_t)gridDim.x * blockDim.x) {
    float G[P];
    gaussP<P>(philox_call((uint64_t)q, id_stream, step, k0, k1), tab, G);
    for (int j = 0; j < P; ++j) {
      const int64_t e = q * P + j;
      if (e >= first && e < first + n) out[e - first] = G[j];
    }
  }
}

// all radius uniforms: bits=32: N = 2n+1, n < 2^23; bits=16: N = (2h+1) << 7, h < 2^16
__global__ void __launch_bounds__(256) debug_radius_kernel(int bits, const RadiusEntry* __restrict__ gtab, float* __restrict__ out) {
  __shared__ RadiusEntry tab[kRadiusTabEntries];
  load_radius_table(tab, gtab);
  __syncthreads();
  const uint32_t total = bits == 32 ? (1u << 23) : (1u << 16);
  for (uint32_t n = blockIdx.x * blockDim.x + threadIdx.x; n < total; n += gridDim.x * blockDim.x) {
    const uint32_t N = bits == 32 ? ((n << 1) | 1u) : (((n << 1) | 1u) << 7);
    out[n] = radius_from_odd24(N << 8, tab);
  }
}

__global__ void __launch_bounds__(256) debug_cossin_kernel(int bits, float* __restrict__ co, float* __restrict__ so) {
  const uint32_t total = bits == 32 ? (1u << 24) : (1u << 16);
  for (uint32_t n = blockIdx.x * blockDim.x + threadIdx.x; n < total; n += gridDim.x * blockDim.x) {
    const uint32_t m = bits == 32 ? n : (n << 8);
    // the fused kernel multiplies (hi, lo) by the radius; with radius 1 the product is the rounded sum
    times_radius(trig_from_u24(m << 8), 1.0f, co[n], so[n]);
  }
}

__global__ void __launch_bounds__(256) copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

// The table lives in static device memory: the library allocates nothing.
__device__ __align__(16) RadiusEntry g_radius_table[kRadiusTabEntries];

}  // namespace

hipError_t ensure_radius_table(const RadiusEntry** dev_ptr, hipStream_t s) {
  static std::mutex mu;
  static const RadiusEntry* cached[64] = {};
  static RadiusEntry host[kRadiusTabEntries];
  static bool host_ready = false;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!cached[dev]) {
    if (!host_ready) {
      for (int E = 0; E < 24; ++E)
        for (int j = 0; j < 64; ++j) {
          const double cj = __builtin_rint(128.0 / (1.0 + (j + 0.5) / 64.0)) / 128.0;
          double hl = 2.0 * __builtin_log(cj) + 2.0 * (24.0 - E) * 0.69314718055994530942;
          if (E == 23 && j == 63) hl = 0.0;        // c = 1/2, N c 2^-23 -> exactly -2 log1p(z)
          RadiusEntry& r = host[E * 64 + j];
          r.H = (float)hl;
          r.L = (float)(hl - (double)r.H);
          r.C = (float)__builtin_ldexp(cj, -E - 8);
        }
      host_ready = true;
    }
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_radius_table));
    if (e != hipSuccess) return e;
    // ordered with the caller's work: on its stream, complete before anything that follows this call is enqueued
    e = hipMemcpyAsync(p, host, sizeof(host), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    cached[dev] = reinterpret_cast<const RadiusEntry*>(p);
  }
  *dev_ptr = cached[dev];
  return hipSuccess;
}

namespace {
// Resident blocks per CU for a persistent kernel: the grid is sized to what the register and
// LDS budget really admits, because a block that has to wait for a slot would start its share of the work
// list only after another block has finished all of its own.
template <typename K>
int resident_blocks_per_cu(K kern, size_t dyn_lds, int cap, int threads = 256) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, threads, dyn_lds) != hipSuccess || nb < 1) nb = 1;
  return nb < cap ? nb : cap;
}

// Launch set-up of one tile-kernel variant: the dynamic-LDS limit (only ever raised, so that contexts with different
// ranks can take turns) and the occupancy at the LDS size asked for (the last answer is kept).
struct TileLaunchCache {
  size_t lds_limit = 0;       // what the kernel's attribute was last set to
  size_t lds = 0;
  int per_cu = 0;
};
template <typename K>
hipError_t tile_launch_setup(K kern, size_t lds, int threads, int cap, TileLaunchCache& cache, int* per_cu) {
  static std::mutex mu;                                  // the caches are shared by every context of the process
  std::lock_guard<std::mutex> lock(mu);
  if (lds > cache.lds_limit) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    cache.lds_limit = lds;
  }
  if (!(cache.per_cu > 0 && cache.lds == lds)) {
    cache.lds = lds;
    cache.per_cu = resident_blocks_per_cu(kern, lds, cap, threads);
  }
  *per_cu = cache.per_cu;
  return hipSuccess;
}

// Grid of a persistent launch: as many computing blocks as there are items, at most the resident capacity, the
// last kPullBlocks of that capacity set aside for pulling the next stage's bases when there are any to pull.
int split_grid(PerturbArgs& a, int items, int capacity) {
  a.pull_blocks = a.n_stage > 0 ? kPullBlocks : 0;
  int compute = capacity - a.pull_blocks;
  if (compute < 1) compute = 1;
  if (compute > items) compute = items;
  return compute + a.pull_blocks;
}

// Whether planes (planes.h) may not hold the entries of b R that a sum of perturbations with these coefficients draws: Gaussians are within 2^-35 and 2^3 of 1 (and all but one in 2^15
// above 2^-15), b within 2^-31 and 2^16.
bool extreme_coefficients(const PerturbArgs& a) {
  float largest = 0.f;
  for (int i = 0; i < a.n_q; ++i) largest = std::max(largest, std::fabs(a.qcoef[i]));
  return largest != 0.f && !(largest >= 0x1p-57f && largest <= 0x1p100f);
}

int mode_of(const PerturbArgs& a) { return a.n_q > 0 ? kBatch : (a.spread ? kSpread : kOne); }

template <typename T, int P>
hipError_t launch_flat_t(const PerturbArgs& a_in, float c, float* zout, hipStream_t s, int n_cu, const RadiusEntry* tab) {
  PerturbArgs a = a_in;
  if (zout) {
    const int grid = a.n_flat < n_cu * 8 ? a.n_flat : n_cu * 8;
    hipLaunchKernelGGL((fill_flat_kernel<T, P>), dim3(grid), dim3(256), 0, s, a, a.descs, a.flat, tab, zout);
    return hipGetLastError();
  }
  const int mode = mode_of(a);
  auto kern = mode == kBatch ? perturb_flat_kernel<T, P, kBatch> : (mode == kSpread ? perturb_flat_kernel<T, P, kSpread> : perturb_flat_kernel<T, P, kOne>);
  static std::atomic<int> per[3];                        // zero-initialised; racing threads compute the same value
  std::atomic<int>& slot = per[mode];
  int nb = slot.load(std::memory_order_relaxed);
  if (nb == 0) { nb = resident_blocks_per_cu(kern, 0, 8); slot.store(nb, std::memory_order_relaxed); }
  const int grid = split_grid(a, a.n_flat, n_cu * nb);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, s, a, a.descs, a.flat, c, tab);
  return hipGetLastError();
}
template <typename T, int P>
hipError_t launch_tile_t(const PerturbArgs& a_in, float c, float* zout, hipStream_t s, int n_cu, const RadiusEntry* tab) {
  PerturbArgs a = a_in;
  const int kp = (a.max_k + 7) & ~7;
  a.extreme = extreme_coefficients(a);
  if (a.min_k >= kMfmaMinK) {
    const size_t lds_m = sizeof(RadiusEntry) * (size_t)kRadiusTabEntries + 6 * (size_t)kp * 32 * P;      // three planes of two bytes
    const int variant = zout ? 3 : mode_of(a);
    const bool whole = a.whole != 0;
    decltype(&perturb_tile_mfma_kernel<T, P, false, kOne, false>) km = perturb_tile_mfma_kernel<T, P, true, kOne, false>;
    switch (variant) {
      case kOne:    km = whole ? perturb_tile_mfma_kernel<T, P, false, kOne, true> : perturb_tile_mfma_kernel<T, P, false, kOne, false>; break;
      case kBatch:  km = whole ? perturb_tile_mfma_kernel<T, P, false, kBatch, true> : perturb_tile_mfma_kernel<T, P, false, kBatch, false>; break;
      case kSpread: km = whole ? perturb_tile_mfma_kernel<T, P, false, kSpread, true> : perturb_tile_mfma_kernel<T, P, false, kSpread, false>; break;
    }
    static TileLaunchCache cache_m[8];
    int per_cu = 1;
    hipError_t e = tile_launch_setup(km, lds_m, 64 * kTileWaves, 4, cache_m[variant + (whole ? 4 : 0)], &per_cu);
    if (e != hipSuccess) return e;
    const int grid_m = split_grid(a, a.n_tiles, n_cu * per_cu);
    hipLaunchKernelGGL(km, dim3(grid_m), dim3(64 * kTileWaves), lds_m, s, a, a.descs, a.tiles, c, tab, zout);
    return hipGetLastError();
  }
  const bool small = a.tile_rows < kTileRowsPerIter;
  const size_t lds = sizeof(float) * ((size_t)kRadiusTabEntries * 3 + (size_t)(small ? kSmallTileRows : kTileRowsPerIter) * kp + (size_t)kp * 32 * P);
  const int variant = (zout ? 3 : mode_of(a)) + (small ? 4 : 0);
  constexpr int RS = kSmallTileRows / 8, RL = kTileRowsPerIter / 8;
  decltype(&perturb_tile_kernel<T, P, false, kOne, RL>) kern = nullptr;
  switch (variant) {
    case kOne:        kern = perturb_tile_kernel<T, P, false, kOne, RL>; break;
    case kBatch:      kern = perturb_tile_kernel<T, P, false, kBatch, RL>; break;
    case kSpread:     kern = perturb_tile_kernel<T, P, false, kSpread, RL>; break;
    case 3:           kern = perturb_tile_kernel<T, P, true, kOne, RL>; break;
    case 4 + kOne:    kern = perturb_tile_kernel<T, P, false, kOne, RS>; break;
    case 4 + kBatch:  kern = perturb_tile_kernel<T, P, false, kBatch, RS>; break;
    case 4 + kSpread: kern = perturb_tile_kernel<T, P, false, kSpread, RS>; break;
    default:          kern = perturb_tile_kernel<T, P, true, kOne, RS>; break;
  }
  static TileLaunchCache cache_v[8];
  int per_cu = 1;
  hipError_t e = tile_launch_setup(kern, lds, 256, 4, cache_v[variant], &per_cu);
  if (e != hipSuccess) return e;
  const int grid = split_grid(a, a.n_tiles, n_cu * per_cu);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, s, a, a.descs, a.tiles, c, tab, zout, kp);
  return hipGetLastError();
}

// The kernel that takes both lists of `a`, and how many of its blocks a CU holds.
struct SmallKernel {
  void (*kern)(PerturbArgs, const TensorDesc*, const WorkItem*, const WorkItem*, float, const RadiusEntry*, int);
  int threads, per_cu;
  size_t lds;
};
template <typename T, int P>
hipError_t small_kernel_t(const PerturbArgs& a, SmallKernel* k) {
  const int kp = (a.max_k + 7) & ~7, mode = mode_of(a);
  const bool mfma = a.min_k >= kMfmaMinK;
  if (mfma) k->kern = mode == kBatch ? perturb_small_mfma_kernel<T, P, kBatch> : (mode == kSpread ? perturb_small_mfma_kernel<T, P, kSpread> : perturb_small_mfma_kernel<T, P, kOne>);
  else      k->kern = mode == kBatch ? perturb_small_kernel<T, P, kBatch> : (mode == kSpread ? perturb_small_kernel<T, P, kSpread> : perturb_small_kernel<T, P, kOne>);
  k->threads = mfma ? 64 * kTileWaves : 256;
  k->lds = sizeof(RadiusEntry) * (size_t)kRadiusTabEntries + (mfma ? 6 * (size_t)kp * 32 * P : sizeof(float) * ((size_t)kSmallTileRows * kp + (size_t)kp * 32 * P));
  static TileLaunchCache cache[6];
  return tile_launch_setup(k->kern, k->lds, k->threads, 2, cache[mode + (mfma ? 0 : 3)], &k->per_cu);
}
hipError_t small_kernel(const PerturbArgs& a, SmallKernel* k) { return a.dtype == 0 ? small_kernel_t<float, 4>(a, k) : small_kernel_t<bf16_t, 4>(a, k); }
}  // namespace

// A block per entry of either list, all of them resident at once and at most two a CU: what a launch of its own costs a list is then all there is to save, and a block has no
// second entry to work ahead for.  Gaussians four to a call; ranks on one side of kMfmaMinK, below it tiles of eight rows.
bool perturb_small(const PerturbArgs& a, int n_cu) {
  if (a.bits != 32 || a.n_flat <= 0 || a.n_tiles <= 0 || a.n_stage != 0 || a.n_flat + a.n_tiles > 2 * n_cu || a.max_k < 1 || a.max_k > kMaxK) return false;
  if (a.min_k < kMfmaMinK && (a.max_k >= kMfmaMinK || a.tile_rows >= kTileRowsPerIter)) return false;
  SmallKernel k;
  return small_kernel(a, &k) == hipSuccess && a.n_flat + a.n_tiles <= k.per_cu * n_cu;
}
hipError_t launch_perturb_small(const PerturbArgs& a_in, float c, hipStream_t s, int n_cu) {
  PerturbArgs a = a_in;
  a.extreme = extreme_coefficients(a);
  if (!perturb_small(a, n_cu) || a.pull_blocks != 0) return hipErrorInvalidValue;
  if (a.n_q < 0 || a.n_q > kMaxBatch || (a.spread && (a.n_q > 0 || a.from_copy)) || ((a.spread || a.from_copy) && !(a.copy[0] && a.copy[1])) || (a.from_copy && a.n_q > 0)) return hipErrorInvalidValue;
  const RadiusEntry* tab = nullptr;
  hipError_t e = ensure_radius_table(&tab, s);
  if (e != hipSuccess) return e;
  SmallKernel k;
  e = small_kernel(a, &k);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k.kern, dim3((unsigned)(a.n_flat + a.n_tiles)), dim3((unsigned)k.threads), k.lds, s, a, a.descs, a.flat, a.tiles, c, tab, (a.max_k + 7) & ~7);
  return hipGetLastError();
}

hipError_t launch_perturb_flat(const PerturbArgs& a, float c, float* zout, hipStream_t s, int n_cu) {
  if (a.n_flat <= 0) return hipSuccess;
  if (a.n_q < 0 || a.n_q > kMaxBatch || (a.n_q > 0 && zout)) return hipErrorInvalidValue;
  if ((a.spread && (a.n_q > 0 || a.from_copy || zout)) || ((a.spread || a.from_copy) && !(a.copy[0] && a.copy[1])) || (a.from_copy && a.n_q > 0)) return hipErrorInvalidValue;
  if (a.n_stage < 0 || a.n_stage > kMaxStage) return hipErrorInvalidValue;
  const RadiusEntry* tab = nullptr;
  hipError_t e = ensure_radius_table(&tab, s);
  if (e != hipSuccess) return e;
  if (a.dtype == 0) return a.bits == 32 ? launch_flat_t<float, 4>(a, c, zout, s, n_cu, tab) : launch_flat_t<float, 8>(a, c, zout, s, n_cu, tab);
  return a.bits == 32 ? launch_flat_t<bf16_t, 4>(a, c, zout, s, n_cu, tab) : launch_flat_t<bf16_t, 8>(a, c, zout, s, n_cu, tab);
}

hipError_t launch_perturb_tile(const PerturbArgs& a, float c, float* zout, hipStream_t s, int n_cu) {
  if (a.n_tiles <= 0) return hipSuccess;
  if (a.max_k < 1 || a.max_k > kMaxK) return hipErrorInvalidValue;
  if (a.n_q < 0 || a.n_q > kMaxBatch || (a.n_q > 0 && zout)) return hipErrorInvalidValue;
  if ((a.spread && (a.n_q > 0 || a.from_copy || zout)) || ((a.spread || a.from_copy) && !(a.copy[0] && a.copy[1])) || (a.from_copy && a.n_q > 0)) return hipErrorInvalidValue;
  if (a.n_stage < 0 || a.n_stage > kMaxStage) return hipErrorInvalidValue;
  if (a.n_stage < 0 || a.n_stage > kMaxStage) return hipErrorInvalidValue;
  const RadiusEntry* tab = nullptr;
  hipError_t e = ensure_radius_table(&tab, s);
  if (e != hipSuccess) return e;
  if (a.dtype == 0) return a.bits == 32 ? launch_tile_t<float, 4>(a, c, zout, s, n_cu, tab) : launch_tile_t<float, 8>(a, c, zout, s, n_cu, tab);
  return a.bits == 32 ? launch_tile_t<bf16_t, 4>(a, c, zout, s, n_cu, tab) : launch_tile_t<bf16_t, 8>(a, c, zout, s, n_cu, tab);
}

hipError_t launch_basis_minmax(const float* U, int64_t rows, int k, int ldu, float* minmax, hipStream_t s) {
  int32_t* mm = reinterpret_cast<int32_t*>(minmax);
  hipLaunchKernelGGL(basis_minmax_init_kernel, dim3(1), dim3(1), 0, s, mm);
  const int64_t n = rows * k;
  const int grid = (int)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024);
  hipLaunchKernelGGL(basis_minmax_kernel, dim3(grid), dim3(256), 0, s, U, rows, k, ldu, mm);
  hipLaunchKernelGGL(basis_minmax_finish_kernel, dim3(1), dim3(1), 0, s, mm);
  return hipGetLastError();
}

hipError_t launch_basis_quantize(const float* U, int64_t rows, int k, int ldu, float lambda, float delta, uint8_t* Uq, int ldq, hipStream_t s) {
  const int64_t n = rows * ((k + 1) / 2);
  const int grid = (int)(n / 256 + 1 < 1024 ? n / 256 + 1 : 1024);
  hipLaunchKernelGGL(basis_quantize_kernel, dim3(grid), dim3(256), 0, s, U, rows, k, ldu, lambda, delta, Uq, ldq);
  return hipGetLastError();
}

hipError_t launch_stage_only(const PerturbArgs& a, hipStream_t s) {
  if (a.n_stage <= 0) return hipSuccess;
  if (a.n_stage > kMaxStage) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stage_only_kernel, dim3(kPullBlocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_debug_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(copy_kernel, dim3(256 * 8), dim3(256), 0, s, reinterpret_cast<uint4*>(dst), reinterpret_cast<const uint4*>(src), bytes / 16);
  return hipGetLastError();
}

hipError_t launch_debug_philox(const uint32_t* ctr, uint32_t k0, uint32_t k1, uint32_t* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(debug_philox_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ctr, k0, k1, out, n);
  return hipGetLastError();
}

hipError_t launch_debug_gauss(uint32_t k0, uint32_t k1, uint32_t step, uint32_t id_stream, int bits, int64_t first, int64_t n,
                              float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const RadiusEntry* tab = nullptr;
  hipError_t e = ensure_radius_table(&tab, s);
  if (e != hipSuccess) return e;
  const int P = bits == 32 ? 4 : 8;
  int64_t blocks = (n / P + 256) / 256;
  if (blocks > 4096) blocks = 4096;
  if (bits == 32) hipLaunchKernelGGL(debug_gauss_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, s, k0, k1, step, id_stream, first, n, tab, out);
  else            hipLaunchKernelGGL(debug_gauss_kernel<8>, dim3((unsigned)blocks), dim3(256), 0, s, k0, k1, step, id_stream, first, n, tab, out);
  return hipGetLastError();
}

hipError_t launch_debug_radius_table(int bits, float* out, hipStream_t s) {
  const RadiusEntry* tab = nullptr;
  hipError_t e = ensure_radius_table(&tab, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(debug_radius_kernel, dim3(bits == 32 ? 2048 : 64), dim3(256), 0, s, bits, tab, out);
  return hipGetLastError();
}

hipError_t launch_debug_cossin_table(int bits, float* c, float* sn, hipStream_t s) {
  hipLaunchKernelGGL(debug_cossin_kernel, dim3(bits == 32 ? 4096 : 64), dim3(256), 0, s, bits, c, sn);
  return hipGetLastError();
}

}  // namespace zgr
