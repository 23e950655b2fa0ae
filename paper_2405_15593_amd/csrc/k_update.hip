// The update kernel for Top-K blocks of up to 4096 elements: the moment
// rebuild from the window and the parameter update, one workgroup per block.
#include "microadam_common.h"

namespace microadam {
namespace {

// ============================================================ update
// One workgroup per block.  A thread's 16 elements are its parameter vectors
// (Vec16: vector v of thread t holds the EV elements from v*EV*NT + t*EV).
// The live rows of the block's window record (contiguous, oldest row first
// from slot0 on) are loaded by every thread at once, NT entries per access,
// and staged in LDS in row order with each entry's index replaced by its
// accumulator word, so that no global load waits inside the row-by-row chain.
// One wave (rotating with the block, at raised priority) adds the rows into
// the one accumulator, several chunks of a row (distinct words) per LDS round
// trip: first sum beta1^r V, later sum beta2^r V^2.  Between and after the two
// chains all waves work on the entries they loaded: each distinct element's
// first entry takes its first sum, then turns both sums into the decrement.
// Word CAP is a sink for lanes without an entry, which keeps the adds free of
// branches.
//
// What bounds it: the chain of n_live LDS round trips, twice, per workgroup,
// which the other workgroups of the compute unit have to cover; hence one
// accumulator (LDS for eight workgroups at m = 10 and 20, k = 41), nothing on
// the chain but add and LDS access, and the decrements (about 20 instructions
// per entry) shared by all waves.  The form before held the entries in the
// adding wave's registers, up to 16 chunks of 64, and that wave computed every
// decrement with the library's square root and division; longer windows were
// read row by row from memory.  Measured, old and new, the update in us per 64 M
// bf16 parameters:
//   B_d = 4096, k = 41:   m = 10   53 ->  51,  m = 20  278 -> 58
//   B_d = 4096, k = 205:  m = 10  466 -> 103
//   B_d = 2048, k = 21:   m = 10  117 ->  52
//   B_d = 1024, k = 11:   m = 10   65 ->  52
constexpr int kStageMax = 24;  // entries per thread at most

// Accumulator word of element i: bf16 parameters are read as pairs of 16-byte
// words by the thread that owns 8 consecutive elements, so every other group
// of 8 threads swaps the two words of its pairs and 16 lanes' reads fall on
// distinct banks; binary32 parameters need no permutation.
template <bool PBF16>
__device__ __forceinline__ uint32_t zswap(uint32_t i) {
  return PBF16 ? i ^ ((i >> 4) & 4u) : i;
}

// lr * (c1 s1) / (eps + sqrt(c2 s2)), the root and the quotient correctly
// rounded in under half of the instructions of the library forms.  After v_rsq
// one Newton step with the exact residual gives the rounded root, and after
// v_rcp one gives the rounded reciprocal (both checked against the IEEE results
// for every float of the ranges below); a quotient from a rounded reciprocal and
// one exact residual is the rounded quotient (Markstein, "Computation of
// elementary functions on the IBM RISC System/6000 processor", 1990).  The
// library forms take the arguments outside the range in which no residual or
// result can under- or overflow (and zeros, infinities and NaN): vh and |mh| in
// [2^-100, 2^50], eps up to 2^24 (uniform).
__device__ __forceinline__ bool range_ok(float mh, float vh) {
  const float a = __builtin_fabsf(mh);
  return (__builtin_fminf(a, vh) >= 0x1p-100f) & (__builtin_fmaxf(a, vh) <= 0x1p50f);
}
__device__ __forceinline__ bool range_eps(float x) { return x <= 0x1p24f; }
__device__ __forceinline__ float decrement_in_range(const StepParams& p, float s1, float s2, bool eps_ok, bool& ok) {
  const float mh = p.c1 * s1;
  const float vh = p.c2 * s2;
  const float r = __builtin_amdgcn_rsqf(vh);
  const float q = vh * r;
  const float root = __builtin_fmaf(__builtin_fmaf(-q, q, vh), 0.5f * r, q);
  const float den = p.eps + root;
  const float y0 = __builtin_amdgcn_rcpf(den);
  const float y = __builtin_fmaf(__builtin_fmaf(-den, y0, 1.0f), y0, y0);
  const float d0 = mh * y;
  ok = range_ok(mh, vh) & eps_ok;
  return p.lr * __builtin_fmaf(__builtin_fmaf(-d0, den, mh), y, d0);
}
__device__ __forceinline__ float decrement_any(const StepParams& p, float s1, float s2) {
  return p.lr * ((p.c1 * s1) / (p.eps + __builtin_sqrtf(p.c2 * s2)));
}
__device__ __forceinline__ float decrement(const StepParams& p, float s1, float s2, bool eps_ok) {
  bool ok;
  const float d = decrement_in_range(p, s1, s2, eps_ok, ok);
  return ok ? d : decrement_any(p, s1, s2);
}

// theta <- theta * decay - decrement over a thread's parameter vectors, the
// decrements in z (the decay factor is skipped by a uniform branch when it
// is 1).
template <int NT, bool PBF16>
__device__ __forceinline__ void apply_decrements(const StepParams& p, Rsrc rp,
                                                 const u32x4 (&th)[Vec16<PBF16>::NV], const float* z, int tid, int s) {
  using V = Vec16<PBF16>;
  constexpr int EV = V::EV;
  const bool full = s == NT * kLaneElems;
  auto apply = [&](auto one_tag) {
    constexpr bool ONE_DECAY = decltype(one_tag)::value;
#pragma unroll
    for (int v = 0; v < V::NV; ++v) {
      const uint32_t e0 = V::template first<NT>(v, tid);  // vectors past s store nothing
      float upd[EV], thf[EV], out[EV];
#pragma unroll
      for (int q = 0; q < EV / 4; ++q) {
        const float4 x = *(const float4*)(z + zswap<PBF16>(e0 + 4 * q));
        upd[4 * q] = x.x;
        upd[4 * q + 1] = x.y;
        upd[4 * q + 2] = x.z;
        upd[4 * q + 3] = x.w;
      }
      V::unpack(th[v], thf);
#pragma unroll
      for (int e = 0; e < EV; ++e) out[e] = (ONE_DECAY ? thf[e] : thf[e] * p.decay) - upd[e];
      V::store(rp, e0, s, full, out);
    }
  };
  if (p.decay_is_one)
    apply(BoolTag<true>{});
  else
    apply(BoolTag<false>{});
}

template <int NT, bool VF>
constexpr size_t staged_lds_bytes(int entries) {
  return (size_t)(NT * kLaneElems + 16) * 4 + (size_t)entries * (VF ? 8 : 4);
}

// Waves per SIMD by the LDS of a full stage of KS entries per thread.
template <int NT, bool VF, int KS>
constexpr int staged_waves_per_eu() {
  const int per_cu = (int)(163840 / staged_lds_bytes<NT, VF>(KS * NT));
  const int w = per_cu * (NT / kWave) / 4;
  return w < 1 ? 1 : w > 8 ? 8 : w;
}

template <int NT, bool PBF16, bool VF32, int KS, int G>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(staged_waves_per_eu<NT, VF32, KS>())))
update_kernel(StepParams p, int64_t first_block, int64_t count) {
  constexpr int NW = NT / kWave;
  constexpr int CAP = NT * kLaneElems;
  using E = Entry<VF32>;
  using ET = typename E::T;
  using V = Vec16<PBF16>;
  typedef __attribute__((address_space(3))) float LdsFloat;
  typedef __attribute__((address_space(3))) uint32_t LdsWord;
  extern __shared__ __align__(16) uint32_t smem[];
  float* const z = (float*)smem;
  ET* const stage = (ET*)(smem + CAP + 16);
  // accumulator words as LDS byte addresses
  const uint32_t z0 = (uint32_t)(uintptr_t)(LdsWord*)smem;
  const uint32_t sink = z0 + (uint32_t)CAP * 4;
  auto at = [](uint32_t a) { return (LdsFloat*)(uintptr_t)a; };

  const int tid = thread_id(), lane = tid & (kWave - 1), wave = (int)sgpr(tid / kWave);
  const int m = p.window, n_live = p.n_live;
  const int slot0 = (p.new_slot + 1 + m - n_live) % m;  // the oldest live row
  const Span u = span_of(p, (int32_t)(first_block + xcd_block(block_id(), count)), PBF16 ? 2 : 4);
  const int s = u.s, kq = u.kq;
  const int n = n_live * kq;    // live entries: the record's first n (slot0 is 0 until the window is full)
  const int old0 = slot0 * kq;  // the oldest row's first entry

  // loads: this thread's window entries, then its parameters
  const Rsrc rw = window_rsrc<VF32 ? 2 : 1>(p, u.gb, kq);
  ET w[KS];
#pragma unroll
  for (int i = 0; i < KS; ++i)
    if (i * NT < n) w[i] = E::template load<kStream>(rw, (uint32_t)(i * NT + tid));  // past the record: 0
  const Rsrc rp = make_rsrc((const void*)u.base, vec_bytes<PBF16>(s));
  u32x4 th[V::NV];
#pragma unroll
  for (int v = 0; v < V::NV; ++v) th[v] = V::load(rp, V::template first<NT>(v, tid));
  const float w1s = constant_ptr(p.wpow)[lane];  // kMaxWindow is one wave's lanes
  const float w2s = constant_ptr(p.wpow)[kMaxWindow + lane];
  static_assert(kMaxWindow == kWave, "one weight per lane");

  {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) *(float4*)(z + q * 4 * NT + tid * 4) = zero;
  }
  uint32_t zp[KS];  // the entry's accumulator word
  {
    // place of entry e: e - old0, or e - old0 + n where that is negative (the
    // smaller of the two as unsigned numbers)
    const uint32_t e0 = (uint32_t)(tid - old0);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      zp[i] = sink;
      if (i * NT < n && i * NT + tid < n) {
        const uint32_t idx = E::word(w[i]);
        zp[i] = idx < (uint32_t)s ? z0 + zswap<PBF16>(idx) * 4u : sink;
        const uint32_t e = e0 + i * NT;
        stage[e < e + (uint32_t)n ? e : e + (uint32_t)n] = E::with_word(w[i], zp[i]);
      }
    }
  }
  lds_sync();

  const bool lead = wave == (u.gb & (NW - 1));
  // adds every live row into z, oldest first: weight * V, or weight * V^2;
  // lanes past the row's end add to the sink word
  auto rebuild = [&](float ws, auto sq_tag) {
    constexpr bool SQ = decltype(sq_tag)::value;
    // U rows of up to 64 G entries at a time (one part of a longer row with
    // U = 1): their words and weighted values are ready in registers before
    // the chain of adds, and the next U rows' entries come during it
    constexpr int U = G == 1 ? 5 : G == 2 ? 2 : 1;
    ET x[U][G];
    auto fetch = [&](int e0) {
      const uint32_t e = (uint32_t)(e0 + lane), top = (uint32_t)n - 1;
#pragma unroll
      for (int r = 0; r < U; ++r)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const uint32_t at_e = e + r * kq + g * kWave;
          x[r][g] = stage[at_e < top ? at_e : top];
        }
    };
    __builtin_amdgcn_s_setprio(3);
    fetch(0);
    int row = 0, col = 0;
    while (row < n_live) {
      uint32_t zo[U][G];
      float add[U][G];
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const float wr = __int_as_float(
            __builtin_amdgcn_readlane(__float_as_int(ws), (n_live - 1 - row - r) & (kMaxWindow - 1)));
        const int left = row + r < n_live ? kq - col : 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          zo[r][g] = g * kWave + lane < left ? E::word(x[r][g]) : sink;
          const float v = E::val(x[r][g]);
          add[r][g] = wr * (SQ ? v * v : v);
        }
      }
      col += U == 1 ? G * kWave : kq;
      if (col >= kq) {
        col = 0;
        row += U;
      }
      fetch(row * kq + col);
#pragma unroll
      for (int r = 0; r < U; ++r) {
        float a[G];
#pragma unroll
        for (int g = 0; g < G; ++g) a[g] = *at(zo[r][g]);
#pragma unroll
        for (int g = 0; g < G; ++g) *at(zo[r][g]) = a[g] + add[r][g];
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };
  if (lead) rebuild(w1s, BoolTag<false>{});
  lds_sync();
  // Each entry takes its word's first sum and leaves -0 (x + -0 is x, so the
  // second sums start from it like from 0; a sum that started at +0 is never
  // -0).  Of the entries of one element the first to come gets the sum and
  // turns the two sums into the decrement; the others get -0 and are done.
  // Lanes without an entry stay out of it, since exchanges of one word, the sink,
  // follow each other (B_d = 4096, 64 M bf16 parameters: k = 41, m = 20 61.6 ->
  // 57.4 us, k = 205, m = 10 104.5 -> 99.3), but for more than 12 entries per
  // thread, where their branches cost more (B_d = 512, k = 128: 316 against 329).
  constexpr uint32_t kTaken = 0x80000000u;
  uint32_t s1[KS];
  {
    const int nn = opaque(n);
#pragma unroll
    for (int i = 0; i < KS; ++i)
      if (i * NT < nn) {
        if (KS <= 12) s1[i] = kTaken;
        if (KS > 12 || zp[i] != sink)
          s1[i] = __hip_atomic_exchange((LdsWord*)(uintptr_t)zp[i], kTaken, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
      }
  }
  lds_sync();
  if (lead) rebuild(w2s, BoolTag<true>{});
  lds_sync();
  {
    const bool eps_ok = range_eps(p.eps);
    const int nn = opaque(n);
#pragma unroll
    for (int i = 0; i < KS; ++i)
      if (i * NT < nn && s1[i] != kTaken)
        *at(zp[i]) = decrement(p, __uint_as_float(s1[i]), *at(zp[i]), eps_ok);
  }
  lds_sync();

  apply_decrements<NT, PBF16>(p, rp, th, z, tid, s);
}

// Blocks of one wave (up to 1024 elements) with few and long rows (the rule is
// at the launch): lane l holds entry l of every live row, oldest first, in
// registers, and no entry passes through a stage.  Each row (distinct words)
// adds to the accumulator in one LDS round trip; rows past the live ones and
// lanes past the row's end add to the sink.  Every entry reads both its sums
// before any word is overwritten, so the entries of one element write the same
// decrement.  All of it is one straight run over KR rows: in a small launch
// that run's latency is the time.  Through the stage and held, update in us,
// B_d = 1024, k = 52, m = 10:
//   bf16      64 M parameters 82 -> 69   1 M 8.9 -> 6.9
//   binary32                             1 M 9.0 -> 6.9
template <bool PBF16, bool VF32, int KR>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(8)))
update_held_kernel(StepParams p, int64_t first_block, int64_t count) {
  constexpr int NT = kWave, CAP = NT * kLaneElems;
  using E = Entry<VF32>;
  using ET = typename E::T;
  using V = Vec16<PBF16>;
  extern __shared__ __align__(16) uint32_t smem[];
  float* const z = (float*)smem;

  const int lane = thread_id();
  const int m = p.window, n_live = p.n_live;
  const Span u = span_of(p, (int32_t)(first_block + xcd_block(block_id(), count)), PBF16 ? 2 : 4);
  const int s = u.s, kq = u.kq;
  const Rsrc rw = window_rsrc<VF32 ? 2 : 1>(p, u.gb, kq);
  ET w[KR];
  int slot = (p.new_slot + 1 + m - n_live) % m;  // the oldest live row
#pragma unroll
  for (int i = 0; i < KR; ++i) {  // (rows past the live ones: any rows of the record)
    w[i] = E::template load<kStream>(rw, (uint32_t)(slot * kq + lane));
    if (++slot == m) slot = 0;
  }
  const Rsrc rp = make_rsrc((const void*)u.base, vec_bytes<PBF16>(s));
  u32x4 th[V::NV];
#pragma unroll
  for (int v = 0; v < V::NV; ++v) th[v] = V::load(rp, V::template first<NT>(v, lane));
  const float w1s = constant_ptr(p.wpow)[lane];  // kMaxWindow is one wave's lanes
  const float w2s = constant_ptr(p.wpow)[kMaxWindow + lane];
  {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) *(float4*)(z + q * 4 * NT + lane * 4) = zero;
  }
  uint32_t zp[KR];  // the entry's accumulator word
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    const uint32_t idx = E::word(w[i]);
    zp[i] = (i < n_live) & (lane < kq) & (idx < (uint32_t)s) ? zswap<PBF16>(idx) : (uint32_t)CAP;
  }
  wave_sync();

  auto rebuild = [&](float ws, bool sq) {
#pragma unroll
    for (int i = 0; i < KR; ++i) {
      const float wr =
          __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ws), (n_live - 1 - i) & (kMaxWindow - 1)));
      const float v = E::val(w[i]);
      z[zp[i]] = z[zp[i]] + wr * (sq ? v * v : v);
    }
  };
  float s1[KR], d[KR];
  rebuild(w1s, false);
#pragma unroll
  for (int i = 0; i < KR; ++i) s1[i] = z[zp[i]];
#pragma unroll
  for (int i = 0; i < KR; ++i) z[zp[i]] = 0.0f;
  rebuild(w2s, true);
  const bool eps_ok = range_eps(p.eps);
  bool out = false;  // an entry outside the range
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    bool ok;
    d[i] = decrement_in_range(p, s1[i], z[zp[i]], eps_ok, ok);
    out |= !ok & (zp[i] != (uint32_t)CAP);
  }
  if (ballot(out) != 0) {
#pragma unroll
    for (int i = 0; i < KR; ++i) d[i] = decrement_any(p, s1[i], z[zp[i]]);
  }
#pragma unroll
  for (int i = 0; i < KR; ++i) z[zp[i]] = d[i];
  wave_sync();
  apply_decrements<NT, PBF16>(p, rp, th, z, lane, s);
}

// Debug export, and the update where the live rows do not fit the stage (more
// than kStageMax entries per thread): two accumulators, sum beta1^r V and sum
// beta2^r V^2, one wave reading the window record row by row.
template <int NT, bool VF>
constexpr size_t update_lds_bytes() {
  return (size_t)2 * (NT * kLaneElems + 16) * 4;
}

template <int NT, bool PBF16, bool VF32, bool EXPORT>
__global__ void __launch_bounds__(NT) update_rows_kernel(StepParams p, int64_t first_block, int64_t count,
                                                         float* mhat, float* vhat) {
  constexpr int NW = NT / kWave;
  constexpr int CAP = NT * kLaneElems;
  using E = Entry<VF32>;
  using ET = typename E::T;
  using V = Vec16<PBF16>;
  constexpr int EV = V::EV;
  extern __shared__ __align__(16) uint32_t smem[];
  float* const z1 = (float*)smem;
  float* const z2 = z1 + CAP + 16;

  const int tid = thread_id(), lane = tid & (kWave - 1), wave = (int)sgpr(tid / kWave);
  const int m = p.window, n_live = p.n_live;
  const int slot0 = (p.new_slot + 1 + m - n_live) % m;  // the oldest live row
  const Span u = span_of(p, (int32_t)(first_block + xcd_block(block_id(), count)), PBF16 ? 2 : 4);
  const int s = u.s, kq = u.kq;
  const Rsrc rw = window_rsrc<VF32 ? 2 : 1>(p, u.gb, kq);
  const Rsrc rp = make_rsrc((const void*)u.base, vec_bytes<PBF16>(s));
  u32x4 th[V::NV];
  if (!EXPORT) {
#pragma unroll
    for (int v = 0; v < V::NV; ++v) th[v] = V::load(rp, V::template first<NT>(v, tid));
  }
  const float w1s = constant_ptr(p.wpow)[lane];  // kMaxWindow is one wave's lanes
  const float w2s = constant_ptr(p.wpow)[kMaxWindow + lane];
  {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      *(float4*)(z1 + q * 4 * NT + tid * 4) = zero;
      *(float4*)(z2 + q * 4 * NT + tid * 4) = zero;
    }
  }
  lds_sync();

  if (wave == (u.gb & (NW - 1))) {
    for (int row = 0, slot = slot0; row < n_live; ++row, slot = (slot + 1 == m) ? 0 : slot + 1) {
      const int r = n_live - 1 - row;
      const float w1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w1s), r));
      const float w2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w2s), r));
      for (int jj = lane; jj < kq; jj += kWave) {
        const ET x = E::load(rw, slot * kq + jj);
        const uint32_t i = E::idx(x);
        const uint32_t zp = i < (uint32_t)s ? zswap<PBF16>(i) : (uint32_t)CAP;
        const float v = E::val(x);
        const float vv = v * v;
        const float x1 = w1 * v, x2 = w2 * vv;
        const float a1 = z1[zp], a2 = z2[zp];
        z1[zp] = a1 + x1;
        z2[zp] = a2 + x2;
      }
    }
    if (!EXPORT) {
      // one 64-entry chunk at a time; z2 = -1 marks a converted word
      const bool eps_ok = range_eps(p.eps);
      for (int row = 0, slot = slot0; row < n_live; ++row, slot = (slot + 1 == m) ? 0 : slot + 1)
        for (int jj = lane; jj < kq; jj += kWave) {
          const uint32_t i = E::idx(E::load(rw, slot * kq + jj));
          if (i < (uint32_t)s) {
            const uint32_t zp = zswap<PBF16>(i);
            const float s2 = z2[zp];
            if (s2 >= 0.0f) {
              z1[zp] = decrement(p, z1[zp], s2, eps_ok);
              z2[zp] = -1.0f;
            }
          }
        }
    }
  }
  lds_sync();

  if (EXPORT) {
#pragma unroll
    for (int v = 0; v < V::NV; ++v) {
#pragma unroll
      for (int e = 0; e < EV; ++e) {
        const uint32_t i = V::template first<NT>(v, tid) + e;
        if ((int)i < s) {
          mhat[u.e0 + i] = p.c1 * z1[zswap<PBF16>(i)];
          vhat[u.e0 + i] = p.c2 * z2[zswap<PBF16>(i)];
        }
      }
    }
    return;
  }
  apply_decrements<NT, PBF16>(p, rp, th, z1, tid, s);
}

template <int NT, bool PB, bool VF, int KS>
hipError_t launch_update_k(const StepParams& p, int64_t first, int64_t count, hipStream_t stream) {
  const size_t lds = staged_lds_bytes<NT, VF>(p.n_live * p.k_full);
  auto go = [&](auto g_tag) {
    constexpr int G = decltype(g_tag)::value;
    hipLaunchKernelGGL((update_kernel<NT, PB, VF, KS, G>), dim3((uint32_t)count), dim3(NT), lds, stream, p,
                       first, count);
    return hipGetLastError();
  };
  if (p.k_full <= kWave) return go(std::integral_constant<int, 1>{});
  if (p.k_full <= 2 * kWave) return go(std::integral_constant<int, 2>{});
  return go(std::integral_constant<int, 4>{});
}

// Whether the live rows of every block fit the stage.
template <int NT, bool VF>
bool fits_stage(const StepParams& p) {
  const int64_t n = (int64_t)p.n_live * p.k_full;
  return n <= (int64_t)kStageMax * NT && staged_lds_bytes<NT, VF>((int)n) <= 65536;
}

// Blocks of one wave with rows of 25 to 64 entries: held in registers, up to 13
// live rows with bf16 parameters and up to 10 with binary32 ones (more take
// registers to scratch: bf16, 16 rows, k = 33, 43 against 34 us per 16.8 M
// parameters).  Shorter rows leave most of every held access empty, and the
// stage's flat accesses win (B_d = 1024, m = 10, 64 M bf16 parameters: k = 11 59
// against 52 us, k = 21 the same, k = 26 66 against 71).  Binary32 parameters
// only in launches that leave the chip's 8192 wave slots unfilled, where one
// block's latency counts: 64 M parameters, k = 41, take 111 us held and 109
// through the stage, 300,000 take 6.3 and 7.5.  Returns false elsewhere.
template <bool PB, bool VF>
bool launch_update_held(const StepParams& p, int64_t first, int64_t count, hipStream_t stream, hipError_t& err) {
  if (p.k_full <= 24 || p.k_full > kWave || p.n_live > (PB ? 13 : 10) || (!PB && count > 8192)) return false;
  auto go = [&](auto kr) {
    hipLaunchKernelGGL((update_held_kernel<PB, VF, decltype(kr)::value>), dim3((uint32_t)count), dim3(kWave),
                       (staged_lds_bytes<kWave, VF>(0)), stream, p, first, count);
    err = hipGetLastError();
    return true;
  };
  if (p.n_live <= 4) return go(std::integral_constant<int, 4>{});
  if (p.n_live <= 7) return go(std::integral_constant<int, 7>{});
  if constexpr (PB) {
    if (p.n_live > 10) return go(std::integral_constant<int, 13>{});
  }
  return go(std::integral_constant<int, 10>{});
}

// The staged kernel wherever every block's live rows fit the stage, else row
// by row (a stage of more entries leaves one or two workgroups per compute
// unit; m * k above 6144 at B_d = 4096 lies outside the method's settings).
template <int NT, bool PB, bool VF>
hipError_t launch_update_t(const StepParams& p, int64_t first, int64_t count, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  if (!fits_stage<NT, VF>(p)) {
    const size_t lds = update_lds_bytes<NT, VF>();
    hipLaunchKernelGGL((update_rows_kernel<NT, PB, VF, false>), dim3((uint32_t)count), dim3(NT), lds, stream, p, first,
                       count, (float*)nullptr, (float*)nullptr);
    return hipGetLastError();
  }
  if constexpr (NT == kWave) {
    hipError_t err;
    if (launch_update_held<PB, VF>(p, first, count, stream, err)) return err;
  }
  const int ks = (p.n_live * p.k_full + NT - 1) / NT;
  if (ks <= 2) return launch_update_k<NT, PB, VF, 2>(p, first, count, stream);
  if (ks <= 4) return launch_update_k<NT, PB, VF, 4>(p, first, count, stream);
  if (ks <= 8) return launch_update_k<NT, PB, VF, 8>(p, first, count, stream);
  if (ks <= 12) return launch_update_k<NT, PB, VF, 12>(p, first, count, stream);
  return launch_update_k<NT, PB, VF, kStageMax>(p, first, count, stream);
}

template <int NT, bool VF>
hipError_t launch_export(const StepParams& p, int64_t first_block, int64_t blocks, float* mh, float* vh,
                         hipStream_t stream) {
  if (blocks <= 0) return hipSuccess;
  const size_t lds = update_lds_bytes<NT, VF>();
  hipLaunchKernelGGL((update_rows_kernel<NT, false, VF, true>), dim3((uint32_t)blocks), dim3(NT), lds, stream, p,
                     first_block, blocks, mh, vh);
  return hipGetLastError();
}

}  // namespace

size_t update_lds_max(int nt) {
  return nt == 64 ? update_lds_bytes<64, true>() : nt == 128 ? update_lds_bytes<128, true>() : update_lds_bytes<256, true>();
}

namespace {
// The launch for a block size and types: f(threads, parameters are bf16,
// window values are binary32), each as a compile-time constant.
template <typename F>
hipError_t by_form(int block, int param_bf16, int value_f32, F f) {
  using Y = std::true_type;
  using N = std::false_type;
  auto types = [&](auto nt) {
    if (param_bf16) return value_f32 ? f(nt, Y{}, Y{}) : f(nt, Y{}, N{});
    return value_f32 ? f(nt, N{}, Y{}) : f(nt, N{}, N{});
  };
  switch (threads_for_block(block)) {
    case 64: return types(std::integral_constant<int, 64>{});
    case 128: return types(std::integral_constant<int, 128>{});
    default: return types(std::integral_constant<int, 256>{});
  }
}
}  // namespace

hipError_t launch_update_blocks(const StepParams& p, int param_bf16, int value_f32, int64_t first, int64_t count,
                                hipStream_t stream) {
  return by_form(p.block, param_bf16, value_f32, [&](auto nt, auto pb, auto vf) {
    return launch_update_t<decltype(nt)::value, decltype(pb)::value, decltype(vf)::value>(p, first, count, stream);
  });
}

hipError_t launch_moments_blocks(const StepParams& p, int64_t first_block, int64_t num_blocks, float* mhat,
                                 float* vhat, int value_f32, hipStream_t stream) {
  return by_form(p.block, 0, value_f32, [&](auto nt, auto, auto vf) {
    return launch_export<decltype(nt)::value, decltype(vf)::value>(p, first_block, num_blocks, mhat, vhat, stream);
  });
}

}  // namespace microadam
