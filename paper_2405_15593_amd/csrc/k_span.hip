// Steps with quantization buckets spanning Top-K blocks: the select kernel's
// partials form, the bucket reduction and the second quantization pass.
#include "select_kernel.h"
#include "select_large_kernel.h"

namespace microadam {
namespace {

// Per bucket of the step (all tensors), by a group of 2^lg lanes: the (min,
// max) over the partials of the blocks it covers, -0 stored as +0, into table
// t mod 2.  The host takes the group from the blocks per bucket: with one
// thread per bucket of 100,000 elements, the 26 loads of a bucket followed
// each other in 16 workgroups (17 us per 405 M parameters; 4 us with 32 lanes).
__global__ void __launch_bounds__(256) bucket_reduce_kernel(StepParams p, int32_t lg) {
  const int64_t cg = ((int64_t)block_id() * 256 + thread_id()) >> lg;
  const int i0 = thread_id() & ((1 << lg) - 1);
  if (cg >= p.total_buckets) return;  // whole groups
  const __attribute__((address_space(4))) TensorDesc* td = constant_ptr(p.tensors);
  int lo = 0, hi = p.n_tensors - 1;  // the last tensor whose buckets start at or before cg
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (td[mid].first_bucket <= cg) lo = mid;
    else hi = mid - 1;
  }
  const TensorDesc d = load_desc(td + lo);
  const int64_t bq = p.big_bucket, B = p.block;
  const int64_t c = cg - d.first_bucket;
  const int64_t e_lo = c * bq;
  const int64_t e_hi = e_lo + bq < d.numel ? e_lo + bq : d.numel;
  const int64_t q_lo = e_lo / B, q_hi = (e_hi - 1) / B;
  // only the bucket's first block can hold another bucket's end before it
  const bool straddles = q_lo * B < e_lo;
  const Rsrc rp = make_rsrc(p.state + p.partial_plane, (uint32_t)(p.total_blocks * 16));
  float mn = __builtin_inff(), mx = -__builtin_inff();
  for (int64_t q = q_lo + i0; q <= q_hi; q += (int64_t)1 << lg) {
    const int64_t gb = q == d.num_blocks - 1 ? d.last_block : d.first_block + q;
    const uint32_t part = q == q_lo && straddles ? 8u : 0u;  // the block's second bucket, or its first
    const u32x2 pr = __builtin_amdgcn_raw_buffer_load_b64(rp, (uint32_t)(gb * 16) + part, 0, 0);
    mn = __builtin_fminf(mn, __uint_as_float(pr[0]));
    mx = __builtin_fmaxf(mx, __uint_as_float(pr[1]));
  }
  for (int x = (1 << lg) >> 1; x > 0; x >>= 1) {
    mn = __builtin_fminf(mn, __shfl_xor(mn, x, kWave));
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, x, kWave));
  }
  if (i0 != 0) return;
  mn = mn + 0.0f;  // a bucket bound of -0 is stored as +0
  mx = mx + 0.0f;
  const uint64_t t = (uint64_t)(p.t & 1);
  float* out = (float*)(p.state + p.stats_plane + t * p.table_bytes) + 2 * cg;
  out[0] = mn;
  out[1] = mx;
}

// e = Q(a with a[I] = 0) for buckets spanning blocks (Algorithm 1; Algorithm
// 2, Q; Lemma 1 with kEfRandom): recomputes a = g + Q^-1(e) exactly as the
// select kernel did (same codes, same pairs), zeroes the elements of the
// block's new window row, and quantizes with the new pairs.  One wave per
// 4096-element sub-block of a block (the whole block up to 4096 elements),
// 64 elements per lane.  Above 4096 the sub-block's entries of the new row
// are those of its four 1024-element quarters, found through the record's
// segment table.
//
// Blocks that are whole sub-blocks come and go as contiguous kilobytes through
// LDS (coalesced_exchange).  Decode and codes take a vector at a time with its
// first element's bucket, and only a vector that holds a bucket's end again with
// the next one (a uniform branch per vector); codes come from two bracketing
// products instead of an IEEE division, as in the select.
// All of a step but its update, 64 M bf16 parameters, with an IEEE division per
// element and uncoalesced accesses, and now: B_q = 100,000 141 -> 113 us, B_q =
// 5003 (a bucket's end in four blocks of five) 128 -> 114.  (Decoding and
// quantizing the whole block a second time where a run straddles: 132 and 216;
// the reloaded inputs of that decode took 53 to 63 registers to scratch.)
template <bool GBF16, bool VF32, int EFM>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
requant_kernel(StepParams p, int64_t first, int64_t count, int32_t nsub) {
  constexpr int EPL = 64, NV = EPL / 8, CAP = kWave * EPL;
  constexpr int CW = (EFM & kEf8) ? 2 : 1;
  constexpr uint32_t kTr = GBF16 ? kTrBytes : kTrBytesF32;
  using E = Entry<VF32>;
  __shared__ __align__(16) uint32_t tr[kTr / 4];
  __shared__ uint32_t kept[CAP / 32];  // bit i: element off + i is in the new row

  const int lane = thread_id();
  const int64_t w = xcd_block(block_id(), count * nsub);
  const int64_t gb = first + w / nsub;
  const uint32_t off = (uint32_t)(w % nsub) * CAP;  // the sub-block's first element
  const uint32_t el = (uint32_t)lane * EPL;         // the lane's first element in the sub-block
  const uint32_t eb = off + el;                     // and in the block
  const uint32_t sub_ef = (EFM & kEf8) ? (uint32_t)CAP : (uint32_t)CAP / 2;
  const uint32_t ef_bytes = (EFM & kEf8) ? (uint32_t)p.block : (uint32_t)(p.block >> 1);
  const bool coal = p.block % CAP == 0;
  const uint32_t ef_off = (EFM & kEf8) ? off : off / 2;
  const uint32_t ef_here = ef_bytes - ef_off < sub_ef ? ef_bytes - ef_off : sub_ef;
  const Rsrc re = make_rsrc(p.state + p.ef_plane + (uint64_t)gb * ef_bytes + ef_off, ef_here);
  LaneIn<EPL, true, GBF16, EFM> in;
  const Block b = locate(p, gb);
  const int s = b.s - (int)off, kq = b.kq;
  if (s <= 0) return;  // a sub-block past the end of a ragged block
  const bool full = s >= CAP;
  const Rsrc rg = make_rsrc((const uint8_t*)b.desc.grad + (b.e0 + off) * (GBF16 ? 2 : 4),
                            vec_bytes<GBF16>(full ? CAP : s));
  const LqBuckets old_b = lq_buckets(p, b, eb, EPL, 0), new_b = lq_buckets(p, b, eb, EPL, 1);
  if (coal) {
    CoalescedIn<GBF16> cx;
    coalesced_load_codes<EFM>(cx, re, lane);
    coalesced_load_grad(cx, rg, lane);
    coalesced_exchange(cx, in, tr, lane);
  } else {
    lane_load_codes(in, re, el, false);
    lane_load_grad(in, rg, el);
  }

  kept[lane] = 0u;
  kept[lane + kWave] = 0u;
  wave_sync();
  const Rsrc rw = window_rsrc<VF32 ? 2 : 1>(p, gb, kq);
  const uint32_t row0 = (uint32_t)p.new_slot * kq;
  // the row's entries of this sub-block: [j0, j1)
  uint32_t j0 = 0, j1 = (uint32_t)kq;
  if (p.block > CAP) {
    constexpr uint32_t EB = VF32 ? 8u : 4u;
    const int nq = (p.block + kQuarter - 1) / kQuarter;
    const int q0 = (int)(off / kQuarter), q1 = q0 + CAP / kQuarter;
    const Rsrc rrec = make_rsrc(p.state + p.win_plane + (uint64_t)gb * p.win_stride, (uint32_t)p.win_stride);
    const uint32_t table = (uint32_t)p.window * p.k_full * EB + (uint32_t)p.new_slot * nq * 4;
    const uint32_t a0 = __builtin_amdgcn_raw_buffer_load_b32(rrec, table + (uint32_t)q0 * 4, 0, 0);
    const uint32_t a1 = q1 < nq ? __builtin_amdgcn_raw_buffer_load_b32(rrec, table + (uint32_t)q1 * 4, 0, 0)
                                : (uint32_t)kq;
    j0 = sgpr(a0 < (uint32_t)kq ? a0 : (uint32_t)kq);  // clamped: any content gives a bounded read
    j1 = sgpr(a1 < (uint32_t)kq ? a1 : (uint32_t)kq);
  }
  for (uint32_t j = j0 + (uint32_t)lane; j < j1; j += kWave) {
    const uint32_t i = E::idx(E::load(rw, row0 + j)) - off;
    if (i < (uint32_t)CAP) atomicOr(&kept[i >> 5], 1u << (i & 31));
  }
  wave_sync();

  float a[NV][8];
  const int rem = s - (int)el;
  const uint32_t k0 = kept[2 * lane], k1 = kept[2 * lane + 1];  // this lane's 64 elements
  const EfStream st{b.e0, b.j, (uint32_t)p.t, p.seed_lo, p.seed_hi};
  uint32_t wv[NV * CW];
  auto zero_kept = [&] {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = 8 * v + e;
        // all ones where the bit is set
        const int32_t m = (int32_t)((i < 32 ? k0 : k1) << (31 - (i & 31))) >> 31;
        a[v][e] = __uint_as_float(__float_as_uint(a[v][e]) & ~(uint32_t)m);
      }
  };
  lane_decode_lq<false>(in, old_b, a, rem, full);
  zero_kept();
  // each vector with its first element's bucket; the vector that the bucket
  // ends inside (wherever a lane has one: a uniform branch) again with the next
  // one, the elements before it at that bucket's lower bound
  const float lo0 = __uint_as_float(new_b.st[0][0]), u0 = ef_step<EFM>(__uint_as_float(new_b.st[0][1]) - lo0);
  const float lo1 = __uint_as_float(new_b.st[1][0]), u1 = ef_step<EFM>(__uint_as_float(new_b.st[1][1]) - lo1);
  const int sp = new_b.sp;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const uint64_t quad = (uint64_t)(b.e0 + eb + 8 * v) >> 2;
    const float lo = 8 * v >= sp ? lo1 : lo0, u = 8 * v >= sp ? u1 : u0;
    uint32_t c[CW];
    vector_codes<EFM>(a[v], lo, u, quad, st, c);
    if (ballot(sp > 8 * v && sp < 8 * v + 8) != 0) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 8 * v + e >= sp ? a[v][e] : lo1;
      uint32_t c1[CW];
      vector_codes<EFM>(x, lo1, u1, quad, st, c1);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t m = (EFM & kEf8) ? 0xFFu << (8 * (e & 3)) : 0xFu << (4 * e);
        uint32_t& w = c[(EFM & kEf8) ? e >> 2 : 0];
        if (8 * v + e >= sp) w = (w & ~m) | (c1[(EFM & kEf8) ? e >> 2 : 0] & m);
      }
    }
#pragma unroll
    for (int h = 0; h < CW; ++h) wv[CW * v + h] = c[h];
  }
  if (!full) {  // codes past the block's end are 0
    const int r = opaque_v(rem);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (8 * v + e >= r) {
          if constexpr (EFM & kEf8) wv[CW * v + (e >> 2)] &= ~(0xFFu << (8 * (e & 3)));
          else wv[v] &= ~(0xFu << (4 * e));
        }
  }
  if (coal) lane_store_codes_coalesced<EFM>(wv, tr, re);
  else if ((int)el < s) lane_store_codes<EPL, EFM>(wv, el, false, re);
}

template <bool GB, bool VF, int EF8>
hipError_t launch_select_partials_t(const StepParams& p, hipStream_t stream) {
  if (p.block > kSubBlock) return launch_select_large<GB, VF, EF8, true>(p, 0, p.total_blocks, stream);
  if (select_dense<64, VF>(p.k_full)) {
    const size_t lds = select_lds<64, GB, !VF>();
    hipLaunchKernelGGL((select_kernel<64, true, GB, VF, EF8, true, !VF>), dim3((uint32_t)p.total_blocks), dim3(kWave),
                       lds, stream, p, (int64_t)0, p.total_blocks);
  } else {
    const size_t lds = select_lds<64, GB, false>();
    hipLaunchKernelGGL((select_kernel<64, true, GB, VF, EF8, true>), dim3((uint32_t)p.total_blocks), dim3(kWave), lds,
                       stream, p, (int64_t)0, p.total_blocks);
  }
  return hipGetLastError();
}

template <bool GB, bool VF>
hipError_t launch_select_partials_d(const StepParams& p, hipStream_t stream) {
  return (p.ef_mode & kEf8) ? launch_select_partials_t<GB, VF, kEf8>(p, stream)
                            : launch_select_partials_t<GB, VF, 0>(p, stream);
}

template <bool GB, bool VF, int EFM>
hipError_t launch_requant_t(const StepParams& p, hipStream_t stream) {
  const int32_t nsub = (p.block + kSubBlock - 1) / kSubBlock;
  hipLaunchKernelGGL((requant_kernel<GB, VF, EFM>), dim3((uint32_t)(p.total_blocks * nsub)), dim3(kWave), 0, stream,
                     p, (int64_t)0, p.total_blocks, nsub);
  return hipGetLastError();
}

template <bool GB, bool VF>
hipError_t launch_requant_d(const StepParams& p, hipStream_t stream) {
  switch (p.ef_mode) {
    case 0: return launch_requant_t<GB, VF, 0>(p, stream);
    case kEf8: return launch_requant_t<GB, VF, kEf8>(p, stream);
    case kEfRandom: return launch_requant_t<GB, VF, kEfRandom>(p, stream);
    case kEf8 | kEfRandom: return launch_requant_t<GB, VF, kEf8 | kEfRandom>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_select_partials(const StepParams& p, int grad_bf16, int value_f32, hipStream_t stream) {
  if (p.total_blocks <= 0) return hipSuccess;
  if (grad_bf16)
    return value_f32 ? launch_select_partials_d<true, true>(p, stream) : launch_select_partials_d<true, false>(p, stream);
  return value_f32 ? launch_select_partials_d<false, true>(p, stream) : launch_select_partials_d<false, false>(p, stream);
}

hipError_t launch_bucket_reduce(const StepParams& p, hipStream_t stream) {
  if (p.total_buckets <= 0) return hipSuccess;
  // lanes per bucket: the blocks a bucket covers, up to a wave (fewer where a
  // launch of 2^32 threads would be reached: tens of millions of tensors)
  int32_t lg = 0;
  while (lg < 6 && (int64_t)p.block << lg < p.big_bucket + p.block && p.total_buckets << (lg + 1) < (1ll << 32) - 256)
    ++lg;
  const uint32_t grid = (uint32_t)(((p.total_buckets << lg) + 255) / 256);
  hipLaunchKernelGGL(bucket_reduce_kernel, dim3(grid), dim3(256), 0, stream, p, lg);
  return hipGetLastError();
}

hipError_t launch_requant(const StepParams& p, int grad_bf16, int value_f32, hipStream_t stream) {
  if (p.total_blocks <= 0) return hipSuccess;
  if (grad_bf16)
    return value_f32 ? launch_requant_d<true, true>(p, stream) : launch_requant_d<true, false>(p, stream);
  return value_f32 ? launch_requant_d<false, true>(p, stream) : launch_requant_d<false, false>(p, stream);
}

}  // namespace microadam
