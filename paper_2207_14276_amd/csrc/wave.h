// Wave-level helpers shared by the per-centre kernels (wave64).
#pragma once

#include "internal.h"
#include "fixed.h"

namespace nnp {

__device__ inline unsigned lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

// A pointer that the kernel read from memory, as one to global memory: the
// compiler knows no more than that it is some address, and would load through
// it with flat instructions, which count as LDS accesses too, so that every
// wait for one waits for all loads in flight.
template <class T> using Global = const __attribute__((address_space(1))) T *;
template <class T> __device__ inline Global<T> as_global(const T *p) { return (Global<T>)p; }
typedef unsigned uintx4_v __attribute__((ext_vector_type(4)));
typedef float floatx4_v __attribute__((ext_vector_type(4)));
template <class T> __device__ inline uint4 load16(Global<T> p) {
  const uintx4_v v = *(Global<uintx4_v>)p;
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ inline float4 load4f(Global<float> p) {
  const floatx4_v v = *(Global<floatx4_v>)p;
  return make_float4(v[0], v[1], v[2], v[3]);
}

// The species bucket of the row tile at r0 (buckets are whole tiles), -1 past
// the last, and in real_end where its rows of atoms end (cnt null: 0).  Lane q
// looks at bucket q, so that a tile waits for memory once: read in turn, the
// buckets were a chain of up to seven waits ahead of a tile's first load
// (a 24-atom call's dE/dG and first layer 8.4 and 13.6 -> 7.9 and 13.0 us with
// the rows' records loaded meanwhile; the chain of a 6,000-atom region with 8
// members 45.2 -> 43.7, its first layer 34.4 -> 33.5).
__device__ inline int tile_bucket(const int *off, const int *cnt, int n_groups, int r0, int lane, int &real_end) {
  static_assert(kMaxSpecies <= kWave, "a lane per bucket");
  const int q = min(lane, n_groups - 1);
  const int from = off[q], to = off[q + 1], n = cnt ? cnt[q] : -from;
  const unsigned long long m = __ballot(lane < n_groups && r0 >= from && r0 < to);
  real_end = 0;
  if (m == 0) return -1;
  const int s = __builtin_ctzll(m);
  real_end = __builtin_amdgcn_readlane(from + n, s);
  return s;
}

// Hardware reciprocal and square root (about 1 ulp), in place of the
// correctly rounded division and square-root sequences.
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Neighbour vector d = r_j + image * L - r_i of entry e of centre i.
__device__ inline float4 entry_vec(const float4 &pi, const float4 &pj, int code, const float L[3]) {
  int ix, iy, iz;
  unpack_image(code, ix, iy, iz);
  float dx = (pj.x - pi.x) + (float)ix * L[0];
  float dy = (pj.y - pi.y) + (float)iy * L[1];
  float dz = (pj.z - pi.z) + (float)iz * L[2];
  return make_float4(dx, dy, dz, fast_sqrt(dx * dx + dy * dy + dz * dz));
}

// Lane reductions on the VALU (DPP) rather than through the LDS crossbar.
template <int CTRL, int ROWS = 0xF> __device__ inline float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}
// sum over aligned groups of 4 / 8 / 16 lanes, result in every lane of the group
__device__ inline float sum4(float v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  return v;
}
__device__ inline float sum8(float v) {
  v = sum4(v);
  v += dpp<0x141>(v);  // row_half_mirror: quads 0 <-> 1 of each half-row
  return v;
}
__device__ inline float sum16(float v) {
  v = sum8(v);
  v += dpp<0x140>(v);  // row_mirror: halves 0 <-> 1 of each row
  return v;
}
// sum over the whole wave, returned in every lane
__device__ inline float wave_sum(float v) {
  v = sum16(v);
  v += dpp<0x142, 0xA>(v);  // row_bcast15 into rows 1 and 3
  v += dpp<0x143, 0xC>(v);  // row_bcast31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// OR over the whole wave, returned in every lane (the steps of wave_sum)
template <int CTRL, int ROWS = 0xF> __device__ inline unsigned dpp_u(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
// sum over this lane and all lanes below it
__device__ inline unsigned wave_scan(unsigned v) {
  v += dpp_u<0x111>(v);  // row_shr:1
  v += dpp_u<0x112>(v);  // row_shr:2
  v += dpp_u<0x114>(v);  // row_shr:4
  v += dpp_u<0x118>(v);  // row_shr:8
  v += dpp_u<0x142, 0xA>(v);  // row_bcast15 into rows 1 and 3
  v += dpp_u<0x143, 0xC>(v);  // row_bcast31 into rows 2 and 3
  return v;
}
__device__ inline unsigned wave_or(unsigned v) {
  v |= dpp_u<0xB1>(v);
  v |= dpp_u<0x4E>(v);
  v |= dpp_u<0x141>(v);
  v |= dpp_u<0x140>(v);
  v |= dpp_u<0x142, 0xA>(v);
  v |= dpp_u<0x143, 0xC>(v);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// The AEV's live halves as they lie in a first layer's input row: gap halves
// follow the rad radial ones (GemmLaunch::rad_gap).
__device__ inline unsigned long long gapped(unsigned long long live, int rad, int gap) {
  const unsigned long long low = (1ull << rad) - 1;
  return (live & low) | (live & ~low) << gap;
}

// Lane r: the r-th set bit of live (bit 63 is not set); and that bit for any
// r, by every lane of the wave.  (In registers: a table in LDS would make the
// compiler wait for all loads to LDS in flight before each read of operands.)
__device__ inline int live_halves(unsigned long long live, int lane) {
  return __builtin_amdgcn_ds_permute(((live >> lane) & 1ull ? (int)lanes_below(live) : 63) << 2, lane);
}
__device__ inline int half_at(int halves, int r) { return __builtin_amdgcn_ds_bpermute(r << 2, halves); }

// Orders this wave's LDS writes before its later LDS reads by other lanes
// (LDS requests of one wave are served in order; this only stops the
// compiler from moving accesses across it).
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace nnp
