// Atomic environment vectors and their gradient (section "ANI models":
// cosine cutoff, radial and angular symmetry functions).
//
// One wavefront per centre atom (or a workgroup of four, where one per centre
// leaves the chip idle); for calls of several systems the waves take
// the centres of the largest systems first (wave_atom), so that no costly
// centre starts last.  The centre's neighbour entries (its list row, or for
// small systems without a list the atoms of its system) are re-derived from
// the packed atom records and sorted by neighbour species into LDS with wave
// ballots.  Then
//   radial:  lanes = 16 radial shifts x 4 neighbour slots, one species block
//            at a time, reduced across the 4 slots with lane shuffles;
//   angular (forward): the species-pair blocks, each padded to a multiple of
//            8 slots, one after another in passes of 64 pair slots:
//            (A) lane per slot: the pair geometry (cos and sin of the angle,
//                the 4 radial Gaussians of the mean distance times the
//                cutoff product) is computed once and staged in a per-wave
//                LDS scratch;
//            (B) lanes = 8 angle shifts x 8 slots, block by block: each lane
//                evaluates the cosine power of its angle shift for a pair
//                and accumulates the 4 radial-shift products; accumulators
//                are reduced across the 8 slots once a block's last pair is
//                done.
//            Blocks without a pair are written as zeros directly.
//   angular (backward): the pairs of all species-pair blocks form one
//            stream, one pair per lane; a lane evaluates all 8 angle shifts
//            of its pair against the block's dE/dG values (read from the
//            centre's row, which stays in the L1/L2 caches), recomputes the
//            angular cutoff of both legs, differentiates through cos, sin,
//            R_j and R_k, and accumulates dE/dd_j and dE/dd_k per neighbour
//            entry in the wave's LDS (float64 atomics, in a fixed order).
//            Forces then go to the accumulators in 64-bit fixed point.
// The backward keeps its LDS per wave near 7 KB (5 waves per SIMD at a
// neighbour capacity of 128) by recomputing the angular cutoffs and reading
// dE/dG from cache; its VALU issue, not memory, sets its time, so every
// instruction saved in the per-pair loop counts.
#include "internal.h"
#include "wave.h"

namespace nnp {

constexpr float kPi = 3.14159265358979323846f;

__device__ inline float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float fast_log2(float x) { return __builtin_amdgcn_logf(x); }


// Wave-uniform per-species counts and offsets of the sorted lists.
struct Lists {
  int cR[8], oR[8];
  int cA[8], oA[8];
};

// LDS layout of one wave's lists (cap entries each), pair-block table and
// pair scratch.
constexpr int kPairPass = kWave;  // neighbour pairs staged per pass
constexpr int kMaxBlocks = kMaxSpecies * (kMaxSpecies + 1) / 2;
constexpr int kMaxAng = kMaxBlocks * kAngBlock;  // 896 angular features

struct WaveLds {
  Lists *ls;       // per-species counts and offsets (wave-uniform)
  float2 *tGeo;    // pair scratch: cos, sin                      (forward)
  float4 *tF2;     // pair scratch: radial Gaussians of Rbar times
                   // fc_j fc_k                                     (forward)
  float4 *rD;      // radial: unit vector d / R and R
  float *rFc;      // radial: fc_rad(R)          (forward)
  float2 *rF2;     // fc(R) and fc'(R): radial cutoff, then (angular entries)
                   // the angular cutoff once the radial stage is done (backward)
  int *rJ;         // radial: neighbour index     (backward)
  double *rG;      // radial: dE/dd accumulators, float64 (backward, 3 per entry)
  int *aIdx;       // angular: position in the radial arrays  (backward)
  unsigned short *aIdx16;  // the same, 16-bit       (forward)
  float *aFc;      // angular: fc_ang(R)          (forward)
};

// Per-wave LDS bytes (a multiple of 16).  Forward entry: rD 16, rFc 4,
// aIdx16 2 (the array padded to 16 bytes), aFc 4: 4,992 bytes per wave at a
// capacity of 128, so that 8 waves per SIMD fit.  Backward entry: rD 16,
// rG 24, rF2 8, rJ 4, aIdx 4; the backward reads the centre's dE/dG row from
// global memory (it stays in the L1/L2 caches) and keeps the angular cutoff
// in the radial cutoff's slots: 7,296 bytes per wave at a capacity of 128
// (5 waves per SIMD).
__host__ __device__ inline size_t aidx16_bytes(int cap) { return ((size_t)cap * 2 + 15) / 16 * 16; }

template <bool BWD>
__host__ __device__ inline size_t wave_lds_bytes(int cap) {
  return sizeof(Lists) + (BWD ? (size_t)cap * (16 + 24 + 4 + 4 + 4 + 4)
                              : (size_t)kPairPass * (8 + 16) +
                                    (size_t)cap * (16 + 4 + 4) + aidx16_bytes(cap));
}

template <bool BWD>
__device__ inline WaveLds carve(char *base, int cap) {
  WaveLds w{};
  char *p = base;
  w.ls = (Lists *)p; p += sizeof(Lists);
  if (BWD) {
    w.rD = (float4 *)p; p += (size_t)cap * 16;
    w.rG = (double *)p; p += (size_t)cap * 24;
    w.rF2 = (float2 *)p; p += (size_t)cap * 8;
    w.rJ = (int *)p; p += (size_t)cap * 4;
    w.aIdx = (int *)p; p += (size_t)cap * 4;
  } else {
    w.tGeo = (float2 *)p; p += (size_t)kPairPass * 8;
    w.tF2 = (float4 *)p; p += (size_t)kPairPass * 16;
    w.rD = (float4 *)p; p += (size_t)cap * 16;
    w.rFc = (float *)p; p += (size_t)cap * 4;
    w.aIdx16 = (unsigned short *)p; p += aidx16_bytes(cap);
    w.aFc = (float *)p; p += (size_t)cap * 4;
  }
  return w;
}

// Lane b (< S (S + 1) / 2) describes species-pair block b of the centre's
// angular pairs, in the upper-triangle order of (sa, sb) that is also the
// feature order: its pair count T and the unrank fields of its two lists
// (a pair is addressed as (x, y), x in the longer species list of length n1,
// y in the shorter of length n2; a same-species block uses the one list for
// both; the angular term is symmetric in its two neighbours): oxy = offsets
// of the x and y lists (16 bits each), ns = n1 | n2 << 16 | same << 31,
// r2 = 1 / n2 (a hardware reciprocal, see unrank).
// Other lanes get T = 0.
__device__ inline void block_words(int lane, const Lists &ls, int S, int &bT, int &bOxy, int &bNs, float &bR2) {
  bT = 0;
  bOxy = 0;
  bNs = 0;
  bR2 = 1.f;
  if (lane < S * (S + 1) / 2) {
    int sa = 0, rem = lane;
#pragma unroll
    for (int s = 0; s < kMaxSpecies - 1; ++s)
      if (sa == s && rem >= S - s) { rem -= S - s; sa = s + 1; }
    const int sb = sa + rem;
    const int na = ls.cA[sa], nb = ls.cA[sb], oa = ls.oA[sa], ob = ls.oA[sb];
    const bool same = sa == sb;
    bT = same ? na * (na - 1) / 2 : na * nb;
    const bool a_long = na >= nb;
    const int n1 = max(na, nb), n2 = min(na, nb);
    bOxy = (a_long ? oa : ob) | ((a_long ? ob : oa) << 16);
    bNs = n1 | (n2 << 16) | (same ? (int)0x80000000u : 0);
    bR2 = fast_rcp((float)max(n2, 1));
  }
}

// List positions (ax, ay) of pair u of a block (ns and r2 as in
// block_words), with u = q n2 + y.  Two species: x = (y + q) mod n1, q < n1.
// One species of n entries (n1 = n2 = n): q < n / 2 and the pair is
// {y, (y + q + 1) mod n}, q + 1 being its distance around the list, so that
// every unordered pair comes once (for even n the last row q = n / 2 - 1
// holds only y < n / 2).  Either way y + q (+ 1) < 2 n1, and neighbouring
// lanes take different entries of both lists (their LDS adds to an entry's
// accumulators do not pile up on one address).  The quotient is that of
// (u + 1/2) r2, cut off: (u + 1/2) / n2 keeps 1 / (2 n2) from any integer,
// more than the rounding of r2 (two ulp) and of the product for every u and n2
// that lists of 1,025 entries allow.
__device__ inline void unrank(int u, int ns, float r2, int oxy, int &ax, int &ay) {
  const int n1 = ns & 0xffff, n2 = (ns >> 16) & 0x7fff;
  const int q = (int)(((float)u + 0.5f) * r2);
  const int y = u - (int)__umul24((unsigned)q, (unsigned)n2);
  const unsigned x = (unsigned)(y + q) + ((unsigned)ns >> 31);
  ax = (oxy & 0xffff) + (int)min(x, x - (unsigned)n1);
  ay = ((oxy >> 16) & 0xffff) + y;
}

// One neighbour entry of a centre: the atom (index within the system's
// records at j0), its species and the vector d (R in w); false for an entry
// past the row or whose stored atom index is not below n_sys (a reused list
// applied to a different system), which is never dereferenced.  self >= 0:
// no list; entry e is the system's atom e (n = n_sys), the centre (local
// index self) excluded.
__device__ __attribute__((always_inline)) inline bool load_entry(int e, int n, const int2 *__restrict__ ent,
                                                                 int self, int j0, int n_sys,
                                                                 const float4 *__restrict__ pos,
                                                                 const float4 &pi, const float L[3], int &sj, int &j,
                                                                 float4 &d) {
  int2 en = make_int2(0, 0);
  if (self >= 0) en = make_int2(e, pack_image(0, 0, 0));
  else if (e < n) en = ent[e];
  const bool v = e < n && (unsigned)en.x < (unsigned)n_sys && en.x != self;
  sj = -1;
  j = 0;
  d = make_float4(0.f, 0.f, 0.f, 1e30f);
  if (v) {
    j = j0 + en.x;
    const float4 pj = pos[j];
    d = entry_vec(pi, pj, en.y, L);
    sj = __float_as_int(pj.w);
  }
  return v;
}

// One entry (vector d, R in w) into slot q of the radial list and slot qa of
// the angular list.
template <bool BWD>
__device__ __attribute__((always_inline)) inline void put_entry(int q, int qa, bool inR, bool inA, int j,
                                                                const float4 &d, float kr, float ka, WaveLds &w) {
  if (inR) {
    float sn, cs;
    __sincosf(kr * d.w, &sn, &cs);
    // the pair geometry and the gradients need only the direction and R
    const float ir = fast_rcp(d.w);
    w.rD[q] = make_float4(d.x * ir, d.y * ir, d.z * ir, d.w);
    if (BWD) {
      w.rF2[q] = make_float2(0.5f * cs + 0.5f, -0.5f * kr * sn);
      w.rJ[q] = j;
    } else {
      w.rFc[q] = 0.5f * cs + 0.5f;
    }
  }
  if (inA) {
    if (BWD) w.aIdx[qa] = q;
    else w.aIdx16[qa] = (unsigned short)q;
    if (!BWD) w.aFc[qa] = 0.5f * __cosf(ka * d.w) + 0.5f;
  }
}

// fill_lists of rows of more than 128 entries: two passes over the entries,
// per-species counts by ballot, then placement.  Per-species tallies live in
// registers (loops over the species slots are fully unrolled; species without
// an entry in a chunk are skipped).
template <bool BWD>
__device__ inline void fill_lists_long(int lane, int n, const int2 *__restrict__ ent, int self, int j0, int n_sys,
                                       const float4 *__restrict__ pos, const float4 &pi,
                                       const float L[3], const AevConst &c, WaveLds &w) {
  const int S = c.S;
  const float rc2 = c.rc_r * c.rc_r;
  int cR[kMaxSpecies], cA[kMaxSpecies];
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s) { cR[s] = 0; cA[s] = 0; }
  for (int b = 0; b < n; b += kWave) {
    int sj, j;
    float4 d;
    load_entry(b + lane, n, ent, self, j0, n_sys, pos, pi, L, sj, j, d);
    const bool inR = sj >= 0 && d.w < c.rc_r && (self < 0 || d.x * d.x + d.y * d.y + d.z * d.z < rc2),
               inA = inR && d.w < c.rc_a;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      cR[s] += __popcll(__ballot(inR && sj == s));
      cA[s] += __popcll(__ballot(inA && sj == s));
    }
  }
  int pR[kMaxSpecies], pA[kMaxSpecies];
  {
    int oR = 0, oA = 0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      pR[s] = oR; oR += cR[s];
      pA[s] = oA; oA += cA[s];
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      w.ls->cR[s] = s < S ? cR[s] : 0; w.ls->oR[s] = pR[s];
      w.ls->cA[s] = s < S ? cA[s] : 0; w.ls->oA[s] = pA[s];
    }
  }
  const float kr = kPi / c.rc_r, ka = kPi / c.rc_a;
  (void)ka;
  for (int b = 0; b < n; b += kWave) {
    int sj, j;
    float4 d;
    load_entry(b + lane, n, ent, self, j0, n_sys, pos, pi, L, sj, j, d);
    const bool inR = sj >= 0 && d.w < c.rc_r && (self < 0 || d.x * d.x + d.y * d.y + d.z * d.z < rc2),
               inA = inR && d.w < c.rc_a;
    // slots of this lane's entry in the two lists (selects per species;
    // the stores below are then issued once, not once per species)
    int q = 0, qa = 0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      const unsigned long long mR = __ballot(inR && sj == s);
      if (!mR) continue;  // (the angular list is a subset of the radial one)
      const unsigned long long mA = __ballot(inA && sj == s);
      if (sj == s) {
        q = pR[s] + (int)lanes_below(mR);
        qa = pA[s] + (int)lanes_below(mA);
      }
      pR[s] += __popcll(mR);
      pA[s] += __popcll(mA);
    }
    put_entry<BWD>(q, qa, inR, inA, j, d, kr, ka, w);
  }
}

// Counts per species slot, a byte each: slots 0 to 3 in lo, 4 to 7 in hi.
struct Bytes8 {
  unsigned lo, hi;
  __device__ inline Bytes8 operator+(const Bytes8 &o) const { return {lo + o.lo, hi + o.hi}; }
};
__device__ inline int byte_of(const Bytes8 &v, int s) {
  return (int)__builtin_amdgcn_ubfe(s < 4 ? v.lo : v.hi, 8u * ((unsigned)s & 3u), 8u);
}
// Per lane: how many of the lanes up to it are in, by species (hi only where
// there can be a slot above 3).
__device__ inline Bytes8 species_scan(bool in, int s, bool many) {
  const unsigned one = in ? 1u << (8u * ((unsigned)s & 3u)) : 0u;
  Bytes8 v = {s < 4 ? one : 0u, 0u};
  v.lo = wave_scan(v.lo);
  if (many) v.hi = wave_scan(s < 4 ? 0u : one);
  return v;
}
__device__ inline Bytes8 last_lane(const Bytes8 &v) {
  return {(unsigned)__builtin_amdgcn_readlane((int)v.lo, kWave - 1),
          (unsigned)__builtin_amdgcn_readlane((int)v.hi, kWave - 1)};
}
// Sums over the slots below each.
__device__ inline Bytes8 slots_below(const Bytes8 &v) {
  return {v.lo * 0x01010100u, v.hi * 0x01010100u + (v.lo * 0x01010101u >> 24) * 0x01010101u};
}

// Builds the species-sorted radial list (R < rc_r) and angular list
// (R < rc_a, a subset) of centre i in LDS from its neighbour row, or (self
// >= 0) from all atoms of its system, keeping those a list would hold (R^2
// below rc_r^2 as the list build tests it).  The wave-uniform counts and
// offsets are published in LDS.
// Rows of up to 128 entries (the common case): the entries stay in registers,
// and an entry's slot is its place among the lanes of its species, by a scan
// over the wave of byte counters (about 40 instructions per 64 entries and
// list, where a ballot per species and pass took 110).
template <bool BWD>
__device__ inline void fill_lists(int lane, int n, const int2 *__restrict__ ent, int self, int j0, int n_sys,
                                  const float4 *__restrict__ pos, const float4 &pi,
                                  const float L[3], const AevConst &c, WaveLds &w) {
  if (n > 2 * kWave) {
    fill_lists_long<BWD>(lane, n, ent, self, j0, n_sys, pos, pi, L, c, w);
    return;
  }
  const float rc2 = c.rc_r * c.rc_r;
  const bool two = n > kWave, many = c.S > 4;
  int s0 = -1, s1 = -1, j_0 = 0, j_1 = 0;
  float4 d0 = make_float4(0.f, 0.f, 0.f, 1e30f), d1 = d0;
  load_entry(lane, n, ent, self, j0, n_sys, pos, pi, L, s0, j_0, d0);
  if (two) load_entry(kWave + lane, n, ent, self, j0, n_sys, pos, pi, L, s1, j_1, d1);
  auto in_radial = [&](int s, const float4 &d) {
    return s >= 0 && d.w < c.rc_r && (self < 0 || d.x * d.x + d.y * d.y + d.z * d.z < rc2);
  };
  const bool r0 = in_radial(s0, d0), a0 = r0 && d0.w < c.rc_a;
  const Bytes8 scR0 = species_scan(r0, s0, many), scA0 = species_scan(a0, s0, many);
  const Bytes8 tR0 = last_lane(scR0), tA0 = last_lane(scA0);
  bool r1 = false, a1 = false;
  Bytes8 scR1 = {0u, 0u}, scA1 = scR1, tR = tR0, tA = tA0;
  if (two) {
    r1 = in_radial(s1, d1);
    a1 = r1 && d1.w < c.rc_a;
    scR1 = species_scan(r1, s1, many);
    scA1 = species_scan(a1, s1, many);
    tR = tR + last_lane(scR1);
    tA = tA + last_lane(scA1);
  }
  const Bytes8 oR = slots_below(tR), oA = slots_below(tA);
  if (lane < 8) {
    w.ls->cR[lane] = byte_of(tR, lane);
    w.ls->oR[lane] = byte_of(oR, lane);
    w.ls->cA[lane] = byte_of(tA, lane);
    w.ls->oA[lane] = byte_of(oA, lane);
  }
  const float kr = kPi / c.rc_r, ka = kPi / c.rc_a;
  put_entry<BWD>(byte_of(scR0 + oR, s0) - 1, byte_of(scA0 + oA, s0) - 1, r0, a0, j_0, d0, kr, ka, w);
  if (two)
    put_entry<BWD>(byte_of(scR1 + (oR + tR0), s1) - 1, byte_of(scA1 + (oA + tA0), s1) - 1, r1, a1, j_1, d1, kr, ka, w);
}

// A workgroup of W waves at one centre (W = 1: a wave on its own): orders the
// LDS writes of all of them before their later reads.
template <int W> __device__ inline void centre_sync() {
  if constexpr (W == 1) {
    wave_lds_sync();
  } else {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// fill_lists by the W waves of a workgroup: wave v takes the row's 64-entry
// chunks v, v + W, ...; the chunks' species counts meet in LDS (cnt, kChunkCounts
// bytes a chunk), and every entry lands where the one-wave form puts it.  The
// counts lie in the forward's pair scratch, and in the backward where the 24
// bytes per entry of dE/dd follow: n entries, at most one more than the
// capacity, come in at most (capacity + 64) / 64 chunks, and no capacity is
// below 4.
constexpr int kMaxChunks = 1024 / kWave + 1;  // rows hold at most 1,024 entries, systems without a list one more
constexpr int kChunkCounts = 16 * sizeof(int);
static_assert(kChunkCounts == kWave && 24 * 4 >= 4 + kChunkCounts, "chunk counts of the backward");
template <bool BWD, int W>
__device__ inline void fill_lists_group(int wave, int lane, int n, const int2 *__restrict__ ent, int self, int j0,
                                        int n_sys, const float4 *__restrict__ pos, const float4 &pi,
                                        const float L[3], const AevConst &c, WaveLds &w, int *cnt) {
  const int S = c.S;
  const float rc2 = c.rc_r * c.rc_r;
  auto load = [&](int b, int &sj, int &j, float4 &d, bool &inR, bool &inA) {
    load_entry(b + lane, n, ent, self, j0, n_sys, pos, pi, L, sj, j, d);
    inR = sj >= 0 && d.w < c.rc_r && (self < 0 || d.x * d.x + d.y * d.y + d.z * d.z < rc2);
    inA = inR && d.w < c.rc_a;
  };
  // the wave's first chunk stays in registers for both passes
  int sj0 = -1, jj0 = 0;
  float4 d0 = make_float4(0.f, 0.f, 0.f, 1e30f);
  bool inR0 = false, inA0 = false;
  const bool many = S > 4;
  Bytes8 scR0 = {0u, 0u}, scA0 = scR0;
  const int b0 = wave * kWave;
  if (b0 < n) load(b0, sj0, jj0, d0, inR0, inA0);
  for (int b = b0; b < n; b += W * kWave) {
    int sj = sj0, j = jj0;
    float4 d = d0;
    bool inR = inR0, inA = inA0;
    if (b != b0) load(b, sj, j, d, inR, inA);
    const Bytes8 scR = species_scan(inR, sj, many), scA = species_scan(inA, sj, many);
    if (b == b0) {
      scR0 = scR;
      scA0 = scA;
    }
    // lane s: radial entries of species s, lane 8 + s: angular ones
    const Bytes8 tR = last_lane(scR), tA = last_lane(scA);
    if (lane < 16) cnt[(b / kWave) * 16 + lane] = byte_of(lane < 8 ? tR : tA, lane & 7);
  }
  centre_sync<W>();
  // lane s / 8 + s: the species' total, then its first slot in the list
  const int chunks = (n + kWave - 1) / kWave;
  int tot = 0;
  if (lane < 16)
    for (int k = 0; k < chunks; ++k) tot += cnt[k * 16 + lane];
  int first = tot;
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    const int y = __shfl_up(first, d, 8);
    if ((lane & 7) >= d) first += y;
  }
  first -= tot;
  if (wave == 0 && lane < 16) {
    int *t = (lane < 8 ? w.ls->cR : w.ls->cA) + (lane & 7);
    t[0] = (lane & 7) < S ? tot : 0;
    t[8] = first;  // oR / oA follow cR / cA
  }
  const float kr = kPi / c.rc_r, ka = kPi / c.rc_a;
  (void)ka;
  int done = 0;  // chunks before b, summed into `first` so far
  for (int b = b0; b < n; b += W * kWave) {
    if (lane < 16)
      for (; done < b / kWave; ++done) first += cnt[done * 16 + lane];
    done = b / kWave;
    int sj = sj0, j = jj0;
    float4 d = d0;
    bool inR = inR0, inA = inA0;
    Bytes8 scR = scR0, scA = scA0;
    if (b != b0) {
      load(b, sj, j, d, inR, inA);
      scR = species_scan(inR, sj, many);
      scA = species_scan(inA, sj, many);
    }
    const int q = __shfl(first, sj & 7) + byte_of(scR, sj) - 1, qa = __shfl(first, 8 + (sj & 7)) + byte_of(scA, sj) - 1;
    put_entry<BWD>(q, qa, inR, inA, j, d, kr, ka, w);
  }
}

// Element k of a small constant table for a lane-dependent k, by selects
// (a dynamically indexed kernel argument would go through scratch memory).
template <int N> __device__ inline float pick(const float (&t)[N], int k) {
  float v = t[0];
#pragma unroll
  for (int q = 1; q < N; ++q) v = k == q ? t[q] : v;
  return v;
}

__device__ inline uint32_t bf16_pair(float lo, float hi) {
  uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
  a += 0x7fffu + ((a >> 16) & 1u);
  b += 0x7fffu + ((b >> 16) & 1u);
  return (a >> 16) | (b & 0xffff0000u);
}

// Eight consecutive features (row offset k, a multiple of 8) from LDS to the
// feature row in one 16-byte (bfloat16) or two 16-byte (float32) stores.
template <bool BF16> __device__ inline void store8(void *row, int k, const float *v);
template <> __device__ inline void store8<true>(void *row, int k, const float *v) {
  uint4 o;
  o.x = bf16_pair(v[0], v[1]); o.y = bf16_pair(v[2], v[3]);
  o.z = bf16_pair(v[4], v[5]); o.w = bf16_pair(v[6], v[7]);
  *(uint4 *)((uint16_t *)row + k) = o;
}
template <> __device__ inline void store8<false>(void *row, int k, const float *v) {
  float4 *d = (float4 *)((float *)row + k);
  d[0] = make_float4(v[0], v[1], v[2], v[3]);
  d[1] = make_float4(v[4], v[5], v[6], v[7]);
}

// One feature (row offset k) to the feature row, rounded to bfloat16 the
// same way as bf16_pair.  The lanes of a wave that store together cover
// contiguous features, so the stores combine into full segments.
template <bool BF16> __device__ inline void store1(void *row, int k, float v);
template <> __device__ inline void store1<true>(void *row, int k, float v) {
  uint32_t a = __float_as_uint(v);
  a += 0x7fffu + ((a >> 16) & 1u);
  ((uint16_t *)row)[k] = (uint16_t)(a >> 16);
}
template <> __device__ inline void store1<false>(void *row, int k, float v) { ((float *)row)[k] = v; }

// Bit p of x (p < 32) to bits 2 p and 2 p + 1.
__device__ inline unsigned long long spread_pairs(unsigned long long x) {
  x &= 0xffffffffull;
  x = (x | (x << 16)) & 0x0000ffff0000ffffull;
  x = (x | (x << 8)) & 0x00ff00ff00ff00ffull;
  x = (x | (x << 4)) & 0x0f0f0f0f0f0f0f0full;
  x = (x | (x << 2)) & 0x3333333333333333ull;
  x = (x | (x << 1)) & 0x5555555555555555ull;
  return x | (x << 1);
}
// The row mask's halves: a radial block is one 16-column half, an angular
// block two, and all of them fit in 64 bits.
static_assert(kNShfRad == 16 && kAngBlock == 32, "row mask halves");
static_assert(kMaxSpecies + kMaxSpecies * (kMaxSpecies + 1) <= 64, "row mask width");

// The issue of vector instructions bounds it (97% of the cycles on 512 ragged
// solutes, 67 neighbours and 830 pairs per centre).  Of 3,900 instructions per
// centre 450 went into the sorted lists and 80 into each pass of pair geometry;
// with byte-counter scans, a quotient that needs no correction and blocks that
// run on over the passes (14 in place of 16.4) there are 3,450: 512 solutes 205
// -> 190 us, 4,096 snapshots of 40 atoms 730 -> 608, a box of 100,002 atoms 197
// -> 169.
//
// Several waves per centre (GROUP): for calls with fewer centres than the chip
// has SIMDs, where a centre's chain of passes is the call's latency, and for
// neighbour capacities whose lists leave too few waves on a compute unit.  The
// waves share the centre's lists; the radial species and the species-pair
// blocks are dealt out over them, each block whole to one wave, so that every
// sum is formed as by one wave.
template <int WPB, bool BF16, bool GROUP>
__global__ void __launch_bounds__(WPB * kWave)
k_aev_fwd(const float4 *__restrict__ pos, const int *__restrict__ sys_of,
          const SysDesc *__restrict__ sys, const int2 *__restrict__ nbr,
          const int *__restrict__ nbr_cnt, int cap, const int *__restrict__ row_of_atom,
          void *__restrict__ G, int ldg, unsigned long long *__restrict__ row_mask,
          const int *__restrict__ wave_atom, int *__restrict__ status, Live N_, int xcd_run, AevConst c) {
  extern __shared__ float4 lds4[];
  const int N = N_.get();
  // the wave index is uniform across the wave: keep it (and the centre's
  // index, descriptors and row pointers) in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  constexpr int W = GROUP ? WPB : 1;  // waves per centre
  const int wv = GROUP ? (int)blockIdx.x : xcd_chunked(blockIdx.x, xcd_run) * WPB + wave;
  const int i = wave_atom && wv < N ? __builtin_amdgcn_readfirstlane(wave_atom[wv]) : wv;
  // an atom without a network row (outside a caller's mask) is skipped
  const bool live = i < N && row_of_atom[i] >= 0;
  WaveLds w = carve<false>((char *)lds4 + (GROUP ? 0 : wave * wave_lds_bytes<false>(cap)), cap);
  int *cnt = nullptr;
  if (GROUP) {
    // the waves' pair scratch follows the lists (the chunk counts use it first)
    char *scratch = (char *)lds4 + wave_lds_bytes<false>(cap);
    cnt = (int *)scratch;
    w.tGeo = (float2 *)(scratch + wave * kPairPass * 24);
    w.tF2 = (float4 *)(scratch + wave * kPairPass * 24 + kPairPass * 8);
  }
  float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
  float L[3] = {0.f, 0.f, 0.f};
  int n = 0, j0 = 0, n_sys = 0, self = -1;
  const int2 *row = nbr;
  if (live) {
    const SysDesc &d = sys[sys_of[i]];
    n_sys = d.n;
    pi = pos[i];
    L[0] = d.L[0]; L[1] = d.L[1]; L[2] = d.L[2];
    j0 = d.atom_off;
    if (nbr) {
      n = min(nbr_cnt[d.state_off + (i - d.atom_off)], cap);
      row = nbr + nbr_row(d, i, cap);
    } else {
      n = n_sys;  // no list: the system's atoms
      self = i - d.atom_off;
    }
  }
  if constexpr (GROUP) fill_lists_group<false, W>(wave, lane, n, row, self, j0, n_sys, pos, pi, L, c, w, cnt);
  else fill_lists<false>(lane, n, row, self, j0, n_sys, pos, pi, L, c, w);
  __syncthreads();
  if (!live) return;
  const Lists &ls = *w.ls;
  // without a list, the largest neighbour count (what the list build
  // records) goes to status[1]: the current value is read here and compared
  // at the end, so that the wave does not wait for it
  int nb_cnt = 0, nb_max = 0;
  if (status && (!GROUP || wave == 0)) {
    for (int s = 0; s < c.S; ++s) nb_cnt += ls.cR[s];
    nb_max = __hip_atomic_load(status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int r_i = row_of_atom[i];
  void *Grow = (char *)G + (size_t)r_i * ldg * (BF16 ? 2 : 4);

  // radial: G[16 s + m] = scale * sum_j exp(-eta (R - Rs_m)^2) fc(R)
  // lanes = 16 shifts x 4 neighbour slots (slot fastest)
  {
    const int m = lane >> 2, slot = lane & 3;
    const float shf = pick(c.shf_r, m);
    const float keta = -c.eta_r * 1.4426950408889634f;
    for (int s = GROUP ? wave : 0; s < c.S; s += W) {
      float acc = 0.f;
      const int o = ls.oR[s];
      const int cnt = ls.cR[s];
      // no branch per entry: slots past the end re-read the last entry
      // and add it with a zero weight
      for (int e0 = 0; e0 < cnt; e0 += 4) {
        const int e = e0 + slot;
        const int q = o + min(e, cnt - 1);
        const float t = w.rD[q].w - shf;
        acc += fast_exp2(keta * t * t) * (e < cnt ? w.rFc[q] : 0.f);
      }
      acc = sum4(acc);
      if (slot == 0) store1<BF16>(Grow, s * kNShfRad + m, acc * c.scale);
    }
  }

  // angular: G[rad_len + 32 p + 8 r + a] = sum over pairs {j, k} of
  //   2^(1-zeta) (1 + cos(theta - theta_a))^zeta exp(-eta (Rbar - Rs_r)^2) fc_j fc_k
  {
    const int a = lane >> 3, t0 = lane & 7;  // phase B: 8 angle shifts x 8 pairs (pair fastest)
    // y = (1 + cos(theta - theta_a)) / 2 in [0, 1] (clamped by its own FMA),
    // so that 2^(1-zeta) (1 + cos)^zeta = 2 y^zeta = 2^(zeta log2 y + 1)
    const float hcz = pick(c.hcz, a), hsz = pick(c.hsz, a);
    const float keta = -c.eta_a * 1.4426950408889634f;
    // lane b: species-pair block b (block_words)
    const int n_blk = c.S * (c.S + 1) / 2;
    int bT, bOxy, bNs;
    float bR2;
    block_words(lane, ls, c.S, bT, bOxy, bNs, bR2);
    const unsigned long long nonempty = __ballot(bT > 0);
    // the row's record of its possibly non-zero halves: radial species with
    // an entry, species pairs with a pair
    if (row_mask) {
      const unsigned long long radial = __ballot(lane < c.S && ls.cR[min(lane, kMaxSpecies - 1)] > 0);
      if (lane == 0 && (!GROUP || wave == 0)) row_mask[r_i] = radial | spread_pairs(nonempty) << c.S;
    }
    // blocks without a pair of their two species are zero: written in one
    // pass of 16-byte stores over the angular part of the row
    {
      constexpr int kChunksPerBlock = kAngBlock * (BF16 ? 2 : 4) / 16;
      uint4 *ang = (uint4 *)((char *)Grow + (size_t)c.rad_len * (BF16 ? 2 : 4));
      for (int k = GROUP ? (int)threadIdx.x : lane; k < n_blk * kChunksPerBlock; k += W * kWave)
        if (!((nonempty >> (k / kChunksPerBlock)) & 1ull)) ang[k] = make_uint4(0u, 0u, 0u, 0u);
    }
    // Passes of 64 pair slots, eight groups of 8, over the stream of the
    // blocks' pairs; every block is padded to whole groups, and a block that
    // does not end in a pass goes on in the next one.
    float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
    int bG = (bT + 7) >> 3;  // lane b: groups of block b
    if constexpr (GROUP) {
      // the blocks whose middle lies in this wave's share of all pair slots
      const int end = 8 * (int)wave_scan((unsigned)bG);
      const int total = __builtin_amdgcn_readlane(end, kWave - 1), mid = end - ((bT + 7) >> 1);
      const bool mine = min((int)((float)mid * (float)W * fast_rcp((float)max(total, 1))), W - 1) == wave;
      bG = mine ? bG : 0;
    }
    const int gEnd = (int)wave_scan((unsigned)bG), gStart = gEnd - bG;
    const int n_groups = __builtin_amdgcn_readlane(gEnd, kWave - 1);
    const unsigned long long todo = __ballot(bG > 0);
    int qb = todo ? __builtin_ctzll(todo) : 0;  // the block of the pass's first group
    for (int base = 0; base < n_groups; base += kPairPass / 8) {
      // this lane's block: the last one that starts at or before its group
      const int gi = base + a;
      int p = qb;
      for (unsigned long long m = todo & (~0ull << (qb + 1)); m; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        const int sr = __builtin_amdgcn_readlane(gStart, r);
        if (sr >= base + kPairPass / 8) break;
        p = gi >= sr ? r : p;
      }
      const int pa = p << 2;
      const int l_oxy = __builtin_amdgcn_ds_bpermute(pa, bOxy);
      const int l_ns = __builtin_amdgcn_ds_bpermute(pa, bNs);
      const float l_r2 = __int_as_float(__builtin_amdgcn_ds_bpermute(pa, __float_as_int(bR2)));
      const int l_T = __builtin_amdgcn_ds_bpermute(pa, bT);
      const int l_u = 8 * (gi - __builtin_amdgcn_ds_bpermute(pa, gStart)) + t0;
      // (A) lane per pair slot; padding slots (and slots past the pass's
      // blocks) repeat a valid pair with a zero cutoff product
      {
        const bool valid = gi < n_groups && l_u < l_T;
        const int tt = min(l_u, l_T - 1);
        int qj, qk;
        unrank(tt, l_ns, l_r2, l_oxy, qj, qk);
        const float4 dj = w.rD[w.aIdx16[qj]], dk = w.rD[w.aIdx16[qk]];  // unit vectors, R
        const float cosv = dj.x * dk.x + dj.y * dk.y + dj.z * dk.z;
        const float cx = dj.y * dk.z - dj.z * dk.y;
        const float cy = dj.z * dk.x - dj.x * dk.z;
        const float cz = dj.x * dk.y - dj.y * dk.x;
        const float sinv = fast_sqrt(cx * cx + cy * cy + cz * cz);
        const float fcc = valid ? w.aFc[qj] * w.aFc[qk] : 0.f;
        const float Rbar = 0.5f * (dj.w + dk.w);
        const float u0 = Rbar - c.shf_a[0], u1 = Rbar - c.shf_a[1];
        const float u2 = Rbar - c.shf_a[2], u3 = Rbar - c.shf_a[3];
        w.tGeo[lane] = make_float2(cosv, sinv);
        w.tF2[lane] = make_float4(fcc * fast_exp2(keta * u0 * u0), fcc * fast_exp2(keta * u1 * u1),
                                  fcc * fast_exp2(keta * u2 * u2), fcc * fast_exp2(keta * u3 * u3));
      }
      wave_lds_sync();
      // (B) per block of the pass, its groups of 8 slots two at a time; a
      // block's accumulators are reduced across the 8 pairs and stored once
      // its last pair is done
      {
        int g = 0;
        const int used = min(n_groups - base, kPairPass / 8);
        while (g < used) {
          const int k = qb, end = __builtin_amdgcn_readlane(gEnd, k) - base;
          const int gend = min(end, used);
          for (; g + 2 <= gend; g += 2) {
            const int q0 = 8 * g + t0, q1 = q0 + 8;
            const float2 geo0 = w.tGeo[q0], geo1 = w.tGeo[q1];
            const float4 f20 = w.tF2[q0], f21 = w.tF2[q1];
            const float y0 = __builtin_amdgcn_fmed3f(fmaf(geo0.x, hcz, fmaf(geo0.y, hsz, 0.5f)), 0.f, 1.f);
            const float y1 = __builtin_amdgcn_fmed3f(fmaf(geo1.x, hcz, fmaf(geo1.y, hsz, 0.5f)), 0.f, 1.f);
            const float v0 = fast_exp2(c.zeta * fast_log2(y0) + 1.0f);
            const float v1 = fast_exp2(c.zeta * fast_log2(y1) + 1.0f);
            acc0 += v0 * f20.x; acc0 += v1 * f21.x;
            acc1 += v0 * f20.y; acc1 += v1 * f21.y;
            acc2 += v0 * f20.z; acc2 += v1 * f21.z;
            acc3 += v0 * f20.w; acc3 += v1 * f21.w;
          }
          if (g < gend) {
            const int q0 = 8 * g + t0;
            const float2 geo = w.tGeo[q0];
            const float4 f2 = w.tF2[q0];
            const float y = __builtin_amdgcn_fmed3f(fmaf(geo.x, hcz, fmaf(geo.y, hsz, 0.5f)), 0.f, 1.f);
            const float v = fast_exp2(c.zeta * fast_log2(y) + 1.0f);
            acc0 += v * f2.x; acc1 += v * f2.y; acc2 += v * f2.z; acc3 += v * f2.w;
            ++g;
          }
          if (end <= used) {
            // sums over the 8 slot lanes of each angle shift, halving the
            // values in flight at each step: the two quads of the 8 lanes
            // swap halves (r 0, 1 stay low, r 2, 3 high), then the lane
            // pairs of a quad, then neighbours add; lane t0 ends with
            // r = 2 (t0 >> 2) + ((t0 >> 1) & 1)
            const bool hi = t0 >= 4, b1 = (t0 >> 1) & 1;
            const float A = (hi ? acc2 : acc0) + dpp<0x141>(hi ? acc0 : acc2);  // row_half_mirror
            const float B = (hi ? acc3 : acc1) + dpp<0x141>(hi ? acc1 : acc3);
            float C = (b1 ? B : A) + dpp<0x4E>(b1 ? A : B);                      // quad_perm [2,3,0,1]
            C += dpp<0xB1>(C);                                                   // quad_perm [1,0,3,2]
            if (!(t0 & 1)) {
              const int r = 2 * (t0 >> 2) + ((t0 >> 1) & 1);
              store1<BF16>(Grow, c.rad_len + k * kAngBlock + kNShfZ * r + a, C);
            }
            acc0 = acc1 = acc2 = acc3 = 0.f;
            const unsigned long long next = todo & (~0ull << (k + 1));
            if (next) qb = __builtin_ctzll(next);
          }
        }
      }
      wave_lds_sync();
    }
  }
  if (status && lane == 0 && nb_cnt > nb_max) atomicMax(status + 1, nb_cnt);
}

// Where the force contributions of a centre go.  Forces accumulate in 64-bit
// fixed point (fixed.h) in the buffer Ffix[N][3], which the caller clears
// first and converts to float32 afterwards: integer sums do not depend on the
// order in which waves add into them, so forces come out the same bit for
// bit whatever else the batch holds.  Atom j of system d accumulates in slot
// j + fix_shift(d) = d.order_off + (j - d.atom_off): the systems in the
// order their centres are launched, so that the waves running together add
// into neighbouring slots (scattered slots made these device atomics
// several times slower).
//   SinkGlobal: device-scope integer atomics straight into Ffix;
//   SinkSys:    an LDS table of one system's atoms (index j - atom_off),
//               added into Ffix once per workgroup;
//   SinkHash:   an LDS hash table keyed by atom index (open addressing,
//               linear probing), added into Ffix once per workgroup; an atom
//               that finds no free slot within kBwdProbe probes goes
//               straight to Ffix.
//   SinkGlobal takes single components (add1): the device atomics bound the
//   backward of a large box, and lanes that take the three components of one
//   atom add into one memory line together.  A wave's adds of an x, then a y,
//   then a z per lane went to three times as many lines: 100,002 atoms in a
//   box 531 -> 301 us, 12,003 68 -> 47, 6,000 of a pair list 63 -> 35.
struct SinkGlobal {
  static constexpr bool kByComponent = true;
  unsigned long long *F;
  int shift;  // fix_shift of the system
  __device__ inline void add1(int j, int k, long long v) const {
    atomicAdd(F + 3 * (size_t)(j + shift) + k, (unsigned long long)v);
  }
  __device__ inline void add(int j, long long x, long long y, long long z) const {
    unsigned long long *p = F + 3 * (size_t)(j + shift);
    atomicAdd(p, (unsigned long long)x);
    atomicAdd(p + 1, (unsigned long long)y);
    atomicAdd(p + 2, (unsigned long long)z);
  }
};
struct SinkSys {
  static constexpr bool kByComponent = false;
  unsigned long long *tab;
  int off;
  __device__ inline void add(int j, long long x, long long y, long long z) const {
    unsigned long long *p = tab + 3 * (j - off);
    atomicAdd(p, (unsigned long long)x);
    atomicAdd(p + 1, (unsigned long long)y);
    atomicAdd(p + 2, (unsigned long long)z);
  }
};
constexpr int kBwdHashBits = 9;
constexpr int kBwdHash = 1 << kBwdHashBits;  // slots: a cell's neighbourhood holds ~300-450 atoms
constexpr int kBwdProbe = 32;
constexpr int kBwdMinCells = 512;  // cells of a grid for the per-cell form
constexpr size_t kBwdStaticLds = 64;  // bytes kept for static LDS of the grouped forms
struct SinkHash {
  static constexpr bool kByComponent = false;
  int *key;
  unsigned long long *val;
  unsigned long long *F;
  int shift;  // fix_shift of the system
  __device__ inline void add(int j, long long x, long long y, long long z) const {
    unsigned h = ((unsigned)j * 2654435761u) >> (32 - kBwdHashBits);
    for (int probe = 0; probe < kBwdProbe; ++probe) {
      int k = key[h];
      if (k == -1) k = atomicCAS(&key[h], -1, j);  // -1: this lane claimed the slot
      if (k == -1 || k == j) {
        unsigned long long *p = val + 3 * h;
        atomicAdd(p, (unsigned long long)x);
        atomicAdd(p + 1, (unsigned long long)y);
        atomicAdd(p + 2, (unsigned long long)z);
        return;
      }
      h = (h + 1) & (kBwdHash - 1);
    }
    SinkGlobal{F, shift}.add(j, x, y, z);
  }
};

// Backward of centre i by one wave (W = 1; wave-uniform i, no workgroup
// barrier, so waves of one workgroup may work on different centres) or by the
// W waves of a workgroup (see k_aev_fwd), which share the lists: dE/dd of every
// radial entry from the radial and angular terms, the centre's virial row
// W_atom[i] = -sum d (x) dE/dd (where asked for), and its force contributions through sink:
// -dE/dd onto each neighbour, the sum of dE/dd onto the centre.
template <int W, class Sink>
__device__ inline void bwd_centre(int i, int wave, int lane, const float4 *__restrict__ pos, const int *__restrict__ sys_of,
                                  const SysDesc *__restrict__ sys, const int2 *__restrict__ nbr,
                                  const int *__restrict__ nbr_cnt, int cap, const int *__restrict__ row_of_atom,
                                  const float *__restrict__ dG, int ldg, const AevConst &c,
                                  float *__restrict__ W_atom, WaveLds &w, const Sink &sink) {
  // an atom without a network row (outside a caller's mask) is skipped; its
  // virial share is zero
  const int r_i = row_of_atom[i];
  if (r_i < 0) {
    if (W_atom && lane < 9 && wave == 0) W_atom[(size_t)9 * i + lane] = 0.f;
    return;
  }
  const SysDesc &d = sys[sys_of[i]];
  const int n_sys = d.n;
  // no list (nbr null): the system's atoms
  const int n = nbr ? min(nbr_cnt[d.state_off + (i - d.atom_off)], cap) : n_sys;
  const int self = nbr ? -1 : i - d.atom_off;
  const float4 pi = pos[i];
  const float L[3] = {d.L[0], d.L[1], d.L[2]};
  const int j0 = d.atom_off;
  const int2 *row = nbr ? nbr + nbr_row(d, i, cap) : nbr;
  // (the chunk counts of a group lie where the dE/dd accumulators follow)
  if constexpr (W > 1) fill_lists_group<true, W>(wave, lane, n, row, self, j0, n_sys, pos, pi, L, c, w, (int *)w.rG);
  else fill_lists<true>(lane, n, row, self, j0, n_sys, pos, pi, L, c, w);
  centre_sync<W>();
  const int first_e = wave * kWave + lane;  // this lane's first entry of a list
  const Lists &ls = *w.ls;
  const float *g = dG + (size_t)r_i * ldg;
  int nR = 0;
  for (int s = 0; s < c.S; ++s) nR += ls.cR[s];
  // radial, lane per neighbour entry: with t_m = R - Rs_m and
  // e_m = exp(-eta t_m^2), dE/dR = scale (fc' sum_m g_m e_m - 2 eta fc
  // sum_m g_m e_m t_m), g being the dE/dG values of the entry's species;
  // dE/dd = dE/dR d / R.  This stage is the first writer of the dE/dd
  // accumulators.
  {
    const float keta = -c.eta_r * 1.4426950408889634f;
    for (int e = first_e; e < nR; e += W * kWave) {
      int sp = 0;
#pragma unroll
      for (int s = 1; s < kMaxSpecies; ++s) sp += e >= ls.oR[s] ? 1 : 0;
      const float4 d = w.rD[e];
      const float2 fc = w.rF2[e];
      const float4 *gs = (const float4 *)(g + sp * kNShfRad);
      float A = 0.f, B = 0.f;
#pragma unroll
      for (int h = 0; h < kNShfRad / 4; ++h) {
        const float4 gv = gs[h];
        const float gm[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float t = d.w - c.shf_r[4 * h + k];
          const float ge = gm[k] * fast_exp2(keta * t * t);
          A += ge;
          B += ge * t;
        }
      }
      const float dEdR = c.scale * (fc.y * A - 2.0f * c.eta_r * fc.x * B);
      double *gg = w.rG + 3 * e;
      gg[0] = (double)(dEdR * d.x); gg[1] = (double)(dEdR * d.y); gg[2] = (double)(dEdR * d.z);
    }
  }
  centre_sync<W>();

  // angular cutoff of every angular entry, into its radial cutoff slot (the
  // radial stage above was the last reader of those)
  {
    const float ka = kPi / c.rc_a;
    int nA = 0;
    for (int s = 0; s < c.S; ++s) nA += ls.cA[s];
    for (int e = first_e; e < nA; e += W * kWave) {
      const int q = w.aIdx[e];
      float sn, cs;
      __sincosf(ka * w.rD[q].w, &sn, &cs);
      w.rF2[q] = make_float2(0.5f * cs + 0.5f, -0.5f * ka * sn);
    }
  }
  centre_sync<W>();

  // angular: lane per neighbour pair over the pair stream of all blocks
  // (the blocks' pairs one after another, in feature order)
  {
    const float *gA = g + c.rad_len;
    // lane b: species-pair block b, with the first pair of the block in the
    // stream (an exclusive prefix sum of the counts over the lanes)
    int bT, bOxy, bNs;
    float bR2;
    block_words(lane, ls, c.S, bT, bOxy, bNs, bR2);
    const int bEnd = (int)wave_scan((unsigned)bT), bStart = bEnd - bT;
    const int P = __builtin_amdgcn_readlane(bEnd, kWave - 1);
    const float zm1 = c.zeta - 1.0f;
    const float keta = -c.eta_a * 1.4426950408889634f;
    const float m2eta = -2.0f * c.eta_a;
    // the non-empty block holding the pass's first pair (wave-uniform);
    // the block searches visit non-empty blocks only
    const unsigned long long nonempty = __ballot(bT > 0);
    int qb = nonempty ? __builtin_ctzll(nonempty) : 0;
    for (int round = 0; round < P; round += W * kPairPass) {
      const int base = round + wave * kPairPass;  // (W > 1: possibly past the end, in the last round)
      for (unsigned long long m = nonempty & (~0ull << (qb + 1)); m; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        if (__builtin_amdgcn_readlane(bStart, r) > base) break;
        qb = r;
      }
      const bool valid = base + lane < P;
      const int t = min(base + lane, P - 1);
      // (the pass's values; the adds below take the waves' passes in turn)
      float gjx = 0.f, gjy = 0.f, gjz = 0.f, gkx = 0.f, gky = 0.f, gkz = 0.f;
      // this lane's block: the last non-empty one starting at or before its
      // pair; the pass's blocks are few, their starts wave-uniform
      int p = qb;
      for (unsigned long long m = nonempty & (~0ull << (qb + 1)); m; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        const int sr = __builtin_amdgcn_readlane(bStart, r);
        if (sr >= base + kPairPass) break;
        p = t >= sr ? r : p;
      }
      const int pa = p << 2;
      const int l_oxy = __builtin_amdgcn_ds_bpermute(pa, bOxy);
      const int l_ns = __builtin_amdgcn_ds_bpermute(pa, bNs);
      const float l_r2 = __int_as_float(__builtin_amdgcn_ds_bpermute(pa, __float_as_int(bR2)));
      const int l_start = __builtin_amdgcn_ds_bpermute(pa, bStart);
      int aj, ak;
      unrank(t - l_start, l_ns, l_r2, l_oxy, aj, ak);
      const int qj = w.aIdx[aj], qk = w.aIdx[ak];
      const float4 dj = w.rD[qj], dk = w.rD[qk];      // unit vectors u, v and R
      const float2 cj2 = w.rF2[qj], ck2 = w.rF2[qk];  // angular fc and fc'
      const float cosv = dj.x * dk.x + dj.y * dk.y + dj.z * dk.z;
      const float cx = dj.y * dk.z - dj.z * dk.y;
      const float cy = dj.z * dk.x - dj.x * dk.z;
      const float cz = dj.x * dk.y - dj.y * dk.x;
      const float sinv = fast_sqrt(cx * cx + cy * cy + cz * cz);
      const float Rbar = 0.5f * (dj.w + dk.w);
      float f2[kNShfAng], ur[kNShfAng];
#pragma unroll
      for (int r = 0; r < kNShfAng; ++r) {
        ur[r] = Rbar - c.shf_a[r];
        f2[r] = fast_exp2(keta * ur[r] * ur[r]);
      }
      // dE/dG of this block: gv[r][a] at gA[32 p + 8 r + a] (global, cached).
      // With p1 = 2^(1-zeta) x^(zeta-1) and f1 = p1 x (x = 1 + cos(theta -
      // theta_a)), the pair's terms are f1 f2[r] fc_j fc_k, so
      //   dE/dx_a   = zeta p1 A_a fc_j fc_k,  A_a = sum_r gv[r][a] f2[r]
      //   dE/dRbar  = sum_r f2'[r] H_r fc_j fc_k,  dE/d(fc_j fc_k) = sum_r f2[r] H_r,
      //   H_r = sum_a gv[r][a] f1_a.
      const float4 *gv = (const float4 *)(gA + p * kAngBlock);
      float dcos = 0.f, dsin = 0.f, H[kNShfAng] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float gq[kNShfAng][4];
#pragma unroll
        for (int r = 0; r < kNShfAng; ++r) {
          const float4 v = gv[2 * r + h];
          gq[r][0] = v.x; gq[r][1] = v.y; gq[r][2] = v.z; gq[r][3] = v.w;
        }
#pragma unroll
        for (int aa = 0; aa < 4; ++aa) {
          const int a = 4 * h + aa;
          // y = x / 2 in [0, 1] (clamped by its own FMA); p1 = y^(zeta-1)
          const float y = __builtin_amdgcn_fmed3f(fmaf(cosv, c.hcz[a], fmaf(sinv, c.hsz[a], 0.5f)), 0.f, 1.f);
          const float p1 = fast_exp2(zm1 * fast_log2(y));
          float A = gq[0][aa] * f2[0];
#pragma unroll
          for (int r = 1; r < kNShfAng; ++r) A += gq[r][aa] * f2[r];
          const float s1 = p1 * A;
          dcos += s1 * c.hcz[a];  // half of dE/dcos: doubled below
          dsin += s1 * c.hsz[a];
          const float f1h = p1 * y;  // f1 / 2: H holds half its value
#pragma unroll
          for (int r = 0; r < kNShfAng; ++r) H[r] += gq[r][aa] * f1h;
        }
      }
      if (valid) {
        float dfc = 0.f, dbar = 0.f;
#pragma unroll
        for (int r = 0; r < kNShfAng; ++r) {
          const float t = f2[r] * H[r];
          dfc += t;
          dbar += ur[r] * t;
        }
        const float fj = cj2.x, fk = ck2.x;
        const float fcc = fj * fk;
        const float zf = 2.0f * c.zeta * fcc;  // the halved cos / sin constants
        dcos *= zf;
        dsin *= zf;
        dbar *= m2eta * fcc;  // via Rbar (dRbar/dR = 1/2, H halved), for each of R_j and R_k
        dfc += dfc;           // H halved
        const float dRj = dbar + dfc * cj2.y * fk;
        const float dRk = dbar + dfc * fj * ck2.y;
        // with c = cos, s = sin of the angle and u, v the unit vectors of
        // the legs j, k: d c / d dj = (v - c u) / Rj and d s / d dj =
        // -(c / s) (v - c u) / Rj (likewise for dk with u and v swapped),
        // so dE/d dj = bj v + (dE/dRj - bj c) u with bj = (dE/dc -
        // dE/ds c / s) / Rj.  Where s vanishes (collinear legs) the sine's
        // term is dropped.
        const float beta = dcos - (sinv > 1e-12f ? dsin * cosv * fast_rcp(sinv) : 0.f);
        const float bj = beta * fast_rcp(dj.w), bk = beta * fast_rcp(dk.w);
        const float uj = dRj - bj * cosv, uk = dRk - bk * cosv;
        gjx = bj * dk.x + uj * dj.x; gjy = bj * dk.y + uj * dj.y; gjz = bj * dk.z + uj * dj.z;
        gkx = bk * dj.x + uk * dk.x; gky = bk * dj.y + uk * dk.y; gkz = bk * dj.z + uk * dk.z;
      }
      // float64 LDS atomics into the centre's own region, a pass after the
      // other: the adds to an entry happen in one fixed order (pass, then
      // program order, then lane order within an instruction) and the sums are
      // the same on every call
      for (int turn = 0; turn < W; ++turn) {
        if ((W == 1 || turn == wave) && valid) {
          double *gj = (double *)((char *)w.rG + __umul24((unsigned)qj, 24u));
          double *gk = (double *)((char *)w.rG + __umul24((unsigned)qk, 24u));
          atomicAdd(gj + 0, (double)gjx);
          atomicAdd(gj + 1, (double)gjy);
          atomicAdd(gj + 2, (double)gjz);
          atomicAdd(gk + 0, (double)gkx);
          atomicAdd(gk + 1, (double)gky);
          atomicAdd(gk + 2, (double)gkz);
        }
        if (W > 1) centre_sync<W>();
      }
    }
    centre_sync<W>();
  }

  // scatter: -dE/dd onto each neighbour, the sum onto the centre (fixed
  // point), per-centre virial -sum d (x) dE/dd
  {
    float fi0 = 0.f, fi1 = 0.f, fi2 = 0.f;
    float vir[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) vir[q] = 0.f;
    static_assert(W == 1 || Sink::kByComponent, "a group's waves share a centre's adds by component");
    if constexpr (Sink::kByComponent) {
      // component t of the entries by lane t (a group: by its waves but the
      // first, which forms the centre's sums, in the one-wave order)
      constexpr int kSend = W > 1 ? W - 1 : 1;
      if (W == 1 || wave > 0)
        for (int t = first_e - (W > 1 ? kWave : 0); t < 3 * nR; t += kSend * kWave) {
          const int e = (int)(((unsigned)t * 43691u) >> 17);  // t / 3 for t < 2^16
          sink.add1(w.rJ[e], t - 3 * e, -to_fix((float)w.rG[t]));
        }
      if (W > 1 && wave > 0) return;
    }
    for (int e = lane; e < nR; e += kWave) {
      const float4 ur = w.rD[e];  // unit vector and R
      const float4 dv = make_float4(ur.x * ur.w, ur.y * ur.w, ur.z * ur.w, ur.w);
      const float gx = (float)w.rG[3 * e], gy = (float)w.rG[3 * e + 1], gz = (float)w.rG[3 * e + 2];
      if (!Sink::kByComponent) sink.add(w.rJ[e], -to_fix(gx), -to_fix(gy), -to_fix(gz));
      fi0 += gx; fi1 += gy; fi2 += gz;
      if (!W_atom) continue;
      vir[0] -= dv.x * gx; vir[1] -= dv.x * gy; vir[2] -= dv.x * gz;
      vir[3] -= dv.y * gx; vir[4] -= dv.y * gy; vir[5] -= dv.y * gz;
      vir[6] -= dv.z * gx; vir[7] -= dv.z * gy; vir[8] -= dv.z * gz;
    }
    fi0 = wave_sum(fi0);
    fi1 = wave_sum(fi1);
    fi2 = wave_sum(fi2);
    if (W_atom) {
#pragma unroll
      for (int q = 0; q < 9; ++q) vir[q] = wave_sum(vir[q]);
    }
    if (lane == 0) sink.add(i, to_fix(fi0), to_fix(fi1), to_fix(fi2));
    if (W_atom && lane < 9) {
      float v = vir[0];
#pragma unroll
      for (int q = 1; q < 9; ++q) v = lane == q ? vir[q] : v;
      W_atom[(size_t)9 * i + lane] = v;
    }
  }
  // the next centre of this wave rewrites the lists
  if (W == 1) wave_lds_sync();
}

// Per-centre form: one wave per centre, or the WPB waves of a workgroup
// (GROUP), forces by device atomics.
template <int WPB, bool GROUP>
__global__ void __launch_bounds__(WPB * kWave)
k_aev_bwd(const float4 *__restrict__ pos, const int *__restrict__ sys_of,
          const SysDesc *__restrict__ sys, const int2 *__restrict__ nbr,
          const int *__restrict__ nbr_cnt, int cap, const int *__restrict__ row_of_atom,
          const float *__restrict__ dG, int ldg, Live N, AevConst c, unsigned long long *__restrict__ Ffix,
          float *__restrict__ W_atom, const int *__restrict__ wave_atom) {
  extern __shared__ float4 lds4[];
  // the wave index is uniform across the wave: keep it (and the centre's
  // index, descriptors and row pointers) in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int wv = GROUP ? (int)blockIdx.x : blockIdx.x * WPB + wave;
  if (wv >= N.get()) return;
  // the centre of this wave (the costliest systems' centres first)
  const int i = wave_atom ? __builtin_amdgcn_readfirstlane(wave_atom[wv]) : wv;
  WaveLds w = carve<true>((char *)lds4 + (GROUP ? 0 : wave * wave_lds_bytes<true>(cap)), cap);
  const SysDesc &d = sys[sys_of[i]];
  bwd_centre<GROUP ? WPB : 1>(i, GROUP ? wave : 0, lane, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, c, W_atom, w,
             SinkGlobal{Ffix, fix_shift(d)});
}

// Next centre of a workgroup's group for the calling wave (an LDS counter:
// waves that finish early take more centres).
__device__ inline int next_centre(int *counter, int lane) {
  int p = 0;
  if (lane == 0) p = atomicAdd(counter, 1);
  return __builtin_amdgcn_readfirstlane(p);
}

// Per-system form (batches of small non-periodic systems): a workgroup takes
// a group of consecutive centres of one system (groups[b] = {first centre,
// count}); the system's forces are summed in an LDS table and added into
// Ffix once.
template <int WPB>
__global__ void __launch_bounds__(WPB * kWave)
k_aev_bwd_sys(const int2 *__restrict__ groups, const float4 *__restrict__ pos, const int *__restrict__ sys_of,
              const SysDesc *__restrict__ sys, const int2 *__restrict__ nbr,
              const int *__restrict__ nbr_cnt, int cap, const int *__restrict__ row_of_atom,
              const float *__restrict__ dG, int ldg, AevConst c, unsigned long long *__restrict__ Ffix,
              float *__restrict__ W_atom, Live n_groups) {
  extern __shared__ float4 lds4[];
  __shared__ int counter;
  if ((int)blockIdx.x >= n_groups.get()) return;  // the whole workgroup leaves together
  const int2 gr = groups[blockIdx.x];
  const SysDesc &d = sys[sys_of[gr.x]];
  const int off = d.atom_off, n3 = 3 * d.n;
  unsigned long long *tab = (unsigned long long *)((char *)lds4 + WPB * wave_lds_bytes<true>(cap));
  for (int t = threadIdx.x; t < n3; t += WPB * kWave) tab[t] = 0ull;
  if (threadIdx.x == 0) counter = 0;
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  WaveLds w = carve<true>((char *)lds4 + wave * wave_lds_bytes<true>(cap), cap);
  const SinkSys sink{tab, off};
  for (int p = next_centre(&counter, lane); p < gr.y; p = next_centre(&counter, lane))
    bwd_centre<1>(gr.x + p, 0, lane, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, c, W_atom, w, sink);
  __syncthreads();
  for (int t = threadIdx.x; t < n3; t += WPB * kWave) {
    const unsigned long long v = tab[t];
    if (v) atomicAdd(Ffix + 3 * (size_t)d.order_off + t, v);
  }
}

// Per-cell form (cell grids): a workgroup takes the centres of one cell;
// they share most of their neighbours, whose forces are summed in an LDS hash
// table and added into Ffix once per cell.
template <int WPB>
__global__ void __launch_bounds__(WPB * kWave)
k_aev_bwd_cells(const int *__restrict__ cell_start, const int *__restrict__ cell_atoms,
                const float4 *__restrict__ pos, const int *__restrict__ sys_of,
                const SysDesc *__restrict__ sys, const int2 *__restrict__ nbr,
                const int *__restrict__ nbr_cnt, int cap, const int *__restrict__ row_of_atom,
                const float *__restrict__ dG, int ldg, AevConst c, unsigned long long *__restrict__ Ffix,
                float *__restrict__ W_atom, Live n_cells) {
  extern __shared__ float4 lds4[];
  __shared__ int counter;
  if ((int)blockIdx.x >= n_cells.get()) return;  // the whole workgroup leaves together
  const int b = cell_start[blockIdx.x], e = cell_start[blockIdx.x + 1];
  if (b == e) return;  // the whole workgroup leaves together
  char *tail = (char *)lds4 + WPB * wave_lds_bytes<true>(cap);
  unsigned long long *hval = (unsigned long long *)tail;
  int *hkey = (int *)(tail + 24 * kBwdHash);
  for (int t = threadIdx.x; t < kBwdHash; t += WPB * kWave) {
    hkey[t] = -1;
    hval[3 * t] = hval[3 * t + 1] = hval[3 * t + 2] = 0ull;
  }
  if (threadIdx.x == 0) counter = 0;
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  WaveLds w = carve<true>((char *)lds4 + wave * wave_lds_bytes<true>(cap), cap);
  // a cell's centres and their neighbours belong to one system
  const int shift = fix_shift(sys[sys_of[cell_atoms[b]]]);
  const SinkHash sink{hkey, hval, Ffix, shift};
  for (int p = next_centre(&counter, lane); b + p < e; p = next_centre(&counter, lane))
    bwd_centre<1>(cell_atoms[b + p], 0, lane, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, c, W_atom, w,
               sink);
  __syncthreads();
  for (int t = threadIdx.x; t < kBwdHash; t += WPB * kWave) {
    const int j = hkey[t];
    if (j < 0) continue;
    unsigned long long *p = Ffix + 3 * (size_t)(j + shift);
    for (int q = 0; q < 3; ++q) {
      const unsigned long long v = hval[3 * t + q];
      if (v) atomicAdd(p + q, v);
    }
  }
}

// Waves per workgroup: the preference (1, 2 or 4) when its LDS fits in
// 64 KB, else one.  One is the default: each wave works on its own centre,
// and single-wave workgroups pack the compute units most freely (it was the
// fastest shape on most measured batches).
template <bool BWD>
static int waves_for_cap(int cap, int pref) {  // centres per workgroup, a wave each
  const size_t per = wave_lds_bytes<BWD>(cap);
  if ((pref == 1 || pref == 2 || pref == 4) && per * pref <= 64 * 1024) return pref;
  return 1;
}

// Several waves per centre where the centres alone leave the chip idle:
//   - at most 1,024 centres (one wave per SIMD).  Forward / backward, one wave
//     and groups: 101 atoms 50 / 51 -> 21 / 27 us, 1,000 in solutes of 20 atoms
//     17 / 12 -> 11 / 11, 900 of a box of water 13 / 15 -> 10 / 12;
//   - up to 4,096 centres of systems without a list whose largest has enough
//     atoms, so that a centre's passes may be many: in the forward more than a
//     300th of the call's; in the backward, whose waves take turns at the adds,
//     more than a 50th and than 48, or 20 up to 1,280 centres, five groups per
//     compute unit (37 solutes of 32 atoms 19 -> 15 us, 43 of them 19 and 18).
//     Of 4,000 atoms in solutes of 10, 20, 40, 64, 100 and 200 (1.2 A n^(1/3) a
//     side) the forward went from 17, 21, 30, 47, 68 and 92 to 20, 22, 29, 36,
//     45 and 59 us, the backward from 12, 18, 32, 56, 87 and 120 to 28, 31, 42,
//     54, 67 and 91; of 1,600 in solutes of 4, 10, 40 and 64 the forward from
//     10, 14, 25 and 36 to 10, 12, 17 and 21, the backward from 8, 9, 22 and 37
//     to 14, 15, 23 and 30.  Open solutes (2.3 A n^(1/3)), whose centres have
//     few passes, lose in the backward: of 100 atoms, 4,000 in all, 17 -> 30;
//   - lists (or systems without one) so long that the LDS holds fewer than
//     eleven one-wave centres per compute unit, or seven in the backward of
//     more than 4,096 centres with lists, where most of a row may lie past the
//     angular cutoff: 30,000 atoms of water at capacities of 304, 400, 448 and
//     600 take 126, 151, 168 and 236 us there one by one and 181, 181, 181 and
//     216 in groups, 120 dense solutes of 10 to 120 atoms at 448 115 and 93; 60
//     dense solutes of 500 atoms without a list 1,305 and 740, open ones 388 and
//     224.  In the forward, those 120 solutes at 600 83 and 63, the water 110
//     and 129.
constexpr int kGroupWaves = 4;
static_assert(kMaxChunks * kChunkCounts <= kGroupWaves * kPairPass * 24, "chunk counts of the forward");
bool aev_grouped(bool bwd, int n_centres, bool list, int cap, size_t max_lds) {
  // (without a list, the capacity is the largest system's other atoms)
  if (n_centres <= (bwd && !list && cap >= 20 ? 1280 : 1024)) return true;
  if (!list && n_centres <= 4096 && (bwd ? cap > 48 && cap * 50 > n_centres : cap * 300 > n_centres)) return true;
  const size_t per = bwd ? wave_lds_bytes<true>(cap) : wave_lds_bytes<false>(cap);
  return per * (bwd && list && n_centres > 4096 ? 7 : 11) > max_lds;
}

template <bool BF16>
static void aev_fwd_t(const float4 *pos, const int *sys_of, const SysDesc *sys, const int2 *nbr,
                      const int *nbr_cnt, int cap, const int *row_of_atom, void *G, int ldg,
                      unsigned long long *row_mask, const int *wave_atom, int *status, Live N, const AevConst &c,
                      int wpb_pref, size_t max_lds, hipStream_t st) {
  if (aev_grouped(false, N.v, nbr != nullptr, cap, max_lds)) {
    const size_t lds = wave_lds_bytes<false>(cap) + kGroupWaves * kPairPass * 24;
    k_aev_fwd<kGroupWaves, BF16, true><<<(unsigned)N.v, kGroupWaves * kWave, lds, st>>>(
        pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg, row_mask, wave_atom, status, N, 1, c);
    return;
  }
  // Runs of 256 centres on one XCD (their system's records and the neighbouring
  // rows' masks stay in its L2) where there are enough rounds of waves to even
  // out: 163,840 centres of 4,096 snapshots 821 -> 792 us per call, 100,002 of
  // a box the same; 32,671 of ragged solutes, largest first, 218 -> 220.
  int wpb = waves_for_cap<false>(cap, wpb_pref);
  const int run = N.v >= 65536 ? 256 / wpb : 1;
  size_t lds = wave_lds_bytes<false>(cap) * wpb;
  unsigned grid = xcd_grid((unsigned)((N.v + wpb - 1) / wpb), run);
  if (wpb == 4)
    k_aev_fwd<4, BF16, false><<<grid, 4 * kWave, lds, st>>>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg,
                                                            row_mask, wave_atom, status, N, run, c);
  else if (wpb == 2)
    k_aev_fwd<2, BF16, false><<<grid, 2 * kWave, lds, st>>>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg,
                                                            row_mask, wave_atom, status, N, run, c);
  else
    k_aev_fwd<1, BF16, false><<<grid, kWave, lds, st>>>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg,
                                                        row_mask, wave_atom, status, N, run, c);
}

void launch_aev_fwd(const float4 *pos, const int *sys_of, const SysDesc *sys, const int2 *nbr,
                    const int *nbr_cnt, int cap, const int *row_of_atom, void *G, bool g_bf16,
                    int ldg, Live N, const AevConst &c, unsigned long long *row_mask, const int *wave_atom,
                    int *status, int wpb_pref, size_t max_lds, hipStream_t st) {
  if (N.v <= 0) return;
  if (g_bf16)
    aev_fwd_t<true>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg, row_mask, wave_atom, status, N, c,
                    wpb_pref, max_lds, st);
  else
    aev_fwd_t<false>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, G, ldg, row_mask, wave_atom, status, N, c,
                     wpb_pref, max_lds, st);
}

template <int WPB>
static void aev_bwd_launch(int form, size_t lds, unsigned grid, const AevBwdGroups &gp, const float4 *pos,
                           const int *sys_of, const SysDesc *sys, const int2 *nbr, const int *nbr_cnt, int cap,
                           const int *row_of_atom, const float *dG, int ldg, Live N, const AevConst &c,
                           unsigned long long *Ffix, float *W_atom, hipStream_t st) {
  if constexpr (WPB >= 4) {  // grouped forms run 4 to 10 waves per workgroup
    if (form == 1) {
      k_aev_bwd_sys<WPB><<<grid, WPB * kWave, lds, st>>>(gp.groups, pos, sys_of, sys, nbr, nbr_cnt, cap,
                                                         row_of_atom, dG, ldg, c, Ffix, W_atom,
                                                         Live(gp.n_groups, gp.live_groups));
      return;
    }
    if (form == 2) {
      k_aev_bwd_cells<WPB><<<grid, WPB * kWave, lds, st>>>(gp.cell_start, gp.cell_atoms, pos, sys_of, sys, nbr,
                                                           nbr_cnt, cap, row_of_atom, dG, ldg, c, Ffix, W_atom,
                                                           Live(gp.n_cells, gp.live_cells));
      return;
    }
  }
  if constexpr (WPB == kGroupWaves) {
    if (form == 3) {
      k_aev_bwd<WPB, true><<<grid, WPB * kWave, lds, st>>>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg,
                                                           N, c, Ffix, W_atom, gp.wave_atom);
      return;
    }
  }
  if constexpr (WPB <= 4)
    k_aev_bwd<WPB, false><<<grid, WPB * kWave, lds, st>>>(pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, N, c,
                                                   Ffix, W_atom, gp.wave_atom);
}

// Chooses the form.  wpb_pref 0 (untuned), 1 or 2: one wave per centre,
// forces straight into Ffix by device atomics, one or two waves per
// workgroup (the fastest form measured on the ragged solutes and on the
// 100k-atom box).  4, 5, 6, 8 or 10: a grouped form when the call has one,
// with that many waves per workgroup (fewer when the LDS does not hold
// them): per system for a batch of small non-periodic systems (gp.groups),
// per cell on a grid of at least kBwdMinCells cells (fewer would leave
// compute units idle).  Without a grouped form: one wave per centre.
// Calls with several waves per centre (aev_grouped) run those whatever
// wpb_pref is.
void launch_aev_bwd(const float4 *pos, const int *sys_of, const SysDesc *sys, const int2 *nbr,
                    const int *nbr_cnt, int cap, const int *row_of_atom, const float *dG, int ldg,
                    Live N, const AevConst &c, unsigned long long *Ffix, float *W_atom, const AevBwdGroups &gp,
                    int wpb_pref, size_t max_lds, hipStream_t st) {
  if (N.v <= 0) return;
  const size_t per = wave_lds_bytes<true>(cap);
  if (aev_grouped(true, N.v, nbr != nullptr, cap, max_lds)) {
    aev_bwd_launch<kGroupWaves>(3, per, (unsigned)N.v, gp, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg,
                                N, c, Ffix, W_atom, st);
    return;
  }
  int form = 0;
  size_t table = 0;
  if (wpb_pref >= 4) {
    if (gp.groups && gp.n_groups > 0) {
      form = 1;
      table = ((size_t)gp.max_sys_atoms * 24 + 15) / 16 * 16;
    } else if (gp.cell_start && gp.n_cells >= kBwdMinCells) {
      form = 2;
      table = (size_t)kBwdHash * 28;
    }
  }
  if (form) {
    // kBwdStaticLds: the kernels' static LDS (the centre counter) comes on
    // top of the dynamic allocation
    int wpb = (wpb_pref == 4 || wpb_pref == 5 || wpb_pref == 6 || wpb_pref == 8 || wpb_pref == 10) ? wpb_pref : 8;
    auto fits = [&](int w) { return per * w + table + kBwdStaticLds <= max_lds; };
    while (wpb >= 4 && !fits(wpb)) wpb = wpb == 10 ? 8 : wpb == 8 ? 6 : wpb - 1;
    if (wpb >= 4) {
      const size_t lds = per * wpb + table;
      const unsigned grid = (unsigned)(form == 1 ? gp.n_groups : gp.n_cells);
#define NNP_BWD_CASE(W)                                                                                     \
  case W:                                                                                                   \
    aev_bwd_launch<W>(form, lds, grid, gp, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, N, c, \
                      Ffix, W_atom, st);                                                                    \
    return;
      switch (wpb) {
        NNP_BWD_CASE(4)
        NNP_BWD_CASE(5)
        NNP_BWD_CASE(6)
        NNP_BWD_CASE(8)
        NNP_BWD_CASE(10)
        default: break;
      }
#undef NNP_BWD_CASE
    }
  }
  const int wpb = waves_for_cap<true>(cap, wpb_pref);
  const size_t lds = per * wpb;
  const unsigned grid = (unsigned)((N.v + wpb - 1) / wpb);
  if (wpb == 4)
    aev_bwd_launch<4>(0, lds, grid, gp, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, N, c, Ffix,
                      W_atom, st);
  else if (wpb == 2)
    aev_bwd_launch<2>(0, lds, grid, gp, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, N, c, Ffix,
                      W_atom, st);
  else
    aev_bwd_launch<1>(0, lds, grid, gp, pos, sys_of, sys, nbr, nbr_cnt, cap, row_of_atom, dG, ldg, N, c, Ffix,
                      W_atom, st);
}

}  // namespace nnp
