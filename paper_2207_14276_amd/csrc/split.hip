// Dense layers of the float32 model on the bfloat16 matrix cores.
//
// A float32 operand x is taken as three bfloat16 parts, x = p1 + p2 + p3, each
// part the rounding of what the earlier ones leave.  Their 3 x 8 significant
// bits are all of x for |x| >= 2^-102, where no part falls below the smallest
// normal bfloat16, 2^-126; below, less than 2^-125 of x is lost.  (Models
// where that could count stay on float32 operands, see below.)  A product x w
// is the six part products down to 2^-18: p1 w1, p1 w2, p2 w1, p2 w2, p1 w3,
// p3 w1; the three left out are below 2^-26 |x w|.  Each of the six is exact
// in the matrix core's float32 accumulation; p1 w1 sums in one
// accumulator and the five small ones in a second, added at the end.  The six
// v_mfma_f32_16x16x32_bf16 take 6/16 of the time of the float32 MFMAs they
// replace, and the main sum is rounded once per 32 products instead of once
// per 2.  The weights' parts are laid out once, when the model is created:
// per row, chunks of 32 columns, each chunk the 32 first, second and third
// parts side by side (192 contiguous bytes).  Activations stay float32 in
// memory and LDS; a wave splits them as it reads its fragments, in the shadow
// of its MFMAs.
//
// A fragment of activations with a value that has no finite first part
// (infinite, or within a rounding of the largest float) takes its products on
// the float32 matrix instruction instead, with the weights put together again
// from their parts (exact), so that overflows come out as they do there.
// Gradients need no such care: none exceeds its network's gain.  Models whose weights
// are not finite, are not whole multiples of 2^-126, or are so large that what
// the smallest activations lose could grow to count (parts_suffice in api.hip),
// or whose widths leave a partial 32-column chunk, stay on the float32 kernels
// of mlp.hip.
#include "internal.h"
#include "split.h"
#include "wave.h"

#include <algorithm>

namespace nnp {

// ------------------------------------------------------------------ weights
// Parts of src [rows][K] (row stride ld) into dst [rows][Kp / 32][3][32], with
// gap zero columns from column gap_at on; columns past those are zeros.
__global__ void __launch_bounds__(256)
k_split_weights(const float *__restrict__ src, int rows, int K, int ld, int Kp, int gap_at, int gap,
                uint16_t *__restrict__ dst) {
  const size_t total = (size_t)rows * Kp;
  for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(t / Kp), k = (int)(t - (size_t)r * Kp);
    const int ks = k < gap_at ? k : k < gap_at + gap ? K : k - gap;
    const float x = ks < K ? src[(size_t)r * ld + ks] : 0.f;
    const __bf16 p1 = (__bf16)x;
    const float a = x - (float)p1;
    const __bf16 p2 = (__bf16)a;
    const __bf16 p3 = (__bf16)(a - (float)p2);
    uint16_t *d = dst + ((size_t)r * (Kp / 32) + k / 32) * kPartChunk + k % 32;
    d[0] = __builtin_bit_cast(uint16_t, p1);
    d[32] = __builtin_bit_cast(uint16_t, p2);
    d[64] = __builtin_bit_cast(uint16_t, p3);
  }
}

void launch_split_weights(const float *src, int rows, int K, int ld, int Kp, int gap_at, int gap, uint16_t *dst,
                          hipStream_t st) {
  const size_t total = (size_t)rows * Kp;
  if (total == 0) return;
  const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 4096);
  k_split_weights<<<blocks, 256, 0, st>>>(src, rows, K, ld, Kp, gap_at, gap, dst);
}

// ------------------------------------------------------------- grouped GEMM
// The grouped GEMM of mlp.hip (same groups, epilogues and row records) for
// the split operands: C[rows, n_out] = sum over K segments of A . B^T, A
// float32, B the weights' parts.  A workgroup of WR x WC waves, each 16 HR
// rows x 16 CB columns, takes a tile of TM rows and TN columns; both operands
// reach LDS by direct global loads in chunks of 32 columns, STAGES chunks in
// a ring.  LDS slots are 16 bytes: A row r's eight slots at 8 r + (slot ^
// aswz(r)), a part's row r's four at 4 r + (slot ^ bswz(r)); the XORs keep the
// fragment reads free of bank conflicts.  Products are formed transposed
// (weights as the first operand), so that a lane ends with four consecutive
// columns of one row.
//
// 128 x 128 tiles (4 x 1 waves of 32 x 128: every activation is split by one
// wave only), two workgroups per compute unit.  16 x 64 tiles (1 x 4 waves of
// 16 x 16) serve small calls (the line: launch_gemm_split): a wave's chain of
// dependent MFMAs is an eighth as long, and the row tiles without a real row are
// skipped.  Where there are at most 256 of them, one per compute unit, they take
// STEP = 2 chunks per barrier from a ring of eight: a chunk is then bound by its
// chain of LDS reads, splitting and five dependent MFMAs (0.39 us), and two
// chunks' reads and splitting run beside each other.  First layer of a call of
// 24 atoms 13.0 -> 11.6 us, of 101 atoms 20.1 -> 17.5; with the ring of eight
// alone 14.2, with more workgroups the 112 KB of LDS would leave one of them
// where two fit.  Every output element sums its products in the same order in
// all.
__device__ inline int aswz(int r) { return (r ^ (r >> 1)) & 7; }
__device__ inline int bswz(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }

constexpr int vm_count(int n) { return 0xF70 | (n & 15) | ((n >> 4) << 14); }
// Waits until at most `ahead` chunks' loads of this wave are outstanding.
template <int LOADS, int MAXA>
__device__ inline void wait_ahead(int ahead) {
  if (MAXA >= 4 && ahead >= 4) __builtin_amdgcn_s_waitcnt(vm_count(4 * LOADS));
  else if (MAXA >= 3 && ahead >= 3) __builtin_amdgcn_s_waitcnt(vm_count(3 * LOADS));
  else if (MAXA >= 2 && ahead >= 2) __builtin_amdgcn_s_waitcnt(vm_count(2 * LOADS));
  else if (MAXA >= 1 && ahead >= 1) __builtin_amdgcn_s_waitcnt(vm_count(LOADS));
  else __builtin_amdgcn_s_waitcnt(vm_count(0));
}

template <int EPI, int HR, int CB, int WR, int WC, int STAGES, int STEP>
__global__ void __launch_bounds__(WR * WC * kWave, 2)
k_gemm_split(GemmLaunch gl) {
  constexpr int TM = 16 * HR * WR, TN = 16 * CB * WC, T = WR * WC * kWave, TK = 32;
  constexpr int A_SLOTS = TM * 8, B_SLOTS = TN * 12;
  // A tiles smaller than one load of the workgroup: its first waves load them
  constexpr int A_LD = (A_SLOTS + T - 1) / T, B_LD = B_SLOTS / T;
  constexpr int A_WAVES = A_SLOTS < T ? A_SLOTS / kWave : WR * WC;
  static_assert(B_SLOTS % T == 0 && (A_SLOTS % T == 0 || A_SLOTS < T), "whole load instructions");
  extern __shared__ uint4 split_lds[];
  const float inv_alpha = 1.f / gl.alpha;

  const int lb = xcd_chunked(blockIdx.x, gl.xcd_chunk);
  if (lb >= gl.n_blocks) return;
  // columns: all members' side by side (member-major, as their weights lie)
  // where the members share A (gl.span), else one member per block
  const int n_ct = gl.col_tiles;
  const int ct = lb % n_ct;
  const int mb = gl.span ? 0 : (lb / n_ct) % gl.n_members;
  const int rt = gl.span ? lb / n_ct : lb / (n_ct * gl.n_members);
  const int r0 = rt * TM;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  // (the rows' records, masked below, on their way meanwhile)
  constexpr bool kMaskK = EPI == kEpiFwd, kMaskN = EPI == kEpiOut;
  constexpr int H_LD = (TM + kWave - 1) / kWave;
  unsigned long long row_h[H_LD];
  if ((kMaskK || kMaskN) && gl.row_mask) {
#pragma unroll
    for (int q = 0; q < H_LD; ++q) row_h[q] = gl.row_mask[r0 + min(lane + q * kWave, TM - 1)];
  }
  int real_end;
  const int s = tile_bucket(gl.bucket_off, gl.bucket_cnt, gl.n_groups, r0, lane, real_end);
  if (s < 0 || r0 >= real_end) return;  // no row of an atom in this tile
  const GemmGroup grp = gl.g[mb * gl.n_groups + s];
  const int n_cols = gl.span ? grp.n_out * gl.n_members : grp.n_out;
  const int c0 = ct * TN;
  if (c0 >= n_cols) return;
  const int K = grp.K, nseg = gl.n_seg, nk = K / TK;

  const int l16 = lane & 15, kq = lane >> 4;
  const int wr = wave / WC, wc = wave % WC;

  // The 16-column halves of the AEV that some row of the tile has (see
  // GemmLaunch::row_mask): a chunk without one is not loaded in the first
  // layer; in the dE/dG product the live halves are the columns, side by side
  // (8 of 63 in a box of water: 12,003 atoms x 8 members 195 -> 133 us).
  unsigned long long live_h = ~0ull;
  const bool masked = gl.row_mask != nullptr && (kMaskN || (kMaskK && nseg == 1 && nk <= 32));
  if (masked) {
    unsigned h_lo = 0, h_hi = 0;
#pragma unroll
    for (int q = 0; q < H_LD; ++q) {
      const bool real = lane + q * kWave < min(TM, real_end - r0);
      h_lo |= real ? (unsigned)row_h[q] : 0u;
      h_hi |= real ? (unsigned)(row_h[q] >> 32) : 0u;
    }
    live_h = ((unsigned long long)wave_or(h_hi) << 32) | wave_or(h_lo);
    if (kMaskK) live_h = gapped(live_h, gl.rad_halves, gl.rad_gap);
  }
  bool wave_live = c0 + wc * 16 * CB < n_cols;
  int n_live = 0, halves_in_order = 0;  // dE/dG, masked: live halves
  bool some_dead = false;
  if (kMaskN && masked) {
    live_h &= ~0ull >> (64 - min(n_cols / 16, 64));
    n_live = __popcll(live_h);
    if (c0 / 16 >= n_live) return;  // uniform over the workgroup, nothing issued yet
    wave_live = (c0 + wc * 16 * CB) / 16 < n_live;
    some_dead = n_live < n_cols / 16;
    if (some_dead) halves_in_order = live_halves(live_h, lane);
  }

  // uniform tile bases and this thread's byte offsets from them
  const char *A = (const char *)((const float *)gl.A + (size_t)r0 * gl.lda + (size_t)mb * gl.a_member_stride);
  const unsigned ldb = (unsigned)(nk * nseg) * (kPartChunk * 2);  // bytes of a row of B
  const char *B = (const char *)grp.B;
  unsigned aoff[A_LD], boff[B_LD];
#pragma unroll
  for (int q = 0; q < A_LD; ++q) {
    const int sl = q * T + tid, row = sl >> 3, ch = (sl & 7) ^ aswz(row);
    aoff[q] = (unsigned)(row * gl.lda + ch * 4) * 4u;
  }
#pragma unroll
  for (int q = 0; q < B_LD; ++q) {
    const int sl = q * T + tid, part = sl / (TN * 4), row = (sl - part * (TN * 4)) >> 2, ch = (sl & 3) ^ bswz(row);
    // past the columns: a valid row, its results are not stored
    int col = min(c0 + row, n_cols - 1);
    if (some_dead) col = 16 * half_at(halves_in_order, min((c0 + row) / 16, n_live - 1)) + (row & 15);
    boff[q] = (unsigned)col * ldb + (part * 32 + ch * 8) * 2;
  }
  const bool loads_a = wave < A_WAVES;  // (wave-uniform)
  auto issue = [&](int c, int stage) {
    const int seg = c / nk;
    const char *ac = A + ((size_t)seg * gl.a_seg_stride + (size_t)(c - seg * nk) * TK) * 4;
    const char *bc = B + (size_t)c * (kPartChunk * 2);
    uint4 *dst = split_lds + stage * (A_SLOTS + B_SLOTS) + wave * kWave;
    if (loads_a) {
#pragma unroll
      for (int q = 0; q < A_LD; ++q)
        __builtin_amdgcn_global_load_lds((const void *)(ac + aoff[q]),
                                         (__attribute__((address_space(3))) void *)(dst + q * T), 16, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < B_LD; ++q)
      __builtin_amdgcn_global_load_lds((const void *)(bc + boff[q]),
                                       (__attribute__((address_space(3))) void *)(dst + A_SLOTS + q * T), 16, 0, 0);
  };

  floatx4 acc[HR][CB], low[HR][CB];  // p1 w1, and the five small products
#pragma unroll
  for (int h = 0; h < HR; ++h)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[h][j] = low[h][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  int total = nk * nseg;
  unsigned long long todo = 0;  // chunks left to issue (masked first layer)
  if (kMaskK && masked) {
    const unsigned long long x = live_h | (live_h >> 1);  // bit 2 c: chunk c has a live half
    for (int c = 0; c < nk; ++c) todo |= ((x >> (2 * c)) & 1ull) << c;
    if (todo == 0) todo = 1;
    total = __builtin_popcountll(todo);
  }
  auto next = [&](int k) {
    if (!(kMaskK && masked)) return k;
    const int c = __builtin_ctzll(todo);
    todo &= todo - 1;
    return c;
  };
  for (int q = 0; q < STAGES - STEP; ++q)
    if (q < total) issue(next(q), q);

  // This wave's rows of A of chunk c (its stage's A slots); whether one of them
  // is an activation without a finite first part.  (128-row tiles look at
  // gradients too, which are never found: without the branch the compiler's
  // schedule makes a workgroup alone on its compute unit 3 to 5% slower, dE/dG
  // of 6,006 atoms x 8 networks of 256 channels 136 -> 143 us.)
  constexpr bool kWide = EPI == kEpiFwd || CB > 1;
  auto take_a = [&](const uint4 *As, Parts (&a)[HR]) {
    float big = 0.f;
#pragma unroll
    for (int h = 0; h < HR; ++h) {
      const int r = (wr * HR + h) * 16 + l16;
      // (typed vector reads: an untyped copy would make the compiler wait for
      // every load to LDS in flight)
      const floatx4 u = *(const floatx4 *)&As[8 * r + ((2 * kq) ^ aswz(r))];
      const floatx4 v = *(const floatx4 *)&As[8 * r + ((2 * kq + 1) ^ aswz(r))];
      const float x[8] = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
      // (padding rows hold whatever an earlier call left there)
      if (kWide) big = fmaxf(big, r0 + r < real_end ? max8(x) : 0.f);
      a[h] = split8(x);
    }
    return kWide && __ballot(big > kPartMax) != 0;
  };
  // block j's fragment of part p: slot(j)[4 TN p] (the XOR of a row depends
  // on its block's parity alone)
  const int br = (wc * CB) * 16 + l16;
  const int xe = kq ^ bswz(br), xo = kq ^ bswz(br + 16);
  auto slot = [&](const uint4 *As, int j) { return As + A_SLOTS + 4 * br + 64 * j + (j & 1 ? xo : xe); };
  auto take_b = [&](const uint4 *As, int j, bf16x8 (&w)[3]) {
#pragma unroll
    for (int p = 0; p < 3; ++p) w[p] = __builtin_bit_cast(bf16x8, slot(As, j)[4 * TN * p]);
  };
  auto products = [&](const Parts (&a)[HR], const bf16x8 (&w)[3], int j) {
#pragma unroll
    for (int h = 0; h < HR; ++h) low[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], a[h].p3, low[h][j], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HR; ++h) low[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2], a[h].p1, low[h][j], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HR; ++h) low[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1], a[h].p2, low[h][j], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HR; ++h) low[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], a[h].p2, low[h][j], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HR; ++h) low[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1], a[h].p1, low[h][j], 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HR; ++h) acc[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], a[h].p1, acc[h][j], 0, 0, 0);
  };
  // a chunk on the float32 instruction
  auto products32 = [&](const uint4 *As) {
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        const float b = joined((const uint16_t *)slot(As, j) + k, 32 * TN);
#pragma unroll
        for (int h = 0; h < HR; ++h) {
          const int r = (wr * HR + h) * 16 + l16;
          const float x = ((const float *)&As[8 * r + ((2 * kq + (k >> 2)) ^ aswz(r))])[k & 3];
          acc[h][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b, x, acc[h][j], 0, 0, 0);
        }
      }
    }
  };

  for (int c = 0; c < total; c += STEP) {
    constexpr int MAXA = STAGES - 2 * STEP;
    if (A_WAVES == WR * WC || loads_a) wait_ahead<A_LD + B_LD, MAXA>(min(total - STEP - c, MAXA));
    else wait_ahead<B_LD, MAXA>(min(total - STEP - c, MAXA));
    // every wave has its part of these chunks and is done with the STEP before
    // them, whose stages the next issues fill
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int q = 0; q < STEP; ++q)
      if (c + STAGES - STEP + q < total) issue(next(c + STAGES - STEP + q), (c + STAGES - STEP + q) % STAGES);
    const uint4 *As = split_lds + (c % STAGES) * (A_SLOTS + B_SLOTS);
    if (!wave_live) continue;
    if (STEP == 2 && c + 1 < total) {
      const uint4 *An = split_lds + ((c + 1) % STAGES) * (A_SLOTS + B_SLOTS);
      Parts a[HR], an[HR];
      bf16x8 w[CB][3], wn[CB][3];
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        take_b(As, j, w[j]);
        take_b(An, j, wn[j]);
      }
      const bool wide = take_a(As, a), wide_n = take_a(An, an);
      if (!wide && !wide_n) {
#pragma unroll
        for (int j = 0; j < CB; ++j) products(a, w[j], j);
#pragma unroll
        for (int j = 0; j < CB; ++j) products(an, wn[j], j);
      } else {
        if (wide) {
          products32(As);
        } else {
#pragma unroll
          for (int j = 0; j < CB; ++j) products(a, w[j], j);
        }
        if (wide_n) {
          products32(An);
        } else {
#pragma unroll
          for (int j = 0; j < CB; ++j) products(an, wn[j], j);
        }
      }
      continue;
    }
    Parts a[HR];
    if (!take_a(As, a)) {
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        bf16x8 w[3];
        take_b(As, j, w);
        products(a, w, j);
      }
    } else {
      products32(As);
    }
  }

  // lane: row l % 16 of each sixteen, columns 4 (l / 16) + 0..3 of each
  // sixteen, which lie within one member (widths are multiples of 32 wherever
  // columns span members)
  if (!wave_live) return;
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    int v16 = c0 + (wc * CB + j) * 16;  // wave-uniform
    if (some_dead) {
      if (v16 / 16 >= n_live) continue;
      v16 = 16 * __builtin_amdgcn_readfirstlane(half_at(halves_in_order, v16 / 16));
    }
    // (a descriptor length may end inside a sixteen; it is a multiple of 4)
    if (v16 + 4 * kq >= n_cols) continue;
    const int om = gl.span ? v16 / grp.n_out : mb;
    const int col = v16 - (gl.span ? om * grp.n_out : 0) + 4 * kq;
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (EPI == kEpiFwd) bias = *(const float4 *)(gl.g[om * gl.n_groups + s].bias + col);
#pragma unroll
    for (int h = 0; h < HR; ++h) {
      const int row = r0 + (wr * HR + h) * 16 + l16;
      const floatx4 v = acc[h][j] + low[h][j];
      float4 o;
      if (EPI == kEpiFwd) {
        o = make_float4(celu32(v[0] + bias.x, gl.alpha, inv_alpha), celu32(v[1] + bias.y, gl.alpha, inv_alpha),
                        celu32(v[2] + bias.z, gl.alpha, inv_alpha), celu32(v[3] + bias.w, gl.alpha, inv_alpha));
      } else if (EPI == kEpiBwd) {
        const float4 x = *(const float4 *)((const float *)gl.H + (size_t)row * gl.ldh + (size_t)om * gl.h_member_stride + col);
        o = make_float4(v[0] * dcelu32(x.x, inv_alpha) * gl.scale, v[1] * dcelu32(x.y, inv_alpha) * gl.scale,
                        v[2] * dcelu32(x.z, inv_alpha) * gl.scale, v[3] * dcelu32(x.w, inv_alpha) * gl.scale);
      } else {
        o = make_float4(v[0] * gl.scale, v[1] * gl.scale, v[2] * gl.scale, v[3] * gl.scale);
      }
      *(float4 *)((float *)gl.C + (size_t)row * gl.ldc + (size_t)om * gl.c_member_stride + col) = o;
    }
  }
}

template <int EPI, int HR, int CB, int WR, int WC, int STAGES, int STEP>
static void gemm_split_t(GemmLaunch gl, int rows, int cols, hipStream_t st) {
  constexpr int TM = 16 * HR * WR, TN = 16 * CB * WC;
  gl.col_tiles = (cols + TN - 1) / TN;
  gl.xcd_chunk = (gl.span ? 1 : gl.n_members) * gl.col_tiles;
  gl.n_blocks = rows / TM * gl.xcd_chunk;
  const size_t lds = (size_t)STAGES * (TM * 8 + TN * 12) * 16;
  k_gemm_split<EPI, HR, CB, WR, WC, STAGES, STEP>
      <<<xcd_grid((unsigned)gl.n_blocks, gl.xcd_chunk), WR * WC * kWave, lds, st>>>(gl);
}

// tn_pref 64: 16-row tiles, 128 or 256: 128-row tiles, else by the work.  A
// product on 128-row tiles takes as long as one tile while the chip holds them
// all.  16-row tiles take a round per two of them and compute unit, for the row
// tiles with a real row (about one per bucket more than a sixteenth of the
// atoms), and bring the weights in more slowly, which for wide layers costs as
// much as 45 more row tiles.  First layer (1,008 columns), one network of 160 to
// 256 channels, 16-row and 128-row tiles: 30 solutes (2,000 atoms) 28 to 42 and
// 61 us, 60 of them 47 to 61 and 61, 100 65 to 82 and 62, 200 109 to 139 and 65
// (the float32 instructions 60 to 98); 3 networks of 256 10 solutes 52 and 66, 25
// 69 and 65; 8 of 128 6 solutes 59 and 69, 20 89 and 69; 8 of 256 one of 65 atoms
// 73 and 60, but one of 24, with 4 of the 7 buckets, 6 us less than wide tiles.
// With 32 or 64 channels (half a wide tile's columns) 200 solutes 47 and 59, 300
// 66 and 61.
// Where the real work is not known here, 16-row tiles until the 128-row ones
// give every compute unit one: in calls with a mask (n_atoms < 0; 1,138 of 11,557
// atoms of a DeepPot call 152 us so, 170 by the rule above), and in dE/dG with row
// records, where the line suits boxes (2,001 atoms of water x 3 networks of 256
// channels 28 and 40 us) and solutes would take the wide tiles sooner (40 of them
// x 3 83 and 42).
void launch_gemm_split(int epi, GemmLaunch gl, int rows, int n_atoms, int max_n_out, int tn_pref, hipStream_t st) {
  if (rows <= 0) return;
  // members side by side where they share A and every 32-column block lies
  // in one member
  gl.span = epi == kEpiFwd && gl.a_member_stride == 0 && gl.n_members > 1;
  int cols = max_n_out;
  if (gl.span) cols *= gl.n_members;
  const long long wide = (long long)((cols + 127) / 128) * (gl.span ? 1 : gl.n_members);
  const long long narrow = (long long)((cols + 63) / 64) * (gl.span ? 1 : gl.n_members);
  const bool few = n_atoms < 0 || (epi == kEpiOut && gl.row_mask)
                       ? rows / 128 * wide < 256
                       : (n_atoms / 16 + gl.n_groups + 45) * narrow <= (narrow > 1 ? 1400 : 920) ||
                             (n_atoms <= 32 && narrow <= 32);
  const bool small = tn_pref == 64 || (tn_pref != 128 && tn_pref != 256 && few);
  // a workgroup per compute unit at most (see above)
  const bool lone = small && rows / 16 * narrow <= 256;
#define NNP_SPLIT(E)                                                    \
  if (lone) gemm_split_t<E, 1, 1, 1, 4, 8, 2>(gl, rows, cols, st);      \
  else if (small) gemm_split_t<E, 1, 1, 1, 4, 4, 1>(gl, rows, cols, st); \
  else gemm_split_t<E, 2, 8, 4, 1, 2, 1>(gl, rows, cols, st)
  if (epi == kEpiFwd) { NNP_SPLIT(kEpiFwd); }
  else if (epi == kEpiBwd) { NNP_SPLIT(kEpiBwd); }
  else { NNP_SPLIT(kEpiOut); }
#undef NNP_SPLIT
}

}  // namespace nnp
