// Fused hidden-layer chain of the element networks (section "Neural Network
// Potentials": one feed-forward network per element, atomic energies summed).
//
// After the first dense layer (a large GEMM over the AEV), the remaining
// layers of a network are narrow (<= 256 wide): run as separate GEMMs their
// activations make several round trips through HBM.  Here one workgroup of
// eight waves takes 16 HR rows of one species bucket for one ensemble member
// and runs the rest of the network on chip:
//   forward   h_l = CELU(h_{l-1} W_l^T + b_l) for the hidden layers l >= 1,
//             E = h_last . w_out + b_out, d_last = w_out * CELU'(h_last) / M;
//   backward  d_{l-1} = (d_l W_l) * CELU'(h_{l-1}) down to d_0,
// keeping every h_l / d_l tile in LDS and writing only d_0 (the input gradient
// the AEV-gradient GEMM needs) and the member's energy per row.  A tile is
// held in P planes: P = 1, bfloat16 models, the values rounded to bfloat16
// exactly where the unfused path stores them; P = 3, float32 models, the three
// bfloat16 parts of the values (split.hip), split once when they are written
// (held as float32 and split by every wave that reads them, the splitting took
// as many cycles as the MFMAs).
//
// What bounds it is the wait for the weights: a layer is only 3 to 8 K steps
// long, and L2 answers in about as long as a layer takes.  So the weights lie
// in fragment order (a wave's load is one contiguous KB, no address work),
// the first steps' fragments of a layer are already on their way while the
// layer before it finishes (the barriers between layers wait for LDS only),
// and the K loop is unrolled for each length, so that every wait counts
// exactly the loads behind it.
#include "internal.h"
#include "split.h"
#include "wave.h"

namespace nnp {

// CELU with the hardware exp2 (about 1 ulp; the result is rounded to
// bfloat16 next), k_exp = log2(e) / alpha; CELU' from h = CELU(z) with
// inv_alpha = 1 / alpha.
__device__ inline float celu_f(float z, float alpha, float k_exp) {
  return z > 0.f ? z : alpha * (__builtin_amdgcn_exp2f(z * k_exp) - 1.f);
}
__device__ inline float dcelu_h(float h, float inv_alpha) { return h > 0.f ? 1.f : 1.f + h * inv_alpha; }

// ------------------------------------------------------------------ weights
// Element k of a row's 32-column chunk c, part p, of a [N][K] matrix (N a
// multiple of 16, K of 32) in fragment order: 16-row block, chunk, part, then
// the MFMA operand's lanes (row % 16, columns 8 (lane / 16) + 0..7).
template <int P>
__global__ void __launch_bounds__(256)
k_weight_frags(const float *__restrict__ src, const uint16_t *__restrict__ src_b, int N, int K,
               uint16_t *__restrict__ dst) {
  const int total = N * K;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
    const int r = t / K, k = t - r * K;
    uint16_t *d = dst + ((size_t)((r / 16) * (K / 32) + k / 32) * P) * 512 + ((k % 32) / 8 * 16 + r % 16) * 8 + k % 8;
    if (P == 1) {
      d[0] = src_b[t];
    } else {
      const float x = src[t];
      const __bf16 p1 = (__bf16)x;
      const float a = x - (float)p1;
      const __bf16 p2 = (__bf16)a;
      d[0] = __builtin_bit_cast(uint16_t, p1);
      d[512] = __builtin_bit_cast(uint16_t, p2);
      d[1024] = __builtin_bit_cast(uint16_t, (__bf16)(a - (float)p2));
    }
  }
}

void launch_weight_frags(const float *src, const uint16_t *src_b, int N, int K, uint16_t *dst, hipStream_t st) {
  const unsigned blocks = (unsigned)((N * K + 255) / 256);
  if (src_b) k_weight_frags<1><<<blocks, 256, 0, st>>>(nullptr, src_b, N, K, dst);
  else k_weight_frags<3><<<blocks, 256, 0, st>>>(src, nullptr, N, K, dst);
}

// -------------------------------------------------------------------- tiles
struct ChainTile {
  uint16_t *p;  // first plane
  int ld;       // row stride, elements (padded by 8: the 16 rows of a fragment read fall on different banks)
  int plane;    // elements between planes
};

// Four consecutive elements of a row: 8 bytes in each plane.  P = 3,
// activations (huge given): a value without a finite first part keeps its
// leading bits there (an infinity nothing else), so that its parts still add up
// to it, and is reported.  (Gradients do not come near it, see split.hip.)
template <int P>
__device__ inline void put4(const ChainTile &t, int row, int col, float (&x)[4], bool *huge = nullptr) {
  uint16_t *d = t.p + row * t.ld + col;
  if (P == 3 && huge) {
    const bool b = fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))) > kPartMax;
    if (__builtin_expect(__ballot(b) != 0, 0)) {
      *huge = *huge || b;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float v = x[k];
        const bool big = fabsf(v) > kPartMax, inf = fabsf(v) > 3.4028235e38f;
        const uint32_t u1 = big ? __float_as_uint(v) >> 16 : round2(v, 0.f) & 0xffffu;
        const float r = inf ? 0.f : v - __uint_as_float(u1 << 16);
        const uint32_t u2 = round2(r, 0.f) & 0xffffu;
        d[k] = (uint16_t)u1;
        d[k + t.plane] = (uint16_t)u2;
        d[k + 2 * t.plane] = (uint16_t)round2(r - __uint_as_float(u2 << 16), 0.f);
      }
      return;
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    uint2 w;
    w.x = round2(x[0], x[1]);
    w.y = round2(x[2], x[3]);
    *(uint2 *)(d + p * t.plane) = w;
    if (p + 1 < P) {
      x[0] -= __uint_as_float(w.x << 16);
      x[1] -= __uint_as_float(w.x & 0xffff0000u);
      x[2] -= __uint_as_float(w.y << 16);
      x[3] -= __uint_as_float(w.y & 0xffff0000u);
    }
  }
}
template <int P>
__device__ inline void get4(const ChainTile &t, int row, int col, float (&x)[4]) {
  const uint16_t *d = t.p + row * t.ld + col;
  uint2 w[P];
#pragma unroll
  for (int p = 0; p < P; ++p) w[p] = *(const uint2 *)(d + p * t.plane);
  x[0] = __uint_as_float(w[P - 1].x << 16);
  x[1] = __uint_as_float(w[P - 1].x & 0xffff0000u);
  x[2] = __uint_as_float(w[P - 1].y << 16);
  x[3] = __uint_as_float(w[P - 1].y & 0xffff0000u);
#pragma unroll
  for (int p = P - 2; p >= 0; --p) {
    x[0] += __uint_as_float(w[p].x << 16);
    x[1] += __uint_as_float(w[p].x & 0xffff0000u);
    x[2] += __uint_as_float(w[p].y << 16);
    x[3] += __uint_as_float(w[p].y & 0xffff0000u);
  }
}

// ----------------------------------------------------------------- products
// C[16 HR x N] = A[16 HR x K] (LDS) . W^T.  Each product is formed transposed
// (weights as the MFMA's first operand), so that a lane ends with four
// consecutive columns of one row: block cb's accumulators hold, of each
// sixteen-row group h, row 16 h + l % 16 and columns 16 cb + 4 (l / 16) + j,
// j = 0..3.  Wave w owns the 16-column blocks w and w + 8 (N <= 256).
constexpr int kChainWaves = 8, kChainBlocks = 2;
constexpr int kChainFirst = 2;  // K steps of the next layer loaded ahead
// K steps loaded ahead within a layer: what the registers hold
template <int P, int HR> constexpr int kChainAhead = P == 3 ? (HR == 1 ? 5 : 3) : (HR == 4 ? 2 : 4);

// The loads above stay above (the scheduler would move them down to their
// uses, and the waits with them).
__device__ inline void pin_loads() { __builtin_amdgcn_sched_barrier(0); }

template <int P, int HR> struct ChainAcc {
  floatx4 v[kChainBlocks][HR];
  floatx4 low[kChainBlocks][P == 3 ? HR : 1];  // P = 3: the small products
};
template <int P> struct ChainFirst {
  uint4 b[kChainFirst][kChainBlocks][P];
};

// One K step: a block's fragments against the row groups'.
template <int P, int NQ, int HR>
__device__ inline void chain_step(const uint16_t *ap, const ChainTile &A, int kb, const uint4 (&w)[NQ][P],
                                  ChainAcc<P, HR> &acc) {
  bf16x8 a[HR][P];
#pragma unroll
  for (int h = 0; h < HR; ++h)
#pragma unroll
    for (int p = 0; p < P; ++p)
      a[h][p] = __builtin_bit_cast(bf16x8, *(const uint4 *)(ap + p * A.plane + 16 * h * A.ld + kb * 32));
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const bf16x8 w1 = __builtin_bit_cast(bf16x8, w[q][0]);
    if constexpr (P == 1) {
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.v[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, a[h][0], acc.v[q][h], 0, 0, 0);
    } else {
      const bf16x8 w2 = __builtin_bit_cast(bf16x8, w[q][1]), w3 = __builtin_bit_cast(bf16x8, w[q][2]);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.low[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, a[h][2], acc.low[q][h], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.low[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3, a[h][0], acc.low[q][h], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.low[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, a[h][1], acc.low[q][h], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.low[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, a[h][1], acc.low[q][h], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.low[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, a[h][0], acc.low[q][h], 0, 0, 0);
#pragma unroll
      for (int h = 0; h < HR; ++h) acc.v[q][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, a[h][0], acc.v[q][h], 0, 0, 0);
    }
  }
}

// All K steps of a layer for NQ blocks of the wave; wp: the wave's first
// fragments, `first` the ones already loaded.
template <int P, int NKB, int NQ, int HR>
__device__ inline void chain_mm(const uint16_t *ap, const ChainTile &A, Global<uint16_t> wp,
                                const ChainFirst<P> &first, ChainAcc<P, HR> &acc) {
  constexpr int AH = kChainAhead<P, HR>;
  uint4 w[NKB][NQ][P];
  auto load = [&](int k) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int p = 0; p < P; ++p) w[k][q][p] = load16(wp + (q * kChainWaves * NKB + k) * (P * 512) + p * 512);
  };
#pragma unroll
  for (int k = 0; k < NKB; ++k) {
    if (k < kChainFirst) {
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int p = 0; p < P; ++p) w[k][q][p] = first.b[k][q][p];
    } else if (k < AH) {
      load(k);
    }
  }
  pin_loads();
#pragma unroll
  for (int k = 0; k < NKB; ++k) {
    if (k + AH < NKB) {
      load(k + AH);
      pin_loads();
    }
    chain_step<P, NQ, HR>(ap, A, k, w[k], acc);
  }
}

template <int P, int HR>
__global__ void __launch_bounds__(kChainWaves * kWave, P == 3 ? 2 : 4)
k_chain(ChainLaunch cl, int n_hidden, int grad) {
  constexpr int R = 16 * HR, T = kChainWaves * kWave;
  const float inv_alpha = 1.f / cl.alpha, k_exp = 1.4426950408889634f * inv_alpha;
  extern __shared__ uint4 chain_lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
  const int l16 = lane & 15, kq = lane >> 4;
  // member-major logical order in chunks of row tiles per XCD: an XCD works
  // through a run of row tiles of one (member, species) network at a time,
  // whose weights then stay in its L2
  const int lb = xcd_chunked(blockIdx.x, cl.xcd_chunk);
  if (lb >= cl.n_blocks) return;
  const int n_rt = cl.n_blocks / cl.n_members;
  const int mb = lb / n_rt;
  const int r0 = (lb - mb * n_rt) * R;
  int real_end;
  const int s = tile_bucket(cl.bucket_off, cl.bucket_cnt, cl.n_groups, r0, lane, real_end);
  if (s < 0 || r0 >= real_end) return;  // padding rows only: their gradients are not read
  const ChainNet &net = cl.nets[mb * cl.n_groups + s];
  auto tile = [&](int l) {  // offsets are of 16 rows
    return ChainTile{(uint16_t *)chain_lds + cl.lds_off[l] * HR, cl.lds_ld[l], R * cl.lds_ld[l]};
  };
  // Layers 1 .. n_hidden forward, then n_hidden .. 1 backward: layer `ph` of
  // 2 n_hidden (weights, K steps, column blocks).
  struct Layer {
    const uint16_t *w;
    int nkb, ncb;
  };
  auto layer = [&](int ph) {
    const int l = ph <= n_hidden ? ph : 2 * n_hidden + 1 - ph;
    if (ph <= n_hidden) return Layer{net.W[l - 1], net.width[l - 1] / 32, net.width[l] / 16};
    return Layer{net.Wt[l - 1], net.width[l] / 32, net.width[l - 1] / 16};
  };
  // the wave's block q of a layer; a block past the end repeats the last one
  auto frags = [&](const Layer &y, int q) {
    return as_global(y.w) + (size_t)min(wave + q * kChainWaves, y.ncb - 1) * y.nkb * (P * 512) + lane * 8;
  };
  ChainFirst<P> first;
  auto load_first = [&](const Layer &y) {
#pragma unroll
    for (int k = 0; k < kChainFirst; ++k)
#pragma unroll
      for (int q = 0; q < kChainBlocks; ++q)
#pragma unroll
        for (int p = 0; p < P; ++p)
          first.b[k][q][p] = load16(frags(y, q) + min(k, y.nkb - 1) * (P * 512) + p * 512);
    pin_loads();
  };
  // every wave's LDS writes are done; loads of weights in flight stay in flight
  auto lds_barrier = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // P = 3: whether h_l holds a value without a finite first part
  __shared__ int huge_tile[kChainMax + 1];
  if (P == 3) {
    if (tid <= kChainMax) huge_tile[tid] = 0;
    lds_barrier();
  }
  auto report = [&](int l, bool huge) {
    if (P == 3 && __builtin_expect(__ballot(huge) != 0, 0)) huge_tile[l] = 1;
  };

  Layer cur = layer(1);
  load_first(cur);
  // h_0 tile (this member's slice of the first layer's output) into LDS
  {
    const ChainTile t0 = tile(0);
    const int w0 = net.width[0];
    bool huge = false;
    if (P == 1) {
      const uint16_t *src = cl.H0 + (size_t)r0 * cl.ldh + (size_t)mb * cl.h_member_stride;
      const int ch = 8 * (tid & 31);
      if (ch < w0)
        for (int row = tid >> 5; row < R; row += T / 32)
          *(uint4 *)(t0.p + row * t0.ld + ch) = *(const uint4 *)(src + (size_t)row * cl.ldh + ch);
    } else {
      const float *src = (const float *)cl.H0 + (size_t)r0 * cl.ldh + (size_t)mb * cl.h_member_stride;
      const int ch = 4 * (tid & 63);
      if (ch < w0) {
#pragma unroll
        for (int row = tid >> 6; row < R; row += T / 64) {
          // (padding rows hold whatever an earlier call left there)
          const float4 v = r0 + row < real_end ? *(const float4 *)(src + (size_t)row * cl.ldh + ch)
                                               : make_float4(0.f, 0.f, 0.f, 0.f);
          float x[4] = {v.x, v.y, v.z, v.w};
          put4<P>(t0, row, ch, x, &huge);
        }
      }
    }
    report(0, huge);
  }
  lds_barrier();

  float *d0 = (float *)cl.D0 + (size_t)r0 * cl.ldd + (size_t)mb * cl.d_member_stride;  // P = 3
  const int n_ph = grad ? 2 * n_hidden : n_hidden;
  for (int ph = 1; ph <= n_ph; ++ph) {
    const bool fwd = ph <= n_hidden;
    const int l_in = fwd ? ph - 1 : 2 * n_hidden + 1 - ph;  // input tile
    const int l_out = fwd ? ph : l_in - 1;                  // output tile
    const ChainTile A = tile(l_in), out = tile(l_out);
    const uint16_t *ap = A.p + l16 * A.ld + 8 * kq;
    const int nq = cur.ncb > wave + kChainWaves ? 2 : cur.ncb > wave ? 1 : 0;
    float4 bias[kChainBlocks];
    if (fwd) {
#pragma unroll
      for (int q = 0; q < kChainBlocks; ++q)
        bias[q] = load4f(as_global(net.b[l_out - 1]) + 16 * min(wave + q * kChainWaves, cur.ncb - 1) + 4 * kq);
    }
    ChainAcc<P, HR> acc;
#pragma unroll
    for (int q = 0; q < kChainBlocks; ++q) {
#pragma unroll
      for (int h = 0; h < HR; ++h) {
        acc.v[q][h] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (P == 3) acc.low[q][h] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
    const bool plain = P == 1 || !fwd || __builtin_amdgcn_readfirstlane(huge_tile[l_in]) == 0;
    if (plain) {
      const Global<uint16_t> wp = frags(cur, 0);
#define NNP_CHAIN_K(NKB)                                                                       \
  case NKB:                                                                                    \
    if (nq == 2) chain_mm<P, NKB, 2, HR>(ap, A, wp, first, acc);                               \
    else if (nq == 1) chain_mm<P, NKB, 1, HR>(ap, A, wp, first, acc);                          \
    break;
      switch (cur.nkb) {
        NNP_CHAIN_K(1)
        NNP_CHAIN_K(2)
        NNP_CHAIN_K(3)
        NNP_CHAIN_K(4)
        NNP_CHAIN_K(5)
        NNP_CHAIN_K(6)
        NNP_CHAIN_K(7)
        default: NNP_CHAIN_K(8)
      }
#undef NNP_CHAIN_K
    } else if constexpr (P == 3) {
#pragma unroll 1
      for (int t = 0; t < 8 * cur.nkb; ++t) {  // element t % 8 of K step t / 8
#pragma unroll
        for (int q = 0; q < kChainBlocks; ++q) {
          const float w = joined(frags(cur, q) + (t >> 3) * (P * 512) + (t & 7), 512);
#pragma unroll
          for (int h = 0; h < HR; ++h)
            acc.v[q][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                w, joined(ap + 16 * h * A.ld + (t >> 3) * 32 + (t & 7), A.plane), acc.v[q][h], 0, 0, 0);
        }
      }
    }
    // the next layer's first weights, before this one's epilogue and barrier
    cur = layer(ph < n_ph ? ph + 1 : ph);
    load_first(cur);

    bool huge = false;
#pragma unroll
    for (int q = 0; q < kChainBlocks; ++q) {
      if (q < nq) {
        const int col = 16 * (wave + q * kChainWaves) + 4 * kq;
#pragma unroll
        for (int h = 0; h < HR; ++h) {
          floatx4 v = acc.v[q][h];
          if (P == 3) v += acc.low[q][h];
          const int row = 16 * h + l16;
          float x[4];
          if (fwd) {
            const float z[4] = {v[0] + bias[q].x, v[1] + bias[q].y, v[2] + bias[q].z, v[3] + bias[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
              x[j] = P == 1 ? celu_f(z[j], cl.alpha, k_exp) : celu32(z[j], cl.alpha, inv_alpha);
          } else {
            get4<P>(out, row, col, x);
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = v[j] * dcelu_h(x[j], inv_alpha);
          }
          if (P == 3 && ph == 2 * n_hidden)  // d_0 straight to memory
            *(float4 *)(d0 + (size_t)row * cl.ldd + col) = make_float4(x[0], x[1], x[2], x[3]);
          else
            put4<P>(out, row, col, x, fwd ? &huge : nullptr);
        }
      }
    }
    if (fwd) report(l_out, huge);
    if (P == 3 && ph == 2 * n_hidden) return;
    lds_barrier();

    // the member's energy of each row, E = h_last . w_out + b_out, and (for
    // forces) d_last = w_out CELU'(h_last) / M in place of h_last.  Eight
    // threads per row, each over the 8-column chunks seg, seg + 8, ..., then
    // summed over the eight: a fixed order, whatever the workgroup's shape.
    if (ph == n_hidden) {
      const int nch = net.width[n_hidden] / 8;
      const ChainTile hl = out;
      // R * 8 is a multiple of 64: every group of eight lanes takes the loop's
      // iterations together
      for (int t8 = tid; t8 < R * 8; t8 += T) {
        const int row = t8 >> 3, seg = t8 & 7;
        float e = 0.f;
        for (int ch = seg; ch < nch; ch += 8) {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int col = ch * 8 + 4 * half;
            float h[4];
            get4<P>(hl, row, col, h);
            const float4 w4 = load4f(as_global(net.w_out) + col);
            const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              e += h[k] * w[k];
              h[k] = w[k] * dcelu_h(h[k], inv_alpha) * cl.inv_m;
            }
            if (grad) put4<P>(hl, row, col, h);
          }
        }
        e = sum8(e);
        if (seg == 0) {
          if (cl.n_members == 1) {
            // a single network: the row's energy is the atomic energy
            const int atom = cl.perm[r0 + row];
            if (atom >= 0) cl.e_atom[atom] = e + net.b_out;
          } else {
            cl.e_mem[(size_t)(r0 + row) * cl.n_members + mb] = e + net.b_out;
          }
        }
      }
      lds_barrier();
    }
  }
  if (!grad) return;

  // d_0 tile to memory (bfloat16, 16-byte stores)
  if (P == 1) {
    const ChainTile t0 = tile(0);
    const int w0 = net.width[0];
    uint16_t *dst = cl.D0 + (size_t)r0 * cl.ldd + (size_t)mb * cl.d_member_stride;
    const int ch = 8 * (tid & 31);
    if (ch < w0)
      for (int row = tid >> 5; row < R; row += T / 32)
        *(uint4 *)(dst + (size_t)row * cl.ldd + ch) = *(const uint4 *)(t0.p + row * t0.ld + ch);
  }
}

// Atomic energies: mean over the members' energies of each row.  Rows past
// the last species bucket carry no atom (and no permutation entry).
__global__ void k_chain_mean(const float *__restrict__ e_mem, int M, const int *__restrict__ perm,
                             const int *__restrict__ bucket_off, int n_groups, int rows, float inv_m,
                             float *__restrict__ e_atom) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= rows || row >= bucket_off[n_groups]) return;
  const int atom = perm[row];
  if (atom < 0) return;
  float e = 0.f;
  for (int m = 0; m < M; ++m) e += e_mem[(size_t)row * M + m];
  e_atom[atom] = e * inv_m;
}

template <int P, int HR>
static void chain_t(ChainLaunch cl, int n_hidden, bool grad, int rows, size_t lds16, hipStream_t st) {
  cl.n_blocks = rows / (16 * HR) * cl.n_members;
  cl.xcd_chunk = 512 / (16 * HR);   // 512 rows of one network per chunk
  k_chain<P, HR><<<xcd_grid((unsigned)cl.n_blocks, cl.xcd_chunk), kChainWaves * kWave, lds16 * HR, st>>>(cl, n_hidden,
                                                                                                      grad ? 1 : 0);
}

// lds16: LDS bytes of the activation tiles of 16 rows.  rows_pref: rows per
// workgroup (16, 32 or 64), 0: by the grid.  More rows amortize the weights'
// trip from L2; fewer fill the compute units sooner.  rows is a multiple of
// 128.
void launch_chain(const ChainLaunch &cl, bool f32, int n_hidden, bool grad, int rows, size_t lds16, int rows_pref,
                  size_t max_lds, hipStream_t st) {
  if (rows <= 0) return;
  const long long all = (long long)rows * cl.n_members;
  int r = rows_pref ? rows_pref : all >= 64 * 512 && !f32 ? 64 : all >= 32 * 256 ? 32 : 16;
  while (r > 16 && lds16 * (r / 16) + 64 > max_lds) r /= 2;
  if (f32) {
    if (r >= 32) chain_t<3, 2>(cl, n_hidden, grad, rows, lds16, st);
    else chain_t<3, 1>(cl, n_hidden, grad, rows, lds16, st);
  } else {
    if (r >= 64) chain_t<1, 4>(cl, n_hidden, grad, rows, lds16, st);
    else if (r >= 32) chain_t<1, 2>(cl, n_hidden, grad, rows, lds16, st);
    else chain_t<1, 1>(cl, n_hidden, grad, rows, lds16, st);
  }
  if (cl.n_members > 1)
    k_chain_mean<<<(rows + 255) / 256, 256, 0, st>>>(cl.e_mem, cl.n_members, cl.perm, cl.bucket_off, cl.n_groups,
                                                      rows, cl.inv_m, cl.e_atom);
}

}  // namespace nnp
