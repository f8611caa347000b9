// Step-wise forward (prefill / decode) of the TNT memory layer from a carried
// state.
//
// Within a chunk every gradient is taken at the chunk-entry weights (Sec. 2.2)
// and folded in with momentum and decay (App. D), so the chunkwise rule has an
// exact token-by-token form once the entry weights are kept beside the
// running ones:
//     u_t = grad_W l(W^; k_t, v_t)           (W^ = weights entering t's chunk)
//     S_t = mom_t S_{t-1} - lr_t u_t,    W_t = (1 - decay_t) W_{t-1} + S_t,
// and W^ <- W at every chunk start.  The global memory reads at its entry
// state, o_G = f(V^, q_t) (Sec. 4.1.2 retrieval box); a local memory resets
// (W^, W, S, M) to (W_init, W_init, 0, 0) at each shard start, adds
// k_t k_t^T / ||k_t||^2 to its Q-K sum M and reads at W_t after the update,
// o_i = f(W_t, M q_t) (Sec. 4.1.1 local update, Sec. 4.1.2; App. C).
//
// The state of every (memory, chain) is split by hidden unit into G slices of
// HS = min(64, hid): slice g owns rows [g HS, (g+1) HS) of W1, S1 and the same
// columns of W2, S2.  Everything that is taken at the entry weights (z = W^1 k,
// y = W^2 s(z), the residual r, delta = (W^2^T r) s'(z), the global retrieval) is
// independent from token to token until the next chunk boundary, and a slice's
// running weights depend on r and its own rows only.  So up to STEP_N tokens that
// no memory's chunk boundary divides, and that the scratch area has room for, take
// two launches:
//   tokens  one workgroup per (slice, chain, memory): y of every token over all
//           hidden units (each slice forms it for itself: no exchange between
//           workgroups), r, the slice's delta; then, token by token with the
//           slice's W1, S1, W2, S2 in registers, the gated update and a local
//           memory's share of W2_t s(W1_t x).  A local memory's queries
//           x = M_t q come from a private copy of its Q-K sum.
//   out     o = the sum of the retrieval shares (global memory first, fixed
//           order); M += k k^T / ||k||^2 of every token.
// A further launch, before them, where a memory's chunk or shard begins: W^ <- W,
// or the reset.
//
// One token by itself, and few of a wide head or of many chains (step_alone), take
//   entry   the slice's z, its share of y and of the global retrieval, and its
//           rows of a local memory's query
//   update  r from the shares, delta, the update and the retrieval share
// instead of the tokens launch: there W^1 is read once and W^2 twice, not G times
// each (from G XCDs: the slices of a chain are neighbours in the grid), and a
// workgroup's registers leave room for several on a CU (the tokens launch takes a
// CU's registers with one workgroup at d 64, and spills at d 128).
//
// The products at the entry weights are fp32 MFMA tiles of 16 tokens (rows past the
// launch's tokens zero), y a sum of one such product per slice in the order of the
// slices, in both forms; a token's row does not depend on the other rows, so every
// cut of a sequence gives bitwise the same results.
//
// Bound by the launches' latency at few chains (entry, update and out: 14.7 us for one
// chain at d 64, hid 256, global + one local) and by the state's bytes at many: its 11
// hid d floats per (memory, chain) and token (W^1, W1, S1, W2, S2 in once, W^2 twice, the
// 4 updated ones out) take 162 us for 512 chains, 4.6 TB/s.  With three
// launches of vector products before, 25 and 196 us.  77 tokens at B 2, H 8: 347 us,
// against 2104 with launches for every token.
#include "tnt_device.h"
#include "tnt_kernels.h"

#include <algorithm>
#include <type_traits>

namespace tnt {

namespace {

constexpr int STEP_THREADS = 256;
// threads of a token launch: 512 at d = 128, where a slice's state, M and the weights
// in flight take twice the registers (135 of them spill all the same)
constexpr int step_threads(int d) { return d == 128 ? 512 : STEP_THREADS; }
constexpr int STEP_MAX_D = 128, STEP_MAX_H = 512;
constexpr int STEP_N = 16;  // tokens of one launch at most: the rows of an MFMA tile

// LDS of the token launch (floats; rows padded by 16 bytes)
struct StepLds {
  int ld, lh, ls;                           // row strides: d, hid, HS
  int k, q, r, x, a, aq, sp, g, z, kk, kq, gt;  // offsets
  int total;
};
__host__ __device__ inline StepLds step_lds(int d, int hid, int HS) {
  StepLds y;
  y.ld = d + 4; y.lh = hid + 4; y.ls = HS + 4;
  int o = 0;
  y.k = o; o += STEP_N * y.ld;
  y.q = o; o += STEP_N * y.ld;
  y.r = o; o += STEP_N * y.ld;
  y.x = o; o += STEP_N * y.ld;
  y.a = o; o += STEP_N * y.lh;   // s(z)
  y.aq = o; o += STEP_N * y.lh;  // s(W^1 q) (global memory)
  y.sp = o; o += STEP_N * y.ls;  // s'(z) of the slice
  y.g = o; o += STEP_N * y.ls;   // delta of the slice
  y.z = o; o += 2 * HS;          // s(W1_t x) of the slice, two tokens in turn
  y.kk = o; o += STEP_N;         // 1 / ||k||^2 (0 for a zero key)
  y.kq = o; o += STEP_N;         // k . q
  y.gt = o; o += 3 * STEP_N;     // lr, mom, decay
  y.total = o;
  return y;
}

// Sum over P 16-byte pieces of a lane's row of B in the product (t, j) -> sum_k A[t][k]
// B[j][k] (16 rows t of A in LDS, 16 rows j of B, both contraction-contiguous): the piece
// at contraction offset k0 + 4 (lane / 16) holds four consecutive k, one per MFMA step (the
// steps sum the same k on both sides).  ONE: the only row is 0, at A.  The pieces are added
// as a tree: in one accumulator, where every step rounds the whole sum, fp32 outputs are
// 2.0 to 2.4e-7 from 64 bits at d 64 and 128, and 1.4 to 1.7e-7 with the tree (as with lane
// sums of vector products).  FINE, for d 16 and 32, halves the chains once more; at wider
// d that costs up to 17 % (d 64, hid 256, 128 chains: 44.6 for 38.3 us) and gains 1 to 6 %.
template <int P, bool ONE, bool FINE>
__device__ __forceinline__ f4 row_sum(const float* A, int lda, int k0, const f4* b) {
  if constexpr (P == 1) {
    const int l = lane_id();
    f4 x = *reinterpret_cast<const f4*>(A + (ONE ? 0 : (l & 15) * lda) + k0 + 4 * (l >> 4));
    if (ONE && (l & 15)) x = zero4();
    constexpr int CHAIN = FINE ? 2 : 4;  // steps in one accumulator
    f4 p[4 / CHAIN];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      p[r / CHAIN] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r], b[0][r], r % CHAIN ? p[r / CHAIN] : zero4(), 0, 0, 0);
    if constexpr (FINE) return p[0] + p[1];
    return p[0];
  } else {
    return row_sum<P / 2, ONE, FINE>(A, lda, k0, b) + row_sum<P - P / 2, ONE, FINE>(A, lda, k0 + 16 * (P / 2), b + P / 2);
  }
}

// Sums over groups of W consecutive lanes (4, 8, 16 or 32, aligned), every lane of a
// group getting the sum, for NU values at once: exchanges inside the quads, then
// mirrors of 8 and 16 lanes (whose quads / halves hold equal values by then).
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
template <int NU>
__device__ __forceinline__ void group_sums(float (&x)[NU], int W) {
#pragma unroll
  for (int u = 0; u < NU; ++u) x[u] += dpp_f<0xB1>(x[u]);  // quad_perm [1, 0, 3, 2]
#pragma unroll
  for (int u = 0; u < NU; ++u) x[u] += dpp_f<0x4E>(x[u]);  // quad_perm [2, 3, 0, 1]
  if (W >= 8)
#pragma unroll
    for (int u = 0; u < NU; ++u) x[u] += dpp_f<0x141>(x[u]);  // row_half_mirror
  if (W >= 16)
#pragma unroll
    for (int u = 0; u < NU; ++u) x[u] += dpp_f<0x140>(x[u]);  // row_mirror
  if (W >= 32)
#pragma unroll
    for (int u = 0; u < NU; ++u) x[u] += __shfl_xor(x[u], 16, WAVE);
}

// The sums below are written as fused products one by one, so that both forms of a
// step round alike (a token's results do not depend on the form that took it).
__device__ __forceinline__ float dot4(const f4& a, const f4& b) {
  return __builtin_fmaf(a[3], b[3], __builtin_fmaf(a[2], b[2], __builtin_fmaf(a[1], b[1], a[0] * b[0])));
}
// w <- keep w + s, s <- beta s - c v
__device__ __forceinline__ void gated(f4& w, f4& s, float beta, float keep, float c, const f4& v) {
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    s[x] = __builtin_fmaf(beta, s[x], -(c * v[x]));  // (the larger product unrounded)
    w[x] = __builtin_fmaf(keep, w[x], s[x]);
  }
}

// One token on a slice's state in registers (pieces tid + u NT of W1, S1 by rows and of
// W2, S2 by rows of the slice's columns): the gated update, and a local memory's share of
// W2_t s(W1_t x).  k, r, x: the token's rows; av, gv: s(z) and delta on the slice; zt:
// HS floats of LDS, no two consecutive tokens' alike.
template <int ACT, int D, int NT, int NU>
__device__ __forceinline__ void slice_token(f4 (&w1)[NU], f4 (&s1)[NU], f4 (&w2)[NU], f4 (&s2)[NU], int HS,
                                            bool global, float eta, float beta, float keep, const float* k,
                                            const float* r, const float* x, const float* av, const float* gv,
                                            float* zt, float* share) {
  constexpr int g4 = D / 4;
  const int tid = threadIdx.x, h4 = HS / 4, n4 = HS * g4;
  const f4 kv = reinterpret_cast<const f4*>(k)[tid % g4];
  const f4 a4 = reinterpret_cast<const f4*>(av)[tid % h4];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int jj = (tid + u * NT) / g4;
    gated(w1[u], s1[u], beta, keep, eta * gv[jj < HS ? jj : 0], kv);
  }
  if (!global) {
    const f4 xv = reinterpret_cast<const f4*>(x)[tid % g4];
    float zp[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) zp[u] = dot4(w1[u], xv);
    group_sums<NU>(zp, g4);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int e = tid + u * NT;
      if (e < n4 && e % g4 == 0) zt[e / g4] = act_f<ACT>(zp[u]);
    }
    __syncthreads();  // (the other token's zt was last read before this barrier)
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int i = (tid + u * NT) / h4;
    gated(w2[u], s2[u], beta, keep, eta * r[i < D ? i : 0], a4);
  }
  if (!global) {
    const f4 zv = reinterpret_cast<const f4*>(zt)[tid % h4];
    float y[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) y[u] = dot4(w2[u], zv);
    group_sums<NU>(y, h4);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int e = tid + u * NT;
      if (e < n4 && e % h4 == 0) share[e / h4] = y[u];
    }
  }
}

// 1 / ||k||^2 (0 for a zero key) of one LDS row, the same in every launch
__device__ __forceinline__ float inv_norm2(const float* k, int d) {
  float s = 0.f;
  for (int i = lane_id(); i < d; i += WAVE) s = __builtin_fmaf(k[i], k[i], s);
  s = wave_sum(s);
  return s > 0.f ? 1.0f / s : 0.f;
}

// One token by itself: the scratch of a (memory, chain), floats: s(z) [hid], s'(z)
// [hid], x [d], then per slice the shares of W^2 s(z) [G][d] and of the retrieval [G][d]
struct StepOne {
  float *a, *sp, *x, *yp, *share;
};
__device__ __forceinline__ StepOne step_one(const StepArgs& a, int chain, int m) {
  float* b = a.scratch + ((size_t)m * a.B * a.H + chain) * a.sc_stride;
  StepOne s;
  s.a = b;
  s.sp = b + a.hid;
  s.x = s.sp + a.hid;
  s.yp = s.x + a.d;
  s.share = s.yp + (size_t)a.G * a.d;
  return s;
}

// the retrieval shares of a launch's tokens, per chain: [n][d] of the global memory
// (if any), then [n][G][d] of every local memory; of one token by itself: [G][d] of each
__device__ __forceinline__ float* step_share(const StepArgs& a, int chain, int m) {
  if (a.one) return step_one(a, chain, m).share;
  float* b = a.scratch + (size_t)chain * a.M * a.sc_stride;
  const size_t nd = (size_t)a.n * a.d;
  if (a.has_global && m == 0) return b;
  return b + (a.has_global ? nd : 0) + (size_t)(m - a.has_global) * a.G * nd;
}

}  // namespace

// A chunk or shard begins at position pos + t0: W^ <- W, or the reset.
__global__ void __launch_bounds__(256) step_boundary_kernel(StepArgs a) {
  const int chain = blockIdx.y, m = blockIdx.z;
  const long long p = a.pos + a.t0;
  const bool global = a.has_global && m == 0;
  const bool reset = !global && p % a.S[m] == 0;
  if (!reset && p % a.C[m] != 0) return;
  const int h = chain % a.H;
  const size_t hd4 = (size_t)a.hid * a.d / 4, dd4 = (size_t)a.d * a.d / 4;
  f4* base = reinterpret_cast<f4*>(a.state + ((size_t)m * a.B * a.H + chain) * a.mem_stride);
  const f4* W1i = reinterpret_cast<const f4*>(a.W1i) + ((size_t)m * a.H + h) * hd4;
  const f4* W2i = reinterpret_cast<const f4*>(a.W2i) + ((size_t)m * a.H + h) * hd4;
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
  for (size_t e = i0; e < hd4; e += st) {
    if (reset) {
      base[e] = base[2 * hd4 + e] = W1i[e];
      base[hd4 + e] = base[3 * hd4 + e] = W2i[e];
      base[4 * hd4 + e] = base[5 * hd4 + e] = zero4();
    } else {
      base[e] = base[2 * hd4 + e];
      base[hd4 + e] = base[3 * hd4 + e];
    }
  }
  if (!global && (reset || a.qk_scope == 1))
    for (size_t e = i0; e < dd4; e += st) base[6 * hd4 + e] = zero4();
}

// Tokens t0 .. t0 + n - 1.  Every weight a workgroup reads is requested before the
// first barrier (hid up to 256; the rest of a larger one in a second round).
template <typename IO, int ACT, int D>
__global__ void __launch_bounds__(step_threads(D), D == 64 ? 1 : 2) step_tokens_kernel(StepArgs a) {
  extern __shared__ __align__(16) float sm[];
  constexpr int d = D, NT = step_threads(D), NW = NT / WAVE;
  constexpr int g4 = D / 4;                    // 16-byte pieces of a row of W1, S1, M
  constexpr int NU = D <= 32 ? 2 : 16 * D / NT;  // pieces of each of the slice's arrays a thread holds
  constexpr int NM = (D * g4 + NT - 1) / NT;  // and of M
  constexpr int ND = D / 16;                   // tiles of d, pieces of a row of W^1
  constexpr bool FINE = D <= 32;
  constexpr int GZ = D == 128 ? 2 : 4;         // row tiles of W^1 a wave requests at a time
  constexpr int GY = D == 128 ? 8 : 16;        // pieces of a row of W^2 likewise
  const int g = blockIdx.x, chain = blockIdx.y, m = blockIdx.z;
  const int H = a.H, hid = a.hid, HS = a.HS, G = a.G, j0 = g * HS, n = a.n;
  const int tid = threadIdx.x, l = lane_id(), w = wave_id(), lg = l >> 4, lc = l & 15;
  const bool global = a.has_global && m == 0;
  const bool proj = !global && a.qk_proj;
  const size_t hd = (size_t)hid * d;
  float* const base = a.state + ((size_t)m * a.B * H + chain) * a.mem_stride;
  const float *Wh1 = base, *Wh2 = base + hd, *Mq = base + 6 * hd;
  float *W1 = base + 2 * hd + (size_t)j0 * d, *W2 = base + 3 * hd + j0;
  float *S1 = base + 4 * hd + (size_t)j0 * d, *S2 = base + 5 * hd + j0;
  const StepLds Y = step_lds(d, hid, HS);
  float *sk = sm + Y.k, *sq = sm + Y.q, *sr = sm + Y.r, *sx = sm + Y.x, *sa = sm + Y.a,
        *saq = sm + Y.aq, *ssp = sm + Y.sp, *sg = sm + Y.g, *sz = sm + Y.z, *skk = sm + Y.kk,
        *skq = sm + Y.kq, *sgt = sm + Y.gt;
  const size_t tok = ((size_t)chain * a.T + a.t0) * d;
  const IO *q = (const IO*)a.q + tok, *k = (const IO*)a.k + tok, *v = (const IO*)a.v + tok;
  const size_t gi = ((size_t)m * a.B * H + chain) * a.T + a.t0;

  for (int e = tid; e < STEP_N * d; e += NT) {
    const int t = e / d, i = e - t * d;
    sk[t * Y.ld + i] = t < n ? to_f(k[e]) : 0.f;
    sq[t * Y.ld + i] = t < n ? to_f(q[e]) : 0.f;
  }
  if (tid < 3 * STEP_N) {
    const int t = tid & (STEP_N - 1);
    const float* p = tid < STEP_N ? a.lr : tid < 2 * STEP_N ? a.mom : a.decay;
    if (t < n) sgt[tid] = p[gi + t];
  }
  // W^1 rows of the wave's first tiles, W^2 rows of its tile, the slice's W^2 columns
  f4 bz[GZ][ND], by[GY], bd[ND];
  auto load_z = [&](int x0) {
#pragma unroll
    for (int x = 0; x < GZ; ++x) {
      const int jt = w + NW * (x0 + x);
      if (jt < hid / 16)
#pragma unroll
        for (int s = 0; s < ND; ++s)
          bz[x][s] = *reinterpret_cast<const f4*>(Wh1 + (size_t)(jt * 16 + lc) * d + 16 * s + 4 * lg);
    }
  };
  auto load_y = [&](int it, int k0) {
#pragma unroll
    for (int s = 0; s < GY; ++s)
      if (k0 + 16 * s < hid)
        by[s] = *reinterpret_cast<const f4*>(Wh2 + (size_t)(it * 16 + lc) * hid + k0 + 16 * s + 4 * lg);
  };
  load_z(0);
  if (w < ND) load_y(w, 0);
  if (w < HS / 16)
#pragma unroll
    for (int s = 0; s < ND; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        bd[s][r] = Wh2[(size_t)(16 * s + 4 * lg + r) * hid + j0 + w * 16 + lc];
  // the slice's state and M
  const int h4 = HS / 4, n4 = HS * g4;
  constexpr int m4 = D * g4;
  f4 w1[NU], s1[NU], w2[NU], s2[NU], mq[NM];
  if (proj)
#pragma unroll
    for (int u = 0; u < NM; ++u) {
      const int e = tid + u * NT;
      if (e < m4) mq[u] = reinterpret_cast<const f4*>(Mq)[e];
    }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    w1[u] = s1[u] = w2[u] = s2[u] = zero4();
    if (e < n4) {
      const size_t o2 = (size_t)(e / h4) * hid + 4 * (e % h4);
      w1[u] = reinterpret_cast<const f4*>(W1)[e];
      s1[u] = reinterpret_cast<const f4*>(S1)[e];
      w2[u] = *reinterpret_cast<const f4*>(W2 + o2);
      s2[u] = *reinterpret_cast<const f4*>(S2 + o2);
    }
  }
  __syncthreads();

  // z = W^1 k of every hidden unit (and the global retrieval's W^1 q).  A product and
  // the reads of its accumulator stay in one basic block here and below: where a
  // branch between them joined, the compiler (ROCm 7.2) left out the wait for the
  // last MFMA on the path that skips it.
  auto z_phase = [&](auto two) {
    constexpr bool TWO = decltype(two)::value;
    for (int x0 = 0; w + NW * x0 < hid / 16; x0 += GZ) {
      if (x0) load_z(x0);
#pragma unroll
      for (int x = 0; x < GZ; ++x) {
        const int jt = w + NW * (x0 + x);
        if (jt >= hid / 16) continue;
        const f4 z = row_sum<ND, false, FINE>(sk, Y.ld, 0, bz[x]);
        f4 zq = zero4();
        if constexpr (TWO) zq = row_sum<ND, false, FINE>(sq, Y.ld, 0, bz[x]);
        const int j = jt * 16 + lc;
        const bool mine = j >= j0 && j < j0 + HS;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int t = 4 * lg + r;
          const ActVals av = act_all<ACT>(z[r]);
          sa[t * Y.lh + j] = av.s;
          if (mine) ssp[t * Y.ls + j - j0] = av.d1;
          if constexpr (TWO) saq[t * Y.lh + j] = act_f<ACT>(zq[r]);
        }
      }
    }
  };
  if (global)
    z_phase(std::true_type{});
  else
    z_phase(std::false_type{});
  if (proj)  // 1 / ||k||^2, k . q
    for (int t = w; t < n; t += NW) {
      const float ik = inv_norm2(sk + t * Y.ld, d);
      float s = 0.f;
      for (int i = l; i < d; i += WAVE) s = __builtin_fmaf(sk[t * Y.ld + i], sq[t * Y.ld + i], s);
      s = wave_sum(s);
      if (l == 0) {
        skk[t] = ik;
        skq[t] = s;
      }
    }
  __syncthreads();
  // r = (2/d) (W^2 s(z) - v); the global retrieval's columns dealt to the slices
  const float rs = 2.0f / (float)d;
  auto y_tile = [&](int it, auto pieces, auto two) {
    constexpr int P = decltype(pieces)::value;  // pieces of a row of W^2 a round
    constexpr bool TWO = decltype(two)::value;
    constexpr int S = P < 4 ? P : 4;  // pieces of a slice, summed slice by slice
    f4 y = zero4(), yq = zero4();
    for (int k0 = 0; k0 < hid; k0 += 16 * P) {
      if (it != w || k0) load_y(it, k0);
#pragma unroll
      for (int s0 = 0; s0 < P; s0 += S) {
        y += row_sum<S, false, FINE>(sa, Y.lh, k0 + 16 * s0, by + s0);
        if constexpr (TWO) yq += row_sum<S, false, FINE>(saq, Y.lh, k0 + 16 * s0, by + s0);
      }
    }
    const int i = it * 16 + lc;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = 4 * lg + r;
      sr[t * Y.ld + i] = t < n ? rs * (y[r] - to_f(v[(size_t)t * d + i])) : 0.f;
      if (TWO && t < n) step_share(a, chain, m)[(size_t)t * d + i] = yq[r];
    }
  };
  auto y_rows = [&](auto pieces) {
    for (int it = w; it < ND; it += NW) {
      if (global && it % G == g)
        y_tile(it, pieces, std::true_type{});
      else
        y_tile(it, pieces, std::false_type{});
    }
  };
  switch (hid / 16) {  // a power of two
    case 1: y_rows(std::integral_constant<int, 1>{}); break;
    case 2: y_rows(std::integral_constant<int, 2>{}); break;
    case 4: y_rows(std::integral_constant<int, 4>{}); break;
    case 8: y_rows(std::integral_constant<int, 8>{}); break;
    default: y_rows(std::integral_constant<int, GY>{}); break;
  }
  // a local memory's queries, token by token: x = M_{t-1} q + k (k . q) / ||k||^2,
  // M_t = M_{t-1} + k k^T / ||k||^2 (or q itself)
  if (proj) {
    for (int t = 0; t < n; ++t) {
      const f4 *k4 = reinterpret_cast<const f4*>(sk + t * Y.ld), *q4 = reinterpret_cast<const f4*>(sq + t * Y.ld);
      const float ik = skk[t], c = skq[t] * ik;
      const f4 qv = q4[tid % g4], kv = k4[tid % g4];  // a thread's pieces share their column
      static_assert(NT % g4 == 0, "one column of pieces per thread");
      float s[NM];
#pragma unroll
      for (int u = 0; u < NM; ++u) s[u] = dot4(mq[u], qv);
      group_sums<NM>(s, g4);
#pragma unroll
      for (int u = 0; u < NM; ++u) {
        const int e = tid + u * NT;
        if (e < m4) {
          const int i = e / g4;
          const float ki = sk[t * Y.ld + i];
          if (e % g4 == 0) sx[t * Y.ld + i] = __builtin_fmaf(ki, c, s[u]);
          const float kn = ki * ik;
#pragma unroll
          for (int x = 0; x < 4; ++x) mq[u][x] = __builtin_fmaf(kn, kv[x], mq[u][x]);
        }
      }
    }
  } else if (!global) {
    for (int e = tid; e < n * d; e += NT) sx[(e / d) * Y.ld + e % d] = sq[(e / d) * Y.ld + e % d];
  }
  __syncthreads();
  // delta = (W^2^T r) s'(z) on the slice's columns (HS / 16 <= 4 tiles, one per wave)
  if (w < HS / 16) {
    const f4 acc = row_sum<ND, false, FINE>(sr, Y.ld, 0, bd);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = 4 * lg + r, j = w * 16 + lc;
      sg[t * Y.ls + j] = acc[r] * ssp[t * Y.ls + j];
    }
  }
  __syncthreads();

  // token by token: the gated update, and a local memory's share of W2_t s(W1_t x)
  float* const share = step_share(a, chain, m);
  for (int t = 0; t < n; ++t)
    slice_token<ACT, D, NT, NU>(w1, s1, w2, s2, HS, global, sgt[t], sgt[STEP_N + t], 1.0f - sgt[2 * STEP_N + t],
                                sk + t * Y.ld, sr + t * Y.ld, sx + t * Y.ld, sa + t * Y.lh + j0, sg + t * Y.ls,
                                sz + (t & 1) * HS, share + ((size_t)t * G + g) * d);
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    if (e < n4) {
      const size_t o2 = (size_t)(e / h4) * hid + 4 * (e % h4);
      reinterpret_cast<f4*>(W1)[e] = w1[u];
      reinterpret_cast<f4*>(S1)[e] = s1[u];
      *reinterpret_cast<f4*>(W2 + o2) = w2[u];
      *reinterpret_cast<f4*>(S2 + o2) = s2[u];
    }
  }
}

// ---------------------------------------------------------------------------
// One token by itself, two launches before `out`: every weight of W^1 is read once and
// of W^2 twice, whatever the number of slices, and a workgroup holds the registers of
// one phase.  The products are the same MFMA tiles with one row that is not zero.
// ---------------------------------------------------------------------------
// entry: z = W^1 k of the slice's rows (and the global retrieval's W^1 q), the slice's
// share of W^2 s(z) (and of W^2 s(W^1 q)); a local memory's query x, its rows dealt to
// the slices
template <typename IO, int ACT, int D>
__global__ void __launch_bounds__(STEP_THREADS) step_entry_kernel(StepArgs a) {
  __shared__ __align__(16) float sk[D], sq[D], sa[64], saq[64];
  constexpr int d = D, g4 = D / 4, ND = D / 16, NW = STEP_THREADS / WAVE, TY = (ND + NW - 1) / NW;
  constexpr bool FINE = D <= 32;
  const int g = blockIdx.x, chain = blockIdx.y, m = blockIdx.z;
  const int hid = a.hid, HS = a.HS, G = a.G, j0 = g * HS;
  const int tid = threadIdx.x, l = lane_id(), w = wave_id(), lg = l >> 4, lc = l & 15;
  const bool global = a.has_global && m == 0;
  const bool proj = !global && a.qk_proj;
  const size_t hd = (size_t)hid * d;
  const float* const base = a.state + ((size_t)m * a.B * a.H + chain) * a.mem_stride;
  const float *Wh1 = base, *Wh2 = base + hd, *Mq = base + 6 * hd;
  const StepOne sc = step_one(a, chain, m);
  const size_t tok = ((size_t)chain * a.T + a.t0) * d;
  const IO *q = (const IO*)a.q + tok, *k = (const IO*)a.k + tok;
  for (int i = tid; i < d; i += STEP_THREADS) {
    sk[i] = to_f(k[i]);
    sq[i] = to_f(q[i]);
  }
  f4 bz[ND], by[TY][4];  // every weight of the workgroup, ahead of the first product
  if (w < HS / 16)
#pragma unroll
    for (int s = 0; s < ND; ++s)
      bz[s] = *reinterpret_cast<const f4*>(Wh1 + (size_t)(j0 + w * 16 + lc) * d + 16 * s + 4 * lg);
#pragma unroll
  for (int y = 0; y < TY; ++y)
    if (w + NW * y < ND)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (16 * s < HS)
          by[y][s] = *reinterpret_cast<const f4*>(Wh2 + (size_t)((w + NW * y) * 16 + lc) * hid + j0 + 16 * s + 4 * lg);
  __syncthreads();
  auto z_tile = [&](auto two) {
    constexpr bool TWO = decltype(two)::value;
    const f4 z = row_sum<ND, true, FINE>(sk, 0, 0, bz);
    f4 zq = zero4();
    if constexpr (TWO) zq = row_sum<ND, true, FINE>(sq, 0, 0, bz);
    if (lg == 0) {
      const int j = w * 16 + lc;
      const ActVals av = act_all<ACT>(z[0]);
      sa[j] = av.s;
      sc.a[j0 + j] = av.s;
      sc.sp[j0 + j] = av.d1;
      if constexpr (TWO) saq[j] = act_f<ACT>(zq[0]);
    }
  };
  if (w < HS / 16) {
    if (global)
      z_tile(std::true_type{});
    else
      z_tile(std::false_type{});
  }
  __syncthreads();
  auto y_tile = [&](int it, const f4(&b)[4], auto pieces, auto two) {
    constexpr int P = decltype(pieces)::value;
    constexpr bool TWO = decltype(two)::value;
    const f4 y = row_sum<P, true, FINE>(sa, 0, 0, b);
    f4 yq = zero4();
    if constexpr (TWO) yq = row_sum<P, true, FINE>(saq, 0, 0, b);
    if (lg == 0) {
      sc.yp[(size_t)g * d + it * 16 + lc] = y[0];
      if constexpr (TWO) sc.share[(size_t)g * d + it * 16 + lc] = yq[0];
    }
  };
  auto y_rows = [&](auto pieces) {
#pragma unroll
    for (int y = 0; y < TY; ++y)
      if (w + NW * y < ND) {
        if (global)
          y_tile(w + NW * y, by[y], pieces, std::true_type{});
        else
          y_tile(w + NW * y, by[y], pieces, std::false_type{});
      }
  };
  switch (HS / 16) {
    case 1: y_rows(std::integral_constant<int, 1>{}); break;
    case 2: y_rows(std::integral_constant<int, 2>{}); break;
    default: y_rows(std::integral_constant<int, 4>{}); break;
  }
  if (global) return;
  if (!proj) {
    for (int i = g * (d / G) + tid; i < (g + 1) * (d / G); i += STEP_THREADS) sc.x[i] = sq[i];
    return;
  }
  const float ik = inv_norm2(sk, d);
  float kq = 0.f;
  for (int i = l; i < d; i += WAVE) kq = __builtin_fmaf(sk[i], sq[i], kq);
  kq = wave_sum(kq);
  const float c = kq * ik;
  const f4 qv = reinterpret_cast<const f4*>(sq)[tid % g4];
  const int e1 = (g + 1) * (d / G) * g4;
  for (int e = g * (d / G) * g4 + tid; e - tid < e1; e += STEP_THREADS) {  // (whole groups of lanes)
    float s[1] = {e < e1 ? dot4(reinterpret_cast<const f4*>(Mq)[e], qv) : 0.f};
    group_sums<1>(s, g4);
    if (e < e1 && e % g4 == 0) sc.x[e / g4] = __builtin_fmaf(sk[e / g4], c, s[0]);
  }
}

// update: r, the slice's delta, the gated update and a local memory's retrieval share
template <typename IO, int ACT, int D>
__global__ void __launch_bounds__(step_threads(D)) step_update_kernel(StepArgs a) {
  __shared__ __align__(16) float sk[D], sr[D], sx[D], sa[64], ssp[64], sg[64], sz[64];
  constexpr int d = D, NT = step_threads(D), g4 = D / 4, ND = D / 16;
  constexpr bool FINE = D <= 32;
  constexpr int NU = D <= 32 ? 2 : 16 * D / NT;
  const int g = blockIdx.x, chain = blockIdx.y, m = blockIdx.z;
  const int H = a.H, hid = a.hid, HS = a.HS, G = a.G, j0 = g * HS;
  const int tid = threadIdx.x, l = lane_id(), w = wave_id(), lg = l >> 4, lc = l & 15;
  const bool global = a.has_global && m == 0;
  const size_t hd = (size_t)hid * d;
  float* const base = a.state + ((size_t)m * a.B * H + chain) * a.mem_stride;
  const float* Wh2 = base + hd;
  float *W1 = base + 2 * hd + (size_t)j0 * d, *W2 = base + 3 * hd + j0;
  float *S1 = base + 4 * hd + (size_t)j0 * d, *S2 = base + 5 * hd + j0;
  const StepOne sc = step_one(a, chain, m);
  const size_t tok = ((size_t)chain * a.T + a.t0) * d;
  const size_t gi = ((size_t)m * a.B * H + chain) * a.T + a.t0;
  const float rs = 2.0f / (float)d;
  f4 bd[ND];  // the slice's W^2 columns
  if (w < HS / 16)
#pragma unroll
    for (int s = 0; s < ND; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) bd[s][r] = Wh2[(size_t)(16 * s + 4 * lg + r) * hid + j0 + w * 16 + lc];
  const int h4 = HS / 4, n4 = HS * g4;
  f4 w1[NU], s1[NU], w2[NU], s2[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    w1[u] = s1[u] = w2[u] = s2[u] = zero4();
    if (e < n4) {
      const size_t o2 = (size_t)(e / h4) * hid + 4 * (e % h4);
      w1[u] = reinterpret_cast<const f4*>(W1)[e];
      s1[u] = reinterpret_cast<const f4*>(S1)[e];
      w2[u] = *reinterpret_cast<const f4*>(W2 + o2);
      s2[u] = *reinterpret_cast<const f4*>(S2 + o2);
    }
  }
  const float eta = a.lr[gi], beta = a.mom[gi], keep = 1.0f - a.decay[gi];
  if (tid < d) {
    sk[tid] = to_f(((const IO*)a.k)[tok + tid]);
    float y = 0.f;
    for (int gg = 0; gg < G; ++gg) y += sc.yp[(size_t)gg * d + tid];
    sr[tid] = rs * (y - to_f(((const IO*)a.v)[tok + tid]));
    if (!global) sx[tid] = sc.x[tid];
  }
  if (tid < HS) {
    sa[tid] = sc.a[j0 + tid];
    ssp[tid] = sc.sp[j0 + tid];
  }
  __syncthreads();
  if (w < HS / 16) {
    const f4 acc = row_sum<ND, true, FINE>(sr, 0, 0, bd);
    if (lg == 0) sg[w * 16 + lc] = acc[0] * ssp[w * 16 + lc];
  }
  __syncthreads();
  slice_token<ACT, D, NT, NU>(w1, s1, w2, s2, HS, global, eta, beta, keep, sk, sr, sx, sa, sg, sz,
                              sc.share + (size_t)g * d);
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    if (e < n4) {
      const size_t o2 = (size_t)(e / h4) * hid + 4 * (e % h4);
      reinterpret_cast<f4*>(W1)[e] = w1[u];
      reinterpret_cast<f4*>(S1)[e] = s1[u];
      *reinterpret_cast<f4*>(W2 + o2) = w2[u];
      *reinterpret_cast<f4*>(S2 + o2) = s2[u];
    }
  }
}

// blockIdx.y = 0: o = the global retrieval, then each local memory's shares (fixed
// order); blockIdx.y = 1 + i: local memory i's Q-K sum after the launch's tokens
template <typename IO>
__global__ void __launch_bounds__(STEP_THREADS) step_out_kernel(StepArgs a) {
  __shared__ __align__(16) float sk[STEP_N * STEP_MAX_D];
  __shared__ float skk[STEP_N];
  const int chain = blockIdx.x, d = a.d, G = a.G, n = a.n;
  const size_t tok = ((size_t)chain * a.T + a.t0) * d;
  if (blockIdx.y == 0) {
    IO* o = (IO*)a.o + tok;
    for (int e = threadIdx.x; e < n * d; e += STEP_THREADS) {
      const int t = e / d, i = e - t * d;
      float acc = a.has_global ? step_share(a, chain, 0)[e] : 0.f;
      if (a.one && a.has_global)
        for (int gg = 1; gg < G; ++gg) acc += step_share(a, chain, 0)[(size_t)gg * d + e];
      for (int m = a.has_global; m < a.M; ++m) {
        const float* sh = step_share(a, chain, m) + (size_t)t * G * d + i;
        for (int gg = 0; gg < G; ++gg) acc += sh[(size_t)gg * d];
      }
      o[e] = from_f<IO>(acc);
    }
    return;
  }
  const int m = a.has_global + (int)blockIdx.y - 1;
  f4* M4 = reinterpret_cast<f4*>(a.state + ((size_t)m * a.B * a.H + chain) * a.mem_stride +
                                 6 * (size_t)a.hid * d);
  for (int e = threadIdx.x; e < n * d; e += STEP_THREADS) sk[e] = to_f(((const IO*)a.k)[tok + e]);
  __syncthreads();
  for (int t = wave_id(); t < n; t += STEP_THREADS / WAVE) {
    const float ik = inv_norm2(sk + t * d, d);
    if (lane_id() == 0) skk[t] = ik;
  }
  __syncthreads();
  const int g4 = d / 4;
  for (int e = threadIdx.x; e < d * g4; e += STEP_THREADS) {
    const int i = e / g4, c4 = e - i * g4;
    f4 x = M4[e];
    for (int t = 0; t < n; ++t) {
      const f4 kv = reinterpret_cast<const f4*>(sk + t * d)[c4];
      const float kn = sk[t * d + i] * skk[t];
#pragma unroll
      for (int y = 0; y < 4; ++y) x[y] = __builtin_fmaf(kn, kv[y], x[y]);
    }
    M4[e] = x;
  }
}

// state blocks of every (memory, chain): W^1 = W1 = W1_init[m][h], W^2 = W2 =
// W2_init[m][h], S = 0, M = 0; with `fin`, a forward's final state [chain][4][hid*d] of
// the global memory (V1, V2, S1, S2), memory 0 starts there: W^1 = W1 = V1, W^2 = W2 = V2,
// S1, S2.  Bound by its bytes, so STEP_INIT_SLICES workgroups write a block together, 16
// bytes a lane: 8 chains at d 64, hid 256, global + one local, took 55 us to set and 91 to
// copy with one workgroup a block and 4 bytes a lane, 5 us now for both.
constexpr int STEP_INIT_SLICES = 16;

__global__ void __launch_bounds__(256) step_init_kernel(StepArgs a, const float* fin) {
  const int chain = blockIdx.x, m = blockIdx.y;
  const int h = chain % a.H;
  const size_t hd = (size_t)a.hid * a.d, n4 = hd / 4;  // (every size is a multiple of 64)
  f4* base = reinterpret_cast<f4*>(a.state + ((size_t)m * a.B * a.H + chain) * a.mem_stride);
  const bool from = fin && m == 0;
  const float* f = from ? fin + (size_t)chain * 4 * hd : nullptr;
  const f4* W1 = reinterpret_cast<const f4*>(from ? f : a.W1i + ((size_t)m * a.H + h) * hd);
  const f4* W2 = reinterpret_cast<const f4*>(from ? f + hd : a.W2i + ((size_t)m * a.H + h) * hd);
  const f4* S = reinterpret_cast<const f4*>(from ? f + 2 * hd : nullptr);
  const size_t first = (size_t)blockIdx.z * blockDim.x + threadIdx.x;
  const size_t step = (size_t)gridDim.z * blockDim.x;
  for (size_t e = first; e < n4; e += step) {
    const f4 w1 = W1[e], w2 = W2[e];
    const f4 s1 = from ? S[e] : zero4(), s2 = from ? S[n4 + e] : zero4();
    base[e] = base[2 * n4 + e] = w1;
    base[n4 + e] = base[3 * n4 + e] = w2;
    base[4 * n4 + e] = s1;
    base[5 * n4 + e] = s2;
  }
  for (size_t e = 6 * n4 + first; e < a.mem_stride / 4; e += step) base[e] = zero4();
}

hipError_t launch_step_from_final(const StepArgs& a, const float* fin, hipStream_t st) {
  hipLaunchKernelGGL(step_init_kernel, dim3(a.B * a.H, a.M, STEP_INIT_SLICES), dim3(256), 0, st, a,
                     a.has_global ? fin : nullptr);
  return hipGetLastError();
}

size_t step_state_floats(int d, int hid) { return 6 * (size_t)hid * d + (size_t)d * d; }

size_t step_scratch_floats(int d, int hid) {
  const int HS = hid < 64 ? hid : 64, G = hid / HS;
  const size_t n = 2 * (size_t)hid + d + 3 * (size_t)G * d;
  return (n + 63) / 64 * 64;
}

hipError_t launch_step_init(const StepArgs& a, hipStream_t st) {
  return launch_step_from_final(a, nullptr, st);
}

// Whether the next token goes by itself (three launches, weights read once or twice)
// rather than with the others of its chunk (two, but every slice reads all of W^1 and W^2
// and a CU holds one workgroup).  One token, us by itself / together:
//   d 64, hid 256, global + one local: 1 chain 14.7 / 17.6, 32 chains 17.7 / 23.3, 128
//   38.5 / 77; d 128, hid 512: 21.5 / 43, 44 / 122, 172 / 514; d 128, hid 128: 1 chain 21 /
//   29; d 32, hid 512: 15.3 / 19.5
//   d 64, hid 128: 1 chain 14.9 / 13.8, 32 15.8 / 15.4, 128 (512 workgroups) 24.7 / 33.7;
//   d 32, hid 128: 15.2 / 12.2, 15.0 / 12.0, 15.9 / 16.2; d 16, hid 32: 1 to 256 chains
//   (up to 512 workgroups) 15.3 / 12.0, 512 chains 14.7 / 14.7
// so: from 64 KB a matrix or d 128 on; from 16 KB where there are more workgroups than
// CUs; below that, four times as many.  Two
// tokens: d 128, hid 512 42 / 46 (1 chain), 87 / 129, 344 / 537; d 64, hid 256 34 / 25 (32
// chains, 256 workgroups), 77 / 84 (128, 1024); three at d 128, hid 512: 64 / 50, 131 /
// 133, 517 / 550.
static bool step_alone(const StepArgs& a) {
  constexpr long cus = 256;  // of the whole card (a query costs the host more than it tells)
  const long grid = (long)a.G * a.B * a.H * a.M;
  const int hd = a.hid * a.d;
  switch (a.n) {
    case 1: return hd >= 16384 || a.d == 128 || (hd >= 4096 && grid > cus) || grid >= 4 * cus;
    case 2: return hd >= 65536 || (hd >= 16384 && grid >= 4 * cus);
    case 3: return hd >= 65536 && grid >= 2 * cus;
    default: return false;
  }
}

template <typename IO, int ACT, int D>
static hipError_t step_run(StepArgs a, hipStream_t st) {
  const size_t lds = (size_t)step_lds(a.d, a.hid, a.HS).total * sizeof(float);
  auto kern = step_tokens_kernel<IO, ACT, D>;
  if (a.d != D || !lds_fits((const void*)kern, lds)) return hipErrorInvalidConfiguration;
  set_lds_limit((const void*)kern);
  const int BH = a.B * a.H, nloc = a.M - a.has_global;
  // tokens whose shares fit a chain's scratch blocks
  const size_t per = (size_t)a.d * (a.has_global + nloc * a.G);
  const int most = std::min<int>(STEP_N, (int)((size_t)a.M * a.sc_stride / per));
  for (int t = 0; t < a.T; t += a.n) {
    a.t0 = t;
    a.n = std::min(most, a.T - t);
    bool bound = false;
    for (int m = 0; m < a.M; ++m) {  // (a shard starts only where a chunk does)
      const long long in = (a.pos + t) % a.C[m];
      bound |= in == 0;
      a.n = (int)std::min<long long>(a.n, a.C[m] - in);
    }
    a.one = step_alone(a) ? 1 : 0;
    if (a.one) a.n = 1;
    if (bound) hipLaunchKernelGGL(step_boundary_kernel, dim3(16, BH, a.M), dim3(256), 0, st, a);
    const dim3 grid(a.G, BH, a.M);
    if (a.one) {
      hipLaunchKernelGGL((step_entry_kernel<IO, ACT, D>), grid, dim3(STEP_THREADS), 0, st, a);
      hipLaunchKernelGGL((step_update_kernel<IO, ACT, D>), grid, dim3(step_threads(D)), 0, st, a);
    } else {
      hipLaunchKernelGGL(kern, grid, dim3(step_threads(D)), lds, st, a);
    }
    hipLaunchKernelGGL(step_out_kernel<IO>, dim3(BH, 1 + nloc), dim3(STEP_THREADS), 0, st, a);
  }
  return hipGetLastError();
}

template <typename IO, int ACT>
static hipError_t step_sizes(const StepArgs& a, hipStream_t st) {
  return a.d == 16   ? step_run<IO, ACT, 16>(a, st)
         : a.d == 32 ? step_run<IO, ACT, 32>(a, st)
         : a.d == 64 ? step_run<IO, ACT, 64>(a, st)
                     : step_run<IO, ACT, 128>(a, st);
}

hipError_t launch_step(const StepArgs& a, hipStream_t st) {
  if (a.d > STEP_MAX_D || a.hid > STEP_MAX_H || a.HS > 64 || a.G * a.HS != a.hid || !a.scratch)
    return hipErrorInvalidValue;
  if (a.bf16)
    return a.act == ACT_SILU ? step_sizes<__bf16, ACT_SILU>(a, st) : step_sizes<__bf16, ACT_GELU>(a, st);
  return a.act == ACT_SILU ? step_sizes<float, ACT_SILU>(a, st) : step_sizes<float, ACT_GELU>(a, st);
}

}  // namespace tnt
